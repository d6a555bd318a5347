// Fields of many chains as one matrix product per problem, H = X A (X the
// chains' 0/1 states, [chains][N]; A the off-diagonal coefficients,
// symmetric), on the int8 matrix cores with exact int32 sums.
//
// An entry of A is a number of up to five signed bytes: the two or four bytes
// of an integer, or for float entries a 39-bit fixed-point number in units of
// the row's own scale, q = rint(a 2^(38 - e)) with |a| < 2^e over the row.
// The sums of the byte planes put together in 64 bits are the exact sums of
// the q (|sum| <= 16384 2^38 < 2^53), so a float field is the exact sum
// rounded once.  A float entry below 2^-14 of its row's largest may have bits
// below that unit: what is left of it, exact in FP64, goes to a short list of
// the row (kRest entries, by column) and is added to the fields of the chains
// whose bit is set.  Rows with more such entries than the list holds are left
// to an FP64 product, 64 fields at a time.
//
// Layout: a workgroup of 2 WM waves computes 64 WM chains x 64 fields, a wave
// 64 chains x 32 fields (4 x 2 tiles of 16 x 16 for every plane).  Per step of
// 64 columns the workgroup loads its 64 x 64 entries once, two steps ahead,
// splits them into the byte planes and puts those and the states into LDS in
// the order in which the lanes read them as operands (16 bytes per lane), two
// buffers with one barrier per step.  Bound: at N = 8192 float32, 1024 chains,
// the matrix cores need 0.14 ms for the five planes, LDS moves 148 KB per
// step (0.13 ms) and the splitting is six VALU instructions an entry (0.09
// ms); the waves of a workgroup go through these in turn rather than at once:
// 0.38 ms, and 0.08 for the row data.  The FP64 product took 2.9 ms (2.0 at
// the rate of a large one).  In all, from states to energies: 4096 chains
// 10.4 -> 1.65 ms, 1024 chains 2.89 -> 0.50; N = 512, 8192 chains 119 -> 46
// us; int16 N = 8192, 1024 chains 1180 -> 209 us (from a product that split
// the entries once per 64 chains); int32 N = 3001, 256 chains 141 -> 67 us.
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "pns_internal.h"

namespace pns {
namespace {

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));

constexpr int kRest = 32;    // entries of a row's list of remainders
constexpr int kUnitBits = 38;  // |q| <= 2^38

// Row data of a float matrix: exponent e of each row, the number of
// remainders (-1: more than kRest), their columns and values.
struct RowPrep {
    int32_t* e;
    int32_t* n;
    int32_t* col;  // [N][kRest]
    double* val;   // [N][kRest]
};

__host__ __device__ inline RowPrep row_prep(void* ws, int64_t N)
{
    RowPrep r;
    r.val = reinterpret_cast<double*>(ws);
    r.col = reinterpret_cast<int32_t*>(r.val + N * kRest);
    r.e = r.col + N * kRest;
    r.n = r.e + N;
    return r;
}

// One workgroup per row of a float matrix.  Memory bound: the row is read
// from HBM once (its second pass finds it in the caches).
__global__ __launch_bounds__(256) void row_prep_kernel(InitArgs a, int32_t cbeg)
{
    const Problem P = a.problems[a.chain_problem[cbeg]];
    const RowPrep rp = row_prep(a.fields_ws, P.N);
    const int row = blockIdx.x;
    if (row >= P.N) return;
    const float4* src = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(P.A) + (int64_t)row * P.pitch);
    const int quads = (int)(P.pitch / 4);
    __shared__ uint32_t smax[4];
    __shared__ int cnt;
    __shared__ int32_t lcol[kRest];
    __shared__ double lval[kRest];
    if (threadIdx.x == 0) cnt = 0;
    uint32_t m = 0;
    for (int q = threadIdx.x; q < quads; q += 256) {
        const float4 v = src[q];
        m = max(m, max(max(__float_as_uint(v.x) & 0x7FFFFFFFu, __float_as_uint(v.y) & 0x7FFFFFFFu),
                       max(__float_as_uint(v.z) & 0x7FFFFFFFu, __float_as_uint(v.w) & 0x7FFFFFFFu)));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, 64));
    if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = m;
    __syncthreads();
    m = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
    int e = 0;
    if (m != 0) (void)frexp((double)__uint_as_float(m), &e);
    const int sh = kUnitBits - e;
    for (int q = threadIdx.x; q < quads; q += 256) {
        const float4 v4 = src[q];
        const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double d = ldexp((double)v[i], sh);
            const double f = d - rint(d);
            if (f != 0.0) {
                const int at = atomicAdd(&cnt, 1);
                if (at < kRest) {
                    lcol[at] = q * 4 + i;
                    lval[at] = ldexp(f, -sh);
                }
            }
        }
    }
    __syncthreads();
    const int n = cnt;
    if (threadIdx.x < 64 && n <= kRest) {
        // by column, so that the sums do not depend on the order of arrival
        const int t = threadIdx.x;
        if (t < n) {
            int rank = 0;
            for (int j = 0; j < n; ++j) rank += lcol[j] < lcol[t] ? 1 : 0;
            rp.col[(int64_t)row * kRest + rank] = lcol[t];
            rp.val[(int64_t)row * kRest + rank] = lval[t];
        }
    }
    if (threadIdx.x == 0) {
        rp.e[row] = e;
        rp.n[row] = n <= kRest ? n : -1;
    }
}

// True if one of the 64 fields from f0 has more remainders than its list
// holds (every lane of the wave takes part).
__device__ __forceinline__ bool needs_f64(const RowPrep& rp, int64_t f0, int64_t N, int lane)
{
    return __ballot(f0 + lane < N && rp.n[f0 + lane] < 0) != 0;
}

// Byte transpose of four words: out[p] = byte p of e[0], e[1], e[2], e[3].
__device__ __forceinline__ void planes4(const uint32_t (&e)[4], uint32_t (&out)[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(e[1], e[0], 0x05010400u), t1 = __builtin_amdgcn_perm(e[3], e[2], 0x05010400u);
    const uint32_t u0 = __builtin_amdgcn_perm(e[1], e[0], 0x07030602u), u1 = __builtin_amdgcn_perm(e[3], e[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(u1, u0, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
}

// Signed bytes of four consecutive entries, plane p of them in out[p].
// Integers: bytes as they are, all but the top one moved by -128 to int8
// (the sums are moved back by 128 times the number of set bits).
__device__ __forceinline__ void split4(const int16_t* v, double, uint32_t (&out)[2])
{
    const uint32_t w0 = reinterpret_cast<const uint32_t*>(v)[0], w1 = reinterpret_cast<const uint32_t*>(v)[1];
    out[0] = __builtin_amdgcn_perm(w1, w0, 0x06040200u) ^ 0x80808080u;
    out[1] = __builtin_amdgcn_perm(w1, w0, 0x07050301u);
}
__device__ __forceinline__ void split4(const int32_t* v, double, uint32_t (&out)[4])
{
    const uint32_t e[4] = {(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
    planes4(e, out);
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] ^= 0x80808080u;
}
// Floats: a 2^(38 - e) rounded to an integer by the addition of 3 2^51 (its
// low 40 bits are then those of q in two's complement), plus 128 in each of
// the four low bytes, which makes the bytes minus 128 signed digits of q.
__device__ __forceinline__ void split4(const float* v, double scale, uint32_t (&out)[5])
{
    uint32_t lo[4], hi[4], pl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double d = fma((double)v[i], scale, 6755399441055744.0 + 2155905152.0);
        lo[i] = (uint32_t)__double2loint(d);
        hi[i] = (uint32_t)__double2hiint(d);
    }
    planes4(lo, pl);
#pragma unroll
    for (int p = 0; p < 4; ++p) out[p] = pl[p] ^ 0x80808080u;
    out[4] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(hi[3], hi[2], 0x0C0C0400u),
                                   __builtin_amdgcn_perm(hi[1], hi[0], 0x0C0C0400u), 0x05040100u);
}

template <typename QT>
constexpr int num_planes()
{
    return std::is_floating_point<QT>::value ? 5 : (int)sizeof(QT);
}

template <typename QT, typename HT, int WM>
__global__ __launch_bounds__(128 * WM, 2) void fields_kernel(InitArgs a, int32_t cbeg, int32_t cend, int32_t nc)
{
    constexpr bool kFloat = std::is_floating_point<QT>::value;
    constexpr int NP = num_planes<QT>();
    constexpr int T = 128 * WM;        // threads
    constexpr int EPT = 64 * 64 / T;   // entries per thread and step: 8 or 16
    constexpr int TPR = 64 / EPT;      // threads per row of A
    constexpr int NL = EPT * (int)sizeof(QT) / 16;  // 16-byte loads per thread and step
    __shared__ i32x4_t bs[2][NP][4][64];
    __shared__ uint4 xs[2][4 * WM][64];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r16 = lane & 15, kg = lane >> 4;
    const Problem P = a.problems[a.chain_problem[cbeg]];
    // The chain blocks of one field block follow each other on one XCD
    // (workgroups go round the eight XCDs), whose L2 then serves their rows.
    const int32_t fblk = ((int32_t)(blockIdx.x >> 3) / nc) * 8 + (int32_t)(blockIdx.x & 7);
    const int32_t cblk = (int32_t)(blockIdx.x >> 3) % nc;
    const int64_t f0 = (int64_t)fblk * 64;
    if (f0 >= P.pitch) return;
    RowPrep rp{};
    if constexpr (kFloat) {
        rp = row_prep(a.fields_ws, P.N);
        if (needs_f64(rp, f0, P.N, lane)) return;
    }
    const int32_t cw = cbeg + cblk * 64 * WM + wm * 64;  // this wave's first chain

    // this thread's entries: EPT columns of row f0 + fl (rows past N: zeros)
    const int fl = tid / TPR, ko = (tid % TPR) * EPT;
    const bool row_ok = f0 + fl < P.N;
    const QT* arow = reinterpret_cast<const QT*>(P.A) + (row_ok ? f0 + fl : 0) * P.pitch + ko;
    double scale = 0.0;
    if constexpr (kFloat) scale = row_ok ? ldexp(1.0, kUnitBits - rp.e[f0 + fl]) : 0.0;
    // (a problem's chains lie one after the other)
    const int64_t off0 = a.foff[cbeg];
    // This thread's state bytes: 16 columns of two chains.  Four lanes read a
    // chain's 64 bytes (read in the operands' order, 16 rows to 16 lanes, the
    // cache would look up 64 lines per load instead of 16: int16 N = 8192,
    // 1024 chains 300 us instead of 209).  Chains past the last: the
    // last one's, computed along and not written.
    const int xr = tid >> 2, xk = tid & 3;
    const uint8_t* xrow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        xrow[i] = a.x + off0 + (int64_t)(min(cbeg + cblk * 64 * WM + xr + i * 32 * WM, cend - 1) - cbeg) * P.pitch + 16 * xk;

    // The column at which the loop's step k0 reads (steps past the end read
    // again from the start, unused).  The field blocks start 5 steps apart:
    // at a power-of-two pitch all rows have the same column on the same L2
    // channel (256 bytes, 16 channels), and workgroups in step with each other
    // would all wait for that one.  (The sums are exact in any order.)
    const int64_t rot = (int64_t)(fblk >> 3) * 5 * 64 % P.pitch;
    auto column = [&](int64_t k0) {
        int64_t k = k0 + rot;
        k -= k >= P.pitch ? P.pitch : 0;
        return k >= P.pitch ? k - P.pitch : k;
    };
    // Entries are loaded two steps ahead (two sets of registers, used in turn),
    // states one: a row comes from HBM, whose latency is longer than a step.
    uint4 araw[2][NL], xnext[2];
    auto load_a = [&](uint4 (&r)[NL], int64_t k0) {
        k0 = column(k0);
#pragma unroll
        for (int l = 0; l < NL; ++l) r[l] = reinterpret_cast<const uint4*>(arow + k0)[l];
    };
    auto load_x = [&](int64_t k0) {
        k0 = column(k0);
#pragma unroll
        for (int i = 0; i < 2; ++i) xnext[i] = *reinterpret_cast<const uint4*>(xrow[i] + k0);
    };
    // (operand lane 16 xk + chain % 16 of its chain tile, the 16 lanes of each
    // xk rotated by 4 xk so that neither side meets bank conflicts)
    auto stage_x = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = xr + i * 32 * WM;
            xs[buf][r >> 4][xk * 16 + ((r + 4 * xk) & 15)] =
                make_uint4(xnext[i].x & 0x01010101u, xnext[i].y & 0x01010101u, xnext[i].z & 0x01010101u,
                           xnext[i].w & 0x01010101u);
        }
    };
    auto stage = [&](uint4 (&r)[NL], int buf) {
        uint32_t pw[NP][EPT / 4];
        if constexpr (!kFloat) {  // (a row past N: scale 0 makes float entries 0)
#pragma unroll
            for (int l = 0; l < NL; ++l) r[l] = row_ok ? r[l] : make_uint4(0u, 0u, 0u, 0u);
        }
        const QT* v = reinterpret_cast<const QT*>(r);
#pragma unroll
        for (int q = 0; q < EPT / 4; ++q) {
            uint32_t o[NP];
            split4(v + 4 * q, scale, o);
#pragma unroll
            for (int p = 0; p < NP; ++p) pw[p][q] = o[p];
        }
        // operand lane (ko / 16) * 16 + fl % 16 of field tile fl / 16
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            char* dst = reinterpret_cast<char*>(&bs[buf][p][fl >> 4][(ko >> 4) * 16 + (fl & 15)]) + (ko & 15);
            if constexpr (EPT == 16) *reinterpret_cast<uint4*>(dst) = make_uint4(pw[p][0], pw[p][1], pw[p][2], pw[p][3]);
            else *reinterpret_cast<uint2*>(dst) = make_uint2(pw[p][0], pw[p][1]);
        }
    };

    i32x4_t acc[NP][4][2];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[p][i][j] = (i32x4_t){0, 0, 0, 0};
    int32_t xsum[4] = {0, 0, 0, 0};

    // one step: the products of the planes in LDS buffer S, then step k0 + 64's
    // entries (register set S ^ 1) into the other buffer
    auto step = [&](int64_t k0, auto sc) {
        constexpr int S = decltype(sc)::value;
        // (the states first: the end of the step waits for them alone, the
        // entries stay in flight)
        load_x(k0 + 64);
        __builtin_amdgcn_sched_barrier(0);
        load_a(araw[S], k0 + 128);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();  // this step's planes are in LDS, and every wave is done with the other buffer
        i32x4_t xop[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 w = xs[S][wm * 4 + i][kg * 16 + ((r16 + 4 * kg) & 15)];
            if constexpr (!kFloat)
                xsum[i] += __builtin_popcount(w.x) + __builtin_popcount(w.y) + __builtin_popcount(w.z) +
                           __builtin_popcount(w.w);
            xop[i] = (i32x4_t){(int)w.x, (int)w.y, (int)w.z, (int)w.w};
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const i32x4_t bop = bs[S][p][wn * 2 + j][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[p][i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xop[i], bop, acc[p][i][j], 0, 0, 0);
            }
        stage(araw[S ^ 1], S ^ 1);
        stage_x(S ^ 1);
    };
    load_a(araw[0], 0);
    load_x(0);
    __builtin_amdgcn_sched_barrier(0);
    load_a(araw[1], 64);
    stage(araw[0], 0);
    stage_x(0);
    for (int64_t k0 = 0; k0 < P.pitch; k0 += 128) {
        step(k0, std::integral_constant<int, 0>{});
        if (k0 + 64 < P.pitch) step(k0 + 64, std::integral_constant<int, 1>{});
    }

    // output register e of a lane: chain 4 kg + e of the chain tile, field r16
    // of the field tile
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t f = f0 + wn * 32 + j * 16 + r16;
        const bool fok = f < P.N;
        int nrest = 0;
        double unit = 0.0;
        if constexpr (kFloat) {
            if (fok) {
                nrest = rp.n[f];
                unit = ldexp(1.0, rp.e[f] - kUnitBits);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // set bits of the 16 operand rows (four lanes hold each)
            int32_t bits = xsum[i];
            if constexpr (!kFloat) {
                bits += __shfl_xor(bits, 16, 64);
                bits += __shfl_xor(bits, 32, 64);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int64_t v = 0;
#pragma unroll
                for (int p = NP - 1; p >= 0; --p) v = v * 256 + (int64_t)acc[p][i][j][e];
                if constexpr (!kFloat) {
                    constexpr int64_t kOff = NP == 2 ? 128 : 128 * (1 + 256 + 65536);
                    v += kOff * (int64_t)__shfl(bits, kg * 4 + e, 64);
                }
                const int32_t c = cw + i * 16 + kg * 4 + e;
                if (c >= cend) continue;
                const int64_t off = off0 + (int64_t)(c - cbeg) * P.pitch;
                if constexpr (kFloat) {
                    double h = (double)v * unit;
                    for (int t = 0; t < nrest; ++t)
                        if (a.x[off + rp.col[f * kRest + t]] & 1u) h += rp.val[f * kRest + t];
                    reinterpret_cast<HT*>(a.h)[off + f] = (HT)h;
                } else {
                    reinterpret_cast<HT*>(a.h)[off + f] = (HT)v;
                }
            }
        }
    }
}

// The 64-field blocks of a float matrix with a row of more than kRest
// remainders (entries spread over many orders of magnitude), on the FP64
// matrix cores: x and A as FP64 (both exact), FP64 accumulation.  A workgroup
// of four waves computes 64 chains x 64 fields; the others' return at once.
// Each lane takes four
// consecutive k of its row (k0 + 4 kg + m); MFMA m of a 16-deep step sums over
// the four lane groups.
__global__ __launch_bounds__(256) void fields_f64_kernel(InitArgs a, int32_t cbeg, int32_t cend)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, kg = lane >> 4;
    const Problem P = a.problems[a.chain_problem[cbeg]];
    const int32_t cw = cbeg + (int32_t)blockIdx.y * 64 + wave * 16;
    const int64_t f0 = (int64_t)blockIdx.x * 64;
    if (!needs_f64(row_prep(a.fields_ws, P.N), f0, P.N, lane)) return;
    const int32_t crow = cw + r16;
    const uint8_t* xrow = crow < cend ? a.x + a.foff[crow] : nullptr;
    const float* A = reinterpret_cast<const float*>(P.A);
    f64x4_t acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    for (int64_t k0 = 0; k0 < P.pitch; k0 += 16) {
        const int64_t k = k0 + 4 * kg;
        uint32_t xw = xrow != nullptr ? *reinterpret_cast<const uint32_t*>(xrow + k) : 0u;
        double xd[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) xd[m] = (k + m < P.N && ((xw >> (8 * m)) & 1u)) ? 1.0 : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t fr = f0 + 16 * t + r16;  // A has N rows: fields past N read zeros
            const float4 av = fr < P.N ? *reinterpret_cast<const float4*>(A + fr * P.pitch + k)
                                       : make_float4(0.f, 0.f, 0.f, 0.f);
            const float am[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
            for (int m = 0; m < 4; ++m)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[m], (double)am[m], acc[t], 0, 0, 0);
        }
    }
    // output register e of a lane holds row kg + 4 e (rows interleaved across
    // the lane groups in the FP64 product), column r16
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int32_t c = cw + kg + 4 * e;
        if (c >= cend) continue;
        double* hc = reinterpret_cast<double*>(a.h) + a.foff[c];
#pragma unroll
        for (int t = 0; t < 4; ++t) hc[f0 + 16 * t + r16] = acc[t][e];
    }
}

template <typename QT, typename HT>
hipError_t launch_typed(int64_t pitch, const InitArgs& a, int32_t cbeg, int32_t cend, hipStream_t st)
{
    if constexpr (std::is_floating_point<QT>::value) {
        // (rows up to the pitch: the workgroups past N return)
        hipLaunchKernelGGL(row_prep_kernel, dim3((unsigned)pitch), dim3(256), 0, st, a, cbeg);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // 256 chains to a workgroup where that still gives every compute unit one
    // (each entry is split once per 256 chains: N = 8192 float32, 1024 chains
    // 0.50 ms, at 128 chains to a workgroup 0.62), else 128 (N = 2000, 100
    // chains: half the lanes of 256 would hold no chain).
    const int64_t nf = pitch / 64, chains = cend - cbeg;
    const bool wide = nf * ((chains + 255) / 256) >= 256;
    const int32_t nc = (int32_t)(wide ? (chains + 255) / 256 : (chains + 127) / 128);
    const dim3 grid((unsigned)((nf + 7) / 8 * 8 * nc));
    if (wide) hipLaunchKernelGGL((fields_kernel<QT, HT, 4>), grid, dim3(512), 0, st, a, cbeg, cend, nc);
    else hipLaunchKernelGGL((fields_kernel<QT, HT, 2>), grid, dim3(256), 0, st, a, cbeg, cend, nc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (std::is_floating_point<QT>::value) {
        hipLaunchKernelGGL(fields_f64_kernel, dim3((unsigned)nf, (unsigned)((chains + 63) / 64)), dim3(256), 0, st, a,
                           cbeg, cend);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

size_t fields_ws_bytes(int64_t N) { return (size_t)N * (kRest * (sizeof(double) + sizeof(int32_t)) + 2 * sizeof(int32_t)); }

hipError_t launch_fields(int32_t qtype, int32_t htype, int64_t pitch, const InitArgs& a, int32_t cbeg, int32_t cend,
                         hipStream_t st)
{
    if (qtype == Q_I16 && htype == H_I32) return launch_typed<int16_t, int32_t>(pitch, a, cbeg, cend, st);
    if (qtype == Q_I32 && htype == H_I32) return launch_typed<int32_t, int32_t>(pitch, a, cbeg, cend, st);
    if (qtype == Q_I32 && htype == H_I64) return launch_typed<int32_t, int64_t>(pitch, a, cbeg, cend, st);
    if (qtype == Q_F32 && htype == H_F64) return launch_typed<float, double>(pitch, a, cbeg, cend, st);
    return hipErrorInvalidConfiguration;
}

}  // namespace pns
