// Kernels of the differentiation path.
//
// * Multiplicity-weighted second moments G = X^T diag(m) X of jump-chain
//   records (x_k, m_k): the estimate of E_pi[x x^T] (times sum_k m_k) whose
//   product with -beta is grad_Q log Z.  Dense contraction over the records
//   on the matrix cores.  Integer weights: v_mfma_i32_16x16x64_i8, x as 0/1
//   bytes and m_k as digits base 128, a pass over the records per digit (the
//   first digit of all of them, a further one only of the steps of 64 records
//   that have it), so that the sums of a workgroup are exact and an entry of G
//   below 2^53 is.  Real weights:
//   v_mfma_f32_16x16x32_bf16 with FP32 accumulation, each weight split into
//   three bf16 pieces.
// * log Z = log sum_x exp(-beta x^T Q x) by enumeration of all 2^N states
//   (N <= 32), 16 states of a lane at a time, FP64 log-sum-exp.
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "pns_internal.h"
#include "pns_step.h"

namespace pns {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Round-to-nearest-even of a float to bf16 (bit pattern).
__device__ __forceinline__ uint16_t bf16_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(r >> 16);
}

__device__ __forceinline__ float bf16_value(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Digits of integer weights, base 128, and their sum.  A step is 64 records;
// digit d of the step's weights is 64 bytes of digits[d], in the order of the
// operand bytes of moments_i8_kernel, and ndig[step] says how many digits the
// step's largest weight has (the others are not written).  Negative weights
// count as 0.  One wave per step; each workgroup's sum goes to psum[block].
constexpr int kDigits = 9;  // 63 bits, 7 bits each

__device__ void weight_digits(const int64_t* __restrict__ m, int64_t K, int64_t steps, uint8_t* __restrict__ digits,
                              uint8_t* __restrict__ ndig, unsigned long long* __restrict__ psum, int block, int blocks)
{
    __shared__ unsigned long long red[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // byte of record `lane` of a step: of word lane / 32 of a column, operand
    // lane group kg and register j take the bits 4 (kg % 2) + j + 8 b
    const int bit = lane & 31, word = lane >> 5;
    const int pos = (word * 2 + ((bit & 7) >> 2)) * 16 + (bit & 3) * 4 + (bit >> 3);
    unsigned long long sum = 0;
    for (int64_t st = (int64_t)block * 4 + wave; st < steps; st += (int64_t)blocks * 4) {
        const int64_t k = st * 64 + lane;
        const int64_t mk = k < K && m[k] > 0 ? m[k] : 0;
        sum += (unsigned long long)mk;
        int nd = 0;
        do {
            digits[(int64_t)nd * steps * 64 + st * 64 + pos] = (uint8_t)((uint64_t)mk >> (7 * nd) & 127u);
            ++nd;
        } while (nd < kDigits && __ballot(((uint64_t)mk >> (7 * nd)) != 0) != 0);
        if (lane == 0) ndig[st] = (uint8_t)nd;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) psum[block] = red[0] + red[1] + red[2] + red[3];
}

// Real (FP64) weights, e.g. the expected multiplicities 1 / p of Thm 3 (5).
// First the largest |w_k| (finite ones; bit patterns of non-negative doubles
// order like the numbers), so that the weights can be scaled by a power of
// two into [-2, 2] before they are rounded to FP32 (relative 2^-24) and split
// exactly into three bf16 pieces; G is scaled back at the end.  Non-finite
// weights count as 0 in G and in the sum.
__global__ __launch_bounds__(256) void moments_absmax_kernel(const double* w, int64_t K, unsigned long long* maxbits)
{
    __shared__ unsigned long long red[4];
    unsigned long long b = 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x) {
        const double v = isfinite(w[k]) ? fabs(w[k]) : 0.0;
        const unsigned long long vb = (unsigned long long)__double_as_longlong(v);
        b = b > vb ? b : vb;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long o = __shfl_xor(b, d, 64);
        b = b > o ? b : o;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t = t > red[i] ? t : red[i];
        atomicMax(maxbits, t);
    }
}

__device__ __forceinline__ int weight_exponent(const unsigned long long* maxbits)
{
    const double mx = __longlong_as_double((long long)*maxbits);
    return mx > 0.0 ? ilogb(mx) : 0;
}

__global__ __launch_bounds__(256) void moments_prep_f64_kernel(const double* w, int64_t K, int64_t kpad,
                                                               uint16_t* pieces, double* sum_w,
                                                               const unsigned long long* maxbits)
{
    __shared__ double red[4];
    const int64_t n = kpad > K ? kpad : K;
    const int e = weight_exponent(maxbits);
    double sv = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        double wk = 0.0;
        if (k < K && isfinite(w[k])) wk = w[k];
        if (k < kpad) {
            float r = (float)ldexp(wk, -e);
            uint16_t b[3];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                b[s] = bf16_bits(r);
                r = r - bf16_value(b[s]);
            }
#pragma unroll
            for (int s = 0; s < 3; ++s) pieces[s * kpad + k] = b[s];
        }
        sv += wk;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sv += __shfl_xor(sv, d, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sv;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
        atomicAdd(sum_w, t);
    }
}

// G *= 2^e, the scale the weights were divided by.
__global__ void moments_unscale_kernel(double* G, int64_t n, const unsigned long long* maxbits)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) G[i] = ldexp(G[i], weight_exponent(maxbits));
}

constexpr int kTile = 64;  // output tile (rows and columns) per wave

// Upper-triangle tile t (row-major over ti <= tj) -> (ti, tj).
__device__ __forceinline__ void upper_tile(int t, int nt, int* ti, int* tj)
{
    int r = 0, rem = t;
    while (rem >= nt - r) {
        rem -= nt - r;
        ++r;
    }
    *ti = r;
    *tj = r + rem;
}

// Records packed column by column: word (w, i) holds bit r = X[32 w + r][i]
// (zero past K), so the records a lane feeds to one MFMA step are bits of one
// word.  One thread per word and column, or four columns (VEC: one 32-bit load
// per record, rows 4-byte aligned: ldx % 4 == 0 and X aligned; npad % 4 == 0).
// The 32 loads of a whole word are issued together.  Bound: the records'
// bytes, read once.
template <bool VEC>
__device__ void pack_columns(const uint8_t* __restrict__ X, int64_t ldx, int64_t K, int32_t N, int32_t npad,
                             int64_t words, uint32_t* __restrict__ Xb, int64_t t)
{
    constexpr int V = VEC ? 4 : 1;
    const int32_t q = npad / V;
    const int64_t w = t / q;
    const int32_t i0 = (int32_t)(t % q) * V;
    if (w >= words) return;
    uint32_t out[V] = {};
    const int64_t k0 = w * 32;
    if (i0 < N && k0 < K) {
        const int rmax = K - k0 < 32 ? (int)(K - k0) : 32;
        const uint8_t* col = X + k0 * ldx + i0;
        auto put = [&](uint32_t bytes, int r) {
#pragma unroll
            for (int v = 0; v < V; ++v) out[v] |= (uint32_t)((bytes >> (8 * v) & 0xFFu) != 0) << r;
        };
        // columns at or past N (inside the row's pitch, or past it when
        // N = ldx) are masked below; a load never goes past the row
        if (VEC && i0 + 4 > ldx) {
            for (int r = 0; r < rmax; ++r) {
                uint32_t b = 0;
                for (int c = 0; c < 4 && i0 + c < ldx; ++c) b |= (uint32_t)col[r * ldx + c] << (8 * c);
                put(b, r);
            }
        } else if (rmax == 32) {
            uint32_t b[32];
#pragma unroll
            for (int r = 0; r < 32; ++r) {
                if constexpr (VEC) b[r] = *reinterpret_cast<const uint32_t*>(col + r * ldx);
                else b[r] = col[r * ldx];
            }
#pragma unroll
            for (int r = 0; r < 32; ++r) put(b[r], r);
        } else {
            for (int r = 0; r < rmax; ++r) {
                if constexpr (VEC) put(*reinterpret_cast<const uint32_t*>(col + r * ldx), r);
                else put(col[r * ldx], r);
            }
        }
#pragma unroll
        for (int v = 1; v < V; ++v)
            if (i0 + v >= N) out[v] = 0;
    }
    if constexpr (VEC) *reinterpret_cast<uint4*>(Xb + w * npad + i0) = make_uint4(out[0], out[1], out[2], out[3]);
    else Xb[w * npad + i0] = out[0];
}

// Workgroups below `prep` form the digits of integer weights, the others pack.
template <bool VEC>
__global__ __launch_bounds__(256) void pack_kernel(const uint8_t* __restrict__ X, int64_t ldx, int64_t K, int32_t N,
                                                   int32_t npad, int64_t words, uint32_t* __restrict__ Xb,
                                                   const int64_t* __restrict__ m, uint8_t* __restrict__ digits,
                                                   uint8_t* __restrict__ ndig, unsigned long long* __restrict__ psum,
                                                   int32_t prep)
{
    if ((int32_t)blockIdx.x < prep)
        weight_digits(m, K, words / 2, digits, ndig, psum, (int)blockIdx.x, prep);
    else
        pack_columns<VEC>(X, ldx, K, N, npad, words, Xb, (int64_t)(blockIdx.x - prep) * 256 + threadIdx.x);
}

// Integer weights.  A workgroup of four waves forms one 64 x 64 tile (ti, tj)
// of the upper triangle over a chunk of steps, each wave a quarter of them, as
// 4 x 4 MFMA tiles of 16 x 16 (v_mfma_i32_16x16x64_i8); MFMA tile a, row r is
// the tile's row 4 r + a, so that a lane's four columns are one 16-byte load.
// Operand lane (l % 16, kg = l / 16) holds 16 records of a column: register j the bits 4 (kg % 2) +
// j + 8 b, b < 4, of the column's word 2 step + kg / 2, as bytes (one shift
// and one mask per four records).  B = x; A = x times the weights' digit: a
// digit d < 128 under the mask 0x80 - x, which is 0x7F where x = 1 and keeps
// nothing of d where x = 0.  The int32 sums are exact (127 per record); the
// waves add theirs, times 128^digit, into the tile in LDS, five digits in 64-bit
// integers (below 2^31 2^28 (1 + 1 / 127) in each of four waves: exact, in any
// order), then, if a weight has more, the other four; the tile goes to
// part[chunk][tile] in FP64.
// Bound: VALU issue: a step of a wave is 130 VALU instructions (60 for A, 28
// for B) and 16 MFMAs, 580 issue cycles against 256 of the matrix cores, two
// waves to a SIMD.  N = 512, K = 131072, weights below 128: 31 us, and 42 with
// weights up to some hundreds (a second pass over the steps that have them);
// the bf16 product of the same weights took 150 us, with 277 VALU instructions
// per 32 records and a load's latency in every step.  The whole call 218 -> 59
// us; K = 32768, N = 20 (8 steps a workgroup instead of 16 a wave) 83 -> 30.
constexpr int kLowDigits = 5;
constexpr int kLd = kTile + 2;  // LDS row of the tile: rows 4 apart on other banks

__global__ __launch_bounds__(256, 2) void moments_i8_kernel(const uint32_t* __restrict__ Xb, int32_t npad, int64_t steps,
                                                         int32_t N, const uint8_t* __restrict__ digits,
                                                         const uint8_t* __restrict__ ndig, int64_t chunk_steps,
                                                         int32_t tiles, double* __restrict__ part)
{
    __shared__ unsigned long long tile[kTile * kLd];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = (int)(blockIdx.x % (unsigned)tiles);
    const int64_t c = blockIdx.x / (unsigned)tiles;
    int ti, tj;
    upper_tile(t, (N + kTile - 1) / kTile, &ti, &tj);
    const int i0 = ti * kTile, j0 = tj * kTile;
    const int64_t s0 = c * chunk_steps;
    const int64_t s1 = s0 + chunk_steps < steps ? s0 + chunk_steps : steps;
    const int64_t quarter = (s1 - s0 + 3) / 4;
    const int64_t w0 = s0 + wave * quarter < s1 ? s0 + wave * quarter : s1;
    const int64_t w1 = w0 + quarter < s1 ? w0 + quarter : s1;
    const int l16 = lane & 15, kg = lane >> 4;
    const int sh = 4 * (kg & 1);
    for (int e = threadIdx.x; e < kTile * kLd; e += 256) tile[e] = 0;
    // digits of this wave's largest weight
    int nd = 0;
    for (int64_t s = w0 + lane; s < w1; s += 64) nd = max(nd, (int)ndig[s]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) nd = max(nd, __shfl_xor(nd, d, 64));
    const bool more = __syncthreads_or(nd > kLowDigits) != 0;  // (of any wave)

    auto pass = [&](int p, int shift) {
        i32x4 acc[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = (i32x4){0, 0, 0, 0};
        // the steps of this pass, from s on
        auto next = [&](int64_t s) {
            if (p > 0)
                while (s < w1 && ndig[s] <= p) ++s;
            return s;
        };
        // three steps in flight: their words and digits come from L2 or beyond
        uint4 ba[3], bb[3], wt[3];
        int64_t at[3];
        auto load = [&](int u, int64_t from) {
            at[u] = next(from);
            const int64_t s = at[u] < w1 ? at[u] : w0;  // (past the end: any step, its digits masked)
            const uint32_t* row = Xb + (2 * s + (kg >> 1)) * npad + 4 * l16;
            ba[u] = *reinterpret_cast<const uint4*>(row + i0);
            bb[u] = *reinterpret_cast<const uint4*>(row + j0);
            wt[u] = *reinterpret_cast<const uint4*>(digits + ((int64_t)p * steps + s) * 64 + kg * 16);
        };
        auto step = [&](int u, int last) {
            constexpr uint32_t kOnes = 0x01010101u;
            const uint32_t wa[4] = {ba[u].x, ba[u].y, ba[u].z, ba[u].w}, wb[4] = {bb[u].x, bb[u].y, bb[u].z, bb[u].w};
            const uint32_t on = at[u] < w1 ? 0x7F7F7F7Fu : 0u;
            const uint32_t dg[4] = {wt[u].x & on, wt[u].y & on, wt[u].z & on, wt[u].w & on};
            i32x4 bop[4];
            uint32_t xa[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t x = wb[b] >> sh;
                bop[b] = (i32x4){(int)(x & kOnes), (int)((x >> 1) & kOnes), (int)((x >> 2) & kOnes),
                                 (int)((x >> 3) & kOnes)};
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) xa[a] = wa[a] >> sh;
            load(u, at[last] + 1);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                i32x4 aop;
#pragma unroll
                for (int j = 0; j < 4; ++j) aop[j] = (int)(dg[j] & (0x80808080u - ((xa[a] >> j) & kOnes)));
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop, bop[b], acc[a][b], 0, 0, 0);
            }
        };
        load(0, w0);
        load(1, at[0] + 1);
        load(2, at[1] + 1);
        while (at[0] < w1) {
            step(0, 2);
            step(1, 0);
            step(2, 1);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (p == 0 || acc[a][b][e] != 0)
                        atomicAdd(&tile[(a * 16 + kg * 4 + e) * kLd + b * 16 + l16],
                                  (unsigned long long)(uint32_t)acc[a][b][e] << shift);
    };
    double* dst = part + (c * tiles + t) * (int64_t)(kTile * kTile);
    auto place = [](int i) { return (i & 3) * 16 + (i >> 2); };  // row or column i in the order of the MFMA tiles
    auto sum = [&](int e) { return (double)tile[place(e / kTile) * kLd + place(e % kTile)]; };
#pragma unroll 1
    for (int p = 0; p < nd && p < kLowDigits; ++p) pass(p, 7 * p);
    __syncthreads();
    for (int e = threadIdx.x; e < kTile * kTile; e += 256) dst[e] = sum(e);
    if (!more) return;
    __syncthreads();
    for (int e = threadIdx.x; e < kTile * kLd; e += 256) tile[e] = 0;
    __syncthreads();
#pragma unroll 1
    for (int p = kLowDigits; p < nd; ++p) pass(p, 7 * (p - kLowDigits));
    __syncthreads();
    for (int e = threadIdx.x; e < kTile * kTile; e += 256) dst[e] += 34359738368.0 * sum(e);  // 128^5
}

// G[i][j] = f times the sum over chunks of the partial tiles (integer weights:
// FP64, exact below 2^53), f = 1 or, scaled, -beta over the sum of the weights.
// One thread per element of an upper-triangle tile; an off-diagonal tile's
// element also gives G[j][i].  Every workgroup adds up the weight sums it
// needs; the first writes the total to *sum.
__global__ __launch_bounds__(256) void moments_int_reduce_kernel(const double* __restrict__ part, int64_t chunks,
                                                                 int32_t tiles, int32_t N, double* __restrict__ G,
                                                                 const unsigned long long* __restrict__ psum,
                                                                 int32_t nsum, bool scaled, double beta,
                                                                 double* __restrict__ sum)
{
    __shared__ unsigned long long red[4];
    double f = 1.0;
    if (scaled || blockIdx.x == 0) {
        unsigned long long v = (int)threadIdx.x < nsum ? psum[threadIdx.x] : 0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        const double total = (double)(red[0] + red[1] + red[2] + red[3]);
        if (scaled) f = -beta / total;
        if (blockIdx.x == 0 && threadIdx.x == 0) *sum = total;
    }
    const int t = (int)(blockIdx.x / (kTile * kTile / 256));
    const int off = (int)(blockIdx.x % (kTile * kTile / 256)) * 256 + (int)threadIdx.x;
    int ti, tj;
    upper_tile(t, (N + kTile - 1) / kTile, &ti, &tj);
    const int i = ti * kTile + off / kTile, j = tj * kTile + off % kTile;
    if (i >= N || j >= N) return;
    const double* src = part + (int64_t)t * (kTile * kTile) + off;
    const int64_t stride = (int64_t)tiles * (kTile * kTile);
    double s = 0.0;
    int64_t c = 0;
    for (; c + 8 <= chunks; c += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(c + u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; c < chunks; ++c) s += src[c * stride];
    s *= f;
    G[(int64_t)i * N + j] = s;
    if (ti != tj) G[(int64_t)j * N + i] = s;
}

// 0xFFFF per set bit of a 2-bit field, in the matching half word.
__device__ __forceinline__ uint32_t half_mask(uint32_t two_bits)
{
    return ((two_bits & 1u) ? 0x0000FFFFu : 0u) | ((two_bits & 2u) ? 0xFFFF0000u : 0u);
}

// One wave computes one 64 x 64 tile (ti, tj) of G over the records
// [32 w0, 32 w1) as 4 x 4 MFMA tiles of 16 x 16 (v_mfma_f32_16x16x32_bf16).
// Lane l supplies row (A) or column (B) l % 16 of each 16-block and the eight
// records 8 (l / 16) .. + 7 of the 32-record step (the same assignment for A
// and B, so their order inside the step does not matter); lane l receives C
// rows 4 (l / 16) + e, column l % 16.  A = diag(piece_s(m)) x, B = x.
// FP32 accumulation; the accumulators go to this wave's slot of `part`.
__global__ __launch_bounds__(256) void moments_kernel(const uint32_t* __restrict__ Xb, int32_t npad, int64_t words,
                                                      int32_t N, const uint16_t* __restrict__ pieces, int64_t kpad,
                                                      int64_t chunk_words, int32_t tiles, float* __restrict__ part)
{
    const int lane = threadIdx.x & 63;
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t chunks = (words + chunk_words - 1) / chunk_words;
    if (gw >= (int64_t)tiles * chunks) return;
    const int t = (int)(gw % tiles);
    const int64_t c = gw / tiles;
    const int nt = (N + kTile - 1) / kTile;
    int ti, tj;
    upper_tile(t, nt, &ti, &tj);
    const int i0 = ti * kTile, j0 = tj * kTile;
    const int64_t w0 = c * chunk_words;
    const int64_t w1 = w0 + chunk_words < words ? w0 + chunk_words : words;
    const int l16 = lane & 15, lg = lane >> 4;

    f32x4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int sh = lg * 8;
    for (int64_t w = w0; w < w1; ++w) {
        const uint32_t* row = Xb + w * npad;
        uint32_t ba[4], bb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) ba[a] = (row[i0 + a * 16 + l16] >> sh) & 0xFFu;
#pragma unroll
        for (int b = 0; b < 4; ++b) bb[b] = (row[j0 + b * 16 + l16] >> sh) & 0xFFu;
        // weights of this lane's eight records, as four pairs per piece
        const int64_t kb = w * 32 + sh;
        uint4 wp[3];
        bool use[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            wp[s] = *reinterpret_cast<const uint4*>(pieces + s * kpad + kb);
            const uint32_t any = (wp[s].x | wp[s].y | wp[s].z | wp[s].w) & 0x7FFF7FFFu;
            use[s] = s == 0 || __ballot(any != 0) != 0;
        }
        bf16x8 bop[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint4 v;
            v.x = half_mask(bb[b]) & 0x3F803F80u;
            v.y = half_mask(bb[b] >> 2) & 0x3F803F80u;
            v.z = half_mask(bb[b] >> 4) & 0x3F803F80u;
            v.w = half_mask(bb[b] >> 6) & 0x3F803F80u;
            bop[b] = __builtin_bit_cast(bf16x8, v);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const uint32_t m0 = half_mask(ba[a]), m1 = half_mask(ba[a] >> 2), m2 = half_mask(ba[a] >> 4),
                           m3 = half_mask(ba[a] >> 6);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                if (!use[s]) continue;
                uint4 v;
                v.x = m0 & wp[s].x;
                v.y = m1 & wp[s].y;
                v.z = m2 & wp[s].z;
                v.w = m3 & wp[s].w;
                const bf16x8 aop = __builtin_bit_cast(bf16x8, v);
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bop[b], acc[a][b], 0, 0, 0);
            }
        }
    }
    // this wave's partial tile: part[c][t][64][64]
    float* dst = part + (c * tiles + t) * (int64_t)(kTile * kTile);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[(a * 16 + lg * 4 + e) * kTile + b * 16 + l16] = acc[a][b][e];
}

// G[i][j] += sum over chunks of the partial tiles (FP64, in chunk order).
// One thread per element of an upper-triangle tile (reads coalesced along the
// tile row); an off-diagonal tile's element also gives G[j][i].
__global__ void moments_reduce_kernel(const float* __restrict__ part, int64_t chunks, int32_t tiles, int32_t N,
                                      double* __restrict__ G)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)tiles * (kTile * kTile)) return;
    const int t = (int)(e / (kTile * kTile));
    const int off = (int)(e % (kTile * kTile));
    const int nt = (N + kTile - 1) / kTile;
    int ti, tj;
    upper_tile(t, nt, &ti, &tj);
    const int i = ti * kTile + off / kTile, j = tj * kTile + off % kTile;
    if (i >= N || j >= N) return;
    double s = 0.0;
    for (int64_t c = 0; c < chunks; ++c) s += (double)part[c * tiles * (int64_t)(kTile * kTile) + e];
    G[(int64_t)i * N + j] += s;
    if (ti != tj) G[(int64_t)j * N + i] += s;
}

// ---- log Z by enumeration ----

template <typename T>
struct Acc {
    using type = int64_t;
};
template <>
struct Acc<float> {
    using type = double;
};

// Lane l of a wave takes the assignment t = 64 u + l of the bits from 4 + MID
// up and enumerates the 2^(4 + MID) states below it: E is linear in the low bits
// but for their own pairs, so that a state is two additions, one product and
// one exponential.  Bits of u are the wave's: their terms are added for set bits
// only.  The (max, sum) of exp(-beta E - max) pairs are block-reduced.
// Bound: FP64 issue, about 30 operations per state (16 states per pass in
// registers).  A call at N = 20 took 280 us and at N = 30 300 ms (2^14 threads
// walking a Gray code with the fields in scratch memory), now 55 us and 1.2 ms;
// MID = 4 from 2^24 states on, where 2^16 lanes are left and the terms of u are
// shared by 16 times the states.
template <typename QT, int MID>
__global__ __launch_bounds__(256) void logz_kernel(const QT* __restrict__ Q, int32_t N, int32_t layout, double beta,
                                                   int64_t count, double* out_max, double* out_sum)
{
    using AT = typename Acc<QT>::type;
    constexpr int L = 4 + MID;  // bits below the lane's six
    __shared__ AT W[32][32];
    __shared__ AT dq[32];
    __shared__ double etab[64][2];
    __shared__ double smax[256], ssum[256];
    const int tid = threadIdx.x;
    int odd = 0;  // an entry is infinite or NaN
    for (int e = tid; e < 32 * 32; e += blockDim.x) {
        const int i = e / 32, j = e % 32;
        AT v = (AT)0;
        if (i < N && j < N) {
            if (i == j) v = (AT)0;
            else if (layout == 0) v = (AT)Q[i * N + j] + (AT)Q[j * N + i];
            else v = i < j ? (AT)Q[i * N + j] : (AT)Q[j * N + i];
        }
        W[i][j] = v;
        if (i == j) v = dq[i] = i < N ? (AT)Q[i * N + i] : (AT)0;
        if constexpr (std::is_floating_point<QT>::value) odd |= !isfinite(v);
    }
    for (int i = tid; i < 128; i += blockDim.x) etab[i >> 1][i & 1] = step::kExp2[i >> 1][i & 1];
    odd = __syncthreads_or(odd);
    const int lane = tid & 63;
    const int states = N < 4 ? 1 << N : 16;
    // the lane's six bits: their pairs, and their terms in the lower bits
    AT Elane = 0, fl[L];
#pragma unroll
    for (int j = 0; j < L; ++j) fl[j] = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        if (!((lane >> i) & 1)) continue;
#pragma unroll
        for (int k = 0; k < i; ++k)
            if ((lane >> k) & 1) Elane += W[L + i][L + k];
#pragma unroll
        for (int j = 0; j < L; ++j) fl[j] += W[L + i][j];
    }
    // pairs of the four lowest bits
    AT pair[16];
    pair[0] = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int st = 0; st < (1 << j); ++st) {
            AT p = pair[st];
#pragma unroll
            for (int k = 0; k < j; ++k)
                if ((st >> k) & 1) p += W[j][k];
            pair[st | (1 << j)] = p;
        }
    }
    double mx = -INFINITY, sm = 0.0;
    bool bad = false;  // a state's -beta E is NaN or infinite
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t u = (int64_t)blockIdx.x * (blockDim.x / 64) + __builtin_amdgcn_readfirstlane(tid >> 6); u * 64 < count; u += waves) {
        AT g[L + 6], E = Elane;
#pragma unroll
        for (int j = 0; j < L + 6; ++j) g[j] = dq[j];
        for (uint32_t m = (uint32_t)u; m; m &= m - 1) {
            const int i = L + 6 + __builtin_ctz(m);
            E += dq[i];
            for (uint32_t r = m & (m - 1); r; r &= r - 1) E += W[i][L + 6 + __builtin_ctz(r)];
#pragma unroll
            for (int j = 0; j < L + 6; ++j) g[j] += W[i][j];
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) E += (lane >> i) & 1 ? g[L + i] : (AT)0;
#pragma unroll
        for (int j = 0; j < L; ++j) g[j] += fl[j];
        if (u * 64 + lane >= count) continue;
#pragma unroll 1
        for (int c = 0; c < (1 << MID); ++c) {
            AT h[4], base = E;
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = g[j];
#pragma unroll
            for (int b = 0; b < MID; ++b) {
                if (!((c >> b) & 1)) continue;
                base += g[4 + b];
#pragma unroll
                for (int k = 0; k < b; ++k)
                    if ((c >> k) & 1) base += W[4 + b][4 + k];
#pragma unroll
                for (int j = 0; j < 4; ++j) h[j] += W[4 + b][j];
            }
            AT e[16];
            e[0] = base;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int st = 0; st < (1 << j); ++st) e[st | (1 << j)] = e[st] + h[j];
            double v[16], top = -INFINITY;
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                v[st] = st < states ? -beta * (double)(e[st] + pair[st]) : -INFINITY;
                top = fmax(top, v[st]);
            }
            // (the maximum passes over NaN, and the exponential takes it for 0)
            if (odd) {
#pragma unroll
                for (int st = 0; st < 16; ++st) bad = bad || (st < states && !(v[st] < INFINITY));
            }
            if (top > mx) {
                sm *= exp(mx - top);
                mx = top;
            }
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                const double w = step::exp_nonpos(v[st] - mx, etab);
                sm += st < states ? w : 0.0;
            }
        }
    }
    smax[tid] = bad ? INFINITY : mx;  // (infinity: the pair outlives the merges)
    ssum[tid] = bad ? NAN : sm;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) {
            const double m1 = smax[tid], m2 = smax[tid + st];
            const double s1 = ssum[tid], s2 = ssum[tid + st];
            const double m = fmax(m1, m2);
            smax[tid] = m;
            ssum[tid] = (m1 == -INFINITY ? 0.0 : s1 * exp(m1 - m)) + (m2 == -INFINITY ? 0.0 : s2 * exp(m2 - m));
        }
        __syncthreads();
    }
    if (tid == 0) {
        out_max[blockIdx.x] = smax[0];
        out_sum[blockIdx.x] = ssum[0];
    }
}

// Final log-sum-exp of the per-block pairs, one workgroup.
__global__ __launch_bounds__(256) void logz_finish_kernel(const double* pm, const double* ps, int32_t n, double* out)
{
    __shared__ double smax[256], ssum[256];
    const int tid = threadIdx.x;
    double mx = -INFINITY, sm = 0.0;
    for (int i = tid; i < n; i += 256) {
        const double m = fmax(mx, pm[i]);
        sm = (mx == -INFINITY ? 0.0 : sm * exp(mx - m)) + (pm[i] == -INFINITY ? 0.0 : ps[i] * exp(pm[i] - m));
        mx = m;
    }
    smax[tid] = mx;
    ssum[tid] = sm;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) {
            const double m1 = smax[tid], m2 = smax[tid + st];
            const double m = fmax(m1, m2);
            ssum[tid] = (m1 == -INFINITY ? 0.0 : ssum[tid] * exp(m1 - m)) +
                        (m2 == -INFINITY ? 0.0 : ssum[tid + st] * exp(m2 - m));
            smax[tid] = m;
        }
        __syncthreads();
    }
    if (tid == 0) out[0] = smax[0] + log(ssum[0]);
}

}  // namespace

hipError_t launch_moments_prep_f64(const double* w, int64_t K, int64_t kpad, uint16_t* pieces, double* sum_w,
                                   unsigned long long* maxbits, hipStream_t st)
{
    const int64_t n = kpad > K ? kpad : K;
    const int64_t blocks = std::min<int64_t>(256, std::max<int64_t>(1, (n + 255) / 256));
    if (K > 0) hipLaunchKernelGGL(moments_absmax_kernel, dim3((unsigned)blocks), dim3(256), 0, st, w, K, maxbits);
    hipLaunchKernelGGL(moments_prep_f64_kernel, dim3((unsigned)blocks), dim3(256), 0, st, w, K, kpad, pieces, sum_w,
                       maxbits);
    return hipGetLastError();
}

// G <- G * (-beta / sum): the weighted second moments to the gradient of
// log Z, the weight sum read on the device.
__global__ void moments_to_grad_kernel(double* G, int64_t n, double beta, const double* sum)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double f = -beta / *sum;
    G[i] = G[i] * f;
}

hipError_t launch_moments_to_grad(double* G, int64_t n, double beta, const double* sum, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(moments_to_grad_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, G, n, beta, sum);
    return hipGetLastError();
}

hipError_t launch_moments_unscale(double* G, int64_t n, const unsigned long long* maxbits, hipStream_t st)
{
    hipLaunchKernelGGL(moments_unscale_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, G, n, maxbits);
    return hipGetLastError();
}

namespace {

// Packing, with `prep` workgroups forming the digits of integer weights m.
hipError_t pack(const uint8_t* X, int64_t ldx, int64_t K, int32_t N, int32_t npad, int64_t words, uint32_t* Xb,
                const int64_t* m, uint8_t* digits, uint8_t* ndig, unsigned long long* psum, int32_t prep,
                hipStream_t st)
{
    const bool vec = ldx % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 3u) == 0 && npad % 4 == 0;
    const int64_t n = words * (vec ? npad / 4 : npad);
    const dim3 grid((unsigned)((n + 255) / 256 + prep));
    if (vec)
        hipLaunchKernelGGL(pack_kernel<true>, grid, dim3(256), 0, st, X, ldx, K, N, npad, words, Xb, m, digits, ndig, psum,
                           prep);
    else
        hipLaunchKernelGGL(pack_kernel<false>, grid, dim3(256), 0, st, X, ldx, K, N, npad, words, Xb, m, digits, ndig,
                           psum, prep);
    return hipGetLastError();
}

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

}  // namespace

hipError_t launch_pack_bits(const uint8_t* X, int64_t ldx, int64_t K, int32_t N, int32_t npad, int64_t words,
                            uint32_t* Xb, hipStream_t st)
{
    return pack(X, ldx, K, N, npad, words, Xb, nullptr, nullptr, nullptr, nullptr, 0, st);
}

hipError_t launch_moments(const uint32_t* Xb, int32_t npad, int64_t words, int32_t N, const uint16_t* pieces,
                          int64_t kpad, int64_t chunk_words, float* part, double* G, hipStream_t st)
{
    const int nt = (N + kTile - 1) / kTile;
    const int32_t tiles = nt * (nt + 1) / 2;
    const int64_t chunks = (words + chunk_words - 1) / chunk_words;
    const int64_t waves = (int64_t)tiles * chunks;
    hipLaunchKernelGGL(moments_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, Xb, npad, words, N, pieces,
                       kpad, chunk_words, tiles, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)tiles * kTile * kTile;
    hipLaunchKernelGGL(moments_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, chunks, tiles,
                       N, G);
    return hipGetLastError();
}

MomentsWorkspace moments_int_workspace(int64_t K, int32_t N, int64_t limit)
{
    MomentsWorkspace w;
    w.npad = (N + kTile - 1) / kTile * kTile;
    w.steps = std::max<int64_t>(1, (K + 63) / 64);
    const int64_t nt = w.npad / kTile;
    w.tiles = nt * (nt + 1) / 2;
    w.digits = align256(w.steps * 2 * w.npad * 4);
    w.ndig = w.digits + align256(w.steps * 64 * kDigits);
    w.psum = w.ndig + align256(w.steps);
    w.part = w.psum + 257 * 8 + 248;
    // At most 512 workgroups where the tiles allow it, two to a compute unit at
    // once (N = 512, K = 131072: 504), of at least 8 steps.
    const int64_t most_chunks = std::max<int64_t>(1, 512 / w.tiles);
    w.chunk_steps = std::max<int64_t>(8, (w.steps + most_chunks - 1) / most_chunks);
    // (a wave's int32 sums: 2^24 records of at most 127)
    w.chunk_steps = std::min<int64_t>(w.chunk_steps, 1 << 20);
    const int64_t tile_bytes = w.tiles * kTile * kTile * 8;
    if (limit > 0) {
        const int64_t most = std::max<int64_t>(1, (limit - w.part) / tile_bytes);
        w.chunk_steps = std::max(w.chunk_steps, (w.steps + most - 1) / most);
    }
    w.bytes = w.part + (w.steps + w.chunk_steps - 1) / w.chunk_steps * tile_bytes;
    return w;
}

hipError_t launch_moments_int(const uint8_t* X, int64_t ldx, const int64_t* m, int64_t K, int32_t N, double* G,
                              double* sum, bool scaled, double beta, const MomentsWorkspace& w, void* ws,
                              hipStream_t st)
{
    uint8_t* b = static_cast<uint8_t*>(ws);
    uint32_t* Xb = reinterpret_cast<uint32_t*>(b);
    uint8_t* digits = b + w.digits;
    uint8_t* ndig = b + w.ndig;
    unsigned long long* psum = reinterpret_cast<unsigned long long*>(b + w.psum);
    double* part = reinterpret_cast<double*>(b + w.part);
    const int64_t chunks = (w.steps + w.chunk_steps - 1) / w.chunk_steps;
    const int32_t prep = (int32_t)std::min<int64_t>(256, (w.steps + 3) / 4);
    hipError_t e = pack(X, ldx, K, N, w.npad, w.steps * 2, Xb, m, digits, ndig, psum, prep, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(moments_i8_kernel, dim3((unsigned)(w.tiles * chunks)), dim3(256), 0, st, Xb, w.npad, w.steps, N,
                       digits, ndig, w.chunk_steps, (int32_t)w.tiles, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(moments_int_reduce_kernel, dim3((unsigned)(w.tiles * (kTile * kTile / 256))), dim3(256), 0, st,
                       part, chunks, (int32_t)w.tiles, N, G, psum, prep, scaled, beta,
                       sum ? sum : reinterpret_cast<double*>(psum + 256));
    return hipGetLastError();
}

// Assignments of the bits above a lane's own, and blocks of 256 lanes for them.
int32_t logz_blocks(int32_t N, int64_t* count)
{
    const int32_t own = N >= 24 ? 8 : std::min(N, 4);
    *count = (int64_t)1 << (N - own);
    return (int32_t)std::min<int64_t>(4096, (*count + 255) / 256);
}

template <typename QT>
void logz_typed(const void* Q, int32_t N, int32_t layout, double beta, double* pm, double* ps, hipStream_t st)
{
    int64_t count = 0;
    const int32_t blocks = logz_blocks(N, &count);
    const QT* q = reinterpret_cast<const QT*>(Q);
    if (N >= 24) hipLaunchKernelGGL((logz_kernel<QT, 4>), dim3(blocks), dim3(256), 0, st, q, N, layout, beta, count, pm, ps);
    else hipLaunchKernelGGL((logz_kernel<QT, 0>), dim3(blocks), dim3(256), 0, st, q, N, layout, beta, count, pm, ps);
}

hipError_t launch_logz(int32_t qtype, const void* Q, int32_t N, int32_t layout, double beta, double* part_max,
                       double* part_sum, int32_t blocks, double* out, hipStream_t st)
{
    if (qtype == Q_I16) logz_typed<int16_t>(Q, N, layout, beta, part_max, part_sum, st);
    else if (qtype == Q_I32) logz_typed<int32_t>(Q, N, layout, beta, part_max, part_sum, st);
    else logz_typed<float>(Q, N, layout, beta, part_max, part_sum, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(logz_finish_kernel, dim3(1), dim3(256), 0, st, part_max, part_sum, blocks, out);
    return hipGetLastError();
}

}  // namespace pns

// ---- moments into a static workspace (pns_moments_noalloc) ----

#include <mutex>

#include "pns.h"

namespace {

// Workspace of pns_moments_noalloc on each GPU: the workspace of one call of
// the integer moments.  A device global holds no valid address on the host:
// host code uses the per-device address from hipGetSymbolAddress, never this
// name.  Calls of up to kCallBytes (packed records, 6 bytes of weights a
// record and 16 KiB per 64 x 64 tile) are taken; what they need at most, with
// 9 digit bytes a record and 32 KiB per tile, fits the array.
constexpr size_t kCallBytes = size_t(32) << 20;
constexpr size_t kScratchBytes = size_t(68) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// Address of `scratch` on the current device, looked up on the first call
// on that device.
int scratch_address(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return pns::set_error(PNS_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return pns::set_error(PNS_EDEVICE, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return pns::set_error(PNS_EDEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PNS_OK;
}

bool on_device(const void* p)
{
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type == hipMemoryTypeDevice;
}

}  // namespace

extern "C" int pns_moments_noalloc(const uint8_t* X, int64_t ldx, const int64_t* m, int64_t K, int32_t N, double* G,
                                   double* sum_m, void* stream)
{
    using namespace pns;
    if (!X || !m || !G) return set_error(PNS_EINVAL, "NULL argument");
    if (N < 1 || N > 32768) return set_error(PNS_EINVAL, "N must be in [1, 32768]");
    if (K < 0) return set_error(PNS_EINVAL, "K must be >= 0");
    if (ldx < N) return set_error(PNS_EINVAL, "ldx must be >= N");
    if (!on_device(X) || !on_device(m) || !on_device(G) || (sum_m && !on_device(sum_m)))
        return set_error(PNS_EINVAL, "X, m, G and sum_m must be device memory (nothing is staged here)");
    const int64_t kpad = std::max<int64_t>(64, (K + 63) / 64 * 64);
    const int32_t npad = (N + 63) / 64 * 64;
    const int64_t words = std::max<int64_t>(1, (K + 31) / 32);
    const int64_t nt = npad / 64;
    const int64_t tiles = nt * (nt + 1) / 2;
    const size_t fixed = align256((size_t)3 * kpad * 2) + 256 + align256((size_t)words * npad * 4);
    const size_t tile_bytes = (size_t)tiles * 64 * 64 * 4;
    if (fixed + tile_bytes > kCallBytes)
        return set_error(PNS_EINVAL,
                         "K = %lld records of N = %d count %zu bytes of workspace; calls of up to %zu are taken "
                         "(use pns_moments)",
                         (long long)K, N, fixed + tile_bytes, kCallBytes);
    const MomentsWorkspace w = moments_int_workspace(K, N, (int64_t)kScratchBytes);
    if (w.bytes > (int64_t)kScratchBytes)
        return set_error(PNS_EINVAL, "K = %lld records of N = %d exceed the static workspace (use pns_moments)",
                         (long long)K, N);
    void* base = nullptr;
    int rc = scratch_address(&base);
    if (rc) return rc;
    hipError_t e = launch_moments_int(X, ldx, m, K, N, G, sum_m, false, 0.0, w, base, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return set_error(PNS_EDEVICE, "moments kernels: %s", hipGetErrorString(e));
    return PNS_OK;
}

