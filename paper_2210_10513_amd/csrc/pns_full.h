// Step kernel of one to eight waves per chain for the runs that weigh every
// bit or a drawn subset: Rejection-Free (Alg 2), Basic PNS (Alg 3), Unbiased
// PNS with random sets (Sec 5) and the optimization runs (Alg 9, 10).
// Included by one translation unit per matrix element type after pns_step.h.
//
// The chain's bits lie as in the step kernel, f = (g * BLOCK + tid) * 4 + v:
// the bits of one wave in one group form a 256-bit segment, numbered in bit
// order, and sums, scans and the choice follow the step kernel's order, so the
// records of the two are equal bit for bit.  What differs:
//   * one wave holds up to 1024 bits (16 fields per lane), so a chain of up to
//     1024 bits has no barrier at all, and the scans, the choice and the record
//     are done once per chain instead of once per 256 bits;
//   * the chain's scalars (energy, budget, counters) are wave-uniform values
//     in scalar registers;
//   * integer problems keep u_j = Q_jj + s h_j, so that dE_j = (1 - 2 x_j) u_j;
//   * a drawn subset is formed from candidates two to a lane, by their ranks
//     among the first occurrences, without clearing the table of occurrences,
//     and (Basic PNS) during the row load of the step before.
// Bound: VALU issue (about 450 vector instructions per wave step of 16 int32
// fields a lane, 4 cycles each) and, with few chains to a SIMD, the latency of
// a step: its table reads, scans and the row of the flip.  us per step, the
// step kernel before and this one: Rejection-Free int16 N = 1024, 1024 chains
// 1.54 -> 1.44, 4096 chains 6.0 -> 3.4; Basic n = 64 3.26 -> 1.97; Basic N = 16,
// one chain 1.87 -> 1.05; Rejection-Free int32 N = 3001, 256 chains 2.95 ->
// 1.76; float N = 512, 8192 chains 9.3 -> 6.1.
#pragma once

#include "pns_step.h"

namespace pns {
namespace full {

using step::kTabHi;
using step::kTabLo;
using step::kTabMax;

// Keys of the table of occurrences: draw number (falling), then position.
constexpr int kPosBits = 20;
constexpr uint32_t kDraws = (1u << (32 - kPosBits)) - 1u;

__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double uniform_f64(double v)
{
    return __longlong_as_double(uniform64(__double_as_longlong(v)));
}
__device__ __forceinline__ bool uniform_bool(bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; }

// Between LDS accesses of different lanes of a chain: a barrier of its waves,
// or with one wave, whose accesses complete in order, a fence for the compiler.
template <int W>
__device__ __forceinline__ void exchange()
{
    if constexpr (W > 1) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Bits of lanes below this one set in m.
__device__ __forceinline__ int count_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Chains of one wave that share a workgroup.  The waves of a workgroup go to
// different SIMDs of a compute unit; workgroups of one wave may meet on one: the
// first launch of 1024 chains after a kernel of larger workgroups took 3.74 ms
// where the later ones took 2.84 (2000 steps, N = 1024 int16).  Up to one chain
// per compute unit there is nothing to share.
constexpr int kMaxShare = 4;
constexpr int share_of(int32_t chains) { return chains <= 256 ? 1 : chains <= 512 ? 2 : kMaxShare; }

constexpr int kTableBytes = 8 * (2 * kTabLo + kTabHi);
typedef const __attribute__((address_space(3))) double* LdsDouble;

// Waves per SIMD asked of the compiler: as many as leave the plain kernels
// without (or nearly without) spilled registers, one fewer for the kernels with
// a budget.  The tile of 512 x 8 has no fewer than two; its 32 64-bit fields a lane
// spill 48 to 242 registers, and it is still ahead of the step kernel's 1024 x 4
// (Rejection-Free floats, N = 10000, us per step: 64 chains 17.7 -> 11.7, 1024 chains
// 87.9 -> 78.4) but for drawn subsets of floats.
template <typename HT, int G, bool PLAIN>
constexpr int waves_per_eu()
{
    constexpr int plain = G == 1 ? 5 : (G == 2 ? 4 : (G <= 4 && sizeof(HT) == 4 ? 3 : 2));
    return PLAIN || plain == 2 ? plain : plain - 1;
}

typedef int16_t v2i16 __attribute__((ext_vector_type(2)));

// The kernel's arguments, read again where they are used: the instrumented
// kernels' many pointers would otherwise be kept in scalar registers across
// the step loop, or spilled to vector lanes and read back in every step.
typedef const __attribute__((address_space(4))) StepArgs* Args;
__device__ __forceinline__ Args args_here()
{
    Args p = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// PLAIN: Rejection-Free or Basic PNS sampling without a time limit, where no
// budget steers the chain; else Unbiased PNS, exact-time and optimization runs.
template <typename QT, typename HT, int W, int G, bool DRAWN, bool INSTR, bool PLAIN>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, W == 1 ? 64 * kMaxShare : 64 * W),
                          amdgpu_waves_per_eu(waves_per_eu<HT, G, PLAIN>())))
void full_kernel(const StepArgs a, const int32_t chains, const int32_t share, const int32_t stride)
{
    // A weight is the rounded product of its two table entries, summed as such.
#pragma clang fp contract(off)
    using step::read_lane;
    using step::small_scan;
    using step::wave_scan;
    constexpr bool kInt = !std::is_floating_point<HT>::value;
    constexpr int BLOCK = 64 * W;
    constexpr int F = 4 * G;
    constexpr int NSEG = G * W;
    // (the sum of all segments is the last lane's of the next power of two, as
    // in every other tile: its order of additions is that of the full tree)
    constexpr int NSEGP = NSEG <= 1 ? 1 : NSEG <= 2 ? 2 : NSEG <= 4 ? 4 : NSEG <= 8 ? 8 : NSEG <= 16 ? 16 : NSEG <= 32 ? 32 : 64;
    static_assert(NSEG <= 64 && F <= 32, "one segment scan, one word of bits per lane");
    using QW = typename step::Wide<QT>::T;

    // One wave: `share` chains to a workgroup, each with its tables in its part
    // (`stride` bytes) of the dynamic LDS; else static tables and one chain.
    __shared__ double tabs[kInt && W > 1 ? 2 * kTabLo + kTabHi : 1];
    __shared__ double etab[kInt ? 1 : 64][2];
    extern __shared__ double lds[];
    const int part_of = W > 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    char* const mine = reinterpret_cast<char*>(lds) + (W > 1 ? 0 : part_of * stride);
    double* const tab_hi = W > 1 ? tabs : reinterpret_cast<double*>(mine);
    double* const tab_lo = tab_hi + kTabHi;  // [kTabLo, 2 kTabLo): zeros, for bits outside the subset
    // exchanges between waves (W > 1), the totals in two buffers (even, odd steps)
    __shared__ double seg_sum[2][W > 1 ? NSEG : 1];
    __shared__ double mx_part[W];
    __shared__ int64_t xchg[2];
    // drawn subsets: the waves' counts of first occurrences (two buffers) and
    // the members' bits per lane; own [pitch] (dynamic) the first occurrences
    __shared__ int32_t cnt[2][W];
    __shared__ uint32_t members[DRAWN && W > 1 ? BLOCK : 1];
    uint32_t* const memw = W > 1 ? members : reinterpret_cast<uint32_t*>(mine + (kInt ? kTableBytes : 0));
    uint32_t* const own = W > 1 ? reinterpret_cast<uint32_t*>(lds) : memw + BLOCK;

    const int tid = W > 1 ? (int)threadIdx.x : (int)threadIdx.x & 63;
    const int lane = tid & 63;
    const int wave = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int index = W > 1 ? (int)blockIdx.x : (int)blockIdx.x * share + part_of;
    if (W == 1 && index >= chains) return;  // (no barrier follows)
    const int chain = a.chain_list ? a.chain_list[index] : a.chain_first + index;
    const Problem P = a.problems[a.chain_problem[chain]];
    const int32_t N = P.N;
    const int64_t pitch = P.pitch;
    const int32_t n = DRAWN ? P.n : N;
    const int s = P.s;
    const int mode = a.mode;
    const int64_t off = a.foff[chain];
    const double beta = uniform_f64(a.beta[chain] * a.inv_temp);  // inv_temp = 1 except in optimization runs
    const uint32_t cid = a.chain_id[chain];
    const uint64_t seed = a.seed;
    const bool unbiased = !PLAIN && DRAWN && mode == step::kModeRand;
    const bool opt = !PLAIN && mode == step::kModeOpt;
    const bool draw_each_step = DRAWN && !unbiased;
    // RF / Basic advancing by exactly a.orig_time original samples (the budget
    // rule of Alg 6 as a stopping time)
    const bool timed = !PLAIN && a.orig_time > 0;
    const bool budget = unbiased || timed;

    if constexpr (kInt) {
        for (int i = tid; i < 2 * kTabLo + kTabHi; i += BLOCK) {
            if (i < kTabLo) tab_lo[i] = exp(-beta * (double)i);
            else if (i < 2 * kTabLo) tab_lo[i] = 0.0;
            else tab_hi[i - 2 * kTabLo] = exp(-beta * (double)(kTabLo * (i - 2 * kTabLo)));
        }
    } else {
        for (int i = tid; i < 128; i += BLOCK) etab[i >> 1][i & 1] = step::kExp2[i >> 1][i & 1];
    }
    if constexpr (DRAWN) {
        for (int64_t i = tid; i < pitch; i += BLOCK) own[i] = 0xFFFFFFFFu;
        memw[tid] = 0u;
    }

    // ---- chain state: fields (integers: u = diag + s h) and bits ----
    HT h[F];
    QW dg[kInt ? 1 : F];
    uint32_t xw = 0, valid = 0;
    HT* hbase = reinterpret_cast<HT*>(a.h) + off;
    const QW* dbase = reinterpret_cast<const QW*>(P.diag);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int64_t fb = ((int64_t)g * BLOCK + tid) * 4;
        const bool in = fb < pitch;
        const step::Four<HT> hv = in ? step::load4(hbase + fb) : step::Four<HT>{};
        const step::Four<QW> dv = in ? step::load4(dbase + fb) : step::Four<QW>{};
        const uint32_t xb = in ? *reinterpret_cast<const uint32_t*>(a.x + off + fb) : 0u;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = g * 4 + v;
            if constexpr (kInt) h[i] = (HT)dv.v[v] + (HT)s * hv.v[v];
            else h[i] = hv.v[v], dg[i] = dv.v[v];
            xw |= ((xb >> (8 * v)) & 1u) << i;
            valid |= (uint32_t)(fb + v < N) << i;
        }
    }

    // ---- chain scalars (wave-uniform) ----
    int64_t k = uniform64(a.step[chain]);
    const int64_t kend = k + a.steps;
    int64_t E = uniform64(a.E[chain]);
    int64_t L = timed ? a.orig_time : uniform64(a.L[chain]);
    int64_t sub = uniform64(a.sub[chain]);
    int32_t last_a = __builtin_amdgcn_readfirstlane(a.last_action[chain]);
    int64_t last_M = uniform64(a.last_M[chain]);
    int64_t last_E = uniform64(a.last_E[chain]);
    int64_t Ebest = 0;
    const bool best = INSTR && !PLAIN && a.xbest != nullptr;
    if (best) Ebest = uniform64(a.Ebest[chain]);
    int64_t c_steps = 0, c_flips = 0, c_stays = 0, c_sat = 0, c_bad = 0;
    int64_t c_sumM = 0;  // the bits of a double
    int32_t snap_n = 0, snap_in = 0;  // snapshots so far; steps to the next one
    if constexpr (INSTR) snap_in = a.snap_every > 0 ? (int32_t)(a.snap_every - k % a.snap_every) : 0;
    if constexpr (INSTR) snap_n = a.snap_every > 0 ? __builtin_amdgcn_readfirstlane(a.snap_count[chain]) : 0;
    const bool n_pow2 = (n & (n - 1)) == 0;
    const double inv_n = 1.0 / (double)n;

    // ---- the subset: this lane's members ----
    uint32_t mem = valid;
    const bool part = N != 4 * BLOCK * G;  // some of the tile's bits do not exist
    const bool masked = DRAWN || part;
    // integer problems: where the zero slots are (bytes), kept with the subset
    const uint32_t tab_at = (uint32_t)(uintptr_t)(LdsDouble)tab_hi;
    const uint32_t zo_at = W > 1 ? 0u : tab_at + (uint32_t)(8 * kTabHi);
    uint32_t zo[kInt ? F : 1];
    auto set_zo = [&]() {
        if constexpr (kInt) {
#pragma unroll
            for (int i = 0; i < F; ++i) zo[i] = (~(mem >> i) & 1u) * (uint32_t)(8 * kTabLo) + zo_at;
        }
    };
    uint32_t tag = kDraws;  // number of the next draw (falling)
    // The first n distinct values of the candidate stream of step kd: candidate
    // s from Philox stream 2^30 | s / 2, its words 0, 1 (even s) or 2, 3, mapped
    // to floor(u64 N / 2^64).  own[f] keeps the smallest key that f met, keys
    // falling from draw to draw; a candidate that finds its own key there is a
    // first occurrence, a member if fewer than n came before it.
    auto draw = [&](int64_t kd) {
        if constexpr (DRAWN) {
            if (tag == 0) {  // keys used up: clear the table
                exchange<W>();
                for (int64_t i = tid; i < pitch; i += BLOCK) own[i] = 0xFFFFFFFFu;
                exchange<W>();
                tag = kDraws;
            }
            const uint32_t key = (tag - 1u) << kPosBits;
            --tag;
            uint32_t c0 = cid, k0 = (uint32_t)kd, k1 = (uint32_t)((uint64_t)kd >> 32);
            int32_t have = 0;
            for (uint32_t round = 0; round < (1u << kPosBits) / (2u * BLOCK); ++round) {
                const uint32_t blk = round * BLOCK + (uint32_t)tid;
                const step::Words o = step::philox(c0, k0, k1, step::kStreamSubset | blk, seed);
                const uint32_t f0 = (uint32_t)__umul64hi(((uint64_t)o.w0 << 32) | o.w1, (uint64_t)(uint32_t)N);
                const uint32_t f1 = (uint32_t)__umul64hi(((uint64_t)o.w2 << 32) | o.w3, (uint64_t)(uint32_t)N);
                const uint32_t key0 = key | (2u * blk), key1 = key | (2u * blk + 1u);
                atomicMin(&own[f0], key0);
                atomicMin(&own[f1], key1);
                exchange<W>();
                const bool first0 = own[f0] == key0, first1 = own[f1] == key1;
                const uint64_t b0 = __ballot(first0), b1 = __ballot(first1);
                int32_t before = have, all = __builtin_popcountll(b0) + __builtin_popcountll(b1);
                if constexpr (W > 1) {
                    if (lane == 0) cnt[round & 1][wave] = all;
                    __syncthreads();
                    all = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const int32_t c = cnt[round & 1][w];
                        before += w < wave ? c : 0;
                        all += c;
                    }
                    all = __builtin_amdgcn_readfirstlane(all);
                }
                const int32_t r0 = before + count_below(b0) + count_below(b1);
                const int32_t r1 = r0 + (first0 ? 1 : 0);
                // lane word (f / 4) % BLOCK, bit 4 (f / (4 BLOCK)) + f % 4
                if (first0 && r0 < n) atomicOr(&memw[(f0 >> 2) & (BLOCK - 1)], 1u << ((f0 / (4 * BLOCK)) * 4 + (f0 & 3u)));
                if (first1 && r1 < n) atomicOr(&memw[(f1 >> 2) & (BLOCK - 1)], 1u << ((f1 / (4 * BLOCK)) * 4 + (f1 & 3u)));
                have += all;
                if (have >= n) break;
            }
            exchange<W>();
            mem = memw[tid];
            memw[tid] = 0u;  // (the next draw's members follow its exchange of occurrences)
        }
    };
    exchange<W>();  // tables ready
    if constexpr (DRAWN) {
        if (!unbiased || k == 0) {
            draw(k);
        } else {
            mem = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int64_t fb = ((int64_t)g * BLOCK + tid) * 4;
                const uint32_t mw = fb < pitch ? *reinterpret_cast<const uint32_t*>(a.rmem + off + fb) : 0u;
#pragma unroll
                for (int v = 0; v < 4; ++v) mem |= ((mw >> (8 * v)) & 1u) << (g * 4 + v);
            }
        }
    }
    set_zo();

    // ---- step uniforms, 64 steps at a time (lane j: step ub_base + j) ----
    int64_t ub_base = k;
    double ubLog = 0.0, ubU2 = 0.0;
    step::batch_uniforms(cid, ub_base, seed, lane, true, &ubLog, &ubU2);

    // Without a budget the multiplicity steers nothing: M of up to 64 steps
    // together, lane j for step ub_base + j, whose escape probability pbuf holds
    // (the instrumented kernels form a step's M also by itself where an output
    // of the step needs it).
    const bool lazy_m = !budget && !opt;
    const bool outputs_every = INSTR && (a.log_cap > 0 || a.hist_w != nullptr);
    const int32_t snap_every = INSTR ? a.snap_every : 0;
    double pbuf = 0.0;
    auto flush_m = [&](int c) {
        const double pj = pbuf;
        double qj;
        if (pj >= 1.0) qj = 0.0;
        else if (pj <= 0.0) qj = INFINITY;
        else qj = ubLog / log1p(-pj);
        const bool act = lane < c;
        const bool satj = act && !(qj < 0x1p63);
        const int64_t mj = satj ? INT64_MAX : (act ? (int64_t)floor(qj) + 1 : 0);
        double tot = act ? (double)mj : 0.0;
        if constexpr (INSTR) {  // (summed in the order of the steps, as the step kernel's instrumented form)
            double sum = __longlong_as_double(c_sumM);
            for (int j = 0; j < c; ++j) sum += read_lane(tot, j);
            c_sumM = uniform64(__double_as_longlong(sum));
        } else {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) tot += __shfl_xor(tot, d, 64);
            c_sumM = uniform64(__double_as_longlong(__longlong_as_double(c_sumM) + tot));
        }
        c_sat += __builtin_popcountll(__ballot(satj));
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mj, c - 1);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(mj >> 32), c - 1);
        last_M = (int64_t)(((uint64_t)hi << 32) | lo);
    };

    double w[F], inc[G], ls[G];

    // energy difference of the lane's bit i
    auto delta = [&](int i) -> HT {
        if constexpr (kInt) {
            const HT m = (HT)(int32_t)__builtin_amdgcn_sbfe(xw, i, 1);  // 0 or -1 (the builtin is unsigned)
            return (h[i] ^ m) - m;
        } else {
            const double e = fma((double)s, h[i], (double)dg[i]);
            return (xw >> i) & 1u ? -e : e;
        }
    };
    // weights of the members (integers: from the tables, past them by the
    // exponential), summed four bits at a time and scanned, every group at
    // once (straight-line: the groups' table reads and scans overlap)
    auto weigh = [&]() {
        if constexpr (kInt) {
            HT e[F], emax = 0;
            double th[F], tl[F];
#pragma unroll
            for (int i = 0; i < F; ++i) {
                e[i] = delta(i);
                emax = emax > e[i] ? emax : e[i];
                const HT e0 = e[i] > 0 ? e[i] : 0;
                const uint32_t ep = (uint32_t)(e0 < (HT)(kTabMax - 1) ? e0 : (HT)(kTabMax - 1));
                // tab_hi[ep >> 6] and tab_lo[ep & 63], or a zero slot, two instructions
                // each: a byte offset from a constant place, or (one wave) a field of
                // ep, which the asm keeps apart, shifted and added to the table's
                if constexpr (W > 1) {
                    const char* ph = reinterpret_cast<const char*>(tab_hi) + ((ep >> 3) & (uint32_t)(8 * (kTabHi - 1)));
                    const char* pl = reinterpret_cast<const char*>(tab_lo) + (((ep << 3) & (uint32_t)(8 * (kTabLo - 1))) | zo[i]);
                    th[i] = *reinterpret_cast<const double*>(ph);
                    tl[i] = *reinterpret_cast<const double*>(pl);
                } else {
                    uint32_t hi = ep >> 6, lo = ep & (uint32_t)(kTabLo - 1);
                    asm("" : "+v"(hi), "+v"(lo));
                    th[i] = *reinterpret_cast<LdsDouble>((uintptr_t)((hi << 3) + tab_at));
                    tl[i] = *reinterpret_cast<LdsDouble>((uintptr_t)((lo << 3) + zo[i]));
                }
            }
#pragma unroll
            for (int i = 0; i < F; ++i) w[i] = th[i] * tl[i];
            if (__ballot(emax >= (HT)kTabMax)) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
#pragma unroll 1
                    for (int v = 0; v < 4; ++v) {
                        const HT ev = v == 0 ? delta(g * 4) : (v == 1 ? delta(g * 4 + 1) : (v == 2 ? delta(g * 4 + 2) : delta(g * 4 + 3)));
                        if (((mem >> (g * 4 + v)) & 1u) && ev >= (HT)kTabMax) {
                            const double x = exp(-beta * (double)ev);
                            if (v == 0) w[g * 4] = x;
                            else if (v == 1) w[g * 4 + 1] = x;
                            else if (v == 2) w[g * 4 + 2] = x;
                            else w[g * 4 + 3] = x;
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < F; ++i) {
                double l = -beta * delta(i);
                l = l < 0.0 ? l : 0.0;
                w[i] = step::exp_nonpos(l, etab);
            }
            if (masked) {
#pragma unroll
                for (int i = 0; i < F; ++i) w[i] = (mem >> i) & 1u ? w[i] : 0.0;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) ls[g] = ((w[g * 4] + w[g * 4 + 1]) + w[g * 4 + 2]) + w[g * 4 + 3];
#pragma unroll
        for (int g = 0; g < G; ++g) inc[g] = ls[g];
#define PNS_SCAN_STEP(CTRL, MASK) \
        _Pragma("unroll") for (int g = 0; g < G; ++g) inc[g] += step::dpp_f64<CTRL, MASK>(inc[g]);
        // (wave_scan of every group, step by step)
        PNS_SCAN_STEP(0x111, 0xF)
        PNS_SCAN_STEP(0x112, 0xF)
        PNS_SCAN_STEP(0x114, 0xF)
        PNS_SCAN_STEP(0x118, 0xF)
        PNS_SCAN_STEP(0x142, 0xA)
        PNS_SCAN_STEP(0x143, 0xC)
#undef PNS_SCAN_STEP
    };

    // segment totals in bit order: lane j (W > 1) or P[j] (one wave), and S
    double sv = 0.0, sinc = 0.0, S = 0.0;
    double tot[W == 1 ? G : 1], pre[W == 1 ? G : 1];
    auto totals = [&]() {
        if constexpr (W == 1) {
#pragma unroll
            for (int g = 0; g < G; ++g) tot[g] = read_lane(inc[g], 63);
            // the order of small_scan over up to four lanes
            pre[0] = tot[0];
            if constexpr (G > 1) pre[1] = tot[1] + tot[0];
            if constexpr (G > 2) pre[2] = (tot[2] + tot[1]) + tot[0];
            if constexpr (G > 3) pre[3] = (tot[3] + tot[2]) + (tot[1] + tot[0]);
            S = G == 3 ? tot[2] + (tot[1] + tot[0]) : pre[G - 1];  // (three: as four, the last one zero)
        } else {
            if (lane == 63) {
#pragma unroll
                for (int g = 0; g < G; ++g) seg_sum[k & 1][g * W + wave] = inc[g];
            }
            __syncthreads();
            sv = lane < NSEG ? seg_sum[k & 1][lane] : 0.0;
            sinc = small_scan<NSEGP>(sv);
            S = read_lane(sinc, NSEGP - 1);
        }
    };
    static_assert(W > 1 || G <= 4, "one wave: the prefix order of up to four segments");

    for (; k < kend; ++k) {
        if (k - ub_base >= 64) {
            if (lazy_m && wave == 0) flush_m(64);
            ub_base = k;
            uint32_t key_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)seed);
            uint32_t key_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(seed >> 32));
            asm volatile("" : "+s"(key_lo), "+s"(key_hi));  // (the round keys are formed here, not kept)
            step::batch_uniforms(cid, ub_base, ((uint64_t)key_hi << 32) | key_lo, lane, true, &ubLog, &ubU2);
        }
        const int uj = (int)(k - ub_base);
        const double U2 = read_lane(ubU2, uj);

        // ---- weights, four-bit sums, segment scans, S ----
        weigh();
        totals();
        double mx = 0.0;
        bool scaled = false;
        if (uniform_bool(S < 0x1p-1000)) {
            // every weight underflowed: rescale by the largest log-weight
            double lm = -INFINITY;
#pragma unroll
            for (int i = 0; i < F; ++i) {
                double l = -beta * (double)delta(i);
                l = l < 0.0 ? l : 0.0;
                if ((mem >> i) & 1u) lm = fmax(lm, l);
            }
            lm = step::wave_max(lm);
            if constexpr (W > 1) {
                if (lane == 0) mx_part[wave] = lm;
                __syncthreads();
                lm = -INFINITY;
                for (int ww = 0; ww < W; ++ww) lm = fmax(lm, mx_part[ww]);
            }
            mx = lm;
            scaled = true;
#pragma unroll
            for (int g = 0; g < G; ++g) {
#pragma unroll 1
                for (int v = 0; v < 4; ++v) {
                    const double e4[4] = {(double)delta(g * 4), (double)delta(g * 4 + 1), (double)delta(g * 4 + 2),
                                          (double)delta(g * 4 + 3)};
                    double l = -beta * (v == 0 ? e4[0] : (v == 1 ? e4[1] : (v == 2 ? e4[2] : e4[3])));
                    l = l < 0.0 ? l : 0.0;
                    double x;
                    if constexpr (kInt) x = exp(l - mx);
                    else x = step::exp_nonpos(l - mx, etab);
                    x = (mem >> (g * 4 + v)) & 1u ? x : 0.0;
                    if (v == 0) w[g * 4] = x;
                    else if (v == 1) w[g * 4 + 1] = x;
                    else if (v == 2) w[g * 4 + 2] = x;
                    else w[g * 4 + 3] = x;
                }
                ls[g] = ((w[g * 4] + w[g * 4 + 1]) + w[g * 4 + 2]) + w[g * 4 + 3];
                inc[g] = wave_scan(ls[g]);
            }
            if constexpr (W > 1) __syncthreads();  // every wave has read this step's totals
            totals();
        }

        // ---- p, and M with the budget decision of Alg 6 where it steers ----
        auto escape = [&]() {
            const double Ss = scaled ? exp(mx) * S : S;
            return n_pow2 ? Ss * inv_n : Ss / (double)n;
        };
        bool snap = false;
        if constexpr (INSTR) snap = snap_every > 0 && --snap_in == 0;
        const bool need_m = budget || (INSTR && !opt && (snap || outputs_every));
        double q = 0.0, pu = 0.0;
        bool sat = false;
        int64_t m = 1;
        if (need_m || (INSTR && outputs_every)) pu = uniform_f64(escape());
        if (need_m) {
            if (pu >= 1.0) q = 0.0;
            else if (pu <= 0.0) q = INFINITY;
            else q = step::geometric_quotient(read_lane(ubLog, uj), pu, budget ? (double)L : -1.0);
            sat = uniform_bool(!(q < 0x1p63));
        }
        const bool stay = budget && uniform_bool(q >= (double)L);
        if (need_m) m = uniform64(sat ? INT64_MAX : (int64_t)floor(q) + 1);
        const int64_t Erec = E, Lrec = L;

        uint32_t rec_idx = 0;
        if constexpr (INSTR) {
            // state index of the record (histograms: N <= 24, lanes 0 .. 5)
            if (outputs_every && args_here()->hist_w != nullptr && wave == 0) rec_idx = step::wave_or(tid < 8 ? (xw & 0xFu) << (4 * tid) : 0u);
            if (snap) {
                const Args r = args_here();
                snap_in = snap_every;
                uint8_t* sx = r->snap_x + ((int64_t)chain * r->snap_cap + snap_n % r->snap_cap) * r->snap_pitch;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int64_t fb = ((int64_t)g * BLOCK + tid) * 4;
                    if (fb < r->snap_pitch) {
                        uint32_t wv = 0;
#pragma unroll
                        for (int v = 0; v < 4; ++v) wv |= ((xw >> (g * 4 + v)) & 1u) << (8 * v);
                        *reinterpret_cast<uint32_t*>(sx + fb) = wv;
                    }
                }
                ++snap_n;
            }
        }

        int32_t action = -1;
        int64_t M = m;
        bool next_set = draw_each_step;
        // the row of a move, added to the fields after the two paths join
        // (defined on both, so that the fields are not copied)
        bool add = false;
        decltype(step::load_raw4(static_cast<const QT*>(nullptr))) raw[G];
        if (stay) {
            // not enough remaining original samples: stay L times and draw the
            // next set (a timed run just ends)
            M = L;
            L = timed ? 0 : uniform64(P.L0);
            ++c_stays;
            sat = false;
            if (!timed) {
                ++sub;
                next_set = true;
            }
#pragma unroll
            for (int i = 0; i < F; ++i) asm volatile("" : "+v"(h[i]));
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if constexpr (sizeof(QT) == 2) asm volatile("" : "=v"(raw[g].x), "=v"(raw[g].y));
                else asm volatile("" : "=v"(raw[g].x), "=v"(raw[g].y), "=v"(raw[g].z), "=v"(raw[g].w));
            }
        } else {
            // ---- proportional choice: first bit whose running sum exceeds
            // U2 S, segment -> lane -> bit ----
            const double t = U2 * S;
            int jstar;
            if constexpr (W == 1) {
                int hit = -1, pos = -1;
#pragma unroll
                for (int g = G - 1; g >= 0; --g) {
                    hit = tot[g] > 0.0 && pre[g] > t ? g : hit;
                    pos = pos < 0 && tot[g] > 0.0 ? g : pos;
                }
                jstar = __builtin_amdgcn_readfirstlane(hit >= 0 ? hit : (pos > 0 ? pos : 0));
            } else {
                const bool pos_seg = lane < NSEG && sv > 0.0;
                const uint64_t bseg = __ballot(pos_seg && sinc > t);
                const uint64_t bpos = __ballot(pos_seg);
                jstar = bseg ? __builtin_ctzll(bseg) : (bpos ? 63 - __builtin_clzll(bpos) : 0);
                jstar = jstar < NSEG ? jstar : NSEG - 1;
            }
            const int gstar = (int)((unsigned)jstar / W), wstar = (int)((unsigned)jstar % W);
            int64_t selc = 0, seld = 0;
            if (W == 1 || wave == wstar) {
                double base = 0.0, my_inc = 0.0, my_ls = 0.0, w4[4] = {0.0, 0.0, 0.0, 0.0};
                HT e4[4] = {};
                if constexpr (W > 1) base = jstar > 0 ? read_lane(sinc, jstar - 1) : 0.0;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (g == gstar) {
                        if constexpr (W == 1) base = g > 0 ? pre[g > 0 ? g - 1 : 0] : 0.0;
                        my_inc = inc[g];
                        my_ls = ls[g];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            w4[v] = w[g * 4 + v];
                            e4[v] = delta(g * 4 + v);
                        }
                    }
                }
                const uint64_t bl = __ballot(my_ls > 0.0 && base + my_inc > t);
                const uint64_t blp = __ballot(my_ls > 0.0);
                const int lstar = bl ? __builtin_ctzll(bl) : (blp ? 63 - __builtin_clzll(blp) : 0);
                double run = lstar > 0 ? base + read_lane(my_inc, lstar - 1) : base;
                int vstar = -1, vlast = -1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool on = w4[v] > 0.0;
                    vlast = on ? v : vlast;
                    run = on ? run + w4[v] : run;
                    vstar = on && vstar < 0 && run > t ? v : vstar;
                }
                if (vstar < 0) vstar = vlast;
                // no positive weight in the chosen lane cannot happen when S > 0;
                // keep the address in range and report it
                vstar = __builtin_amdgcn_readlane(vstar, lstar);
                int64_t bad = 0;
                if (vstar < 0) {
                    vstar = 0;
                    bad = 1;
                }
                const HT ec = vstar == 0 ? e4[0] : (vstar == 1 ? e4[1] : (vstar == 2 ? e4[2] : e4[3]));
                int32_t c = (gstar * BLOCK + wave * 64 + lstar) * 4 + vstar;
                if (c >= N) {
                    c = 0;
                    bad = 1;
                }
                const uint32_t xl = (uint32_t)__builtin_amdgcn_readlane((int)xw, lstar);
                selc = (int64_t)c | ((int64_t)((xl >> (gstar * 4 + vstar)) & 1u) << 40) | (bad << 41);
                if constexpr (kInt && sizeof(HT) == 4) {
                    seld = __builtin_amdgcn_readlane((int)ec, lstar);
                } else {
                    int64_t eb;
                    if constexpr (kInt) eb = ec;
                    else eb = __double_as_longlong(ec);
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)eb, lstar);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)eb >> 32), lstar);
                    seld = (int64_t)(((uint64_t)hi << 32) | lo);
                }
                if constexpr (W > 1) {
                    if (lane == 0) {
                        xchg[0] = selc;
                        xchg[1] = seld;
                    }
                }
            }
            if constexpr (W > 1) {
                // (the next write of xchg follows the next step's segment
                // barrier, which every wave passes after these reads)
                __syncthreads();
                selc = uniform64(xchg[0]);
                seld = uniform64(xchg[1]);
            }
            const int32_t c = (int32_t)(selc & 0xFFFFFFFFll);
            const bool xc = (selc >> 40) & 1;
            c_bad += (selc >> 41) & 1;
            // ---- move: the row of c, loaded while the next subset is drawn
            // (Basic PNS); lanes past the pitch read the row's start and drop it ----
            const QT* row = reinterpret_cast<const QT*>(P.A) + (int64_t)(uint32_t)c * pitch;
            if (!part) {
#pragma unroll
                for (int g = 0; g < G; ++g) raw[g] = step::load_raw4(row + (g * BLOCK + tid) * 4);
            } else {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int32_t fb = (g * BLOCK + tid) * 4;
                    raw[g] = step::load_raw4(row + (fb < (int32_t)pitch ? fb : 0));
                }
            }
            const int ci = (int)(((uint32_t)c >> 2) / BLOCK) * 4 + (c & 3);
            if (tid == ((c >> 2) & (BLOCK - 1))) xw ^= 1u << ci;
            if constexpr (kInt) E = uniform64(E + seld);
            else E = uniform64(__double_as_longlong(__longlong_as_double(E) + __longlong_as_double(seld)));
            if (budget) L -= m;
            action = c;
            ++c_flips;
            if constexpr (INSTR) {
                if (best) {
                    const bool better = kInt ? E < Ebest : __longlong_as_double(E) < __longlong_as_double(Ebest);
                    if (better) {
                        Ebest = E;
                        uint8_t* xbest = args_here()->xbest;
#pragma unroll
                        for (int g = 0; g < G; ++g) {
                            const int64_t fb = ((int64_t)g * BLOCK + tid) * 4;
                            if (fb < pitch) {
                                uint32_t wv = 0;
#pragma unroll
                                for (int v = 0; v < 4; ++v) wv |= ((xw >> (g * 4 + v)) & 1u) << (8 * v);
                                *reinterpret_cast<uint32_t*>(xbest + off + fb) = wv;
                            }
                        }
                    }
                }
            }
            add = !xc;
        }
        if (lazy_m && wave == 0) {
            const double p = escape();
            pbuf = lane == uj ? p : pbuf;
        }
        if constexpr (DRAWN) {
            if (next_set) {
                draw(k + 1);
                set_zo();
            }
        }
        if (!stay) {
            // (fields of bits that do not exist: rows read there are not theirs,
            // but their weights are masked and they are not written back)
            if (part) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if ((g * BLOCK + tid) * 4 >= (int32_t)pitch) raw[g] = {};
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if constexpr (kInt && sizeof(QT) == 2) {
                    // coefficients times +-1 or +-2: two-term 16-bit dot products,
                    // the pair of coefficients against (mult, 0) or (0, mult)
                    const int16_t mult = (int16_t)(add ? s : -s);
                    const v2i16 mlo = {mult, 0}, mhi = {0, mult};
                    const v2i16 p0 = __builtin_bit_cast(v2i16, raw[g].x), p1 = __builtin_bit_cast(v2i16, raw[g].y);
                    h[g * 4 + 0] = __builtin_amdgcn_sdot2(p0, mlo, h[g * 4 + 0], false);
                    h[g * 4 + 1] = __builtin_amdgcn_sdot2(p0, mhi, h[g * 4 + 1], false);
                    h[g * 4 + 2] = __builtin_amdgcn_sdot2(p1, mlo, h[g * 4 + 2], false);
                    h[g * 4 + 3] = __builtin_amdgcn_sdot2(p1, mhi, h[g * 4 + 3], false);
                } else {
                    const auto r = step::widen4(raw[g]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        HT d = (HT)r.v[v];
                        if constexpr (kInt) {
                            d = s == 2 ? (HT)(d + d) : d;
                            h[g * 4 + v] += add ? d : -d;
                        } else {
                            h[g * 4 + v] += add ? d : -d;  // (a sum's rounding does not depend on the sign)
                        }
                    }
                }
            }
        }

        // ---- record k: the state before the step and M ----
        ++c_steps;
        last_a = action;
        last_E = Erec;
        if (!lazy_m) {
            c_sat += sat ? 1 : 0;
            c_sumM = uniform64(__double_as_longlong(__longlong_as_double(c_sumM) + (double)M));
            last_M = M;
        }
        if constexpr (INSTR) {
            double wrb = 1.0;
            if (!opt && (snap || outputs_every)) wrb = step::expected_multiplicity(pu, Lrec, budget);
            if (tid == 0 && (snap || outputs_every)) {
                const Args r = args_here();
                if (r->log_cap > 0) {
                    const int64_t slot = (int64_t)chain * r->log_cap + (k % r->log_cap);
                    r->log_action[slot] = action;
                    r->log_M[slot] = M;
                    r->log_E[slot] = Erec;
                    r->log_p[slot] = pu;
                    r->log_w[slot] = wrb;
                }
                if (r->hist_w != nullptr) {
                    atomicAdd(&r->hist_w[rec_idx], (unsigned long long)M);
                    atomicAdd(&r->hist_v[rec_idx], 1ull);
                    atomicAdd(&r->hist_rb[rec_idx], wrb);
                }
                if (snap) {
                    const int64_t slot = (int64_t)chain * r->snap_cap + (snap_n - 1) % r->snap_cap;
                    r->snap_M[slot] = M;
                    r->snap_E[slot] = Erec;
                    r->snap_w[slot] = wrb;
                }
            }
        }
        if (timed && stay) {
            ++k;  // the cut record was the run's last
            break;
        }
    }
    if (lazy_m && wave == 0 && k > ub_base) flush_m((int)(k - ub_base));

    // ---- chain state back to memory (integers: h = (u - diag) / s) ----
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));  // (addresses formed here, not kept across the loop)
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int64_t fb = ((int64_t)g * BLOCK + tid_e) * 4;
        if (fb < pitch) {
            HT hv[4];
            uint32_t xb = 0, mw = 0;
            [[maybe_unused]] step::Four<QW> dv{};
            if constexpr (kInt) dv = step::load4(dbase + fb);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = g * 4 + v;
                hv[v] = h[i];
                if constexpr (kInt) {
                    hv[v] -= (HT)dv.v[v];
                    hv[v] = s == 2 ? hv[v] >> 1 : hv[v];
                }
                xb |= ((xw >> i) & 1u) << (8 * v);
                mw |= ((mem >> i) & 1u) << (8 * v);
            }
            step::store4(hbase + fb, hv);
            *reinterpret_cast<uint32_t*>(a.x + off + fb) = xb;
            if (unbiased) *reinterpret_cast<uint32_t*>(a.rmem + off + fb) = mw;
        }
    }
    if (tid == 0) {
        a.step[chain] = k;
        a.E[chain] = E;
        a.L[chain] = L;
        a.sub[chain] = sub;
        a.last_action[chain] = last_a;
        a.last_M[chain] = last_M;
        a.last_E[chain] = last_E;
        if constexpr (INSTR) {
            if (a.snap_every > 0) a.snap_count[chain] = snap_n;
            if (best) a.Ebest[chain] = Ebest;
        }
        int64_t* cn = a.counters + (int64_t)chain * 6;
        cn[0] += c_steps;
        cn[1] += c_flips;
        cn[2] += c_stays;
        cn[3] += c_sat;
        cn[4] = __double_as_longlong(__longlong_as_double(cn[4]) + __longlong_as_double(c_sumM));
        cn[5] += c_bad;
    }
}

template <typename QT, typename HT, int W, int G, bool DRAWN, bool INSTR>
hipError_t launch_one(int32_t grid, size_t dyn, hipStream_t st, const StepArgs& a)
{
    // dyn: the table of first occurrences
    const int32_t share = W == 1 ? share_of(grid) : 1;
    const bool tables = W == 1 && !std::is_floating_point<HT>::value;
    const size_t stride = (tables ? kTableBytes : 0) + (DRAWN ? (W == 1 ? 4 * 64 : 0) + dyn : 0);
    const dim3 blocks((grid + share - 1) / share), threads(64 * W * share);
    if (a.mode <= step::kModeBasic && a.orig_time == 0)
        hipLaunchKernelGGL((full_kernel<QT, HT, W, G, DRAWN, INSTR, true>), blocks, threads, share * stride, st, a, grid, share, (int32_t)stride);
    else
        hipLaunchKernelGGL((full_kernel<QT, HT, W, G, DRAWN, INSTR, false>), blocks, threads, share * stride, st, a, grid, share, (int32_t)stride);
    return hipGetLastError();
}

#define PNS_FULL_CASE(B, GG)                                                             \
    if (block == B && groups == GG)                                                      \
        return instr ? launch_one<QT, HT, B / 64, GG, DRAWN, true>(grid, dyn, st, a)     \
                     : launch_one<QT, HT, B / 64, GG, DRAWN, false>(grid, dyn, st, a);

// The tiles of a field type and of all bits or drawn subsets (pns_internal.h).
template <typename QT, typename HT, bool DRAWN>
hipError_t launch_tile(bool instr, int block, int groups, int grid, size_t dyn, hipStream_t st, const StepArgs& a)
{
    if constexpr (std::is_floating_point<HT>::value) {
        if constexpr (DRAWN) { PNS_FULL_TILES_F64_DRAWN(PNS_FULL_CASE) }
        else { PNS_FULL_TILES_F64_ALL(PNS_FULL_CASE) }
    } else if constexpr (sizeof(HT) == 8) {
        if constexpr (DRAWN) { PNS_FULL_TILES_I64_DRAWN(PNS_FULL_CASE) }
        else { PNS_FULL_TILES_I64_ALL(PNS_FULL_CASE) }
    } else {
        if constexpr (DRAWN) { PNS_FULL_TILES_I32_DRAWN(PNS_FULL_CASE) }
        else { PNS_FULL_TILES_I32_ALL(PNS_FULL_CASE) }
    }
    return hipErrorInvalidConfiguration;
}

}  // namespace full
}  // namespace pns
