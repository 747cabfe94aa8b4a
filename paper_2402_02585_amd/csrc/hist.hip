// Level-space ("effective space") G-QAOA, App. C "Optimization".
//
// From |s>, every amplitude depends on z only through the level C(z) = k, so
// the state is one amplitude b_k per occupied level with weight
// w_k = N_k / 2^n. A round (Eq. (3)) is b_k <- e^{-i gamma k} b_k, then
// b_k <- b_k + (e^{-i beta} - 1) S with S = sum_k w_k b_k (= <s|psi>).
// Readouts: P_sol = w_t |b_t|^2, E = sum_k k w_k |b_k|^2 (Eq. (4)).
//
// gqaoa_hist_evolve: one instance, float64, one wave; lanes own levels and
// S is a wave reduction per round.
// gqaoa_scan_batched: the single-angle-pair protocol (Eq. (5)) for every
// (instance, gamma, beta) triple, float32. A wave takes one (instance, gamma,
// 64-beta tile) work item from a global counter; gamma is wave-uniform, so the
// phase/weight table lives in LDS and is read as broadcasts, while each lane
// holds its own beta's K level amplitudes in registers. Instances are
// bucketed by padded level count (a register-array size per kernel
// instantiation) and, inside a bucket, ordered by level count descending so
// the dynamic queue ends with the short items.
#include "batch.h"
#include "stream_pool.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <optional>
#include <string>
#include <utility>
#include <vector>

namespace gqaoa {

// ---- single instance, float64 ------------------------------------------------------
// rounds[j] = {cos g_j, -sin g_j, cos b_j - 1, -sin b_j} is not enough for exact
// phases at every level, so the host passes, per round, e^{-i gamma_j 2^t} for
// t = 0..7 (each reduced mod 2 pi in double); level k multiplies the powers
// selected by its bits.
struct HistRound {
    double pw[8][2];   // e^{-i gamma 2^t}
    double mix[2];     // e^{-i beta} - 1
    int same_gamma;    // gamma equal to the previous round's: phases unchanged
    int pad;
};

__global__ void __launch_bounds__(64)
hist_evolve_kernel(const unsigned long long *__restrict__ hist, int m, int n, int p,
                   const HistRound *__restrict__ rounds, int target, double *__restrict__ out) {
    const int lane = threadIdx.x;
    constexpr int kPer = 4;  // levels per lane: k = lane + 64 i
    const double invN = std::ldexp(1.0, -n);
    double w[kPer], br[kPer], bi[kPer], pr[kPer], pi_[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int k = lane + 64 * i;
        w[i] = k <= m ? (double)hist[k] * invN : 0.0;
        br[i] = 1.0;
        bi[i] = 0.0;
        pr[i] = 1.0;
        pi_[i] = 0.0;
    }
    auto readout = [&](int j) {
        double P = 0, E = 0, Nn = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int k = lane + 64 * i;
            const double pb = w[i] * (br[i] * br[i] + bi[i] * bi[i]);
            Nn += pb;
            E += (double)k * pb;
            P += k == target ? pb : 0.0;
        }
        P = wave_sum_dpp(P);  // the one-wave block is converged here
        E = wave_sum_dpp(E);
        Nn = wave_sum_dpp(Nn);
        if (lane == 0) {
            out[3 * j] = P;
            out[3 * j + 1] = E;
            out[3 * j + 2] = Nn;
        }
    };
    readout(0);
    for (int j = 0; j < p; ++j) {
        const HistRound &R = rounds[j];
        if (!R.same_gamma) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int k = lane + 64 * i;
                double xr = 1.0, xi = 0.0;
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if ((k >> t) & 1) {
                        const double yr = xr * R.pw[t][0] - xi * R.pw[t][1];
                        xi = xr * R.pw[t][1] + xi * R.pw[t][0];
                        xr = yr;
                    }
                pr[i] = xr;
                pi_[i] = xi;
            }
        }
        double sr = 0, si = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const double nr = pr[i] * br[i] - pi_[i] * bi[i];
            bi[i] = pr[i] * bi[i] + pi_[i] * br[i];
            br[i] = nr;
            sr += w[i] * br[i];
            si += w[i] * bi[i];
        }
        sr = wave_sum_dpp(sr);
        si = wave_sum_dpp(si);
        const double cr = R.mix[0] * sr - R.mix[1] * si, ci = R.mix[0] * si + R.mix[1] * sr;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            br[i] += cr;
            bi[i] += ci;
        }
        readout(j + 1);
    }
}

int run_hist_evolve(int n, int m, const uint64_t *hist, int p, const double *beta,
                    const double *gamma, int target, double *psol, double *energy, double *norm,
                    hipStream_t st) {
    std::vector<HistRound> rounds((size_t)std::max(p, 1));
    const double two_pi = 2.0 * M_PI;
    for (int j = 0; j < p; ++j) {
        HistRound &R = rounds[j];
        for (int t = 0; t < 8; ++t) {
            const double a = std::fmod(gamma[j] * (double)(1 << t), two_pi);
            R.pw[t][0] = std::cos(a);
            R.pw[t][1] = -std::sin(a);
        }
        R.mix[0] = std::cos(beta[j]) - 1.0;
        R.mix[1] = -std::sin(beta[j]);
        R.same_gamma = (j > 0 && gamma[j] == gamma[j - 1]) ? 1 : 0;
        R.pad = 0;
    }
    const size_t rb = sizeof(HistRound) * rounds.size();
    const size_t ob = sizeof(double) * 3 * (size_t)(p + 1);
    AsyncScratch guard(st);
    GQ_HIP(guard.alloc(rb + ob + 256));
    char *base = reinterpret_cast<char *>(guard.ptr);
    double *d_out = reinterpret_cast<double *>(base + ((rb + 255) & ~size_t(255)));
    GQ_HIP(hipMemcpyAsync(base, rounds.data(), rb, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(hist_evolve_kernel, dim3(1), dim3(64), 0, st,
                       reinterpret_cast<const unsigned long long *>(hist), m, n, p,
                       reinterpret_cast<const HistRound *>(base), target, d_out);
    GQ_LAUNCH_CHECK();
    std::vector<double> o((size_t)3 * (p + 1));
    GQ_HIP(hipMemcpyAsync(o.data(), d_out, ob, hipMemcpyDeviceToHost, st));
    GQ_HIP(hipStreamSynchronize(st));
    for (int j = 0; j <= p; ++j) {
        if (psol) psol[j] = o[3 * j];
        if (energy) energy[j] = o[3 * j + 1];
        if (norm) norm[j] = o[3 * j + 2];
    }
    return GQAOA_OK;
}

// ---- batched single-angle-pair scan, float32 -------------------------------------------
constexpr int kScanMaxWaves = 4;
// Tables up to kScanHoist4 levels stay in registers whole (cos, -sin, sin, w:
// every instruction of a level-round has two VGPR operands); up to
// kScanHoist3 levels as (cos, sin, w), with the one negated product of a
// level-round as a three-operand fma, which gives the same value; larger
// tables are re-read from LDS every round.
constexpr int kScanHoist4 = 24;
constexpr int kScanHoist3 = 36;

// Per item, each wave's table in LDS: tab[k] = {cos(gamma l_k), -sin(gamma l_k),
// sin(gamma l_k), w_k}; the energy weights l_k w_k (read only at readouts) go
// from the lanes that compute them to scalar registers. The target level,
// when occupied, is level 0 of the instance's compacted order, so the
// crossing readout reads one amplitude.
//
// A level-round is eight two-operand VALU instructions on VGPR operands (the
// form gfx950 issues at twice the rate of instructions with an SGPR or a third
// source): the phase multiply as two products and two fused accumulates, the
// weighted sum for <s|phi> as two fused accumulates, the mixer as two adds.
// Dual issue needs two waves with VALU work on a SIMD, so an item's loads
// (its descriptor, levels and weights) are issued one item ahead, while the
// previous item's rounds run, instead of stalling the wave between items.

// The work item's coordinates: beta tile, gamma index and slot.
struct ScanItem {
    int tile, g;
    unsigned slot;
};
__device__ __forceinline__ ScanItem scan_decode(const ScanArgs &a, unsigned item) {
    const unsigned rest = item / (unsigned)a.ntiles;
    return ScanItem{(int)(item % (unsigned)a.ntiles), (int)(rest % (unsigned)a.ng), rest / (unsigned)a.ng};
}

// The lane's share of an instance's levels: level k = lane + 64 i.
template <int NL>
__device__ __forceinline__ void scan_load_levels(const ScanArgs &a, const ScanSlot &sl, int lane, int (&lv)[NL],
                                                 float (&wk)[NL]) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int k = lane + 64 * i;
        lv[i] = k < sl.K ? a.lev[sl.lev_off + k] : 0;
        wk[i] = k < sl.K ? a.w[sl.lev_off + k] : 0.f;
    }
}

// Writes the item's table (phases in float64, rounded once) to LDS.
template <int KMAX, int NL>
__device__ __forceinline__ void scan_table(const ScanArgs &a, const ScanSlot &sl, int g, int lane, const int (&lv)[NL],
                                           const float (&wk)[NL], float4 *tab, float (&kwl)[NL]) {
    const double gam = a.gammas[(a.per_inst ? (size_t)sl.inst * a.ng : 0) + g];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int k = lane + 64 * i;
        if (k < KMAX) {
            float4 e = {1.f, 0.f, 0.f, 0.f};
            float ew = 0.f;
            if (k < sl.K) {
                double sn, cs;
                sincos(gam * (double)lv[i], &sn, &cs);
                e = {(float)cs, (float)-sn, (float)sn, wk[i]};
                ew = wk[i] * (float)lv[i];
            }
            tab[k] = e;
            kwl[i] = ew;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// How far a round can bring a state to the target level. With x^2 = P = <psi|Pi_t|psi>
// and theta = asin x, the phase leaves theta as it is, and the mixer, a unitary
// M, moves the angle between psi and the target state |t> by at most the angle
// between |t> and M^dagger |t>: cos d = |<t|M|t>| = |1 + (e^{-i beta} - 1) w_t|, so
// sin d = |e^{-i beta} - 1| sqrt(w_t (1 - w_t)). A lane whose theta + r d stays
// below asin sqrt(S) with r rounds left cannot cross any more. The margins
// (1% and 1e-6 per round of P, 1e-4) are wide of what float32 rounding moves.
constexpr int kReachEvery = 16;  // rounds between the checks (under 1% of their arithmetic)
struct ScanReach {
    float th, d, rel;  // th and rel in scalar registers: the rounds have no vector register to spare
    static __device__ __forceinline__ float uniform(float x) {
        return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
    }
    __device__ __forceinline__ ScanReach(const ScanSlot &sl, float S, float w0, float mr, float mi) {
        th = uniform(sl.unit ? asinf(sqrtf(fminf(fmaxf(S, 0.f), 1.f))) : 0.f);  // th = 0: always within reach
        d = asinf(fminf(sqrtf(w0 * (1.f - w0) * (mr * mr + mi * mi)), 1.f));
        rel = uniform(0.99f - 1e-6f * (float)sl.pmax);
    }
    // P after a round with r more to come
    __device__ __forceinline__ bool out_of_reach(float P, int r) const {
        const float t = th - (float)r * d;
        const float s = __sinf(t);  // 0 < t <= pi/2: good to 1e-6, far within the margins
        return t > 0.f && P < rel * s * s - 1e-4f;
    }
};

// The rounds of one item for this lane's beta (mixer e^{-i beta} - 1 = mr + i mi).
template <int KMAX, bool CROSS>
__device__ __forceinline__ void scan_rounds(const ScanArgs &a, const ScanSlot &sl, const ScanItem &it, int lane,
                                            float mr, float mi, const float4 *tab,
                                            const float (&kwl)[(KMAX + 63) / 64]) {
    // l_k w_k of every level, for the energy readout: the same in every lane,
    // so held in scalar registers (read out of the lane that computed it)
    float kw[CROSS ? 1 : KMAX];
    if constexpr (!CROSS) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            kw[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(kwl[k / 64]), k % 64));
    }
    const int b = it.tile * 64 + lane;
    const bool active = b < a.nb;
    const float w0 = sl.t_idx == 0 ? tab[0].w : 0.f;   // weight of the target level (index 0)
    // The lane keeps the phased amplitudes phi_k of the current round and the
    // mixer's correction c of the round before, and forms b_k = phi_k + c at
    // the start of the next round: the same adds on the same operands as
    // applying the mixer at the end of each round, with one level's
    // temporaries live at a time instead of all of them.
    float pr[KMAX], pi[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        pr[k] = 1.f;
        pi[k] = 0.f;
    }
    float cr = 0.f, ci = 0.f;
    // One round: phases, <s|phi> and the mixer's correction. Small tables stay in
    // registers across rounds (the crossing form's, whose rounds come in runs, by
    // name: the compiler would load them once a run); larger ones are re-read from
    // LDS (broadcast) each round to bound register use.
    constexpr bool kHeld = CROSS && KMAX <= kScanHoist3;
    float4 held[kHeld ? KMAX : 1];
    if constexpr (kHeld)
#pragma unroll
        for (int k = 0; k < KMAX; ++k) held[k] = tab[k];
    auto round = [&]() {
        if constexpr (KMAX > kScanHoist3) asm volatile("" ::: "memory");
        float sr = 0.f, si = 0.f;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const float4 e = kHeld ? held[kHeld ? k : 0] : tab[k];
            const float xr = pr[k] + cr, xi = pi[k] + ci;               // b_k after the last mixer
            const float nr = __builtin_fmaf(e.x, xr, e.z * xi);         // cos br + sin bi
            float ni;                                                    // cos bi - sin br
            if constexpr (KMAX <= kScanHoist4)
                ni = __builtin_fmaf(e.x, xi, e.y * xr);
            else
                ni = __builtin_fmaf(e.x, xi, -(e.z * xr));
            pr[k] = nr;
            pi[k] = ni;
            sr = __builtin_fmaf(e.w, nr, sr);
            si = __builtin_fmaf(e.w, ni, si);
        }
        // Which product is rounded first is written out: first crossings are whole
        // numbers, compared exactly, and each size keeps the order it has had.
        cr = __builtin_fmaf(mr, sr, -(mi * si));
        if constexpr (CROSS && KMAX >= 20 && KMAX <= 32) ci = __builtin_fmaf(mi, sr, mr * si);
        else ci = __builtin_fmaf(mr, si, mi * sr);
    };
    auto target_prob = [&]() {
        const float b0r = pr[0] + cr, b0i = pi[0] + ci;
        return w0 * __builtin_fmaf(b0r, b0r, b0i * b0i);
    };
    if constexpr (CROSS) {
        // The reach is checked between runs of rounds: inside the round loop the
        // check cost every round its schedule (one instance of 10 levels, 1,000
        // rounds: 320 us without a check, 354 with; in runs, and the round's own test
        // without branches, 306).
        const ScanReach reach(sl, a.threshold, w0, mr, mi);
        const int pmax = __builtin_amdgcn_readfirstlane(sl.pmax);  // and so j and stop: scalar
        int found = 0;
        // (wave-uniform; P again from its amplitude, which is there anyway)
        for (int j = 0; __ballot(active && found == 0 && !reach.out_of_reach(target_prob(), pmax - j)) != 0;) {
            const int stop = min(pmax, j + kReachEvery);
            while (j < stop) {
                round();
                ++j;
                const bool hit = (found == 0) & (target_prob() >= a.threshold);
                found = hit ? j : found;
                if (__builtin_amdgcn_ballot_w64(active & (found == 0)) == 0) break;  // wave-uniform
            }
            if (j >= pmax) break;
        }
        if (active) a.first_p[((size_t)sl.inst * a.ng + it.g) * a.nb + b] = found;
    } else {
        int q = 0;
        int next_p = a.p_list[0];   // next readout round, kept in a register
        for (int j = 1; j <= sl.pmax; ++j) {
            round();
            if (j != next_p) continue;
            float E = 0.f;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const float br = pr[k] + cr, bi = pi[k] + ci;
                E = __builtin_fmaf(kw[k], __builtin_fmaf(br, br, bi * bi), E);
            }
            const float P = target_prob();
            if (active) {
                const size_t o = (((size_t)sl.inst * a.num_p + q) * a.ng + it.g) * a.nb + b;
                a.psol[o] = P;
                if (a.energy) a.energy[o] = E;
            }
            ++q;
            next_p = q < a.num_p ? a.p_list[q] : 0;
        }
    }
}

// Mixer factor of this lane's beta, recomputed only when the beta row changes
// (the grid is shared, or the instance's own).
__device__ __forceinline__ void scan_mixer(const ScanArgs &a, const ScanSlot &sl, int tile, int lane, long long &key,
                                           float &mr, float &mi) {
    const long long k = (long long)(a.per_inst ? sl.inst : 0) * a.ntiles + tile;
    if (k == key) return;
    key = k;
    const int b = tile * 64 + lane;
    double sb, cb;
    sincos(a.betas[(a.per_inst ? (size_t)sl.inst * a.nb : 0) + (b < a.nb ? b : 0)], &sb, &cb);
    mr = (float)(cb - 1.0);
    mi = (float)(-sb);
}

// Waves per SIMD a crossing kernel is held to. Two waves can keep a SIMD issuing,
// but only while neither waits for a result; a third covers that. Without a bound
// the compiler keeps the constants of the tables' sines in registers from item to
// item (185 for KMAX = 20, 209 for 24, 205 for 28: two waves); held to 168 it
// reloads what it has to once an item, never in a round. 128 instances, 360 x 181
// pairs: n = 12..20 of density 4.6..8 8,500 -> 7,980 us, of 3..5 6,300 -> 5,800, the
// buckets one after another; 32 levels at three waves would spill in their rounds
// (8,900 us). The fixed rounds of
// the other kernels are too short for it: 1,024 instances of 64 x 64 pairs, 64
// rounds within 1%, 16 rounds 413 -> 430 us.
constexpr int scan_waves_per_simd(int kmax) { return kmax <= 12 ? 4 : kmax <= 28 ? 3 : 1; }

// CROSS = false: P_sol (and E) after each p in p_list. Every item of a bucket
// costs the same (same padded level count, same rounds), so wave w of the
// grid takes items w, w + W, w + 2W, ... (W waves), and the next item's
// descriptor and levels are loaded while the current one runs.
// CROSS = true: the first round j <= p_i with P >= threshold; a wave stops
// once every lane has crossed, so items differ in length and come from a
// global queue (the next index is fetched while the current item runs).
template <int KMAX, bool CROSS>
__global__ void __launch_bounds__(kScanMaxWaves * 64, CROSS ? scan_waves_per_simd(KMAX) : 1) scan_kernel(ScanArgs a) {
    constexpr int NL = (KMAX + 63) / 64;
    __shared__ float4 tab_s[kScanMaxWaves][KMAX];
    const int lane = threadIdx.x & 63;
    float4 *tab = tab_s[threadIdx.x >> 6];
    float kwl[NL];
    long long mix_key = -1;
    float mr = 0.f, mi = 0.f;
    unsigned item;
    if constexpr (CROSS) {
        unsigned v = 0;
        if (lane == 0) v = atomicAdd(a.counter, 1u);
        item = __builtin_amdgcn_readfirstlane(__shfl(v, 0, 64));
    } else {
        item = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    }
    if (item >= a.total_items) return;  // whole waves
    const unsigned W = gridDim.x * (blockDim.x >> 6);
    ScanItem it = scan_decode(a, item);
    ScanSlot sl = a.slots[it.slot];
    int lv[NL];
    float wk[NL];
    scan_load_levels<NL>(a, sl, lane, lv, wk);
    unsigned nxt = CROSS ? 0u : item + W;
    ScanSlot sl_n = sl;
    if constexpr (!CROSS)
        if (nxt < a.total_items) sl_n = a.slots[scan_decode(a, nxt).slot];
    for (;;) {
        scan_table<KMAX, NL>(a, sl, it.g, lane, lv, wk, tab, kwl);
        // loads for the next item, consumed after this item's rounds
        int lv_n[NL];
        float wk_n[NL];
        unsigned nn = 0;
        ScanSlot sl_nn = sl_n;
        if constexpr (CROSS) {
            unsigned v = 0;
            if (lane == 0) v = atomicAdd(a.counter, 1u);
            nxt = __builtin_amdgcn_readfirstlane(__shfl(v, 0, 64));
        } else {
            if (nxt < a.total_items) scan_load_levels<NL>(a, sl_n, lane, lv_n, wk_n);
            nn = nxt + W;
            if (nn < a.total_items) sl_nn = a.slots[scan_decode(a, nn).slot];
        }
        scan_mixer(a, sl, it.tile, lane, mix_key, mr, mi);
        scan_rounds<KMAX, CROSS>(a, sl, it, lane, mr, mi, tab, kwl);
        // the next item rewrites tab: keep every lane's reads of this one first
        __builtin_amdgcn_wave_barrier();
        if (nxt >= a.total_items) break;
        it = scan_decode(a, nxt);
        if constexpr (CROSS) {
            sl = a.slots[it.slot];
            scan_load_levels<NL>(a, sl, lane, lv, wk);
        } else {
            sl = sl_n;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                lv[i] = lv_n[i];
                wk[i] = wk_n[i];
            }
            sl_n = sl_nn;
            nxt = nn;
        }
    }
}

__global__ void zero_counters_kernel(unsigned int *c, int n) {
    const int i = threadIdx.x;
    if (i < n) c[i] = 0u;
}

// Register-array sizes of the scan kernel instantiations: every multiple of
// 4 up to 64 (an instance pays for at most 3 padding levels, which carry
// weight 0), then steps of 16.
static const int kBuckets[] = {4, 8, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48, 52, 56, 60, 64, 80, 96, 112, 128};
constexpr int kNumBuckets = sizeof(kBuckets) / sizeof(kBuckets[0]);
constexpr int kScanMaxK = 128;

typedef void (*ScanFn)(ScanArgs);
template <bool CROSS, int... KS>
static ScanFn scan_fn_pick(int kmax, std::integer_sequence<int, KS...>) {
    ScanFn f = nullptr;
    ((f = (KS == kmax ? scan_kernel<KS, CROSS> : f)), ...);
    return f;
}
template <bool CROSS>
static ScanFn scan_fn_t(int bucket) {
    return scan_fn_pick<CROSS>(kBuckets[bucket], std::integer_sequence<int, 4, 8, 12, 16, 20, 24, 28, 32, 36, 40, 44, 48,
                                                                       52, 56, 60, 64, 80, 96, 112, 128>{});
}
static ScanFn scan_fn(int bucket, bool cross) { return cross ? scan_fn_t<true>(bucket) : scan_fn_t<false>(bucket); }

int scan_max_levels() { return kScanMaxK; }

// ---- autotuned launch shape -----------------------------------------------------------
// Candidates: waves per block in {1, 2, 4} x blocks per CU in {2, 4, 8, 16}. A
// candidate is timed on the bucket's real work (a prefix of the queue) and
// the best is cached per (device arch, bucket, beta tiles) for the process;
// GQAOA_TUNE_CACHE names an optional text file that persists the choices.
static std::mutex g_tune_mu;
static std::map<std::string, TileChoice> g_tune;
static bool g_tune_loaded = false;

static void tune_load_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char *path = getenv("GQAOA_TUNE_CACHE");
    if (!path) return;
    FILE *f = fopen(path, "r");
    if (!f) return;
    tune_cache_read(f, g_tune);  // shapes outside the accepted range are dropped and retuned
    fclose(f);
}

static void tune_store_locked() {
    const char *path = getenv("GQAOA_TUNE_CACHE");
    if (!path) return;
    FILE *f = fopen(path, "w");
    if (!f) return;
    tune_cache_write(f, g_tune);
    fclose(f);
}

int scan_launch_bucket(int bucket, const TileChoice &tc, const DeviceInfo &dev, ScanArgs a, unsigned int *counter,
                       hipStream_t st) {
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, st, counter, 1);
    GQ_LAUNCH_CHECK();
    a.counter = counter;
    const unsigned want = (a.total_items + tc.waves - 1) / tc.waves;
    const unsigned blocks = std::max(1u, std::min<unsigned>(want, (unsigned)(dev.num_cus * tc.blocks_per_cu)));
    hipLaunchKernelGGL(scan_fn(bucket, a.first_p != nullptr), dim3(blocks), dim3(64 * tc.waves), 0, st, a);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

static int tune_bucket(int bucket, const DeviceInfo &dev, const ScanArgs &a, unsigned int *counter,
                       hipStream_t st, TileChoice *out) {
    const std::string key = std::string(dev.arch) + ":k" + std::to_string(kBuckets[bucket]) + ":t" +
                            std::to_string(a.ntiles) + ":p" + std::to_string(a.p_list[a.num_p - 1] > 16 ? 64 : 16);
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        tune_load_locked();
        auto it = g_tune.find(key);
        if (it != g_tune.end()) {
            *out = it->second;
            return GQAOA_OK;
        }
    }
    // time a prefix of the items that fills the device a few times over
    ScanArgs t = a;
    t.total_items = std::min<unsigned>(a.total_items, (unsigned)dev.num_cus * 64);
    const int waves_c[] = {1, 2, 4};
    const int bpc_c[] = {2, 4, 8, 16};
    hipEvent_t e0, e1;
    GQ_HIP(hipEventCreate(&e0));
    GQ_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    TileChoice bestc{4, 4};
    for (int wv : waves_c)
        for (int bpc : bpc_c) {
            TileChoice tc{wv, bpc};
            int s = scan_launch_bucket(bucket, tc, dev, t, counter, st);  // warm-up
            if (s) return s;
            GQ_HIP(hipEventRecord(e0, st));
            for (int r = 0; r < 3; ++r)
                if ((s = scan_launch_bucket(bucket, tc, dev, t, counter, st))) return s;
            GQ_HIP(hipEventRecord(e1, st));
            GQ_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            GQ_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (ms < best) {
                best = ms;
                bestc = tc;
            }
        }
    GQ_HIP(hipEventDestroy(e0));
    GQ_HIP(hipEventDestroy(e1));
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[key] = bestc;
    tune_store_locked();
    *out = bestc;
    return GQAOA_OK;
}

size_t scan_workspace_bytes(int num_inst, int hist_stride, int nb, int ng, int num_p, int per_inst) {
    (void)num_p;
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const size_t lv = (size_t)num_inst * std::min(hist_stride, kScanMaxK);
    const size_t ga = per_inst ? (size_t)num_inst : 1;
    return al(sizeof(ScanSlot) * (size_t)num_inst) + al(4 * lv) + al(4 * lv) + al(8 * (size_t)nb * ga) +
           al(8 * (size_t)ng * ga) + al(4 * kNumBuckets) + 256;
}

int scan_num_buckets() { return kNumBuckets; }

ScanDev scan_dev_tables(void *ws, int num_inst, int hist_stride, int nb, int ng, int per_inst) {
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const size_t lv = (size_t)num_inst * std::min(hist_stride, kScanMaxK);
    const size_t ga = per_inst ? (size_t)num_inst : 1;
    char *p = reinterpret_cast<char *>(ws);
    ScanDev d;
    d.slots = reinterpret_cast<ScanSlot *>(p);
    p += al(sizeof(ScanSlot) * (size_t)num_inst);
    d.lev = reinterpret_cast<int32_t *>(p);
    p += al(4 * lv);
    d.w = reinterpret_cast<float *>(p);
    p += al(4 * lv);
    d.betas = reinterpret_cast<double *>(p);
    p += al(8 * (size_t)nb * ga);
    d.gammas = reinterpret_cast<double *>(p);
    p += al(8 * (size_t)ng * ga);
    d.counters = reinterpret_cast<unsigned int *>(p);
    return d;
}

int scan_host_tables(int num_inst, const int32_t *n_host, const int32_t *m_host, const uint64_t *hists,
                     int hist_stride, const int32_t *target_host, const int32_t *pmax_host, int pmax_all,
                     ScanHost *out) {
    // compact the occupied levels of every instance
    std::vector<int32_t> K(num_inst), tidx(num_inst), off(num_inst), unit(num_inst);
    out->lev.clear();
    out->w.clear();
    for (int i = 0; i < num_inst; ++i) {
        const uint64_t *h = hists + (size_t)i * hist_stride;
        const int t = target_host ? target_host[i] : 0;
        off[i] = (int32_t)out->lev.size();
        tidx[i] = -1;
        const double invN = std::ldexp(1.0, -n_host[i]);
        uint64_t total = 0;
        // the target level (when occupied) first, then the others in level order
        if (t <= m_host[i] && h[t]) {
            tidx[i] = 0;
            total += h[t];
            out->lev.push_back(t);
            out->w.push_back((float)((double)h[t] * invN));
        }
        for (int k = 0; k <= m_host[i]; ++k)
            if (h[k] && k != t) {
                total += h[k];
                out->lev.push_back(k);
                out->w.push_back((float)((double)h[k] * invN));
            }
        K[i] = (int32_t)out->lev.size() - off[i];
        unit[i] = n_host[i] < 64 && total == 1ull << n_host[i];
        if (K[i] > kScanMaxK) return fail(GQAOA_ERANGE, "instance %d has %d occupied levels (max %d)", i, K[i], kScanMaxK);
    }
    // buckets, each ordered by K descending
    std::vector<std::vector<int>> members(kNumBuckets);
    for (int i = 0; i < num_inst; ++i) {
        int bk = 0;
        while (kBuckets[bk] < std::max(1, K[i])) ++bk;
        members[bk].push_back(i);
    }
    out->slots.clear();
    out->bucket_first.assign(kNumBuckets + 1, 0);
    for (int bk = 0; bk < kNumBuckets; ++bk) {
        auto &mb = members[bk];
        std::stable_sort(mb.begin(), mb.end(), [&](int x, int y) { return K[x] > K[y]; });
        out->bucket_first[bk] = (int)out->slots.size();
        for (int i : mb)
            out->slots.push_back(
                ScanSlot{i, off[i], K[i], tidx[i], pmax_host ? pmax_host[i] : pmax_all, unit[i], {0, 0}});
    }
    out->bucket_first[kNumBuckets] = (int)out->slots.size();
    return GQAOA_OK;
}

int scan_choose_tile(int bucket, const DeviceInfo &dev, const ScanArgs &a, unsigned int *counter,
                     const int32_t *tile, hipStream_t st, TileChoice *out) {
    if (tile) {
        *out = TileChoice{tile[0], tile[1]};
        return GQAOA_OK;
    }
    if (a.first_p) {
        // The crossing form takes its items from a queue. Long items want two waves
        // per SIMD and gain nothing from more; short ones wait for the queue's
        // counter, the longer the more waves ask for it. Blocks of one wave, which
        // the hardware spreads best: 256 instances, 230 x 92 pairs, 1 round 1,262 us
        // at 1 wave per CU, 1,309 at 2, 1,520 at 8, 2,266 at 32; 32 rounds 2,051 at
        // 2, 1,612 at 4, 1,704 at 8; 64 rounds 3,716 at 2, 2,478 at 4, 2,475 at 8,
        // 3,188 at 32; 128 unsatisfiable instances, 360 x 181 pairs, caps of 400
        // 9,528 at 2, 7,056 at 4, 7,005 at 8, 7,495 at 32 (blocks of four waves).
        // Timing a prefix of the queue cannot tell: items run from one round to
        // their cap, and a prefix of one fill chose one wave per SIMD.
        const int cap = a.p_list[a.num_p - 1];
        *out = TileChoice{1, cap <= 16 ? 2 : cap <= 50 ? 4 : 8};
        return GQAOA_OK;
    }
    return tune_bucket(bucket, dev, a, counter, st, out);
}

// Streams of a call's own beside the caller's: forked from it behind what it has
// enqueued so far, joined to it at the end. They come from the device's pool and go
// back when their work has ended, also when the call fails.
struct SideStreams {
    int device;
    std::vector<hipStream_t> streams;
    hipEvent_t ev = nullptr;
    SideStreams(int d) : device(d) {}
    SideStreams(const SideStreams &) = delete;
    SideStreams &operator=(const SideStreams &) = delete;
    int fork(size_t n, hipStream_t st) {
        // a pooled stream never joins a caller's capture (the call fails at its
        // synchronization and would give it back inside one): none then
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
            (void)hipGetLastError();
            return GQAOA_OK;
        }
        if (const int s = stream_pool_take(n, &streams)) return s;
        GQ_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        GQ_HIP(hipEventRecord(ev, st));
        for (hipStream_t x : streams) GQ_HIP(hipStreamWaitEvent(x, ev, 0));
        return GQAOA_OK;
    }
    int join(hipStream_t st) {
        for (hipStream_t x : streams) {
            GQ_HIP(hipEventRecord(ev, x));
            GQ_HIP(hipStreamWaitEvent(st, ev, 0));
        }
        return GQAOA_OK;
    }
    ~SideStreams() {
        for (hipStream_t x : streams) (void)hipStreamSynchronize(x);
        if (!streams.empty()) stream_pool_give(device, streams);
        if (ev) (void)hipEventDestroy(ev);
    }
};

// Side streams of a crossing scan over the buckets `used`: as many as run beside
// the caller's, none where the fork and join cost more than the overlap can give
// (about 16 us and 14 more per stream). A bucket alone takes about 3 us and 0.1 +
// 0.02 us per round and level for every fill of the device (8 waves per CU); the
// overlap saves what exceeds the longest one and an even share. 16 instances of 10
// to 60 levels, 90 x 45 pairs: 1 round 184 us forked and 142 in turn, 4 rounds 184
// and 193, 16 rounds 195 and 353; 2 instances, 64 rounds 119 and 121.
static size_t crossing_side_streams(const ScanHost &H, const std::vector<int> &used, unsigned items_per_slot,
                                    const DeviceInfo &dev) {
    const size_t ways = std::min<size_t>(used.size(), 4);
    double total = 0.0, longest = 0.0;
    for (int bk : used) {
        int cap = 0;
        for (int i = H.bucket_first[bk]; i < H.bucket_first[bk + 1]; ++i) cap = std::max(cap, H.slots[i].pmax);
        const double fills = (double)(H.bucket_first[bk + 1] - H.bucket_first[bk]) * items_per_slot / (8.0 * dev.num_cus);
        const double us = std::max(1.0, fills) * (3.0 + cap * (0.1 + 0.02 * kBuckets[bk]));
        total += us;
        longest = std::max(longest, us);
    }
    const double saves = total - std::max(longest, total / (double)std::max<size_t>(ways, 1));
    return ways > 1 && saves > 16.0 + 14.0 * (double)(ways - 1) ? ways - 1 : 0;
}

int run_scan(int num_inst, const int32_t *n_host, const int32_t *m_host, const uint64_t *hists,
             int hist_stride, const int32_t *target_host, int nb, const double *betas, int ng,
             const double *gammas, int per_inst, int num_p, const int32_t *p_list, float *psol, float *energy,
             float threshold, int32_t *first_p, const int32_t *pmax_host, const int32_t *tile, void *ws,
             hipStream_t st) {
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    ScanHost H;
    if ((s = scan_host_tables(num_inst, n_host, m_host, hists, hist_stride, target_host, pmax_host,
                              p_list[num_p - 1], &H)))
        return s;
    const ScanDev D = scan_dev_tables(ws, num_inst, hist_stride, nb, ng, per_inst);
    const size_t ga = per_inst ? (size_t)num_inst : 1;
    GQ_HIP(hipMemcpyAsync(D.slots, H.slots.data(), sizeof(ScanSlot) * H.slots.size(), hipMemcpyHostToDevice, st));
    GQ_HIP(hipMemcpyAsync(D.lev, H.lev.data(), 4 * H.lev.size(), hipMemcpyHostToDevice, st));
    GQ_HIP(hipMemcpyAsync(D.w, H.w.data(), 4 * H.w.size(), hipMemcpyHostToDevice, st));
    GQ_HIP(hipMemcpyAsync(D.betas, betas, 8 * (size_t)nb * ga, hipMemcpyHostToDevice, st));
    GQ_HIP(hipMemcpyAsync(D.gammas, gammas, 8 * (size_t)ng * ga, hipMemcpyHostToDevice, st));

    ScanArgs a{};
    a.lev = D.lev;
    a.w = D.w;
    a.betas = D.betas;
    a.gammas = D.gammas;
    a.psol = psol;
    a.energy = energy;
    a.first_p = first_p;
    a.threshold = threshold;
    a.nb = nb;
    a.ng = ng;
    a.ntiles = (nb + 63) / 64;
    a.num_p = num_p;
    a.per_inst = per_inst;
    for (int q = 0; q < num_p; ++q) a.p_list[q] = p_list[q];
    // The crossing form's buckets run side by side on up to four streams, the most
    // levels first: its items end anywhere between one round and their cap, so a
    // bucket ends with few waves, and one of a few instances never fills the device
    // (16 instances of 10 to 60 levels, 90 x 45 pairs, 64 rounds 980 -> 359 us; 256 of
    // them 2,050 -> 875). The scan's items are equal and its buckets end full: one
    // after another.
    std::vector<int> used;
    for (int bk = kNumBuckets - 1; bk >= 0; --bk)
        if (H.bucket_first[bk + 1] > H.bucket_first[bk]) used.push_back(bk);
    if (!first_p) std::reverse(used.begin(), used.end());
    SideStreams side(dev.device);
    const size_t nside = first_p ? crossing_side_streams(H, used, (unsigned)ng * (unsigned)a.ntiles, dev) : 0;
    // buckets side by side are timed as one, from fork to join
    std::optional<ProfScope> all;
    if (nside) {
        all.emplace("scan", st);
        if ((s = side.fork(nside, st))) return s;
    }
    for (size_t u = 0; u < used.size(); ++u) {
        const int bk = used[u];
        const size_t branch = u % (side.streams.size() + 1);
        const hipStream_t bs = branch ? side.streams[branch - 1] : st;
        ScanArgs ab = a;
        ab.slots = D.slots + H.bucket_first[bk];
        ab.total_items = (unsigned)(H.bucket_first[bk + 1] - H.bucket_first[bk]) * (unsigned)ng * (unsigned)ab.ntiles;
        TileChoice tc;
        if ((s = scan_choose_tile(bk, dev, ab, D.counters + bk, tile, bs, &tc))) return s;
        std::optional<ProfScope> one;
        if (!all) one.emplace("scan", bs);
        if ((s = scan_launch_bucket(bk, tc, dev, ab, D.counters + bk, bs))) return s;
        if (one) one->end();
    }
    if ((s = side.join(st))) return s;
    if (all) all->end();
    GQ_HIP(hipStreamSynchronize(st));  // host staging vectors end here
    if (prof_on()) prof_collect();
    return GQAOA_OK;
}

}  // namespace gqaoa
