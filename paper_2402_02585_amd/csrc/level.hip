// Rounds from |s> in the level form.
//
// From |s> an amplitude depends on z only through its level C(z) = k (App. C,
// "Optimization"): psi_j(z) = 2^{-n/2} b_k(j). A round, Eq. (3), is
// b_k <- e^{-i gamma k} b_k, then b_k <- b_k + (e^{-i beta} - 1) S with
// S = sum_k w_k b_k, w_k = N_k / 2^n. So an evolution from |s> is one pass that
// counts the levels of the given cost table, a float64 recursion over the
// occupied levels, and one pass that writes 2^{-n/2} b_{C(z)}(p) to every z:
// 1 byte read per amplitude twice and the state written once, whatever p,
// where p round passes read and write the state p times. Every readout
// (P_sol, E, norm of each round) comes from the recursion.
//
// The costs are counted from the table itself, so any table is taken as it
// is; entries above m (which the caller promises not to pass) get the phase
// factor 0 that the round passes' tables hold there.
//
// complex128 only: its results agree with the round passes' to their rounding.
// A complex64 evolution rounds its state to float32 in every round, and that
// rounding is part of its results (its readouts would move by 4e-7).
#include "level.h"

#include <algorithm>
#include <cmath>

namespace gqaoa {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kLevels = 256;
constexpr int kCols = kWave;             // LDS counter columns: one per lane
constexpr int kCountThreads = 1024;
constexpr int kRunThreads = 512;         // wave 0 runs the rounds, the others feed it
constexpr int kRunWaves = kRunThreads / kWave;
constexpr size_t kCountBytes = sizeof(uint32_t) * kLevels * kCols;  // 64 KiB
constexpr int kChunkStates = 1024;       // amplitudes of one chunk buffer (16 KiB)

// ---- level counts -----------------------------------------------------------------
// Lane l of every wave counts in column l of h[level][64]: a wave's 64 adds
// fall in 64 different banks whatever the levels, so concentrated costs (a
// random instance has most assignments on about 15 levels) tally at the
// conflict-free rate of LDS adds.
__device__ __forceinline__ void tally4(uint32_t *h, uint32_t v) {
#pragma unroll
    for (int b = 0; b < 4; ++b) atomicAdd(h + ((v >> (8 * b)) & 0xFFu) * kCols, 1u);
}

// Counts costs [0, N) of which this block takes every nblocks-th run.
template <int THREADS>
__device__ __forceinline__ void count_levels(const uint8_t *__restrict__ c, uint64_t N, int block, int nblocks,
                                             uint32_t *h) {
    for (int i = threadIdx.x; i < kLevels * kCols; i += THREADS) h[i] = 0u;
    __syncthreads();
    uint32_t *col = h + (threadIdx.x & (kCols - 1));
    const uint64_t step = (uint64_t)nblocks * THREADS, first = (uint64_t)block * THREADS + threadIdx.x;
    if (N >= 16 && (reinterpret_cast<uintptr_t>(c) & 15) == 0) {
        const u32x4 *q = reinterpret_cast<const u32x4 *>(c);
        const uint64_t nq = N >> 4;
        constexpr int U = 4;  // 64 bytes in flight per lane
        uint64_t i = first;
        for (; i + (U - 1) * step < nq; i += U * step) {
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = q[i + u * step];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                tally4(col, v[u].x);
                tally4(col, v[u].y);
                tally4(col, v[u].z);
                tally4(col, v[u].w);
            }
        }
        for (; i < nq; i += step) {
            const u32x4 v = q[i];
            tally4(col, v.x);
            tally4(col, v.y);
            tally4(col, v.z);
            tally4(col, v.w);
        }
    } else {
        for (uint64_t i = first; i < N; i += step) atomicAdd(col + (uint32_t)c[i] * kCols, 1u);
    }
    __syncthreads();
}

// Total of level t over the columns: 16-byte reads, rotated by the level so
// that the lanes of a wave spread over the banks.
__device__ __forceinline__ uint32_t level_total(const uint32_t *h, int t) {
    const u32x4 *r = reinterpret_cast<const u32x4 *>(h + t * kCols);
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kCols / 4; ++i) {
        const u32x4 v = r[(i + t) & (kCols / 4 - 1)];
        s += (v.x + v.y) + (v.z + v.w);
    }
    return s;
}

// Block (b, i): counts of instance i's costs, one row of 256 per block. Bound
// by the read of the costs (n = 28: 256 MiB in 45 us, 6 TB/s); 1024 threads of
// 64 bytes in flight on 64 KiB of LDS fill a CU with one block, so at most 256
// rows are left to sum.
__global__ void __launch_bounds__(kCountThreads) level_count_kernel(const uint8_t *__restrict__ cost, uint64_t N,
                                                                    uint32_t *__restrict__ rows) {
    __shared__ __attribute__((aligned(16))) uint32_t h[kLevels * kCols];
    count_levels<kCountThreads>(cost + (uint64_t)blockIdx.y * N, N, blockIdx.x, gridDim.x, h);
    if (threadIdx.x < kLevels)
        rows[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kLevels + threadIdx.x] = level_total(h, threadIdx.x);
}

// ---- the recursion --------------------------------------------------------------------
// One block. Wave 0 holds the level amplitudes (lane l: compacted levels
// l + 64 i, i < LPL) and runs a chunk of rounds from a table of phases and
// mixer factors in LDS, one pair of wave sums per round; meanwhile the other
// waves compute the next chunk's table (float64 sincos) and the readouts of
// the chunk before from the states wave 0 left in LDS. One barrier per
// chunk. The serial chain per round is the two wave sums and four fused
// operations; everything else is off it (p = 20 at n = 10: 8 us with the counts
// and the write of the state; p = 64 at n = 28: 17 us with the sum of 256 rows).
struct LevelLds {
    double w[kLevels];
    int lev[kLevels];
    int K, t_idx;
    int wave_cnt[4];
    double2 mix[2][16];
    double ang[2 * kLevelInlineRounds];
};

struct LevelRunArgs {
    const uint8_t *cost;
    const uint32_t *rows;
    int nrows, n, m, p, target;
    const double *angles;  // device: beta[p], gamma[p]; null: the inline angles
    double2 *psi;
    double2 *table;
    double *readout;
};

template <int ROUNDS>
struct LevelAngles {
    double v[2 * ROUNDS];  // beta[p], gamma[p]
};

// Compacts the occupied levels (thread t < 256 holds level t's count) into
// L.w / L.lev in level order; every thread of the block calls this.
__device__ __forceinline__ void compact_levels(LevelLds &L, uint64_t count, int n, int target) {
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    const bool on = t < kLevels && count != 0;
    const uint64_t mask = __ballot(on);
    if (t == 0) L.t_idx = -1;
    if (wave < 4 && lane == 0) L.wave_cnt[wave] = __popcll(mask);
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) base += w < wave ? L.wave_cnt[w] : 0;
    if (t == 0) L.K = L.wave_cnt[0] + L.wave_cnt[1] + L.wave_cnt[2] + L.wave_cnt[3];
    if (on) {
        const int pos = base + __popcll(mask & ((1ull << lane) - 1ull));
        L.lev[pos] = t;
        L.w[pos] = ldexp((double)count, -n);  // exact: a count times a power of two
        if (t == target) L.t_idx = pos;
    }
    __syncthreads();
}

// All p rounds; returns in wave 0 the final amplitudes of its levels.
template <int LPL>
__device__ __forceinline__ void level_rounds(const LevelRunArgs &a, LevelLds &L, double2 *buf, const double *beta,
                                             const double *gamma, double (&br)[LPL], double (&bi)[LPL]) {
    constexpr int KP = kWave * LPL, R = kChunkStates / KP;  // R = 16, 8, 4 rounds per chunk
    double2 *ph = buf, *bs = buf + 2 * kChunkStates;        // [2][R][KP] each
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int K = L.K, p = a.p, nchunk = (p + R - 1) / R;
    double w[LPL], lv[LPL];
    bool on[LPL];
#pragma unroll
    for (int i = 0; i < LPL; ++i) {
        const int k = lane + kWave * i;
        on[i] = k < K;
        w[i] = on[i] ? L.w[k] : 0.0;
        lv[i] = on[i] ? (double)L.lev[k] : 0.0;
        br[i] = on[i] ? 1.0 : 0.0;
        bi[i] = 0.0;
    }
    // phases e^{-i gamma l} and mixer factors of chunk c, by nw waves (w0: this wave's index among them)
    auto tables = [&](int c, int w0, int nw) {
        const int j0 = c * R, nr = min(R, p - j0);
        for (int r = w0; r < nr; r += nw)
#pragma unroll
            for (int i = 0; i < LPL; ++i)
                if (on[i]) {
                    double s, cs;
                    sincos(gamma[j0 + r] * lv[i], &s, &cs);
                    const bool in = lv[i] <= (double)a.m;
                    ph[((c & 1) * R + r) * KP + lane + kWave * i] = in ? double2{cs, -s} : double2{0.0, 0.0};
                }
        if (w0 == nw - 1 && lane < nr) {
            double s, cs;
            sincos(beta[j0 + lane], &s, &cs);
            L.mix[c & 1][lane] = double2{cs - 1.0, -s};
        }
    };
    // readout of the state after round j (1-based) from amplitudes x
    auto readout = [&](int j, const double2 (&x)[LPL]) {
        double E = 0.0, N = 0.0;
        double *ro = a.readout + 3 * (size_t)j;
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            const double pb = on[i] ? w[i] * (x[i].x * x[i].x + x[i].y * x[i].y) : 0.0;
            N += pb;
            E += lv[i] * pb;
            if (lane + kWave * i == L.t_idx) ro[0] = pb;
        }
        E = wave_sum_dpp(E);
        N = wave_sum_dpp(N);
        if (lane == 0) {
            ro[1] = E;
            ro[2] = N;
            if (L.t_idx < 0) ro[0] = 0.0;
        }
    };
    if (nchunk > 0) tables(0, wave, kRunWaves);
    __syncthreads();
    for (int c = 0; c <= nchunk; ++c) {
        if (wave == 0) {
            if (c < nchunk) {
                const int nr = min(R, p - c * R);
                const double2 *e0 = ph + (c & 1) * R * KP + lane;
                double2 *o0 = bs + (c & 1) * R * KP + lane;
                double2 e[LPL], m = L.mix[c & 1][0];
#pragma unroll
                for (int i = 0; i < LPL; ++i) e[i] = on[i] ? e0[kWave * i] : double2{0.0, 0.0};
                for (int r = 0; r < nr; ++r) {
                    double sr = 0.0, si = 0.0;
#pragma unroll
                    for (int i = 0; i < LPL; ++i) {
                        const double nb = e[i].x * br[i] - e[i].y * bi[i];
                        bi[i] = e[i].x * bi[i] + e[i].y * br[i];
                        br[i] = nb;
                        sr += w[i] * br[i];
                        si += w[i] * bi[i];
                    }
                    const double2 mc = m;
                    const int rn = min(r + 1, nr - 1);  // the next round's table, loaded under the sums
#pragma unroll
                    for (int i = 0; i < LPL; ++i) e[i] = on[i] ? e0[rn * KP + kWave * i] : double2{0.0, 0.0};
                    m = L.mix[c & 1][rn];
                    sr = wave_sum_dpp(sr);
                    si = wave_sum_dpp(si);
                    const double dr = mc.x * sr - mc.y * si, di = mc.x * si + mc.y * sr;
#pragma unroll
                    for (int i = 0; i < LPL; ++i) {
                        br[i] += dr;
                        bi[i] += di;
                        o0[r * KP + kWave * i] = double2{br[i], bi[i]};
                    }
                }
            }
        } else {
            if (c + 1 < nchunk) tables(c + 1, wave - 1, kRunWaves - 1);
            if (c == 0) {
                if (wave == kRunWaves - 1) {
                    double2 one[LPL];
#pragma unroll
                    for (int i = 0; i < LPL; ++i) one[i] = double2{1.0, 0.0};
                    readout(0, one);
                }
            } else {
                const int j0 = (c - 1) * R, nr = min(R, p - j0);
                for (int r = wave - 1; r < nr; r += kRunWaves - 1) {
                    double2 x[LPL];
#pragma unroll
                    for (int i = 0; i < LPL; ++i) x[i] = bs[(((c - 1) & 1) * R + r) * KP + lane + kWave * i];
                    readout(j0 + r + 1, x);
                }
            }
        }
        __syncthreads();
    }
}

template <int LPL>
__device__ __forceinline__ void level_run(const LevelRunArgs &a, LevelLds &L, double2 *buf, const double *beta,
                                          const double *gamma, double2 *tab) {
    double br[LPL], bi[LPL];
    level_rounds<LPL>(a, L, buf, beta, gamma, br, bi);
    if (threadIdx.x < kWave) {
        const double amp = sqrt(ldexp(1.0, -a.n));
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            const int k = threadIdx.x + kWave * i;
            if (k < L.K) tab[L.lev[k]] = double2{amp * br[i], amp * bi[i]};
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void put(double2 x, double2 *p) {
    __builtin_nontemporal_store(f64x2{x.x, x.y}, reinterpret_cast<f64x2 *>(p));
}

// FUSED: the whole evolution of one small state in this block (counts, rounds,
// final state). Otherwise: counts from the counting launch's rows, and the
// final table to a.table for the expansion.
template <bool FUSED, int INLINE>
__global__ void __launch_bounds__(kRunThreads) level_run_kernel(LevelRunArgs a, LevelAngles<INLINE> in) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kCountBytes];  // counters, then the chunk buffers
    __shared__ LevelLds L;
    __shared__ double2 tab[kLevels];
    static_assert(4 * kChunkStates * sizeof(double2) <= kCountBytes, "chunk buffers");
    const int t = threadIdx.x;
    if (t < kLevels) tab[t] = double2{0.0, 0.0};
    if constexpr (INLINE > 1)
        for (int i = t; i < 2 * a.p; i += kRunThreads) L.ang[i] = in.v[i];
    uint64_t count = 0;
    if constexpr (FUSED) {
        uint32_t *h = reinterpret_cast<uint32_t *>(smem);
        count_levels<kRunThreads>(a.cost, 1ull << a.n, 0, 1, h);
        if (t < kLevels) count = level_total(h, t);
    } else {
        uint64_t *half = reinterpret_cast<uint64_t *>(smem);
        const uint32_t *r = a.rows + (t & (kLevels - 1));
        int b = t / kLevels;
        constexpr int U = 16;  // rows in flight per thread: the sum is a few memory latencies long
        for (; b + (U - 1) * 2 < a.nrows; b += 2 * U) {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = r[(size_t)(b + 2 * u) * kLevels];
#pragma unroll
            for (int u = 0; u < U; ++u) count += v[u];
        }
        for (; b < a.nrows; b += 2) count += r[(size_t)b * kLevels];
        if (t >= kLevels) half[t - kLevels] = count;
        __syncthreads();
        if (t < kLevels) count += half[t];
    }
    compact_levels(L, count, a.n, a.target);  // its barriers also end the counters' use of smem
    const double *beta = INLINE > 1 ? L.ang : a.angles;
    const double *gamma = beta + a.p;
    double2 *buf = reinterpret_cast<double2 *>(smem);
    if (L.K <= kWave) level_run<1>(a, L, buf, beta, gamma, tab);
    else if (L.K <= 2 * kWave) level_run<2>(a, L, buf, beta, gamma, tab);
    else level_run<4>(a, L, buf, beta, gamma, tab);
    if constexpr (FUSED) {
        for (uint32_t z = t; z < (1u << a.n); z += kRunThreads) put(tab[a.cost[z]], a.psi + z);
    } else {
        if (t < kLevels) a.table[t] = tab[t];
    }
}

// psi[z] = table[C(z)]. Bound by the write of the state; each lane stores 16
// bytes per group, a wave 1 KiB of consecutive memory, nontemporal (n = 28:
// 4.3 GB written and 0.27 GB read in 0.84 ms, 5.4 TB/s).
constexpr int kExpThreads = 256, kExpU = 4;
__global__ void __launch_bounds__(kExpThreads) level_expand_kernel(const uint8_t *__restrict__ cost,
                                                                   const double2 *__restrict__ table, uint64_t N,
                                                                   double2 *__restrict__ psi) {
    __shared__ double2 tab[kLevels];
    tab[threadIdx.x] = table[threadIdx.x];
    __syncthreads();
    constexpr uint64_t kTile = (uint64_t)kExpThreads * kExpU;
    for (uint64_t base = blockIdx.x * kTile; base < N; base += gridDim.x * kTile) {
        uint8_t c[kExpU];  // N is a power of two and at least one tile
#pragma unroll
        for (int u = 0; u < kExpU; ++u) c[u] = cost[base + u * kExpThreads + threadIdx.x];
#pragma unroll
        for (int u = 0; u < kExpU; ++u) put(tab[c[u]], psi + base + u * kExpThreads + threadIdx.x);
    }
}
static_assert((2u << kLevelFusedMaxN) >= kExpThreads * kExpU, "one expansion tile");

template <bool FUSED>
static void launch_run(const LevelRunArgs &r, const LevelEvolve &e, bool inl, hipStream_t st) {
    if (inl) {
        LevelAngles<kLevelInlineRounds> in;
        std::copy(e.beta_host, e.beta_host + e.p, in.v);
        std::copy(e.gamma_host, e.gamma_host + e.p, in.v + e.p);
        hipLaunchKernelGGL((level_run_kernel<FUSED, kLevelInlineRounds>), dim3(1), dim3(kRunThreads), 0, st, r, in);
    } else {
        hipLaunchKernelGGL((level_run_kernel<FUSED, 1>), dim3(1), dim3(kRunThreads), 0, st, r, LevelAngles<1>{});
    }
}

int level_evolve(const LevelEvolve &e, bool captured, hipStream_t st) {
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    const bool inl = !captured && e.p <= kLevelInlineRounds;
    if (!captured && !inl) {
        GQ_HIP(hipMemcpyAsync(e.angles_dev, e.beta_host, 8 * (size_t)e.p, hipMemcpyHostToDevice, st));
        GQ_HIP(hipMemcpyAsync(e.angles_dev + e.p, e.gamma_host, 8 * (size_t)e.p, hipMemcpyHostToDevice, st));
    }
    double2 *psi = reinterpret_cast<double2 *>(e.psi), *table = reinterpret_cast<double2 *>(e.table);
    LevelRunArgs r{e.cost, e.rows, 0, e.n, e.m, e.p, e.target, inl ? nullptr : e.angles_dev, psi, table, e.readout};
    if (e.n <= kLevelFusedMaxN) {
        ProfScope ps("sv_resident_c128", st);
        launch_run<true>(r, e, inl, st);
        ps.end();
        GQ_LAUNCH_CHECK();
        return GQAOA_OK;
    }
    const uint64_t N = 1ull << e.n;
    r.nrows = (int)std::min<uint64_t>(kLevelMaxRows, std::max<uint64_t>(1, N / 16 / kCountThreads));
    hipLaunchKernelGGL(level_count_kernel, dim3(r.nrows, 1), dim3(kCountThreads), 0, st, e.cost, N, e.rows);
    GQ_LAUNCH_CHECK();
    launch_run<false>(r, e, inl, st);
    GQ_LAUNCH_CHECK();
    const unsigned blocks = (unsigned)std::min<uint64_t>(N / (kExpThreads * kExpU), (uint64_t)dev.num_cus * 64);
    hipLaunchKernelGGL(level_expand_kernel, dim3(blocks), dim3(kExpThreads), 0, st, e.cost, table, N, psi);
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

}  // namespace gqaoa
