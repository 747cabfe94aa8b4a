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
// A given state takes the same form. With a_k the mean of psi_0 over level k, the
// deviations psi_0(z) - a_{C(z)} sum to zero on every level, so they only rotate:
//     psi_j(z) = e^{-i Gamma_j k} (psi_0(z) - a_k) + 2^{-n/2} b_k(j),  k = C(z),
// with Gamma_j = gamma_1 + .. + gamma_j and the b_k above started from
// 2^{n/2} a_k. Level k holds the probability V_k + w_k |b_k|^2, V_k the sum of its
// squared deviations. One pass takes the level sums of psi_0 and |psi_0|^2, the
// recursion is the same, and one pass applies e^{-i Gamma_p k} x + l_k in place.
//
// The costs are counted from the table itself, so any table is taken as it
// is; entries above m (which the caller promises not to pass) get the phase
// factor 0 that the round passes' tables hold there, from |s> and from a given
// state. Their amplitudes are all the same after the first round, so the sums of
// a given state keep one slot m + 1 for all of them (none at m = 255).
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

// A given state's level means (times 2^{n/2}) and squared deviations, by compacted
// level; the slot above m holds the sum of |psi_0|^2 as its deviation, for round 0
// alone, and the mean of its levels.
struct GivenLds {
    double2 b0[kLevels];
    double var[kLevels];
    double lev[kLevels];
    double e_above, c_above;  // sums of C(z) |psi_0(z)|^2 and C(z) over the slot above m
    bool above;               // the slot is occupied
};

struct LevelRunArgs {
    const uint8_t *cost;
    const double *sums;    // given state: [slots][4] sums of re, im, |.|^2 and counts (level_sums_kernel)
    const uint32_t *rows;
    int nrows, n, m, p, target;
    const double *angles;  // device: beta[p], gamma[p]; null: the inline angles
    double2 *psi;
    double2 *table;
    double *readout;
};

// Slots of a given state's sums: levels 0..m and one for what is above.
__host__ __device__ constexpr int given_slots(int m) { return m < kLevels - 1 ? m + 2 : kLevels; }

template <int ROUNDS>
struct LevelAngles {
    double v[2 * ROUNDS];  // beta[p], gamma[p]
};

// Thread t < 256: the sum of column t of the counting blocks' rows (tmp: 256 words of LDS).
__device__ __forceinline__ uint64_t sum_rows(const uint32_t *rows, int nrows, uint64_t *tmp) {
    const int t = threadIdx.x;
    const uint32_t *r = rows + (t & (kLevels - 1));
    uint64_t count = 0;
    int b = t / kLevels;
    constexpr int U = 16;  // rows in flight per thread: the sum is a few memory latencies long
    for (; b + (U - 1) * 2 < nrows; b += 2 * U) {
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = r[(size_t)(b + 2 * u) * kLevels];
#pragma unroll
        for (int u = 0; u < U; ++u) count += v[u];
    }
    for (; b < nrows; b += 2) count += r[(size_t)b * kLevels];
    if (t >= kLevels) tmp[t - kLevels] = count;
    __syncthreads();
    if (t < kLevels) count += tmp[t];
    return count;
}
static_assert(kRunThreads == 2 * kLevels, "two threads per level");

// Compacts the occupied levels (thread t < 256 holds level t's count) into
// L.w / L.lev in level order and returns the level's place, -1 if it is not
// occupied; every thread of the block calls this.
__device__ __forceinline__ int compact_levels(LevelLds &L, uint64_t count, int n, int target) {
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
    const int pos = on ? base + __popcll(mask & ((1ull << lane) - 1ull)) : -1;
    if (on) {
        L.lev[pos] = t;
        L.w[pos] = ldexp((double)count, -n);  // exact: a count times a power of two
        if (t == target) L.t_idx = pos;
    }
    __syncthreads();
    return pos;
}

// All p rounds; returns in wave 0 the final amplitudes of its levels and, for
// a given state, the products e[] of its phases.
template <int LPL, bool GIVEN>
__device__ __forceinline__ void level_rounds(const LevelRunArgs &a, LevelLds &L, const GivenLds *G, double2 *buf,
                                             const double *beta, const double *gamma, double (&br)[LPL],
                                             double (&bi)[LPL], double2 (&ep)[LPL]) {
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
        if constexpr (GIVEN) {
            lv[i] = on[i] ? G->lev[k] : 0.0;
            br[i] = on[i] ? G->b0[k].x : 0.0;
            bi[i] = on[i] ? G->b0[k].y : 0.0;
        }
        ep[i] = double2{1.0, 0.0};
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
            double pb = on[i] ? w[i] * (x[i].x * x[i].x + x[i].y * x[i].y) : 0.0;
            if constexpr (GIVEN)
                if (on[i]) {
                    const bool above = lv[i] > (double)a.m;
                    if (!above || j == 0) pb += G->var[lane + kWave * i];
                    if (above && j == 0) E += G->e_above - lv[i] * pb;
                }
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
                        if constexpr (GIVEN)
                            ep[i] = double2{e[i].x * ep[i].x - e[i].y * ep[i].y, e[i].x * ep[i].y + e[i].y * ep[i].x};
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
                    double2 x[LPL];
#pragma unroll
                    for (int i = 0; i < LPL; ++i) x[i] = double2{br[i], bi[i]};
                    readout(0, x);
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

// tab: the final amplitude of each level; for a given state the pair
// (e^{-i Gamma k}, l_k = 2^{-n/2} (b_k(p) - e^{-i Gamma k} b_k(0))).
template <int LPL, bool GIVEN>
__device__ __forceinline__ void level_run(const LevelRunArgs &a, LevelLds &L, const GivenLds *G, double2 *buf,
                                          const double *beta, const double *gamma, double2 *tab) {
    double br[LPL], bi[LPL];
    double2 ep[LPL];
    level_rounds<LPL, GIVEN>(a, L, G, buf, beta, gamma, br, bi, ep);
    if (threadIdx.x < kWave) {
        const double amp = sqrt(ldexp(1.0, -a.n));
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            const int k = threadIdx.x + kWave * i;
            if (k >= L.K) continue;
            if constexpr (GIVEN) {
                const double2 b0 = G->b0[k], e = ep[i];
                tab[2 * L.lev[k]] = e;
                tab[2 * L.lev[k] + 1] = double2{amp * (br[i] - (e.x * b0.x - e.y * b0.y)),
                                                amp * (bi[i] - (e.x * b0.y + e.y * b0.x))};
            } else {
                tab[L.lev[k]] = double2{amp * br[i], amp * bi[i]};
            }
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void put(double2 x, double2 *p) {
    __builtin_nontemporal_store(f64x2{x.x, x.y}, reinterpret_cast<f64x2 *>(p));
}

// What a run starts from: kFused, |s>, the whole evolution of one small state in
// this block (counts, rounds, final state); kRows, |s> with the counts in the
// counting launch's rows; kGiven, the level sums of a given state. The latter
// two leave the final table in a.table.
enum LevelStart { kFused = 0, kRows = 1, kGiven = 2 };
template <int START, int INLINE>
__global__ void __launch_bounds__(kRunThreads) level_run_kernel(LevelRunArgs a, LevelAngles<INLINE> in) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kCountBytes];  // counters, then the chunk buffers
    __shared__ LevelLds L;
    constexpr bool GIVEN = START == kGiven;
    constexpr int kTab = GIVEN ? 2 : 1;
    __shared__ double2 tab[kTab * kLevels];
    __shared__ GivenLds given[1];
    const GivenLds *G = GIVEN ? given : nullptr;
    static_assert(4 * kChunkStates * sizeof(double2) <= kCountBytes, "chunk buffers");
    const int t = threadIdx.x;
    if (t < kTab * kLevels) tab[t] = double2{0.0, 0.0};
    if constexpr (INLINE > 1)
        for (int i = t; i < 2 * a.p; i += kRunThreads) L.ang[i] = in.v[i];
    uint64_t count = 0;
    double2 sum{0.0, 0.0};
    double sq = 0.0;
    if constexpr (GIVEN) {
        if (t < given_slots(a.m)) {
            sum = double2{a.sums[4 * t], a.sums[4 * t + 1]};
            sq = a.sums[4 * t + 2];
            count = (uint64_t)a.sums[4 * t + 3];
        }
        if (t == a.m + 1) given[0].above = count != 0;  // (read behind the barriers below)
    } else if constexpr (START == kFused) {
        uint32_t *h = reinterpret_cast<uint32_t *>(smem);
        count_levels<kRunThreads>(a.cost, 1ull << a.n, 0, 1, h);
        if (t < kLevels) count = level_total(h, t);
    } else {
        count = sum_rows(a.rows, a.nrows, reinterpret_cast<uint64_t *>(smem));
    }
    const int pos = compact_levels(L, count, a.n, a.target);  // its barriers also end the counters' use of smem
    if constexpr (GIVEN) {
        if (given[0].above) {
            // the table breaks its promise: this block reads it for the sums of the
            // levels above m, which the sums kernel has no time for (+8%)
            __shared__ double red[2 * kRunWaves];
            double v[2] = {0.0, 0.0};
            for (uint64_t z = t; z < 1ull << a.n; z += kRunThreads) {
                const int c = a.cost[z];
                if (c <= a.m) continue;
                const double2 x = a.psi[z];
                v[0] += (double)c * (x.x * x.x + x.y * x.y);
                v[1] += (double)c;
            }
            block_sum<2, kRunThreads>(v, red);
            if (t == 0) {
                given[0].e_above = v[0];
                given[0].c_above = v[1];
            }
            __syncthreads();
        }
        if (pos >= 0) {
            const double inv = 1.0 / (double)count, root = sqrt(ldexp(1.0, a.n));
            if (t <= a.m) {
                given[0].b0[pos] = double2{root * (sum.x * inv), root * (sum.y * inv)};
                given[0].var[pos] = fmax(sq - (sum.x * sum.x + sum.y * sum.y) * inv, 0.0);
                given[0].lev[pos] = (double)t;
            } else {
                given[0].b0[pos] = double2{0.0, 0.0};
                given[0].var[pos] = sq;
                given[0].lev[pos] = given[0].c_above * inv;
            }
        }
        __syncthreads();
    }
    const double *beta = INLINE > 1 ? L.ang : a.angles;
    const double *gamma = beta + a.p;
    double2 *buf = reinterpret_cast<double2 *>(smem);
    if (L.K <= kWave) level_run<1, GIVEN>(a, L, G, buf, beta, gamma, tab);
    else if (L.K <= 2 * kWave) level_run<2, GIVEN>(a, L, G, buf, beta, gamma, tab);
    else level_run<4, GIVEN>(a, L, G, buf, beta, gamma, tab);
    if constexpr (START == kFused) {
        for (uint32_t z = t; z < (1u << a.n); z += kRunThreads) put(tab[a.cost[z]], a.psi + z);
    } else {
        if (t < kTab * kLevels) a.table[t] = tab[t];
    }
}

// ---- level sums of a given state ------------------------------------------------------
// Sums of re, im, |psi|^2 and the count of every level, one row per block. A
// wave adds into tables of its own in LDS, [3][levels][C] doubles, C columns
// for its 64 lanes, which take turns: C lanes per add instruction, so no two
// lanes of an instruction share an address and a wave's adds to one address
// keep their order. The sums then do not depend on timing, and concentrated
// levels cost no conflicts. C is the largest of 16, 8 and 4 that fits the LDS
// of four waves (up to 99, 190 and 256 slots). Bound by the read of the state
// and by the LDS adds; each wave keeps its next 8 vectors' loads in flight (n =
// 22, m = 92: 22 us, 3.3 TB/s from the 64 MiB state).
constexpr int kSumThreads = 256, kSumWaves = kSumThreads / kWave, kSumU = 8;
static size_t level_sums_lds(int ns, int C) {
    return sizeof(double) * kSumWaves * 3 * (size_t)ns * C + sizeof(uint32_t) * (size_t)ns * 16;
}
static int level_sums_cols(int ns) {
    for (int C : {16, 8})
        if (level_sums_lds(ns, C) <= 155 * 1024) return C;
    return 4;
}

template <int C>
__global__ void __launch_bounds__(kSumThreads) level_sums_kernel(const uint8_t *__restrict__ cost,
                                                                 const double2 *__restrict__ psi, uint64_t N, int m,
                                                                 double *__restrict__ rows) {
    const int ns = given_slots(m);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_sums[];
    double *all = reinterpret_cast<double *>(smem_sums);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(all + (size_t)kSumWaves * 3 * ns * C);
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    for (int i = t; i < kSumWaves * 3 * ns * C; i += kSumThreads) all[i] = 0.0;
    for (int i = t; i < ns * 16; i += kSumThreads) cnt[i] = 0u;
    __syncthreads();
    double *mine = all + (size_t)wave * 3 * ns * C + lane % C;
    const int plane = ns * C;
    const uint64_t step = (uint64_t)gridDim.x * kSumWaves * kWave * kSumU;
    uint64_t base = ((uint64_t)blockIdx.x * kSumWaves + wave) * kWave * kSumU;
    double2 nx[kSumU];
    uint8_t nc[kSumU];
    auto load = [&](uint64_t b0) {
#pragma unroll
        for (int u = 0; u < kSumU; ++u) {
            const uint64_t z = b0 + (uint64_t)u * kWave + lane;
            if (z < N) {
                nc[u] = cost[z];
                const f64x2 v = __builtin_nontemporal_load(reinterpret_cast<const f64x2 *>(psi + z));
                nx[u] = double2{v.x, v.y};
            }
        }
    };
    if (base < N) load(base);
    for (; base < N; base += step) {
        double2 x[kSumU];
        int c[kSumU];
#pragma unroll
        for (int u = 0; u < kSumU; ++u) {
            x[u] = nx[u];
            c[u] = min((int)nc[u], ns - 1);
        }
        if (base + step < N) load(base + step);
#pragma unroll
        for (int u = 0; u < kSumU; ++u) {
            const bool ok = base + (uint64_t)u * kWave + lane < N;
            const double q = x[u].x * x[u].x + x[u].y * x[u].y;
            if (ok) atomicAdd(cnt + c[u] * 16 + (lane & 15), 1u);
            double *p = mine + c[u] * C;
#pragma unroll
            for (int g = 0; g < kWave / C; ++g) {
                if (ok && lane / C == g) {
                    (void)__hip_atomic_fetch_add(p, x[u].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    (void)__hip_atomic_fetch_add(p + plane, x[u].y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    (void)__hip_atomic_fetch_add(p + 2 * plane, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                asm volatile("" ::: "memory");  // the turns stay apart and in order
            }
        }
    }
    __syncthreads();
    double *row = rows + (size_t)blockIdx.x * kLevels * 4;
    for (int i = t; i < 4 * ns; i += kSumThreads) {
        const int l = i >> 2, v = i & 3;
        double s = 0.0;
        if (v < 3) {
            for (int w = 0; w < kSumWaves; ++w)
                for (int k = 0; k < C; ++k) s += all[((size_t)w * 3 + v) * plane + l * C + (k + l) % C];
        } else {
            uint32_t n = 0;
            for (int k = 0; k < 16; ++k) n += cnt[l * 16 + (k + l) % 16];
            s = (double)n;
        }
        row[i] = s;
    }
}

// Block l: the sums of slot l over at most 256 rows, in a fixed order.
__global__ void __launch_bounds__(kSumThreads) level_sums_fold_kernel(const double *__restrict__ rows, int nrows,
                                                                      double *__restrict__ sums) {
    __shared__ double red[4 * kSumWaves];
    const int l = blockIdx.x, t = threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (t < nrows)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = rows[((size_t)t * kLevels + l) * 4 + k];
    block_sum<4, kSumThreads>(v, red);
    if (t == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) sums[4 * l + k] = v[k];
}

// psi[z] <- e_k psi[z] + l_k, k = C(z) (or the slot above m), in place: one read
// and one write of the state (n = 22: 27 us, 5.1 TB/s).
constexpr int kApplyThreads = 256, kApplyU = 4;
__global__ void __launch_bounds__(kApplyThreads) level_apply_kernel(const uint8_t *__restrict__ cost,
                                                                    const double2 *__restrict__ table, uint64_t N,
                                                                    int ns, double2 *__restrict__ psi) {
    __shared__ double2 tab[2 * kLevels];
    tab[threadIdx.x] = table[threadIdx.x];
    tab[threadIdx.x + kLevels] = table[threadIdx.x + kLevels];
    __syncthreads();
    constexpr uint64_t kTile = (uint64_t)kApplyThreads * kApplyU;
    for (uint64_t base = blockIdx.x * kTile; base < N; base += gridDim.x * kTile) {
        f64x2 x[kApplyU];
        uint8_t c[kApplyU];
#pragma unroll
        for (int u = 0; u < kApplyU; ++u) {
            const uint64_t z = base + (uint64_t)u * kApplyThreads + threadIdx.x;
            if (z < N) {
                c[u] = cost[z];
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const f64x2 *>(psi + z));
            }
        }
#pragma unroll
        for (int u = 0; u < kApplyU; ++u) {
            const uint64_t z = base + (uint64_t)u * kApplyThreads + threadIdx.x;
            if (z >= N) continue;
            const int k = min((int)c[u], ns - 1);
            const double2 e = tab[2 * k], l = tab[2 * k + 1];
            put(double2{e.x * x[u].x - e.y * x[u].y + l.x, e.x * x[u].y + e.y * x[u].x + l.y}, psi + z);
        }
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

template <int START>
static void launch_run(const LevelRunArgs &r, const LevelEvolve &e, bool inl, hipStream_t st) {
    if (inl) {
        LevelAngles<kLevelInlineRounds> in;
        std::copy(e.beta_host, e.beta_host + e.p, in.v);
        std::copy(e.gamma_host, e.gamma_host + e.p, in.v + e.p);
        hipLaunchKernelGGL((level_run_kernel<START, kLevelInlineRounds>), dim3(1), dim3(kRunThreads), 0, st, r, in);
    } else {
        hipLaunchKernelGGL((level_run_kernel<START, 1>), dim3(1), dim3(kRunThreads), 0, st, r, LevelAngles<1>{});
    }
}

int level_evolve(const LevelEvolve &e, hipStream_t st) {
    DeviceInfo dev;
    int s = device_info(&dev);
    if (s) return s;
    const bool inl = e.p <= kLevelInlineRounds;
    if (!inl) {
        GQ_HIP(hipMemcpyAsync(e.angles_dev, e.beta_host, 8 * (size_t)e.p, hipMemcpyHostToDevice, st));
        GQ_HIP(hipMemcpyAsync(e.angles_dev + e.p, e.gamma_host, 8 * (size_t)e.p, hipMemcpyHostToDevice, st));
    }
    double2 *psi = reinterpret_cast<double2 *>(e.psi), *table = reinterpret_cast<double2 *>(e.table);
    const uint64_t N = 1ull << e.n;
    double *sums = reinterpret_cast<double *>(e.rows), *sum_rows = sums + 4 * kLevels;
    uint32_t *rows = reinterpret_cast<uint32_t *>(e.rows);
    LevelRunArgs r{e.cost, sums, rows, 0, e.n, e.m, e.p, e.target, inl ? nullptr : e.angles_dev, psi, table, e.readout};
    if (!e.init_uniform) {
        ProfScope ps("level_evolve", st);
        const int ns = given_slots(e.m);
        const unsigned blocks =
            (unsigned)std::min<uint64_t>(kLevelMaxRows, std::max<uint64_t>(1, N / (kSumThreads * kSumU)));
        const int C = level_sums_cols(ns);
        const size_t lds = level_sums_lds(ns, C);
        if (lds > dev.lds_per_block) return fail(GQAOA_EINVAL, "internal: level sums need %zu bytes of LDS", lds);
        const auto fn = C == 16 ? level_sums_kernel<16> : C == 8 ? level_sums_kernel<8> : level_sums_kernel<4>;
        hipLaunchKernelGGL(fn, dim3(blocks), dim3(kSumThreads), lds, st, e.cost, psi, N, e.m, sum_rows);
        GQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(level_sums_fold_kernel, dim3(ns), dim3(kSumThreads), 0, st, sum_rows, (int)blocks, sums);
        GQ_LAUNCH_CHECK();
        launch_run<kGiven>(r, e, inl, st);
        GQ_LAUNCH_CHECK();
        const unsigned ab = (unsigned)std::min<uint64_t>(
            std::max<uint64_t>(1, N / (kApplyThreads * kApplyU)), (uint64_t)dev.num_cus * 1024);
        hipLaunchKernelGGL(level_apply_kernel, dim3(ab), dim3(kApplyThreads), 0, st, e.cost, table, N, ns, psi);
        GQ_LAUNCH_CHECK();
        ps.end();
        return GQAOA_OK;
    }
    if (e.n <= kLevelFusedMaxN) {
        ProfScope ps("sv_resident_c128", st);
        launch_run<kFused>(r, e, inl, st);
        ps.end();
        GQ_LAUNCH_CHECK();
        return GQAOA_OK;
    }
    ProfScope ps("level_evolve", st);
    r.nrows = (int)std::min<uint64_t>(kLevelMaxRows, std::max<uint64_t>(1, N / 16 / kCountThreads));
    hipLaunchKernelGGL(level_count_kernel, dim3(r.nrows, 1), dim3(kCountThreads), 0, st, e.cost, N, rows);
    GQ_LAUNCH_CHECK();
    launch_run<kRows>(r, e, inl, st);
    GQ_LAUNCH_CHECK();
    const unsigned blocks = (unsigned)std::min<uint64_t>(N / (kExpThreads * kExpU), (uint64_t)dev.num_cus * 64);
    hipLaunchKernelGGL(level_expand_kernel, dim3(blocks), dim3(kExpThreads), 0, st, e.cost, table, N, psi);
    GQ_LAUNCH_CHECK();
    ps.end();
    return GQAOA_OK;
}

// ---- adjoint gradient -----------------------------------------------------------------
// The reverse sweep of the adjoint gradient in the level space, one block per
// instance, split as the rounds above: wave 0 carries the amplitudes, the
// other waves compute the tables of the next chunk and sum the dgamma terms of
// the chunk before. Forward: phi_k = e^{-i gamma_k l} psi_{k-1}, S_k = sum_l w_l
// phi_l, psi_k = phi_k + (e^{-i beta_k} - 1) S_k. Reverse, from lambda_p = Pi_t psi_p:
//   s = sum_l w_l lambda_l,  mu = lambda + (e^{+i beta_k} - 1) s
//   dP/dbeta_k  = 2 Re(-i e^{-i beta_k} conj(s) S_k)
//   dP/dgamma_k = 2 sum_l w_l l Im(conj(mu_l) phi_l)
//   lambda <- e^{+i gamma_k l} mu.
// The forward states are not stored: phi_k = psi_k - (e^{-i beta_k} - 1) S_k
// with the S_k of the forward sweep (kept in the gradient arrays until round
// k's entries replace them), psi_{k-1} = e^{+i gamma_k l} phi_k. So the serial
// chain is one pair of wave sums per round in each direction: 0.56 us per round
// for both (200 instances, p = 100: 56 us, where one wave per instance doing
// everything by itself took 182 us). 128 registers keep two blocks on a CU
// (512 instances, p = 100: 260 us a call against 307 us with 168 registers and
// one block; one wave per instance 374 us; from 2048 instances on the two
// splits meet, so there is one kernel for all).
struct LevelGradRun {
    LevelGrad g;
    int nrows;
};

struct GradLds {
    double2 S[2][16];  // S_k of the chunk in reverse and of the next one
};

template <int LPL>
__device__ __forceinline__ void level_grad_rounds(LevelLds &L, GradLds &G, double2 *ph, double *qb, int m, int p,
                                                  const double *beta, const double *gamma, double *db, double *dg,
                                                  double *psol) {
    constexpr int KP = kWave * LPL, R = kChunkStates / KP;  // R = 16, 8, 4 rounds per chunk
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int K = L.K, nchunk = (p + R - 1) / R;
    double w[LPL], lv[LPL], br[LPL], bi[LPL];
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
    auto tables = [&](int c, int w0, int nw, bool sums) {
        const int j0 = c * R, nr = min(R, p - j0);
        for (int r = w0; r < nr; r += nw)
#pragma unroll
            for (int i = 0; i < LPL; ++i)
                if (on[i]) {
                    double s, cs;
                    sincos(gamma[j0 + r] * lv[i], &s, &cs);
                    const bool in = lv[i] <= (double)m;
                    ph[((c & 1) * R + r) * KP + lane + kWave * i] = in ? double2{cs, -s} : double2{0.0, 0.0};
                }
        if (w0 == nw - 1 && lane < nr) {
            double s, cs;
            sincos(beta[j0 + lane], &s, &cs);
            L.mix[c & 1][lane] = double2{cs - 1.0, -s};
            if (sums) G.S[c & 1][lane] = double2{db[j0 + lane], dg[j0 + lane]};
        }
    };
    tables(0, wave, kRunWaves, false);
    __syncthreads();
    for (int c = 0; c < nchunk; ++c) {
        if (wave == 0) {
            const int j0 = c * R, nr = min(R, p - j0);
            const double2 *e0 = ph + (c & 1) * R * KP + lane;
            double2 e[LPL], mx = L.mix[c & 1][0];
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
                const double2 mc = mx;
                const int rn = min(r + 1, nr - 1);
#pragma unroll
                for (int i = 0; i < LPL; ++i) e[i] = on[i] ? e0[rn * KP + kWave * i] : double2{0.0, 0.0};
                mx = L.mix[c & 1][rn];
                sr = wave_sum_dpp(sr);
                si = wave_sum_dpp(si);
                if (lane == 0) {
                    db[j0 + r] = sr;
                    dg[j0 + r] = si;
                }
                const double dr = mc.x * sr - mc.y * si, di = mc.x * si + mc.y * sr;
#pragma unroll
                for (int i = 0; i < LPL; ++i) {
                    br[i] += dr;
                    bi[i] += di;
                }
            }
        } else if (c + 1 < nchunk) {
            tables(c + 1, wave - 1, kRunWaves - 1, false);
        }
        __syncthreads();
    }
    // P, lambda_p, and the last chunk's S (its phases and factors are still in place)
    double lr[LPL], li[LPL];
    if (wave == 0) {
        double P = 0.0;
#pragma unroll
        for (int i = 0; i < LPL; ++i) {
            const bool t = lane + kWave * i == L.t_idx;
            lr[i] = t ? br[i] : 0.0;
            li[i] = t ? bi[i] : 0.0;
            P += t ? w[i] * (br[i] * br[i] + bi[i] * bi[i]) : 0.0;
        }
        P = wave_sum_dpp(P);
        if (lane == 0) *psol = P;
    } else if (wave == 1) {
        const int j0 = (nchunk - 1) * R;
        if (lane < p - j0) G.S[(nchunk - 1) & 1][lane] = double2{db[j0 + lane], dg[j0 + lane]};
    }
    __syncthreads();
    for (int c = nchunk - 1; c >= -1; --c) {
        if (wave == 0) {
            if (c >= 0) {
                const int j0 = c * R, nr = min(R, p - j0);
                const double2 *e0 = ph + (c & 1) * R * KP + lane;
                double *q0 = qb + (c & 1) * R * kWave + lane;
                double2 e[LPL], mx = L.mix[c & 1][nr - 1], S = G.S[c & 1][nr - 1];
#pragma unroll
                for (int i = 0; i < LPL; ++i) e[i] = on[i] ? e0[(nr - 1) * KP + kWave * i] : double2{0.0, 0.0};
                for (int r = nr - 1; r >= 0; --r) {
                    double sr = 0.0, si = 0.0;
#pragma unroll
                    for (int i = 0; i < LPL; ++i) {
                        sr += w[i] * lr[i];
                        si += w[i] * li[i];
                    }
                    const double2 mc = mx, Sc = S;
                    double2 ec[LPL];
                    const int rn = max(r - 1, 0);
#pragma unroll
                    for (int i = 0; i < LPL; ++i) {
                        ec[i] = e[i];
                        e[i] = on[i] ? e0[rn * KP + kWave * i] : double2{0.0, 0.0};
                    }
                    mx = L.mix[c & 1][rn];
                    S = G.S[c & 1][rn];
                    const double dr = mc.x * Sc.x - mc.y * Sc.y, di = mc.x * Sc.y + mc.y * Sc.x;
                    sr = wave_sum_dpp(sr);
                    si = wave_sum_dpp(si);
                    // (e^{+i beta} - 1) s
                    const double ur = mc.x * sr + mc.y * si, ui = mc.x * si - mc.y * sr;
                    double q = 0.0;
#pragma unroll
                    for (int i = 0; i < LPL; ++i) {
                        const double fr = br[i] - dr, fi = bi[i] - di;   // phi
                        const double ar = lr[i] + ur, ai = li[i] + ui;   // mu
                        q += w[i] * lv[i] * (ar * fi - ai * fr);
                        // times e^{+i gamma l} = conj(ec)
                        br[i] = ec[i].x * fr + ec[i].y * fi;
                        bi[i] = ec[i].x * fi - ec[i].y * fr;
                        lr[i] = ec[i].x * ar + ec[i].y * ai;
                        li[i] = ec[i].x * ai - ec[i].y * ar;
                    }
                    q0[r * kWave] = q;
                    // conj(s) S, times -i e^{-i beta} = (-sin beta, -cos beta)
                    const double zr = sr * Sc.x + si * Sc.y, zi = sr * Sc.y - si * Sc.x;
                    if (lane == 0) db[j0 + r] = 2.0 * (mc.y * zr + (mc.x + 1.0) * zi);
                }
            }
        } else {
            if (c > 0) tables(c - 1, wave - 1, kRunWaves - 1, true);
            if (c + 1 < nchunk) {
                const int j0 = (c + 1) * R, nr = min(R, p - j0);
                for (int r = wave - 1; r < nr; r += kRunWaves - 1) {
                    const double q = wave_sum_dpp(qb[(((c + 1) & 1) * R + r) * kWave + lane]);
                    if (lane == 0) dg[j0 + r] = 2.0 * q;
                }
            }
        }
        __syncthreads();
    }
}

enum LevelSource { kFromCosts = 0, kFromRows = 1, kCompacted = 2 };

template <int SRC>
__global__ void __launch_bounds__(kRunThreads, 4) level_grad_kernel(LevelGradRun a) {
    constexpr size_t kWork = 2 * kChunkStates * sizeof(double2) + 2 * 16 * kWave * sizeof(double);
    __shared__ __attribute__((aligned(16))) unsigned char smem[SRC == kFromCosts ? kCountBytes : kWork];
    static_assert(kWork <= kCountBytes, "chunk buffers");
    __shared__ LevelLds L;
    __shared__ GradLds G;
    const LevelGrad &g = a.g;
    const int t = threadIdx.x;
    int inst = blockIdx.x, p = g.pstride, m = kLevels;
    if constexpr (SRC == kCompacted) {
        const HistGradSlot sl = g.slots[blockIdx.x];
        inst = sl.inst;
        p = sl.p;
        for (int k = t; k < sl.K; k += kRunThreads) {
            L.lev[k] = g.lev[sl.lev_off + k];
            L.w[k] = g.w[sl.lev_off + k];
        }
        if (t == 0) {
            L.K = sl.K;
            L.t_idx = sl.t_idx;
        }
        __syncthreads();
    } else {
        uint64_t count = 0;
        if constexpr (SRC == kFromCosts) {
            uint32_t *h = reinterpret_cast<uint32_t *>(smem);
            count_levels<kRunThreads>(g.cost + ((uint64_t)inst << g.n), 1ull << g.n, 0, 1, h);
            if (t < kLevels) count = level_total(h, t);
        } else {
            count = sum_rows(g.rows + (size_t)inst * a.nrows * kLevels, a.nrows, reinterpret_cast<uint64_t *>(smem));
        }
        m = g.m[inst];
        compact_levels(L, count, g.n, g.target[inst]);
    }
    double2 *ph = reinterpret_cast<double2 *>(smem);
    double *qb = reinterpret_cast<double *>(ph + 2 * kChunkStates);
    const size_t o = (size_t)inst * g.pstride;
    double *db = g.dbeta + o, *dg = g.dgamma + o;
    if (L.K <= kWave) level_grad_rounds<1>(L, G, ph, qb, m, p, g.beta + o, g.gamma + o, db, dg, g.psol + inst);
    else if (L.K <= 2 * kWave) level_grad_rounds<2>(L, G, ph, qb, m, p, g.beta + o, g.gamma + o, db, dg, g.psol + inst);
    else level_grad_rounds<4>(L, G, ph, qb, m, p, g.beta + o, g.gamma + o, db, dg, g.psol + inst);
    for (int r = p + t; r < g.pstride; r += kRunThreads) db[r] = dg[r] = 0.0;  // rounds beyond this instance's p
}

int level_grad(const LevelGrad &g, hipStream_t st) {
    LevelGradRun a{g, 0};
    const dim3 grid(g.num_inst), block(kRunThreads);
    if (!g.cost) {
        hipLaunchKernelGGL(level_grad_kernel<kCompacted>, grid, block, 0, st, a);
    } else if (g.n <= kLevelFusedMaxN) {
        hipLaunchKernelGGL(level_grad_kernel<kFromCosts>, grid, block, 0, st, a);
    } else {
        // counting blocks: two per CU over the batch while each has 16 KiB to read
        DeviceInfo dev;
        int s = device_info(&dev);
        if (s) return s;
        const uint64_t N = 1ull << g.n;
        const int want = std::max(1, 2 * dev.num_cus / g.num_inst);
        a.nrows = (int)std::min<uint64_t>(std::min(want, std::min(g.row_cap, kLevelMaxRows)), N / 16 / kCountThreads);
        hipLaunchKernelGGL(level_count_kernel, dim3(a.nrows, g.num_inst), dim3(kCountThreads), 0, st, g.cost, N,
                           g.rows);
        GQ_LAUNCH_CHECK();
        hipLaunchKernelGGL(level_grad_kernel<kFromRows>, grid, block, 0, st, a);
    }
    GQ_LAUNCH_CHECK();
    return GQAOA_OK;
}

}  // namespace gqaoa
