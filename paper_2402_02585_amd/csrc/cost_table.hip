// Cost table C(z) and level histogram N_k by bit-sliced clause evaluation.
//
// C(z) is the number of clauses left unsatisfied by assignment z, i.e. the
// diagonal of H_P (Sec. II.A, the clause energy that follows Eq. (1); App. B).
// N_k = #{z : C(z) = k} is the per-level state count of App. C. The word
// layout and clause records are described in cost_bits.h.
//
// Each lane evaluates one 32-assignment word per tile. The clauses whose mask
// varies over word bits and lanes (class A) are tested against the tile's high
// bits 64 at a time; the active ones are compacted into wave-private LDS and
// folded, 16 at a time, into bit planes by a carry-save adder tree (one LDS
// broadcast, a bit extract and an AND per clause). The other classes' sums are
// the same along lanes or word bits: a wave forms them for up to 64 tiles at
// once, one tile per lane, and each tile reads its own back as scalars (the
// starting planes of the adder tree, and lane masks added at its end).
// Three 8x8 bit transposes turn the planes into byte costs. The histogram is
// counted from the planes and written as per-block rows, which a second kernel
// sums in a fixed order.
#include "internal.h"
#include "cost_bits.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

namespace gqaoa {

constexpr int kCostThreads = 256;
constexpr int kCostWaves = kCostThreads / kWave;
// LDS histogram copies per block: four per wave (by lane & 3). Copies are
// kHistStride = 257 words apart, so one level in different copies falls in
// different LDS banks: lanes of different copies tallying the same level
// neither share an address nor a bank.
constexpr int kHistCopies = kCostWaves * 4;
constexpr int kHistStride = 257;

// A clause's masks as each half-wave reads them: entry [c][h] = {P, bits
// 32h..32h+31 of L}.
struct EffEntry {
    uint32_t P, Lhalf;
};

// Dynamic LDS of a cost block: clause records, per-wave entries of the active
// clauses [waves][neff][2], and the histogram copies [copies][kHistStride].
struct CostLds {
    EffEntry *eff;
    ClauseRec *rec;
    uint32_t *hist;
    __device__ CostLds(unsigned char *smem, int neff)
        : eff(reinterpret_cast<EffEntry *>(smem)),
          rec(reinterpret_cast<ClauseRec *>(smem + sizeof(EffEntry) * 2 * kCostWaves * neff)),
          hist(reinterpret_cast<uint32_t *>(smem + sizeof(EffEntry) * 2 * kCostWaves * neff +
                                            sizeof(ClauseRec) * kMaxRecs)) {}
    __device__ EffEntry (*wave_eff(int neff))[2] {
        return reinterpret_cast<EffEntry(*)[2]>(eff + (size_t)2 * neff * (threadIdx.x / kWave));
    }
};

// Entries a wave may hold: every clause of the classes it evaluates per tile.
static inline int eff_entries(int m) { return (m + kHalfGroup - 1) / kHalfGroup * kHalfGroup; }

size_t cost_lds_bytes(int m) {
    return sizeof(EffEntry) * 2 * kCostWaves * eff_entries(m) + sizeof(ClauseRec) * kMaxRecs +
           sizeof(uint32_t) * kHistCopies * kHistStride;
}

__device__ __forceinline__ uint32_t *wave_copies(CostLds &s) {
    return s.hist + (threadIdx.x / kWave) * 4 * kHistStride;
}
__device__ __forceinline__ uint32_t *hist_copy(CostLds &s) { return wave_copies(s) + (threadIdx.x & 3) * kHistStride; }

// Sums of classes B, C and D for up to 64 tiles, lane t holding tile tile0 + t:
// b: bit planes over the word bits of B's sum plus D's count; c[0], c[1]: bit
// planes over lanes 0..31 and 32..63 of C's sum.
struct TileSums {
    uint32_t b[8], c[2][8];
};

__device__ __forceinline__ void tile_sums(const ClauseRec *rec, const ClauseCounts &n, uint32_t tile0, TileSums &s) {
    const uint32_t tile = tile0 + (threadIdx.x & (kWave - 1));
    SlicedCounter sb;
    sb.clear();
    for (int g = 0; g < n.n[kClassB]; g += kHalfGroup) {
        uint32_t f[kHalfGroup];
#pragma unroll
        for (int i = 0; i < kHalfGroup; ++i) {
            const ClauseRec &r = rec[n.first[kClassB] + g + i];
            f[i] = high_literals_false(tile, r.hv, r.hn) ? r.P : 0u;
        }
        sb.add8(f);
    }
    uint32_t u = 0;
    for (int g = 0; g < n.n[kClassD]; ++g) {
        const ClauseRec &r = rec[n.first[kClassD] + g];
        u += high_literals_false(tile, r.hv, r.hn) ? 1u : 0u;
    }
    sb.add_scalar(u);
#pragma unroll
    for (int b = 0; b < 8; ++b) s.b[b] = sb.p[b];
    SlicedCounter lo, hi;
    lo.clear();
    hi.clear();
    for (int g = 0; g < n.n[kClassC]; g += kHalfGroup) {
        uint32_t fl[kHalfGroup], fh[kHalfGroup];
#pragma unroll
        for (int i = 0; i < kHalfGroup; ++i) {
            const ClauseRec &r = rec[n.first[kClassC] + g + i];
            const uint64_t L = high_literals_false(tile, r.hv, r.hn) ? r.L : 0ull;
            fl[i] = (uint32_t)L;
            fh[i] = (uint32_t)(L >> 32);
        }
        lo.add8(fl);
        hi.add8(fh);
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        s.c[0][b] = lo.p[b];
        s.c[1][b] = hi.p[b];
    }
}

// Costs of the 32 assignments of word w = tile*64 + lane as bit planes: bit j
// of v[b] is bit b of C(z) for the assignment at word bit j. Every lane of the
// wave must call this with the same tile. SUMS: the sums of classes B, C and D
// come from s (lane `slot`); otherwise their clauses are evaluated with class
// A's (they follow it in rec).
template <bool SUMS>
__device__ __forceinline__ void eval_planes(const ClauseRec *rec, const ClauseCounts &n, uint32_t tile,
                                            const TileSums &s, int slot, EffEntry (*eff)[2], uint32_t (&v)[8]) {
    const int lane = threadIdx.x & (kWave - 1);
    const int ncand = SUMS ? n.n[kClassA] : n.first[kClassD];
    // 1) the active clauses, compacted
    int active = 0;
    for (int c0 = 0; c0 < ncand; c0 += kWave) {
        const int c = c0 + lane;
        ClauseRec r{0u, 0u, 0u, 0u, 0ull};
        if (c < ncand) r = rec[c];
        const bool on = r.P != 0u && r.L != 0ull && high_literals_false(tile, r.hv, r.hn);
        const uint64_t mask = __ballot(on);
        if (on) {
            const int at = active + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            eff[at][0] = EffEntry{r.P, (uint32_t)r.L};
            eff[at][1] = EffEntry{r.P, (uint32_t)(r.L >> 32)};
        }
        active += __popcll(mask);
    }
    const int padded = (active + kHalfGroup - 1) & ~(kHalfGroup - 1);
    if (lane < padded - active) {
        eff[active + lane][0] = EffEntry{0u, 0u};
        eff[active + lane][1] = EffEntry{0u, 0u};
    }
    SlicedCounter cnt;
    uint32_t u = 0;
    if constexpr (SUMS) {
#pragma unroll
        for (int b = 0; b < 8; ++b) cnt.p[b] = __builtin_amdgcn_readlane(s.b[b], slot);
    } else {
        cnt.clear();
        for (int c0 = 0; c0 < n.n[kClassD]; c0 += kWave) {
            const int c = n.first[kClassD] + c0 + lane;
            const bool f = c0 + lane < n.n[kClassD] && high_literals_false(tile, rec[c].hv, rec[c].hn);
            u += (uint32_t)__popcll(__ballot(f));
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // 2) per active clause: the lane's bit of L selects P; 16 (then 8) clauses per adder tree
    const int half = lane >> 5, bit = lane & 31;
    int g = 0;
    for (; g + kGroup <= padded; g += kGroup) {
        uint32_t f[kGroup];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
            const EffEntry e = eff[g + i][half];
            f[i] = e.P & (uint32_t)__builtin_amdgcn_sbfe((int)e.Lhalf, bit, 1);
        }
        cnt.add16(f);
    }
    if (g < padded) {
        uint32_t f[kHalfGroup];
#pragma unroll
        for (int i = 0; i < kHalfGroup; ++i) {
            const EffEntry e = eff[g + i][half];
            f[i] = e.P & (uint32_t)__builtin_amdgcn_sbfe((int)e.Lhalf, bit, 1);
        }
        cnt.add8(f);
    }
    // 3) no overflow: every count <= m <= 255
    if constexpr (SUMS) {
        uint32_t carry = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t lanes = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(s.c[1][b], slot) << 32 |
                                   (uint32_t)__builtin_amdgcn_readlane(s.c[0][b], slot);
            const uint32_t add = __builtin_amdgcn_inverse_ballot_w64(lanes) ? 0xFFFFFFFFu : 0u;
            uint32_t c;
            csa(c, v[b], cnt.p[b], add, carry);
            carry = c;
        }
    } else {
        cnt.add_scalar(u);
#pragma unroll
        for (int b = 0; b < 8; ++b) v[b] = cnt.p[b];
    }
    // the next tile rewrites eff: every lane's reads of this one come first
    __builtin_amdgcn_wave_barrier();
}

// Planes to bytes: out[r] byte q = C of word bit 8q + r, i.e. C(32 w + 4 r + q).
__device__ __forceinline__ void planes_to_bytes(const uint32_t (&v)[8], uint32_t (&out)[8]) {
    SlicedCounter c;
#pragma unroll
    for (int b = 0; b < 8; ++b) c.p[b] = v[b];
    c.transpose_to_bytes();
#pragma unroll
    for (int r = 0; r < 8; ++r) out[r] = c.p[r];
}

// Per-lane level counters for NB aligned blocks of 32 levels starting at
// level 32 a0, fed straight from the bit planes. A block's word bits are those
// where planes 5..7 spell a; cnt[S] counts the ones where the planes of the
// set S (of 0..4) are all set, one AND and one popcount a set, and the level
// counts follow by inclusion and exclusion once, at the flush. That is 58
// instructions a block where a mask for each level takes 80, and the sets of
// plane 4 (levels 16..31), or of planes 3 and 4 (24..31), are skipped where no
// lane has them. Levels outside the window are returned as a word-bit mask for
// the caller.
template <int NB>
struct LevelWindow {
    uint32_t cnt[NB][32];
    int a0;
    __device__ __forceinline__ void clear(int a) {
        a0 = a;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int k = 0; k < 32; ++k) cnt[i][k] = 0;
    }
    __device__ __forceinline__ uint32_t add(const uint32_t (&v)[8]) {
        uint32_t in = 0;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int a = a0 + i;  // uniform
            const uint32_t hi = (v[5] ^ ((a & 1) ? 0u : ~0u)) & (v[6] ^ ((a & 2) ? 0u : ~0u)) &
                                (v[7] ^ ((a & 4) ? 0u : ~0u));
            in |= hi;
            uint32_t p[16];  // p[S]: the planes of S and hi
            p[0] = hi;
#pragma unroll
            for (int s = 1; s < 16; ++s) {
                const int top = s >= 8 ? 3 : s >= 4 ? 2 : s >= 2 ? 1 : 0, rest = s ^ (1 << top);
                p[s] = v[top] & p[rest];
            }
#pragma unroll
            for (int s = 0; s < 16; ++s) cnt[i][s] += (uint32_t)__builtin_popcount(p[s]);
            if (__ballot((v[4] & hi) != 0u) == 0) continue;
#pragma unroll
            for (int s = 0; s < 8; ++s) cnt[i][16 + s] += (uint32_t)__builtin_popcount(v[4] & p[s]);
            if (__ballot((v[4] & p[8]) != 0u) == 0) continue;
#pragma unroll
            for (int s = 8; s < 16; ++s) cnt[i][16 + s] += (uint32_t)__builtin_popcount(v[4] & p[s]);
        }
        return ~in;
    }
    // Add the counters into an LDS histogram (levels < 256): summed over each
    // row of 16 lanes first (DPP shifts), so a level costs four LDS adds to four
    // copies instead of 64 to 4. Every lane of the wave calls this.
    __device__ __forceinline__ void flush(uint32_t *h) const {
        const int lane = threadIdx.x & (kWave - 1);
        uint32_t *copy = h + (lane >> 4) * kHistStride;  // h: the wave's first copy
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            uint32_t lev[32];  // sets to levels: exactly S = S less S and one more plane
#pragma unroll
            for (int k = 0; k < 32; ++k) lev[k] = cnt[i][k];
#pragma unroll
            for (int b = 0; b < 5; ++b)
#pragma unroll
                for (int k = 0; k < 32; ++k)
                    if (!((k >> b) & 1)) lev[k] -= lev[k | (1 << b)];
#pragma unroll
            for (int k = 0; k < 32; ++k) {
                if (a0 + i >= 8 || __ballot(lev[k] != 0u) == 0) continue;
                int s = (int)lev[k];
                s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, true);  // row_shr:1
                s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, true);  // row_shr:2
                s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, true);  // row_shr:4
                s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, true);  // row_shr:8
                if ((lane & 15) == 15) atomicAdd(copy + 32 * (a0 + i) + k, (uint32_t)s);
            }
        }
    }
};

// Tally the word bits of `mask` one by one from the cost bytes (the rare
// levels outside the window).
__device__ __forceinline__ void tally_bits(uint32_t *h, const uint32_t (&t)[8], uint32_t mask) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((mask >> (8 * q + r)) & 1u) atomicAdd(h + ((t[r] >> (8 * q)) & 0xFFu), 1u);
}

__device__ __forceinline__ void tally(uint32_t *h, uint32_t v) {
    atomicAdd(h + (v & 0xFFu), 1u);
    atomicAdd(h + ((v >> 8) & 0xFFu), 1u);
    atomicAdd(h + ((v >> 16) & 0xFFu), 1u);
    atomicAdd(h + (v >> 24), 1u);
}

__device__ __forceinline__ void tally_word(uint32_t *h, const uint32_t (&t)[8], uint32_t nbits) {
    if (nbits == 32u) {
#pragma unroll
        for (int r = 0; r < 8; ++r) tally(h, t[r]);
    } else {
        for (uint32_t z = 0; z < nbits; ++z) atomicAdd(h + ((t[z >> 2] >> (8 * (z & 3))) & 0xFFu), 1u);
    }
}

// Tiles tile0 .. tile0 + ntiles of one instance by one wave: cost bytes to
// `cost` (when not null), levels to win and, outside its window, to h.
template <int NB, bool SUMS>
__device__ __forceinline__ void wave_tiles(const ClauseRec *rec, const ClauseCounts &n, EffEntry (*eff)[2],
                                           uint32_t tile0, uint32_t ntiles, int nvars, uint8_t *cost,
                                           LevelWindow<NB> &win, uint32_t *h) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t nwords = nvars >= kLowBits ? (1ull << (nvars - kLowBits)) : 1;
    TileSums s;
    if constexpr (SUMS) tile_sums(rec, n, tile0, s);
    for (uint32_t t0 = 0; t0 < ntiles; ++t0) {
        const uint32_t tile = tile0 + t0;
        uint32_t v[8], t[8];
        eval_planes<SUMS>(rec, n, tile, s, (int)t0, eff, v);
        const uint64_t w = (uint64_t)tile * kWave + lane;
        if (w >= nwords) continue;
        if (nvars >= kLowBits) {
            const uint32_t outside = win.add(v);
            if (outside || cost) planes_to_bytes(v, t);
            if (cost) {
                typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
                u32x4 *dst = reinterpret_cast<u32x4 *>(cost + (w << kLowBits));
                dst[0] = u32x4{t[0], t[1], t[2], t[3]};
                dst[1] = u32x4{t[4], t[5], t[6], t[7]};
            }
            if (outside) tally_bits(h, t, outside);
        } else {
            const uint32_t N = 1u << nvars;
            planes_to_bytes(v, t);
            if (cost)
                for (uint32_t z = 0; z < N; ++z) cost[z] = (uint8_t)((t[z >> 2] >> (8 * (z & 3))) & 0xFFu);
            tally_word(h, t, N);
        }
    }
}

// A wave takes runs of `run` tiles (at most 64). SUMS pays for itself from a
// run of 8 on: the sums of a run cost about two tiles' work and save half of
// every tile's.
template <int NB, bool SUMS>
__global__ void __launch_bounds__(kCostThreads)
cost_table_kernel(const ClauseRec *__restrict__ recs, ClauseCounts cc, int neff, int n, uint32_t run,
                  uint8_t *__restrict__ cost, uint32_t *__restrict__ block_hist, int hist_len, int win_a0) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    CostLds lds(smem, neff);
    for (int i = threadIdx.x; i < kHistCopies * kHistStride; i += kCostThreads) lds.hist[i] = 0;
    for (int i = threadIdx.x; i < kMaxRecs; i += kCostThreads) lds.rec[i] = recs[i];
    __syncthreads();
    uint32_t *h = hist_copy(lds);
    EffEntry(*eff)[2] = lds.wave_eff(neff);
    const uint32_t ntiles = n > kHighBit0 ? 1u << (n - kHighBit0) : 1u;
    const uint32_t step = gridDim.x * kCostWaves * run;
    LevelWindow<NB> win;
    win.clear(win_a0);
    for (uint32_t t0 = (blockIdx.x * kCostWaves + threadIdx.x / kWave) * run; t0 < ntiles; t0 += step)
        wave_tiles<NB, SUMS>(lds.rec, cc, eff, t0, min(run, ntiles - t0), n, cost, win, h);
    win.flush(wave_copies(lds));
    __syncthreads();
    for (int k = threadIdx.x; k < hist_len; k += kCostThreads) {
        uint32_t s = 0;
        for (int c = 0; c < kHistCopies; ++c) s += lds.hist[c * kHistStride + k];
        block_hist[(size_t)blockIdx.x * hist_len + k] = s;
    }
}

// hist[k] = sum over blocks of block_hist[b][k]: one block per level k, every
// thread sums a strided subset of rows (integer sums, so the order is free).
__global__ void __launch_bounds__(256) hist_reduce_kernel(const uint32_t *__restrict__ block_hist,
                                                          int nblocks, int hist_len,
                                                          unsigned long long *__restrict__ hist) {
    __shared__ unsigned long long red[256];
    const int k = blockIdx.x;
    unsigned long long s = 0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += block_hist[(size_t)b * hist_len + k];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) hist[k] = red[0];
}

// ---- many instances, histograms only ---------------------------------------
// Clause ingest runs on the device here: each block builds its instance's
// records from the raw literals straight into LDS, so the host uploads 12
// bytes per clause and packs nothing.
// The kernel is bound by its vector instructions (76% of the issue slots at 4096
// instances of n = 8..20). NB, the 32-level blocks of the counting window, is 1
// for m <= 128: 126 registers and four waves a SIMD against 160 and three, and
// half the counting; with the sets of LevelWindow 330 -> 190 us.
struct HistInst {
    uint32_t lit_off;   // first clause of the instance in the literal array
    int32_t n, m;
    int32_t win_a0;     // first 32-level block of the counting window
    uint64_t cost_off;  // byte offset of the instance's cost table (when costs are written)
};
struct HistUnit {
    uint32_t inst, tile0, ntiles, pad;
};

constexpr uint32_t kSumsRun = 8;  // shortest run of tiles per wave that takes the class sums

template <int NB>
__global__ void __launch_bounds__(kCostThreads)
hist_batched_kernel(const HistInst *__restrict__ insts, const HistUnit *__restrict__ units,
                    const int32_t *__restrict__ lits, int neff, unsigned long long *__restrict__ hists,
                    int hist_stride, uint8_t *__restrict__ costs) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int cls_n[kCostWaves][kClasses];
    const HistUnit unit = units[blockIdx.x];
    const HistInst in = insts[unit.inst];
    CostLds lds(smem, neff);
    const int32_t *L = lits + 3 * (size_t)in.lit_off;
    const int c = threadIdx.x, wave = threadIdx.x / kWave;
    for (int i = c; i < kHistCopies * kHistStride; i += kCostThreads) lds.hist[i] = 0;
    for (int i = c; i < kMaxRecs; i += kCostThreads) lds.rec[i] = ClauseRec{0u, 0u, 0u, 0u, 0ull};
    // thread c ingests clause c (m <= 255): its record goes behind those of its
    // class with a lower index
    int cls = -1, below = 0;
    ClauseRec r;
    if (c < in.m) r = make_record(L[3 * c], L[3 * c + 1], L[3 * c + 2], &cls);
#pragma unroll
    for (int k = 0; k < kClasses; ++k) {
        const uint64_t mask = __ballot(cls == k);
        if (cls == k) below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if ((c & (kWave - 1)) == 0) cls_n[wave][k] = __popcll(mask);
    }
    __syncthreads();
    int tot[kClasses];
#pragma unroll
    for (int k = 0; k < kClasses; ++k) {
        tot[k] = 0;
#pragma unroll
        for (int w = 0; w < kCostWaves; ++w) {
            if (cls == k && w < wave) below += cls_n[w][k];
            tot[k] += cls_n[w][k];
        }
        tot[k] = __builtin_amdgcn_readfirstlane(tot[k]);
    }
    const ClauseCounts cc = clause_layout(tot[0], tot[1], tot[2], tot[3]);
    if (cls >= 0) lds.rec[cc.first[cls] + below] = r;
    __syncthreads();
    uint32_t *h = hist_copy(lds);
    EffEntry(*eff)[2] = lds.wave_eff(neff);
    LevelWindow<NB> win;
    win.clear(in.win_a0);
    // the unit's tiles in equal runs, one per wave
    const uint32_t run = (unit.ntiles + kCostWaves - 1) / kCostWaves;
    const uint32_t t0 = wave * run;
    uint8_t *cost = costs ? costs + in.cost_off : nullptr;
    if (t0 < unit.ntiles) {
        const uint32_t nt = min(run, unit.ntiles - t0);
        if (run >= kSumsRun) wave_tiles<NB, true>(lds.rec, cc, eff, unit.tile0 + t0, nt, in.n, cost, win, h);
        else wave_tiles<NB, false>(lds.rec, cc, eff, unit.tile0 + t0, nt, in.n, cost, win, h);
    }
    win.flush(wave_copies(lds));
    __syncthreads();
    for (int k = threadIdx.x; k <= in.m; k += kCostThreads) {
        uint32_t s = 0;
        for (int q = 0; q < kHistCopies; ++q) s += lds.hist[q * kHistStride + k];
        if (s && hists) atomicAdd(hists + (size_t)unit.inst * hist_stride + k, (unsigned long long)s);
    }
}

// ---- host launchers (arguments already validated) ---------------------------
// Counting window for an instance with m clauses: C has mean m/8 over all
// assignments (each clause is false on 1/8 of them) and, for random clauses,
// a spread of about sqrt(7m/64); the window is the aligned 32-level blocks
// covering mean +- 4 spreads, at most two. Levels outside it are still
// counted exactly, one by one.
static void level_window(int m, int *a0, int *nb) {
    const double mu = m / 8.0, sd = std::sqrt(m * 7.0 / 64.0);
    const int lo = std::max(0, (int)std::floor(mu - 4.0 * sd));
    const int hi = std::min(m, (int)std::ceil(mu + 4.0 * sd));
    *a0 = lo / 32;
    *nb = std::min(2, hi / 32 - *a0 + 1);
}

// Runs of tiles per wave and blocks of a cost table: the longest run (at most
// 64) that still gives 4096 waves, and single tiles where that leaves runs
// shorter than kSumsRun.
struct CostGrid {
    uint32_t run;
    int blocks;
};
static CostGrid cost_grid(int n, const DeviceInfo &dev, int cap) {
    const uint32_t ntiles = n > kHighBit0 ? 1u << (n - kHighBit0) : 1u;
    CostGrid g{1, 0};
    if (ntiles / 4096 >= kSumsRun) g.run = std::min(64u, ntiles / 4096);
    const uint32_t want = (ntiles / g.run + kCostWaves - 1) / kCostWaves;
    g.blocks = (int)std::min<uint32_t>(want, (uint32_t)std::min(dev.num_cus * 8, cap));
    return g;
}

template <int NB>
static void launch_cost_kernel(bool sums, int m, const CostGrid &g, const ClauseRec *recs, const ClauseCounts &cc,
                               int n, uint8_t *cost, uint32_t *d_bh, int a0, hipStream_t stream) {
    const dim3 grid(g.blocks), block(kCostThreads);
    if (sums)
        hipLaunchKernelGGL((cost_table_kernel<NB, true>), grid, block, cost_lds_bytes(m), stream, recs, cc,
                           eff_entries(m), n, g.run, cost, d_bh, m + 1, a0);
    else
        hipLaunchKernelGGL((cost_table_kernel<NB, false>), grid, block, cost_lds_bytes(m), stream, recs, cc,
                           eff_entries(m), n, g.run, cost, d_bh, m + 1, a0);
}

// Cost kernel and histogram reduce on records already on the device.
static int enqueue_cost_kernels(int n, int m, const CostGrid &g, const ClauseCounts &cc, const ClauseRec *d_rec,
                                uint32_t *d_bh, uint8_t *cost, uint64_t *hist, hipStream_t stream) {
    const int hist_len = m + 1;
    int a0 = 0, nb = 1;
    level_window(m, &a0, &nb);
    ProfScope ps("cost_table", stream);
    if (nb == 1) launch_cost_kernel<1>(g.run >= kSumsRun, m, g, d_rec, cc, n, cost, d_bh, a0, stream);
    else launch_cost_kernel<2>(g.run >= kSumsRun, m, g, d_rec, cc, n, cost, d_bh, a0, stream);
    ps.end();
    GQ_LAUNCH_CHECK();
    if (hist) {
        hipLaunchKernelGGL(hist_reduce_kernel, dim3(hist_len), dim3(256), 0, stream, d_bh, g.blocks, hist_len,
                           reinterpret_cast<unsigned long long *>(hist));
        GQ_LAUNCH_CHECK();
    }
    return GQAOA_OK;
}

constexpr size_t kRecBytes = sizeof(ClauseRec) * kMaxRecs;

int launch_cost_table(int n, int m, const int32_t *lits, uint8_t *cost, uint64_t *hist,
                      hipStream_t stream) {
    DeviceInfo dev;
    int st = device_info(&dev);
    if (st) return st;
    ClauseRec rec[kMaxRecs];
    const ClauseCounts cc = pack_clauses(m, lits, rec);
    const CostGrid g = cost_grid(n, dev, 1 << 30);
    const size_t rec_bytes = (kRecBytes + 255) & ~size_t(255);
    AsyncScratch guard(stream);
    GQ_HIP(guard.alloc(rec_bytes + sizeof(uint32_t) * (size_t)g.blocks * (m + 1)));
    char *scratch = reinterpret_cast<char *>(guard.ptr);
    GQ_HIP(hipMemcpyAsync(scratch, rec, kRecBytes, hipMemcpyHostToDevice, stream));
    GQ_HIP(hipStreamSynchronize(stream));  // the records are host stack memory of this call
    return enqueue_cost_kernels(n, m, g, cc, reinterpret_cast<const ClauseRec *>(scratch),
                                reinterpret_cast<uint32_t *>(scratch + rec_bytes), cost, hist, stream);
}

// ---- allocation-free form: scratch in a static device array --------------------------------
// The clause records and the per-block histogram rows of gqaoa_cost_table,
// for callers that cannot allocate device memory. The grid is capped at
// kStaticBlocks blocks (the kernel's loop over tiles covers any n), so every
// valid (n, m) fits: 8 KiB of records and at most 2 MiB of rows. Each GPU
// holds its own copy of the array until the process ends; host code reaches it
// only through the address hipGetSymbolAddress returns on that device.
constexpr int kStaticBlocks = 2048;
constexpr size_t kStaticRecBytes = 8192;
static_assert(kRecBytes <= kStaticRecBytes, "records");
constexpr size_t kStaticRowBytes = sizeof(uint32_t) * (size_t)kStaticBlocks * 256;
constexpr size_t kStaticScratchBytes = kStaticRecBytes + kStaticRowBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static std::mutex g_scratch_mu;
static std::map<int, unsigned char *> g_scratch_addr;  // device -> device address of `scratch`

// Device address of this device's copy of `scratch`, looked up once per
// device (with that device current).
static int static_scratch(unsigned char **out) {
    int dev = -1;
    GQ_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch_addr.find(dev);
    if (it == g_scratch_addr.end()) {
        void *ptr = nullptr;
        GQ_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        it = g_scratch_addr.emplace(dev, reinterpret_cast<unsigned char *>(ptr)).first;
    }
    *out = it->second;
    return GQAOA_OK;
}

int launch_cost_table_noalloc(int n, int m, const int32_t *lits, uint8_t *cost, uint64_t *hist,
                              hipStream_t stream) {
    DeviceInfo dev;
    int st = device_info(&dev);
    if (st) return st;
    unsigned char *base = nullptr;
    if ((st = static_scratch(&base))) return st;
    ClauseRec rec[kMaxRecs];
    const ClauseCounts cc = pack_clauses(m, lits, rec);
    const CostGrid g = cost_grid(n, dev, kStaticBlocks);
    const size_t row_bytes = sizeof(uint32_t) * (size_t)g.blocks * (size_t)(m + 1);
    if (row_bytes > kStaticRowBytes)
        return fail(GQAOA_ERANGE, "cost table n=%d m=%d needs %zu scratch bytes, more than the static %zu", n, m,
                    row_bytes, kStaticRowBytes);
    GQ_HIP(hipMemcpyAsync(base, rec, kRecBytes, hipMemcpyHostToDevice, stream));
    GQ_HIP(hipStreamSynchronize(stream));  // the records are host stack memory of this call
    // every block writes its whole row of hist_len counts, so no row needs clearing
    return enqueue_cost_kernels(n, m, g, cc, reinterpret_cast<const ClauseRec *>(base),
                                reinterpret_cast<uint32_t *>(base + kStaticRecBytes), cost, hist, stream);
}

// Byte offset of each instance's cost table in the concatenated output: the
// tables follow each other in instance order, each starting at a multiple of
// 64 bytes.
uint64_t batched_cost_offset(int i, const int32_t *n_host) {
    uint64_t off = 0;
    for (int j = 0; j < i; ++j) off += ((1ull << n_host[j]) + 63) & ~63ull;
    return off;
}

int launch_hist_batched(int num_inst, const int32_t *n_host, const int32_t *m_host,
                        const int32_t *lits, uint64_t *hists, int hist_stride, uint8_t *costs, hipStream_t stream) {
    std::vector<HistInst> insts(num_inst);
    std::vector<HistUnit> units;
    // tiles of a unit: runs of up to 32 per wave while the batch still gives
    // 4096 of them
    uint64_t all_tiles = 0;
    for (int i = 0; i < num_inst; ++i) all_tiles += n_host[i] > kHighBit0 ? 1ull << (n_host[i] - kHighBit0) : 1;
    uint32_t unit_tiles = 4 * kCostWaves;
    while (unit_tiles < 32 * kCostWaves && all_tiles / (unit_tiles * 2) * kCostWaves >= 4096) unit_tiles *= 2;
    size_t off = 0;
    int max_m = 1;
    for (int i = 0; i < num_inst; ++i) max_m = std::max(max_m, m_host[i]);
    uint64_t cost_off = 0;
    int win_a0[256], win_nb[256];  // by m, filled as they occur
    std::fill(win_a0, win_a0 + 256, -1);
    units.reserve((size_t)num_inst + all_tiles / unit_tiles);
    // Units in the order of their launches (windows of one 32-level block, then
    // of two) and by falling n in each, so that the last blocks to start are the
    // shortest. start[key]: where the instances of a key begin in `order`.
    auto key = [&](int i) { return (win_nb[m_host[i]] - 1) * 32 + 31 - n_host[i]; };
    int start[65] = {0};
    for (int i = 0; i < num_inst; ++i) {
        int &a0 = win_a0[m_host[i]];
        if (a0 < 0) level_window(m_host[i], &a0, &win_nb[m_host[i]]);
        insts[i] = HistInst{(uint32_t)off, n_host[i], m_host[i], a0, cost_off};
        cost_off += ((1ull << n_host[i]) + 63) & ~63ull;
        off += (size_t)m_host[i];
        ++start[key(i) + 1];
    }
    for (int k = 0; k < 64; ++k) start[k + 1] += start[k];
    const int num_one = start[32];
    std::vector<int32_t> order(num_inst);
    for (int i = 0; i < num_inst; ++i) order[start[key(i)]++] = i;
    size_t units_one = 0;
    for (int o = 0; o < num_inst; ++o) {
        const int i = order[o];
        const uint32_t ntiles = n_host[i] > kHighBit0 ? 1u << (n_host[i] - kHighBit0) : 1u;
        for (uint32_t t0 = 0; t0 < ntiles; t0 += unit_tiles)
            units.push_back(HistUnit{(uint32_t)i, t0, std::min(unit_tiles, ntiles - t0), 0u});
        if (o + 1 == num_one) units_one = units.size();
    }
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const size_t b_inst = sizeof(HistInst) * insts.size();
    const size_t b_unit = sizeof(HistUnit) * units.size();
    const size_t b_lits = sizeof(int32_t) * 3 * off;
    const size_t o_unit = al(b_inst), o_lits = o_unit + al(b_unit);
    AsyncScratch guard(stream);
    GQ_HIP(guard.alloc(o_lits + al(b_lits)));
    void *scratch = guard.ptr;
    char *base = reinterpret_cast<char *>(scratch);
    GQ_HIP(hipMemcpyAsync(base, insts.data(), b_inst, hipMemcpyHostToDevice, stream));
    GQ_HIP(hipMemcpyAsync(base + o_unit, units.data(), b_unit, hipMemcpyHostToDevice, stream));
    GQ_HIP(hipMemcpyAsync(base + o_lits, lits, b_lits, hipMemcpyHostToDevice, stream));
    if (hists) GQ_HIP(hipMemsetAsync(hists, 0, sizeof(uint64_t) * (size_t)num_inst * hist_stride, stream));
    auto launch = [&](auto kernel, size_t first, size_t count) -> int {
        if (!count) return GQAOA_OK;
        hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(kCostThreads), cost_lds_bytes(max_m), stream,
                           reinterpret_cast<const HistInst *>(base),
                           reinterpret_cast<const HistUnit *>(base + o_unit) + first,
                           reinterpret_cast<const int32_t *>(base + o_lits), eff_entries(max_m),
                           reinterpret_cast<unsigned long long *>(hists), hist_stride, costs);
        GQ_LAUNCH_CHECK();
        return GQAOA_OK;
    };
    int s;
    if ((s = launch(hist_batched_kernel<1>, 0, units_one))) return s;
    if ((s = launch(hist_batched_kernel<2>, units_one, units.size() - units_one))) return s;
    GQ_HIP(hipStreamSynchronize(stream));  // the host tables above end with this call
    return GQAOA_OK;
}

}  // namespace gqaoa
