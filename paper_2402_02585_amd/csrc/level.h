// Level form of the rounds that start from |s> (level.hip), shared with the
// statevector entry points (sv.hip).
#pragma once

#include "internal.h"

namespace gqaoa {

constexpr int kLevelFusedMaxN = 15;      // largest n evolved in one launch of one block
constexpr int kLevelMaxRows = 256;       // blocks of a counting launch per instance
constexpr int kLevelInlineRounds = 112;  // rounds whose angles travel as kernel arguments

struct LevelEvolve {
    int n, m, p, target;
    int init_uniform;
    const uint8_t *cost;
    void *psi;              // [2^n] complex128: the initial state unless init_uniform, the final one
    const double *beta_host, *gamma_host;  // p host angles each
    double *angles_dev;     // beta[p], gamma[p]: scratch of calls of more than kLevelInlineRounds
    void *rows;             // [kLevelMaxRows + 1][256][4] doubles: counts or level sums of the blocks
    void *table;            // [512] complex128: the final level table
    double *readout;        // [p+1][3]
};

// Enqueues the whole evolution. beta_host and gamma_host must stay valid until
// the stream has been synchronized.
int level_evolve(const LevelEvolve &e, hipStream_t st);

// Adjoint gradient of P_sol in the level space: the occupied levels of one
// instance per block, counted from its cost table or given compacted.
struct HistGradSlot {
    int32_t inst;     // caller's instance index
    int32_t lev_off;  // first compacted level of the instance
    int32_t K;        // occupied levels
    int32_t t_idx;    // position of the target level among them, -1 if unoccupied
    int32_t p;        // rounds of this instance
    int32_t pad[3];
};

struct LevelGrad {
    int num_inst, pstride;         // angles and gradients: [inst][pstride]
    // counted: every instance has n variables, costs cost + i 2^n, p = pstride rounds
    int n;
    const uint8_t *cost;
    const int32_t *m, *target;     // [inst], device
    uint32_t *rows;                // [inst][row_cap][256] (n > kLevelFusedMaxN)
    int row_cap;
    // compacted: slots [num_inst] with their levels and weights (cost null)
    const HistGradSlot *slots;
    const int32_t *lev;
    const double *w;
    const double *beta, *gamma;    // device
    double *psol, *dbeta, *dgamma; // device: [inst], [inst][pstride] each
};

int level_grad(const LevelGrad &g, hipStream_t st);

}  // namespace gqaoa
