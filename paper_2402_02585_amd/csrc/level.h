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
    const uint8_t *cost;
    void *psi;              // [2^n] complex128, written
    const double *beta_host, *gamma_host;  // eager calls: p host angles each
    double *angles_dev;     // beta[p], gamma[p]: read by captured calls, scratch of long eager ones
    uint32_t *rows;         // [kLevelMaxRows][256] counts (n > kLevelFusedMaxN)
    void *table;            // [256] complex128 (n > kLevelFusedMaxN)
    double *readout;        // [p+1][3]
};

// Enqueues the whole evolution. captured: the angles are read from
// angles_dev when the launches run; otherwise from beta_host / gamma_host,
// which must stay valid until the stream has been synchronized.
int level_evolve(const LevelEvolve &e, bool captured, hipStream_t st);

}  // namespace gqaoa
