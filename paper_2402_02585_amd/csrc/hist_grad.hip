// Level-space adjoint gradient of P_sol for many instances (float64): the
// reverse sweep of the adjoint gradient (dP/dbeta_k, dP/dgamma_k for every
// round) in the effective space of App. C, "Optimization", for full G-QAOA
// (all 2p angles, App. C) at the sizes the paper simulates. The host compacts
// the occupied levels of the given histograms; the sweep is level.hip's, one
// block per instance.
#include "level.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

namespace gqaoa {

constexpr int kHistGradMaxK = 256;
constexpr size_t kPackBytes = 1 << 20;  // larger batches' arrays are copied one by one, without a host copy

static size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

size_t hist_grad_workspace_bytes(int num_inst, int hist_stride, int pstride) {
    const size_t I = (size_t)num_inst;
    const size_t lv = I * (size_t)std::min(hist_stride, kHistGradMaxK);
    const size_t ang = I * (size_t)pstride * sizeof(double);
    return al256(sizeof(HistGradSlot) * I) + al256(4 * lv) + al256(8 * lv) + 2 * al256(ang) +
           al256(8 * I) + 2 * al256(ang);
}

int run_hist_grad(int num_inst, const int32_t *n_host, const int32_t *m_host, const uint64_t *hists,
                  int hist_stride, const int32_t *target_host, int pstride, const int32_t *p_host,
                  const double *beta, const double *gamma, double *psol, double *dbeta, double *dgamma,
                  void *ws, hipStream_t st) {
    // compact the occupied levels
    size_t cap = 0;
    for (int i = 0; i < num_inst; ++i) cap += (size_t)m_host[i] + 1;
    const std::unique_ptr<int32_t[]> lev(new (std::nothrow) int32_t[cap]);
    const std::unique_ptr<double[]> w(new (std::nothrow) double[cap]);
    if (!lev || !w) return fail(GQAOA_EINVAL, "out of host memory");
    std::vector<HistGradSlot> slots((size_t)num_inst);
    size_t nl = 0;
    for (int i = 0; i < num_inst; ++i) {
        const uint64_t *h = hists + (size_t)i * hist_stride;
        const int t = target_host ? target_host[i] : 0;
        const double invN = std::ldexp(1.0, -n_host[i]);
        HistGradSlot s{i, (int32_t)nl, 0, -1, p_host ? p_host[i] : pstride, {0, 0, 0}};
        for (int k = 0; k <= m_host[i]; ++k)
            if (h[k]) {
                if (k == t) s.t_idx = (int32_t)nl - s.lev_off;
                lev[nl] = k;
                w[nl++] = (double)h[k] * invN;  // exact: a count times a power of two
            }
        s.K = (int32_t)nl - s.lev_off;
        slots[i] = s;
    }

    const size_t I = (size_t)num_inst;
    const size_t ang = I * (size_t)pstride * sizeof(double);
    // tables and angles back to back in the workspace (each at most its share
    // of hist_grad_workspace_bytes), then the results; a small batch's go up
    // and come down in one copy each
    const size_t o_lev = al256(sizeof(HistGradSlot) * I), o_w = o_lev + al256(4 * nl);
    const size_t o_beta = o_w + al256(8 * nl), o_gamma = o_beta + al256(ang), o_psol = o_gamma + al256(ang);
    const size_t o_db = o_psol + al256(8 * I), o_dg = o_db + al256(ang), o_end = o_dg + ang;
    char *base = reinterpret_cast<char *>(ws);
    const bool packed = o_end <= kPackBytes;
    const std::unique_ptr<char[]> pack(packed ? new (std::nothrow) char[o_end] : nullptr);
    if (packed && !pack) return fail(GQAOA_EINVAL, "out of host memory");
    const struct {
        size_t at;
        const void *src;
        size_t bytes;
    } parts[] = {{0, slots.data(), sizeof(HistGradSlot) * I}, {o_lev, lev.get(), 4 * nl}, {o_w, w.get(), 8 * nl},
                 {o_beta, beta, ang}, {o_gamma, gamma, ang}};
    for (const auto &q : parts) {
        if (packed) memcpy(pack.get() + q.at, q.src, q.bytes);
        else if (q.bytes) GQ_HIP(hipMemcpyAsync(base + q.at, q.src, q.bytes, hipMemcpyHostToDevice, st));
    }
    if (packed) GQ_HIP(hipMemcpyAsync(base, pack.get(), o_psol, hipMemcpyHostToDevice, st));

    LevelGrad g{};
    g.num_inst = num_inst;
    g.pstride = pstride;
    g.slots = reinterpret_cast<const HistGradSlot *>(base);
    g.lev = reinterpret_cast<const int32_t *>(base + o_lev);
    g.w = reinterpret_cast<const double *>(base + o_w);
    g.beta = reinterpret_cast<const double *>(base + o_beta);
    g.gamma = reinterpret_cast<const double *>(base + o_gamma);
    g.psol = reinterpret_cast<double *>(base + o_psol);
    g.dbeta = reinterpret_cast<double *>(base + o_db);
    g.dgamma = reinterpret_cast<double *>(base + o_dg);
    int s = level_grad(g, st);
    if (s) return s;

    if (packed) {
        GQ_HIP(hipMemcpyAsync(pack.get() + o_psol, base + o_psol, o_end - o_psol, hipMemcpyDeviceToHost, st));
        GQ_HIP(hipStreamSynchronize(st));
        if (psol) memcpy(psol, pack.get() + o_psol, 8 * I);
        if (dbeta) memcpy(dbeta, pack.get() + o_db, ang);
        if (dgamma) memcpy(dgamma, pack.get() + o_dg, ang);
        return GQAOA_OK;
    }
    if (psol) GQ_HIP(hipMemcpyAsync(psol, g.psol, 8 * I, hipMemcpyDeviceToHost, st));
    if (dbeta) GQ_HIP(hipMemcpyAsync(dbeta, g.dbeta, ang, hipMemcpyDeviceToHost, st));
    if (dgamma) GQ_HIP(hipMemcpyAsync(dgamma, g.dgamma, ang, hipMemcpyDeviceToHost, st));
    GQ_HIP(hipStreamSynchronize(st));  // host tables above and the outputs
    return GQAOA_OK;
}

}  // namespace gqaoa
