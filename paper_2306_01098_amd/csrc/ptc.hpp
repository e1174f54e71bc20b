// Parallel-transport convolution (PTC) network: shared definitions.
//
// Layer: out_c(x) = sum_{c'} sum_{p} w[c][c'][p] (T_p in_{c'})(x) with the
// nine paths p = 0 (identity), 1 + 2 mu (hop +mu: X_mu(x) in(x+mu)) and
// 2 + 2 mu (hop -mu: X_mu(x-mu)^+ in(x-mu)); time-boundary sign on wraps.
// Network 1 -> 8 -> 8 -> 1 channels, no bias, no nonlinearity, acting on the
// whole lattice; its input is an even-site field extended by zero.
#pragma once

#include "common.hpp"

namespace hisq {

constexpr int PTC_PATHS = 9;
constexpr int PTC_CH = 8;
constexpr int PTC_W1 = 0;                            // layer 1: [8][1][9]
constexpr int PTC_W2 = PTC_W1 + PTC_CH * 1 * PTC_PATHS;  // layer 2: [8][8][9]
constexpr int PTC_W3 = PTC_W2 + PTC_CH * PTC_CH * PTC_PATHS;  // layer 3: [1][8][9]
constexpr int PTC_NW = PTC_W3 + 1 * PTC_CH * PTC_PATHS;  // 720 complex weights
constexpr int PTC_BLOCK = 256;

// The folded network (ptc.hip): 65 double2 of the map, 65 of its adjoint; the
// gradient with respect to it: 64 complex correlations and K0 as doubles.
constexpr int PTC_NFOLD = 130;
constexpr int PTC_ADJOINT = 65;  // where the adjoint network starts
constexpr int PTC_C0 = 64;       // c0 in each of the two
constexpr int PTC_NK = 130;
constexpr int PTC_COLS = 4;  // training pairs per launch

// skip (nullable): the launch does nothing while *skip != 0.
hipError_t ptc_fold(const float2 *w, double2 *fold, float2 *keep, hipStream_t st, const int *skip = nullptr);
// Columns col0 .. col0 + ncols - 1 of an ncol-column field; s: 24 vh float2 a column.
hipError_t ptc_spread(const Geom &g, const char *links, const double2 *fold, const void *in, int ncol, int col0,
                      int ncols, float2 *s, hipStream_t st, const int *skip = nullptr);
hipError_t ptc_gather(const Geom &g, const double2 *c0, const void *in, const float2 *s, void *out, void *keep,
                      hipStream_t st, const int *skip = nullptr);
hipError_t ptc_error(const Geom &g, const double2 *c0, const void *b32, int ncol, int col0, int ncols, const float2 *s,
                     const void *x64, void *e, double *partials, hipStream_t st);
// Column cin + k of `in` with column k of the ncols-column field gr.
hipError_t ptc_correlate(const Geom &g, const char *links, const void *in, int nin, int cin, const void *gr, int ncols,
                         double *partials, hipStream_t st);
hipError_t ptc_correlate_sum(const Geom &g, int ncols, const double *partials, bool first, double *K, const double *xb,
                             double inv_batch, const double *dot, int ndot, double *loss, hipStream_t st);
hipError_t ptc_chain(const float2 *wf, const float2 *wb, const double *K, double2 *grad, hipStream_t st);
hipError_t ptc_chain_adam(const float2 *w, const double *K, double2 *w_master, float2 *w_f32, double2 *m, double2 *v,
                          int step, double lr, double b1, double b2, double eps, hipStream_t st);
int ptc_correlate_blocks(const Geom &g, int ncols);
int ptc_error_blocks(const Geom &g);
hipError_t ptc_adam(double2 *w_master, float2 *w_f32, const double2 *grad, double2 *m, double2 *v, int step,
                    double lr, double b1, double b2, double eps, hipStream_t st);

}  // namespace hisq
