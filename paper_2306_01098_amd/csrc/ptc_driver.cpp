// C ABI of the PTC preconditioner network: apply, backward, Adam, and one
// training step (forward, loss, backward over a batch of (source, solution)
// pairs, then Adam), all on the caller's device buffers.
#include <cmath>

#include "api_util.hpp"
#include "dslash.hpp"
#include "ptc.hpp"

namespace hisq {

namespace {

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace: the input of the last forward pass (a0), the half-network vectors
// s, the training chunk's error fields e, t = D_oe e and A e, all for up to
// PTC_COLS columns, the small arrays (folded map, weights of the last forward
// pass and of the training step, correlations, loss) and the block partials of
// <e, A e>, <x, b> and the correlations.
struct PtcLayout {
    size_t a0, s, e, t, ae, fold, keep, keep0, k, scal, dot_part, xb_part, corr_part, total;
};

PtcLayout ptc_layout(const Geom &g) {
    PtcLayout L;
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off = a256(off + b);
        return o;
    };
    const size_t h32 = field_bytes(g, HISQ_FP32, 1), cols32 = field_bytes(g, HISQ_FP32, PTC_COLS);
    L.a0 = take(h32);
    L.s = take(8 * PTC_COLS * h32);  // eight vectors on half the sites per column
    L.e = take(cols32);
    L.t = take(cols32);
    L.ae = take(cols32);
    L.fold = take(sizeof(double2) * PTC_NFOLD);
    L.keep = take(sizeof(float2) * PTC_NW);
    L.keep0 = take(sizeof(float2) * PTC_NW);
    L.k = take(sizeof(double) * PTC_NK);
    L.scal = take(sizeof(double));
    L.dot_part = take(sizeof(double) * PTC_COLS * (g.vh / 4 + 1));  // a Dslash block holds at least 4 sites
    L.xb_part = take(sizeof(double) * PTC_COLS * ptc_error_blocks(g));
    L.corr_part = take(sizeof(double) * PTC_COLS * PTC_NK * ptc_correlate_blocks(g, PTC_COLS));  // fewer columns take no more
    L.total = off;
    return L;
}

struct Ptc {
    Geom g;
    PtcLayout L;
    char *ws;
    const char *links;
    hipStream_t st;
    template <typename T> T *at(size_t o) const { return reinterpret_cast<T *>(ws + o); }
};

// out_even = N(in_even); skip (nullable): every launch does nothing while
// *skip != 0.  keep: leave the input and the weights for the backward pass.
hipError_t forward(const Ptc &P, const float2 *w, const void *in_even, void *out_even, bool keep,
                   const int *skip = nullptr) {
    double2 *fold = P.at<double2>(P.L.fold);
    hipError_t e = ptc_fold(w, fold, keep ? P.at<float2>(P.L.keep) : nullptr, P.st, skip);
    if (e == hipSuccess)
        e = ptc_spread(P.g, P.links, fold, in_even, 1, 0, 1, P.at<float2>(P.L.s), P.st, skip);
    if (e == hipSuccess)
        e = ptc_gather(P.g, fold + PTC_C0, in_even, P.at<float2>(P.L.s), out_even, keep ? P.at<void>(P.L.a0) : nullptr,
                       P.st, skip);
    return e;
}

// From the output gradient g_out on the even sites: weight gradients += into
// grad, input gradient into g_in if non-NULL.
hipError_t backward(const Ptc &P, const float2 *w, const void *g_out, double2 *grad, void *g_in) {
    double *part = P.at<double>(P.L.corr_part), *K = P.at<double>(P.L.k);
    hipError_t e = ptc_correlate(P.g, P.links, P.at<void>(P.L.a0), 1, 0, g_out, 1, part, P.st);
    if (e == hipSuccess)
        e = ptc_correlate_sum(P.g, 1, part, true, K, nullptr, 0.0, nullptr, 0, nullptr, P.st);
    if (e == hipSuccess)
        e = ptc_chain(P.at<float2>(P.L.keep), w, K, grad, P.st);
    if (e == hipSuccess && g_in) {
        double2 *fold = P.at<double2>(P.L.fold), *adj = fold + PTC_ADJOINT;
        float2 *s = P.at<float2>(P.L.s);
        e = ptc_fold(w, fold, nullptr, P.st);
        if (e == hipSuccess)
            e = ptc_spread(P.g, P.links, adj, g_out, 1, 0, 1, s, P.st);
        if (e == hipSuccess)
            e = ptc_gather(P.g, adj + PTC_C0, g_out, s, g_in, nullptr, P.st);
    }
    return e;
}

hisq_status common_checks(const hisq_lattice *lat, const void *links, const void *w, const void *ws, size_t ws_bytes,
                          Ptc *P, hisq_context *ctx, void *stream) {
    hisq_status s = check_lattice(lat);
    if (s == HISQ_OK) s = check_ptr(links, "links_f32");
    if (s == HISQ_OK) s = check_ptr(w, "weights");
    if (s == HISQ_OK) s = check_ptr(ws, "ws");
    if (s == HISQ_OK) s = set_device(ctx);
    if (s != HISQ_OK)
        return s;
    P->g = make_geom(*lat);
    P->L = ptc_layout(P->g);
    if (ws_bytes < P->L.total)
        return fail(HISQ_ERR_WORKSPACE, "workspace holds %zu bytes, needs %zu", ws_bytes, P->L.total);
    P->ws = static_cast<char *>(const_cast<void *>(ws));
    P->links = static_cast<const char *>(links);
    P->st = static_cast<hipStream_t>(stream);
    return HISQ_OK;
}

}  // namespace

// Internal entry used by the flexible CG: z = N(r) on even sites; the launches
// do nothing while skip (nullable) points to a nonzero value.
hisq_status ptc_apply_internal(const hisq_lattice *lat, const void *links_f32, const void *weights, const void *in,
                               void *out, void *ws, size_t ws_bytes, hipStream_t st, const int *skip) {
    Ptc P;
    hisq_status s = common_checks(lat, links_f32, weights, ws, ws_bytes, &P, nullptr, st);
    if (s != HISQ_OK)
        return s;
    const hipError_t e = forward(P, static_cast<const float2 *>(weights), in, out, false, skip);
    return e == hipSuccess ? HISQ_OK : device_fail(e, "ptc forward");
}

size_t ptc_workspace(const Geom &g) { return ptc_layout(g).total; }

}  // namespace hisq

using namespace hisq;

extern "C" {

size_t hisq_ptc_workspace_bytes(const hisq_lattice *lat) {
    if (check_lattice(lat) != HISQ_OK)
        return 0;
    return ptc_layout(make_geom(*lat)).total;
}

hisq_status hisq_ptc_forward(hisq_context *ctx, const hisq_lattice *lat, const void *links_f32, const void *weights,
                             const void *in_even, void *out_even, void *ws, size_t ws_bytes, void *stream) {
    Ptc P;
    hisq_status s = common_checks(lat, links_f32, weights, ws, ws_bytes, &P, ctx, stream);
    if (s == HISQ_OK) s = check_ptr(in_even, "in_even");
    if (s == HISQ_OK) s = check_ptr(out_even, "out_even");
    if (s != HISQ_OK)
        return s;
    const hipError_t e = forward(P, static_cast<const float2 *>(weights), in_even, out_even, true);
    return e == hipSuccess ? HISQ_OK : device_fail(e, "ptc forward");
}

hisq_status hisq_ptc_backward(hisq_context *ctx, const hisq_lattice *lat, const void *links_f32,
                              const void *weights, const void *g_out_even, void *g_in_even, void *grad, void *ws,
                              size_t ws_bytes, void *stream) {
    Ptc P;
    hisq_status s = common_checks(lat, links_f32, weights, ws, ws_bytes, &P, ctx, stream);
    if (s == HISQ_OK) s = check_ptr(g_out_even, "g_out_even");
    if (s == HISQ_OK) s = check_ptr(grad, "grad");
    if (s != HISQ_OK)
        return s;
    const hipError_t e = backward(P, static_cast<const float2 *>(weights), g_out_even, static_cast<double2 *>(grad),
                                  g_in_even);
    return e == hipSuccess ? HISQ_OK : device_fail(e, "ptc backward");
}

hisq_status hisq_ptc_adam_step(hisq_context *ctx, void *w_master, void *w_f32, const void *grad, void *m, void *v,
                               int32_t step, double lr, double beta1, double beta2, double eps, void *stream) {
    hisq_status s = check_ptr(w_master, "w_master");
    if (s == HISQ_OK) s = check_ptr(w_f32, "w_f32");
    if (s == HISQ_OK) s = check_ptr(grad, "grad");
    if (s == HISQ_OK) s = check_ptr(m, "m");
    if (s == HISQ_OK) s = check_ptr(v, "v");
    if (s == HISQ_OK && step < 1)
        s = fail(HISQ_ERR_INVALID_ARG, "step = %d must be >= 1", step);
    if (s == HISQ_OK && !(lr > 0.0 && beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && eps > 0.0))
        s = fail(HISQ_ERR_INVALID_ARG, "invalid Adam hyper-parameters");
    if (s == HISQ_OK) s = set_device(ctx);
    if (s != HISQ_OK)
        return s;
    const hipError_t e = ptc_adam(static_cast<double2 *>(w_master), static_cast<float2 *>(w_f32),
                                  static_cast<const double2 *>(grad), static_cast<double2 *>(m),
                                  static_cast<double2 *>(v), step, lr, beta1, beta2, eps,
                                  static_cast<hipStream_t>(stream));
    return e == hipSuccess ? HISQ_OK : device_fail(e, "ptc adam");
}

hisq_status hisq_ptc_train_step(hisq_context *ctx, const hisq_lattice *lat, double mass, const void *links_f32,
                                void *w_master, void *w_f32, void *m, void *v, int32_t step, int32_t batch,
                                const void *src_f32, const void *sol_f64, double lr, double beta1, double beta2,
                                double eps, double *loss, void *ws, size_t ws_bytes, void *stream) {
    Ptc P;
    hisq_status s = common_checks(lat, links_f32, w_f32, ws, ws_bytes, &P, ctx, stream);
    if (s == HISQ_OK) s = check_ptr(src_f32, "src_f32");
    if (s == HISQ_OK) s = check_ptr(sol_f64, "sol_f64");
    if (s == HISQ_OK && batch < 1)
        s = fail(HISQ_ERR_INVALID_ARG, "batch = %d must be >= 1", batch);
    if (s == HISQ_OK && (!std::isfinite(mass) || mass * mass <= 0.0))
        s = fail(HISQ_ERR_INVALID_ARG, "mass^2 must be positive (mass = %g)", mass);
    if (s != HISQ_OK)
        return s;
    const float2 *w = static_cast<const float2 *>(w_f32);
    double *sum = P.at<double>(P.L.scal);  // the loss
    float2 *w0 = P.at<float2>(P.L.keep0);  // the weights before the update
    double *K = P.at<double>(P.L.k);
    double2 *fold = P.at<double2>(P.L.fold);
    float2 *half = P.at<float2>(P.L.s);
    hipError_t e = ptc_fold(w, fold, w0, P.st);
    // PTC_COLS pairs at a time: the columns share every launch
    for (int k = 0; k < batch && e == hipSuccess; k += PTC_COLS) {
        const int n = batch - k < PTC_COLS ? batch - k : PTC_COLS;
        double *xb = P.at<double>(P.L.xb_part), *corr = P.at<double>(P.L.corr_part);
        e = ptc_spread(P.g, P.links, fold, src_f32, batch, k, n, half, P.st);
        if (e == hipSuccess)
            e = ptc_error(P.g, fold + PTC_C0, src_f32, batch, k, n, half, sol_f64, P.at<void>(P.L.e), xb, P.st);
        // A e = m^2 e - D_eo D_oe e (FP32 links) with <e, A e>
        const DslashShape shape = pick_shape(ctx, P.g, HISQ_FP32, HISQ_FP32, n);
        DslashParams prm{};
        prm.g = P.g;
        prm.nrhs = n;
        prm.links = P.links;
        prm.out_parity = 1;
        prm.in = P.at<void>(P.L.e);
        prm.out = P.at<void>(P.L.t);
        if (e == hipSuccess) e = launch_dslash(prm, HISQ_FP32, HISQ_FP32, EPI_PLAIN, shape, P.st);
        prm.out_parity = 0;
        prm.in = P.at<void>(P.L.t);
        prm.out = P.at<void>(P.L.ae);
        prm.y = P.at<void>(P.L.e);
        prm.ad = -1.0;
        prm.ay = mass * mass;
        prm.partials = P.at<double>(P.L.dot_part);
        prm.dot_out = nullptr;  // summed with the correlations
        if (e == hipSuccess) e = launch_dslash(prm, HISQ_FP32, HISQ_FP32, EPI_AXPY_DOT, shape, P.st);
        // the output gradient of pair k is 2 A e_k / (B <x_k, b_k>): A e_k here, the factor in the sum
        if (e == hipSuccess)
            e = ptc_correlate(P.g, P.links, src_f32, batch, k, P.at<void>(P.L.ae), n, corr, P.st);
        if (e == hipSuccess)
            e = ptc_correlate_sum(P.g, n, corr, k == 0, K, xb, 1.0 / batch, prm.partials,
                                  dslash_partial_blocks(P.g, shape), sum, P.st);
    }
    if (e == hipSuccess)
        e = ptc_chain_adam(w0, K, static_cast<double2 *>(w_master), static_cast<float2 *>(w_f32),
                           static_cast<double2 *>(m), static_cast<double2 *>(v), step, lr, beta1, beta2, eps, P.st);
    if (e == hipSuccess && loss) {
        e = hipMemcpyAsync(loss, sum, sizeof(double), hipMemcpyDeviceToHost, P.st);
        if (e == hipSuccess)
            e = hipStreamSynchronize(P.st);
    }
    return e == hipSuccess ? HISQ_OK : device_fail(e, "ptc train step");
}

}  // extern "C"
