// The Dslash autotuner: times every supported launch shape on the caller's
// buffers with HIP events and keeps the fastest per (extents, precisions,
// nrhs) in the context.
#include <algorithm>
#include <iterator>
#include <vector>

#include "api_util.hpp"
#include "dslash.hpp"

namespace hisq {

// Launch time of a shape on a lattice of a few ten thousand sites per parity:
// the latency of its chain of loads, which grows with the right-hand sides a
// thread carries, and a time per 1000 sites and group of right-hand sides
// (microseconds, fitted to 14 lattices from 4^4 to 48^3x12 at 1 to 16
// right-hand sides; within 10 % of nearly all of them below 49152 sites).
struct ShapeCost {
    int variant, nin;
    double fixed, per;
};
constexpr ShapeCost COST_FP64[] = {{VAR_DIR, 1, 3.5, 0.239}, {VAR_DIR, 2, 4.1, 0.34},  {VAR_SITE, 1, 4.8, 0.129},
                                   {VAR_SITE, 2, 6.3, 0.184}, {VAR_SITE, 4, 9.7, 0.295}};
constexpr ShapeCost COST_FP32[] = {{VAR_DIR, 1, 3.5, 0.148}, {VAR_DIR, 2, 3.8, 0.16},   {VAR_SITE, 1, 4.8, 0.06},
                                   {VAR_SITE, 2, 6.2, 0.083}, {VAR_SITE, 4, 8.7, 0.141}, {VAR_LDS, 4, 8.2, 0.135}};
constexpr ShapeCost COST_FP16[] = {{VAR_DIR, 1, 3.5, 0.074}, {VAR_SITE, 1, 4.4, 0.036}};

// Several right-hand sides on a lattice that one thread per site and group of
// right-hand sides spreads over too few wavefronts.
DslashShape small_multi_shape(const Geom &g, int fp, int nrhs) {
    const ShapeCost *c = fp == HISQ_FP64 ? COST_FP64 : fp == HISQ_FP32 ? COST_FP32 : COST_FP16;
    const int n = fp == HISQ_FP64 ? (int)std::size(COST_FP64)
                  : fp == HISQ_FP32 ? (int)std::size(COST_FP32) : (int)std::size(COST_FP16);
    DslashShape best{};
    double least = 1e30;
    for (int k = 0; k < n; ++k) {
        DslashShape s{c[k].variant, c[k].nin, 64, 1};
        if (s.variant == VAR_LDS)
            s = DslashShape{VAR_LDS, s.nin, LDS_BAND * g.hx, 2};
        else if (fp == HISQ_FP16N && s.variant == VAR_SITE && g.vh >= 16384)
            s.block = 256;
        if (s.nin >= 2 * nrhs || (s.variant == VAR_LDS && (nrhs < 4 || !dslash_shape_fits(s, g, fp))))
            continue;
        if (fp == HISQ_FP64 && s.variant == VAR_SITE && s.nin == 1 && g.vh > 8192)
            continue;  // 12288 and 16800 sites: 10-30 % slower than two a thread
        if (s.variant == VAR_SITE && g.vh >= 32768 && g.nz % 8 == 0)
            s.xcd_remap = 2;
        const double t = c[k].fixed + c[k].per * 1e-3 * g.vh * ((nrhs + s.nin - 1) / s.nin);
        if (t < least) {
            least = t;
            best = s;
        }
    }
    return best;
}

// Several right-hand sides on lattices that fill the chip.  The lines lie
// between measured launches at 48^3x12, 32^3x8, 24^3x12 (times below in this
// order; z-slab order in 8-row y-bands where N_z allows it), a few at 20^3x24,
// 32^3x16, 48^3x8, 32^2x48x12, 32^2x64x8, 48^2x32x8, 64x32^2x8 and 64^3x6.
//
// FP32 fields: groups of eight columns, or of four where that leaves fewer
// empty places, staged in LDS once links and vectors exceed the MALL (the
// neighbour rows then come from HBM), else through the caches:
// FP32 links, 16 rhs: staged 4 / staged 8 / site 8: 414 / 380 / 425, 79 / 84 /
// 72, - / - / 54 us; 8 rhs: 251 / 212 / 238, 46 / 47 / 43 and site 4 41, site 4
// / 8 31 / 36; 5 rhs staged 8 190, site 8 205; 40; 26.  FP32R12 links, 16 rhs:
// 355 / 340 / 379, 70 / 77 / 69; FP32W14 402 / 369 / 411, 79 / 81 / 72.
DslashShape large_multi_fp32(const Geom &g, int lp, int nrhs) {
    const int remap = g.nz % 8 == 0 ? 2 : 1;
    const bool large = links_bytes(g, lp) + 2 * field_bytes(g, HISQ_FP32, nrhs) > MALL_BYTES;
    const int eights = (nrhs + 7) / 8 * 8 - nrhs <= 3;  // 5 .. 8, 13 .. 16
    // (from ten columns staged in any case: a solver moves more between two
    // launches; 32^3x8 at 16 rhs is not large by itself, 72 us with eight through
    // the caches, but 60 iterations of its CG take 20.7 ms then and 20.0 staged)
    if (large || nrhs > 9) {
        const DslashShape l{VAR_LDS, nrhs == 2 ? 2 : eights && large ? 8 : 4, LDS_BAND * g.hx, 2};
        if (dslash_shape_fits(l, g, HISQ_FP32))
            return l;
        // (64x32^2x8, which fits four columns, not eight: staged 4 / site 8, 8
        // rhs 114 / 101, 16 rhs 225 / 225)
        if (eights && large && lp != HISQ_FP32R12)  // FP32R12, 16 rhs at 44x36x28x14: site 4 / 8 196 / 204
            return DslashShape{VAR_SITE, 8, g.vh >= (1 << 22) ? 256 : 128, remap};
    }
    if (nrhs == 5 || nrhs == 6)
        return DslashShape{VAR_SITE, 8, 128, remap};
    if (nrhs == 2 || (nrhs == 9 && !large))  // 9: 40.5 us against 49 as 4 + 4 + 1
        return DslashShape{VAR_SITE, 2, 128, remap};
    return DslashShape{VAR_SITE, 4, nrhs <= 4 || nrhs > 12 ? 128 : 256, remap};
}

// FP64 fields: four columns a thread, staged in LDS once the links exceed the
// MALL (16 rhs, site 4 / staged 4: FP64 918 / 906, 203 / 190 us; 8 rhs 538 / 519,
// 117 / 111; 16 rhs FP64R12 834 / 749, FP64W14 890 / 870, 196 / 179).  Five and
// six: eight a thread, in registers beyond the first 256, which saves a pass
// over the links (6 rhs, site 4 / 8: 468 / 406, 100 / 84; 8 rhs gained at two
// lattices and lost at 24x16x32x44, 236 / 263).  Links within the MALL: two a
// thread where groups of four would be half empty (6 rhs at 24^3x12: 65 / 55,
// FP64R12 57 / 45; 14 rhs 112 / 100, 104 / 85, on small lattices only: 32^3x8
// FP64R12 153 / 164).
DslashShape large_multi_fp64(const Geom &g, int lp, int nrhs) {
    const int remap = g.nz % 8 == 0 ? 2 : 1;
    // (two at 18x16x18x14: blocks of 128 19.6 us, of 64 15.2; 24^3x12 34.6 / 35.6)
    const DslashShape four{VAR_SITE, nrhs == 2 ? 2 : 4, nrhs == 2 && g.vh < 65536 ? 64 : 128, remap};
    const bool half = nrhs % 4 == 1 || nrhs % 4 == 2;
    if (nrhs <= 3)  // three as one group of four: 24^3x12 57 -> 42 us
        return four;
    if (links_bytes(g, lp) < MALL_BYTES)
        return half && (nrhs <= 10 || g.vh < 98304) ? DslashShape{VAR_SITE, 2, 64, remap} : four;
    if (lp != HISQ_FP64R12 && (nrhs == 5 || nrhs == 6))
        return DslashShape{VAR_SITE, 8, 128, remap};
    if (lp != HISQ_FP64R12 && nrhs > 4 && half)  // 14 rhs, site 4 / staged 4: 821 / 864
        return four;
    const DslashShape l{VAR_LDS, 4, LDS_BAND * g.hx, 2};
    return dslash_shape_fits(l, g, HISQ_FP64) ? l : four;
}

// FP16N fields: two columns a thread; two and three columns one by one below
// 262144 sites (2 rhs, one / two: 32^3x8 15.1 / 19.5 us, 48^3x12 - / 87).
DslashShape large_multi_fp16(const Geom &g, int nrhs) {
    return DslashShape{VAR_SITE, nrhs <= 3 && g.vh < 262144 ? 1 : 2, 256, g.nz % 8 == 0 ? 2 : 1};
}

// Built-in shapes (measured on MI355X): one thread per site (four lanes per
// site on lattices too small to fill the chip); with several right-hand sides
// large_multi_*, on small lattices small_multi_shape.
DslashShape default_shape(const Geom &g, int lp, int fp, int nrhs) {
    // At one right-hand side the z-slab block order (when N_z allows it) keeps
    // the t-hops inside each XCD: 32^3x8 FP64 53.1 -> 48.1 us.
    DslashShape s;
    s.variant = VAR_SITE;
    s.xcd_remap = 1;
    if (nrhs == 1) {
        s.nin = 1;
        // Small lattices cannot fill 256 CUs with one thread per site in
        // blocks of 256: up to 16384 sites per parity (49152 for FP32 and
        // FP16N links) four lanes per site (8^4 .. 16^3x8: 9.6-16.1 -> 9.2-9.3
        // us FP64; 16^4 FP32 12.2 -> 9.4 us), below 131072 blocks of 64
        // (24^3x6 FP64 19.4 -> 16.6 us).  FP64 at 20x12x14x10 (16800): 12.5 ->
        // 9.0 us, FP64R12 9.6 -> 7.5; at 32768 the two tie.
        const bool wide = lp == HISQ_FP64 || lp == HISQ_FP64R12 || lp == HISQ_FP64W14;
        if (g.vh <= (wide ? 24576 : 49152)) {
            s.variant = VAR_DIR;
            // inside the CG graph blocks of 64 spread these lattices over more
            // CUs (8^4 FP64 CG 17.3 -> 15.6 ms; the isolated launch is the same)
            s.block = 64;
            return s;
        }
        if (g.vh < 131072) {
            s.block = 64;
            s.xcd_remap = g.nz % 8 == 0 ? 2 : 1;
            return s;
        }
        if (g.nz % 8 == 0) {
            // FP16N links too: the CG's fused scalar step sums 4x fewer block
            // partials (32^3x8 FP16N-link CG 7.53 -> 7.41 ms; the Dslash alone
            // the same within 1 %)
            s.xcd_remap = 2;
            s.block = 256;
        } else {
            s.block = 128;
        }
        return s;
    }
    // 5 and 16 rhs at 8^4: FP32 11.0 -> 4.6 and 18.4 -> 5.8 us, FP64 13.0 -> 5.8
    // and 13.2 -> 6.7; 3 rhs at 20x12x14x10: FP32 9.0 -> 7.7, FP16N 11.2 ->
    // 5.2.  From 49152 sites (FP64: 32768) the shapes below are as fast.  The
    // smallest lattices that the LDS staging fits (16x8x8x8) keep it: the
    // solver's test of the staged kernels runs there.
    const bool staged = fp == HISQ_FP32 && nrhs >= 4 && g.vh <= 4096 &&
                        dslash_shape_fits(DslashShape{VAR_LDS, 4, LDS_BAND * g.hx, 2}, g, fp);
    // three FP32 columns: two a thread from 40960 sites (one / two: FP32 links
    // 16x8x32x22 16.8 / 14.1 us, FP32R12 10x18x20x26 14.0 / 12.2, 16^3x22 13.8 /
    // 12.4, at 14^2x18x20 11.0 / 11.5)
    if (fp == HISQ_FP32 && nrhs == 3 && g.vh >= 40960 && g.vh < 49152)
        return DslashShape{VAR_SITE, 2, 128, g.nz % 8 == 0 ? 2 : 1};
    if (!staged && g.vh < (fp == HISQ_FP64 ? 32768 : 49152))
        return small_multi_shape(g, fp, nrhs);
    if (staged)
        return DslashShape{VAR_LDS, 4, LDS_BAND * g.hx, 2};
    return fp == HISQ_FP64   ? large_multi_fp64(g, lp, nrhs)
           : fp == HISQ_FP32 ? large_multi_fp32(g, lp, nrhs)
                             : large_multi_fp16(g, nrhs);
}

std::vector<DslashShape> candidate_shapes(const Geom &g, int nrhs, int lp, int fp) {
    std::vector<DslashShape> out;
    // LDS-staged neighbours: one block per piece of rows, block size fixed
    // by N_x, z-slab order
    for (int nin : {1, 2, 4, 8}) {
        const DslashShape s{VAR_LDS, nin, LDS_BAND * g.hx, 2};
        if (nin <= nrhs && dslash_shape_fits(s, g, fp) &&
            !((lp == HISQ_FP64 || lp == HISQ_FP64R12 || lp == HISQ_FP64W14) && nin > 4))
            out.push_back(s);
    }
    for (int var : {VAR_SITE, VAR_DIR, VAR_HOP})
        for (int nin : {1, 2, 4, 8}) {
            if (nin > 1 && nin > nrhs)
                continue;
            if (var == VAR_HOP && nin > 2)
                continue;
            for (int block : {64, 128, 256})
                for (int remap : {0, 1, 2})
                    if (remap != 2 || g.nz % 8 == 0)
                        out.push_back(DslashShape{var, nin, block, remap});
        }
    return out;
}

// Median time (ms) of `reps` launches of one shape; <0 on a launch error.
static float time_shape(const DslashParams &prm, int lp, int fp, DslashShape s, hipStream_t st, int reps,
                        hipEvent_t e0, hipEvent_t e1, hipError_t *err) {
    std::vector<float> t;
    for (int k = 0; k < 2; ++k) {  // warm-up
        *err = launch_dslash(prm, lp, fp, EPI_PLAIN, s, st);
        if (*err != hipSuccess)
            return -1.f;
    }
    for (int k = 0; k < reps; ++k) {
        hipEventRecord(e0, st);
        *err = launch_dslash(prm, lp, fp, EPI_PLAIN, s, st);
        hipEventRecord(e1, st);
        if (*err != hipSuccess)
            return -1.f;
        *err = hipEventSynchronize(e1);
        if (*err != hipSuccess)
            return -1.f;
        float ms = 0.f;
        hipEventElapsedTime(&ms, e0, e1);
        t.push_back(ms);
    }
    std::sort(t.begin(), t.end());
    return t[t.size() / 2];
}

hisq_status tune_dslash(hisq_context *ctx, const Geom &g, int lp, int fp, int nrhs, const void *links,
                        const void *in, void *out, hipStream_t st, DslashShape *best_out) {
    DslashParams prm{};
    prm.g = g;
    prm.out_parity = 0;
    prm.nrhs = nrhs;
    prm.links = static_cast<const char *>(links);
    prm.in = in;
    prm.out = out;
    hipEvent_t e0, e1;
    hipError_t e = hipEventCreate(&e0);
    if (e != hipSuccess)
        return device_fail(e, "hipEventCreate");
    e = hipEventCreate(&e1);
    if (e != hipSuccess) {
        hipEventDestroy(e0);
        return device_fail(e, "hipEventCreate");
    }
    DslashShape best = default_shape(g, lp, fp, nrhs);
    float best_ms = 1e30f;
    hisq_status status = HISQ_OK;
    for (const DslashShape &s : candidate_shapes(g, nrhs, lp, fp)) {
        hipError_t err = hipSuccess;
        const float ms = time_shape(prm, lp, fp, s, st, 5, e0, e1, &err);
        if (err != hipSuccess) {
            status = device_fail(err, "tune_dslash");
            break;
        }
        if (ms < best_ms) {
            best_ms = ms;
            best = s;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (status != HISQ_OK)
        return status;
    ctx->store(g, lp, fp, nrhs, best);
    if (best_out)
        *best_out = best;
    return HISQ_OK;
}

}  // namespace hisq

using namespace hisq;

extern "C" {

hisq_status hisq_tune_dslash(hisq_context *ctx, const hisq_lattice *lat, hisq_prec prec, int32_t nrhs,
                             const void *links, const void *in, void *out, void *stream) {
    if (!ctx)
        return fail(HISQ_ERR_INVALID_ARG, "ctx is NULL (the tuned shape is kept in the context)");
    hisq_status s = check_lattice(lat);
    if (s == HISQ_OK) s = check_prec(prec);
    if (s == HISQ_OK) s = check_nrhs(nrhs);
    if (s == HISQ_OK) s = check_ptr(links, "links");
    if (s == HISQ_OK) s = check_ptr(in, "in");
    if (s == HISQ_OK) s = check_ptr(out, "out");
    if (s == HISQ_OK && in == out)
        s = fail(HISQ_ERR_INVALID_ARG, "in and out must not alias");
    if (s == HISQ_OK) s = set_device(ctx);
    if (s != HISQ_OK)
        return s;
    return tune_dslash(ctx, make_geom(*lat), prec, field_prec_of(prec), nrhs, links, in, out, static_cast<hipStream_t>(stream),
                       nullptr);
}

hisq_status hisq_get_dslash_shape(hisq_context *ctx, const hisq_lattice *lat, hisq_prec prec, int32_t nrhs,
                                  hisq_dslash_shape *shape) {
    hisq_status s = check_lattice(lat);
    if (s == HISQ_OK) s = check_prec(prec);
    if (s == HISQ_OK) s = check_nrhs(nrhs);
    if (s == HISQ_OK) s = check_ptr(shape, "shape");
    if (s != HISQ_OK)
        return s;
    const DslashShape d = pick_shape(ctx, make_geom(*lat), prec, field_prec_of(prec), nrhs);
    shape->variant = d.variant;
    shape->nin = d.nin;
    shape->block = d.block;
    shape->xcd_remap = d.xcd_remap;
    return HISQ_OK;
}

hisq_status hisq_set_dslash_shape(hisq_context *ctx, const hisq_lattice *lat, hisq_prec prec, int32_t nrhs,
                                  const hisq_dslash_shape *shape) {
    if (!ctx)
        return fail(HISQ_ERR_INVALID_ARG, "ctx is NULL");
    hisq_status s = check_lattice(lat);
    if (s == HISQ_OK) s = check_prec(prec);
    if (s == HISQ_OK) s = check_nrhs(nrhs);
    if (s == HISQ_OK) s = check_ptr(shape, "shape");
    if (s != HISQ_OK)
        return s;
    DslashShape d{shape->variant, shape->nin, shape->block, shape->xcd_remap};
    if (d.variant == VAR_LDS) {  // block size and order follow from the lattice
        const Geom g = make_geom(*lat);
        d.block = LDS_BAND * g.hx;
        d.xcd_remap = 2;
        const int fp = prec == HISQ_FP16N ? HISQ_FP32 : field_prec_of(prec);
        if (!dslash_shape_fits(d, g, fp))
            return fail(HISQ_ERR_INVALID_ARG,
                        "the LDS-staged Dslash needs N_z and N_y divisible by 8, N_x in {16, 32, 48, 64}, FP64 or "
                        "FP32 fields and at most 64 KiB of staging for nin = %d",
                        d.nin);
    }
    if (!dslash_shape_supported(d))
        return fail(HISQ_ERR_INVALID_ARG, "unsupported shape (variant %d, nin %d, block %d, remap %d)", d.variant,
                    d.nin, d.block, d.xcd_remap);
    if (!dslash_shape_fits(d, make_geom(*lat)))
        return fail(HISQ_ERR_INVALID_ARG, "block order 2 needs N_z divisible by 8 (N_z = %d)", lat->dims[2]);
    ctx->store(make_geom(*lat), prec, field_prec_of(prec), nrhs, d);
    if (prec == HISQ_FP16N)  // also the FP16-link, FP32-field Dslash inside mixed-precision CG
        ctx->store(make_geom(*lat), prec, HISQ_FP32, nrhs, d);
    return HISQ_OK;
}

}  // extern "C"
