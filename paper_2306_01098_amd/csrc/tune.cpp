// The Dslash autotuner: times every supported launch shape on the caller's
// buffers with HIP events and keeps the fastest per (extents, precisions,
// nrhs) in the context.
#include <algorithm>
#include <iterator>
#include <vector>

#include "api_util.hpp"
#include "dslash.hpp"

namespace hisq {

// Several right-hand sides below 49152 sites per parity, where a launch is a
// chain of loads, longer the more columns a thread carries, and a time per 1000
// sites and group of columns.  The two constants of each shape (microseconds)
// are those whose least sum picks best among the shapes as measured on 23
// lattices from 4^3x8 to 10x18x20x26 with 2 to 16 right-hand sides: within 1.5 %
// of the fastest on average (2 % FP32R12), at worst 20 %.  A launch time by
// itself is met within 10 to 15 % only.
struct ShapeCost {
    int variant, nin;
    double fixed, per;
};
constexpr ShapeCost COST_FP64[] = {{VAR_DIR, 1, 0.52, 0.3697},  {VAR_DIR, 2, 1.48, 0.4520},  {VAR_SITE, 1, 3.75, 0.1131},
                                   {VAR_SITE, 2, 4.74, 0.1673}, {VAR_SITE, 4, 7.44, 0.2526}, {VAR_LDS, 4, 7.65, 0.2481}};
constexpr ShapeCost COST_FP64R12[] = {{VAR_DIR, 1, 2.56, 0.2299},  {VAR_DIR, 2, 4.12, 0.2066},
                                      {VAR_SITE, 1, 4.62, 0.1034}, {VAR_SITE, 2, 4.99, 0.1417},
                                      {VAR_SITE, 4, 11.72, 0.2120}, {VAR_LDS, 4, 7.95, 0.2179}};
constexpr ShapeCost COST_FP32[] = {{VAR_DIR, 1, 1.95, 0.2409},  {VAR_DIR, 2, 2.53, 0.2152},  {VAR_SITE, 1, 4.31, 0.0634},
                                   {VAR_SITE, 2, 5.33, 0.0773}, {VAR_SITE, 4, 7.30, 0.1068}, {VAR_LDS, 4, 7.83, 0.0959}};
constexpr ShapeCost COST_FP32R12[] = {{VAR_DIR, 1, 2.26, 0.1771},  {VAR_DIR, 2, 3.60, 0.1360},
                                      {VAR_SITE, 1, 4.31, 0.0536}, {VAR_SITE, 2, 5.61, 0.0677},
                                      {VAR_SITE, 4, 7.74, 0.1036}, {VAR_LDS, 4, 8.77, 0.0894}};
constexpr ShapeCost COST_FP16[] = {{VAR_DIR, 1, 2.49, 0.0897}, {VAR_SITE, 1, 4.18, 0.0369}, {VAR_SITE, 2, 5.36, 0.0627}};

DslashShape small_multi_shape(const Geom &g, int lp, int fp, int nrhs) {
    const ShapeCost *c = COST_FP32;
    int n = (int)std::size(COST_FP32);
    if (fp == HISQ_FP64)
        c = lp == HISQ_FP64R12 ? COST_FP64R12 : COST_FP64;  // as many entries as COST_FP32
    else if (fp == HISQ_FP16N)
        c = COST_FP16, n = (int)std::size(COST_FP16);
    else if (lp == HISQ_FP32R12)
        c = COST_FP32R12;
    DslashShape best{};
    double least = 1e30;
    for (int k = 0; k < n; ++k) {
        // blocks of 64 in plain order: the z-slab order gains from 55000 sites on
        DslashShape s{c[k].variant, c[k].nin, 64, 1};
        if (s.variant == VAR_LDS)
            s = DslashShape{VAR_LDS, s.nin, LDS_BAND * g.hx, 2};
        else if (fp == HISQ_FP16N && s.nin == 2)
            s = DslashShape{VAR_SITE, 2, 256, g.nz % 8 == 0 ? 2 : 1};
        if (s.nin >= 2 * nrhs || (s.variant == VAR_LDS && (nrhs < 4 || !dslash_shape_fits(s, g, fp))))
            continue;
        if (lp == HISQ_FP16N && fp == HISQ_FP32 && (s.nin == 4 || (s.variant == VAR_SITE && s.nin == 2 && nrhs == 3)))
            continue;  // four: see large_multi_fp32; three columns, one / two a thread at 16^4: 20.5 / 23.1 us
        if (fp == HISQ_FP64 && lp != HISQ_FP64R12 && s.variant == VAR_SITE && s.nin == 1 && g.vh > 8192)
            continue;  // 13440 and 16384 sites, two and three columns: 8 to 25 % slower than two a thread
        const double t = c[k].fixed + c[k].per * 1e-3 * g.vh * ((nrhs + s.nin - 1) / s.nin);
        if (t < least) {
            least = t;
            best = s;
        }
    }
    return best;
}

// Several right-hand sides on larger lattices.  The lines lie between launches
// measured at 16 lattices from 49152 to 331776 sites with 2 to 16 right-hand
// sides (z-slab order in 8-row y-bands where N_z allows it); times below in
// microseconds.
//
// FP32 fields: groups of eight columns, or of four where that leaves fewer
// empty places, staged in LDS once links and vectors exceed the MALL (the
// neighbour rows then come from HBM), else through the caches.  16 rhs at
// 48^3x12, staged 4 / staged 8 / site 8: 414 / 380 / 425, FP32R12 355 / 340 /
// 379, FP32W14 402 / 369 / 411.  From ten columns staged in any case: a solver
// moves more between two launches (32^3x8 at 16 rhs, 60 iterations of CG: site 8
// 20.7 ms, staged 20.0); FP32W14 from seven (48x16^2x24, 8 rhs: site 4 59.2,
// staged 4 52.7; 32^3x8 43.0 / 42.6).
// Five and six columns within the MALL: two a thread with FP32R12 (48x16^2x24
// 41.6, site 8 50.1; 24^3x12 23.1 / 24.7), else eight, which saves a pass over
// the links (24^3x12, site 2 / 4 / 8: 28.5 / 36.0 / 27.1), but two below 73728
// sites (24x16^3 19.4 / 19.7 / 20.6, FP32W14 18.6 / 18.8 / 20.5).  FP32R12 beyond
// the MALL two a thread, staged (32^3x16, 2 / 4 / 8: 70.7 / 84.1 / 72.8), where that
// does not fit two below 262144 sites, eight above (site 2 / 8, 28x26x24x18 43.9 /
// 49.7, 44x36x28x14 107.0 / 101.6, 36^3x16 130.8 / 119.7).
// Three columns: two a thread, blocks of 64, between 43008 and 53248 sites (24x16^3,
// one / two / four a thread: 17.0 / 13.8 / 15.2; 10x18x20x26 16.8 / 12.8 / 13.6,
// FP32R12 13.9 / 12.2 / 13.7).
// FP16N links (both halves of the operator): two a thread, whose loads go out
// ahead of the arithmetic within 128 registers, staged in LDS where that fits,
// from 262144 sites four (48^2x24x12, staged 2 / staged 4 / site 8: 6 rhs 173 / 177 /
// 212; 16 rhs 416 / 367 / 462; 32^3x8, 16 rhs 138 / 152 / 173; 24^3x12, site 2 / 4 /
// 8: 6 rhs 47 / 57 / 56, 16 rhs 102 / 111 / 128).
DslashShape large_multi_fp32(const Geom &g, int lp, int nrhs) {
    const int remap = g.nz % 8 == 0 ? 2 : 1;
    const bool large = links_bytes(g, lp) + 2 * field_bytes(g, HISQ_FP32, nrhs) > MALL_BYTES;
    const bool r12 = lp == HISQ_FP32R12, five_six = nrhs == 5 || nrhs == 6;
    const auto staged = [&](int nin) { return DslashShape{VAR_LDS, nin, LDS_BAND * g.hx, 2}; };
    if (lp == HISQ_FP16N && nrhs >= 4) {
        const DslashShape l = staged(g.vh >= (1 << 18) && nrhs >= 7 ? 4 : 2);
        return dslash_shape_fits(l, g, HISQ_FP32) ? l : DslashShape{VAR_SITE, 2, 128, remap};
    }
    if (five_six && (r12 || g.vh < 73728)) {
        if (large && dslash_shape_fits(staged(2), g, HISQ_FP32))
            return staged(2);
        return DslashShape{VAR_SITE, g.vh >= (1 << 18) ? 8 : 2, 128, remap};
    }
    const bool eights = large && (nrhs + 7) / 8 * 8 - nrhs <= 3;  // 5 .. 8, 13 .. 16
    if (large || nrhs > 9 || (lp == HISQ_FP32W14 && nrhs >= 7)) {
        const DslashShape l = staged(nrhs == 2 ? 2 : eights ? 8 : 4);
        if (dslash_shape_fits(l, g, HISQ_FP32))
            return l;
        // (64x32^2x8, which fits four columns, not eight: staged 4 / site 8, 8
        // rhs 114 / 101, 16 rhs 225 / 225)
        if (eights && !r12)  // FP32R12, 16 rhs at 44x36x28x14: site 4 / 8 196 / 204
            return DslashShape{VAR_SITE, 8, g.vh >= (1 << 22) ? 256 : 128, remap};
    }
    if (five_six)
        return DslashShape{VAR_SITE, 8, 128, remap};
    // (9: 24^3x12 40.5 against 49 as 4 + 4 + 1; 3, FP32R12: 24^3x8, two / four 13.4 / 14.6)
    if (nrhs == 2 || (nrhs == 9 && !large) || (nrhs == 3 && r12 && g.vh < 73728))
        return DslashShape{VAR_SITE, 2, 128, remap};
    // blocks of 256: four columns, 24^3x8 128 / 256 16.0 / 14.9, but 24^3x12 22.1 / 24.1;
    // 14 columns, 24^3x8 36.0 / 34.5
    return DslashShape{VAR_SITE, 4, g.vh < 73728 || (nrhs > 4 && nrhs <= 12) ? 256 : 128, remap};
}

// FP64 fields: four columns a thread, staged in LDS once the links exceed the
// MALL (48^3x12 and 32^3x8, 16 rhs, site 4 / staged 4: FP64 918 / 906, 203 / 190;
// 8 rhs 538 / 519, 117 / 111; 16 rhs FP64R12 834 / 749, FP64W14 890 / 870, 196 /
// 179).  Where groups of four would be half empty (5, 6, 9, 10, 13, 14): two a
// thread while the links leave room for the vectors in the MALL (24^3x12, 14
// rhs, two / four: 103 / 114; 6 rhs FP64R12 45 / 57), beyond that four (30x28x26x10,
// 9 rhs: 130 / 107, FP64W14 112 / 97, 6 rhs 87 / 82) and five and six eight, in
// registers beyond the first 256, which saves a pass over the links (30x28x26x10,
// 6 rhs 79; 48^3x12 468 / 406); FP64R12 staged or, where that does not fit, four
// in blocks of 64 (28x26x24x18, 9 rhs, two / four 153 / 133; five and six columns
// stay two a thread up to 256 MB of links: 48x16^2x24, 6 rhs 91 / 98).
DslashShape large_multi_fp64(const Geom &g, int lp, int nrhs) {
    const int remap = g.nz % 8 == 0 ? 2 : 1;
    // (two at 18x16x18x14: blocks of 128 19.6 us, of 64 15.2; 24^3x12 34.6 / 35.6)
    const DslashShape four{VAR_SITE, nrhs == 2 ? 2 : 4, nrhs == 2 && g.vh < 65536 ? 64 : 128, remap};
    if (nrhs <= 3)  // three as one group of four: 24^3x12 57 -> 42 us
        return four;
    const bool r12 = lp == HISQ_FP64R12, half = nrhs % 4 == 1 || nrhs % 4 == 2;
    const size_t links = links_bytes(g, lp);
    const DslashShape l{VAR_LDS, 4, LDS_BAND * g.hx, 2};
    const bool fits = dslash_shape_fits(l, g, HISQ_FP64);
    if (half) {
        if (links < (r12 && nrhs <= 6 ? MALL_BYTES : (size_t)200000000))
            return DslashShape{VAR_SITE, 2, 64, r12 ? remap : 1};
        if (nrhs <= 6 && !r12)
            return DslashShape{VAR_SITE, 8, 128, remap};
        if (r12 && fits)
            return l;
        return links < MALL_BYTES || r12 ? DslashShape{VAR_SITE, 4, 64, 1} : four;
    }
    return links >= MALL_BYTES && fits ? l : four;
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
        // blocks of 256: up to 24576 sites per parity (49152 for FP32 and
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
    // The smallest lattices that the LDS staging fits keep it by contract, not for
    // its speed: 16x8x8x8, 6 FP32 columns 10.0 us and 31.7 ms in a CG solve against
    // 5.0 and 21.7 by the cost table (16 columns 8.9 and 30.5 against 8.8 and 31.4).
    const DslashShape staged{VAR_LDS, 4, LDS_BAND * g.hx, 2};
    if (fp == HISQ_FP32 && nrhs >= 4 && g.vh <= 4096 && dslash_shape_fits(staged, g, fp))
        return staged;
    if (fp == HISQ_FP32 && nrhs == 3 && g.vh >= 43008 && g.vh < 53248)  // see large_multi_fp32
        return DslashShape{VAR_SITE, 2, 64, 1};
    if (g.vh < 49152)
        return small_multi_shape(g, lp, fp, nrhs);
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
