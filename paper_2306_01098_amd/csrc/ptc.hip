// PTC network kernels: the network as a folded linear map, its gradient, the
// training loss and Adam.  FP32 fields, FP64 reductions.
//
// The network is linear in its input and its weights do not depend on the
// site, its input lives on the even sites and only the even sites of its output
// are read, and every path is the identity or one hop.  So of all products of
// three paths only those with no hop or with two remain, and the network is
//   out(x) = c0 in(x) + sum_p' T_p' u_p'(x),   u_p'(y) = sum_p C[p'][p] (T_p in)(y)
// over the eight hops p, p' and the odd sites y, with (paths 0 = identity)
//   c0       = sum_dc w3[d][0] w2[d][c][0] w1[c][0]
//   C[p'][p] = sum_dc ( w3[d][0] w2[d][c][p'] w1[c][p] + w3[d][p'] w2[d][c][0] w1[c][p]
//                     + w3[d][p'] w2[d][c][p] w1[c][0] ).
// The folding (FP64, from the FP32 weights, once per call) replaces the layers
// 1 -> 8 -> 8 -> 1: a site takes 192 complex multiply-adds instead of about
// 2000, and no 8-channel activation is written.  C and c0 stay FP64 and are
// applied in FP64: a product of three weights may lie outside the range of FP32
// where every activation of the layers lies inside.  The gradient with respect to
// C and c0 is one 8 x 8 correlation over the odd sites,
//   K[p'][p] = sum_y <(T_p in)(y), (T_p'^+ g)(y)>,   K0 = sum_x <in(x), g(x)>,
// and the gradients of the 720 weights follow from it by the chain rule.
//
// Bound: memory.  At 32^4 the forward pass reads the links once (302 MB),
// writes and reads the eight half-lattice vectors (101 MB in all, each way) and
// takes 118 to 127 us (fold 5, spread 86, 4.8 TB/s, gather 24, 4.8 TB/s); layer by
// layer it took 753 us, 460 of them FP32 arithmetic of the 8 -> 8 layer.  The
// backward pass with input gradient 2.2 ms -> 208 us (correlation 81); training
// on four pairs at 16^4 1656 -> 132 us, small lattices bound by the launches.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dslash.hpp"
#include "internal.hpp"
#include "ptc.hpp"
#include "reduce.hpp"

namespace hisq {

namespace {

constexpr int PB = PTC_BLOCK;
constexpr int NHOP = PTC_PATHS - 1;  // hop 2 mu: +mu, 2 mu + 1: -mu; the adjoint of hop q is hop q ^ 1

// Hop q of the odd site i: the even site it reads and its link.
struct Hop {
    int nb;
    int lblk, lidx;  // link parity block and index
    float sg;        // boundary sign
};

__device__ __forceinline__ Hop odd_hop(const Geom &g, const Site &s, int i, int q) {
    const int mu = q >> 1;
    const bool fwd = (q & 1) == 0;
    const int c = mu == 0 ? s.x : mu == 1 ? s.y : mu == 2 ? s.z : s.t;
    const int n = mu == 0 ? g.nx : mu == 1 ? g.ny : mu == 2 ? g.nz : g.nt;
    const int stride = mu == 1 ? g.hx : mu == 2 ? g.hx * g.ny : g.hx * g.ny * g.nz;
    Hop h;
    neighbour<float>(g, i, c, n, stride, mu, fwd ? +1 : -1, h.nb, h.sg);
    h.lblk = fwd ? 1 : 0;
    h.lidx = fwd ? i : h.nb;
    return h;
}

// t = m v, or m^+ v
template <bool ADJ>
__device__ __forceinline__ void transport(const float (&m)[18], const cplx<float> (&v)[3], cplx<float> (&t)[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        t[a].re = t[a].im = 0.f;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (!ADJ)
                cmac(t[a], m[6 * a + 2 * b], m[6 * a + 2 * b + 1], v[b]);
            else
                cmac_conj(t[a], m[6 * b + 2 * a], m[6 * b + 2 * a + 1], v[b]);
        }
    }
}

// The link times the boundary sign of its hop.
__device__ __forceinline__ void load_link(const char *links, int vh, int mu, const Hop &h, float (&m)[18]) {
    LinkIO<HISQ_FP32>::load<false>(links + link_block<HISQ_FP32>(0, h.lblk, mu, vh), vh, h.lidx, m);
#pragma unroll
    for (int k = 0; k < 18; ++k)
        m[k] *= h.sg;
}

// Site block of this workgroup: XCD b mod 8 takes a contiguous range of sites.
__device__ __forceinline__ int site_block() {
    const int b = blockIdx.x, G = gridDim.x, q = G >> 3, r = G & 7, k = b & 7;
    return k * q + min(k, r) + (b >> 3);
}

__device__ __forceinline__ double2 dmul(double2 a, double2 b) {
    return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ void dmac(double2 &s, double2 a, double2 b) {
    s.x = fma(a.x, b.x, fma(-a.y, b.y, s.x));
    s.y = fma(a.x, b.y, fma(a.y, b.x, s.y));
}
__device__ __forceinline__ double2 wide(float2 a) { return make_double2(a.x, a.y); }

// The weights in shared memory, NT threads.
template <int NT> __device__ __forceinline__ void stage_weights(const float2 *w, float2 *lds) {
    for (int k = threadIdx.x; k < PTC_NW; k += NT)
        lds[k] = w[k];
    __syncthreads();
}

__device__ __forceinline__ double2 w1_(const float2 *w, int c, int p) { return wide(w[PTC_W1 + c * PTC_PATHS + p]); }
__device__ __forceinline__ double2 w2_(const float2 *w, int d, int c, int p) {
    return wide(w[PTC_W2 + (d * PTC_CH + c) * PTC_PATHS + p]);
}
__device__ __forceinline__ double2 w3_(const float2 *w, int d, int p) { return wide(w[PTC_W3 + d * PTC_PATHS + p]); }

// The folded map: fold[8 p' + p] = C[p'][p] and fold[64] = c0; the adjoint
// network in the same form, C'[p'][p] = conj(C[p ^ 1][p' ^ 1]), at fold + 65.
// Eight lanes (the channel d) per entry.  keep (nullable): a copy of the
// weights.
__global__ void __launch_bounds__(576) fold_kernel(const float2 *weights, double2 *fold, float2 *keep,
                                                   const int *skip) {
    if (skip && *skip)
        return;
    __shared__ float2 w[PTC_NW];
    stage_weights<576>(weights, w);
    if (keep)
        for (int k = threadIdx.x; k < PTC_NW; k += 576)
            keep[k] = w[k];
    const int e = threadIdx.x >> 3, d = threadIdx.x & 7;
    const int po = (e >> 3) + 1, pi = (e & 7) + 1;  // paths of the outer and the inner hop
    double2 sum = make_double2(0.0, 0.0);
    if (e < 64) {
        double2 a = make_double2(0.0, 0.0), b = a;
        for (int c = 0; c < PTC_CH; ++c) {
            dmac(a, w2_(w, d, c, po), w1_(w, c, pi));
            dmac(b, w2_(w, d, c, 0), w1_(w, c, pi));
            dmac(b, w2_(w, d, c, pi), w1_(w, c, 0));
        }
        dmac(sum, w3_(w, d, 0), a);
        dmac(sum, w3_(w, d, po), b);
    } else if (e == 64) {
        double2 a = make_double2(0.0, 0.0);
        for (int c = 0; c < PTC_CH; ++c)
            dmac(a, w2_(w, d, c, 0), w1_(w, c, 0));
        dmac(sum, w3_(w, d, 0), a);
    }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) {
        sum.x += __shfl_xor(sum.x, o, 64);
        sum.y += __shfl_xor(sum.y, o, 64);
    }
    if (d != 0 || e > 64)
        return;
    fold[e] = sum;
    fold[65 + (e < 64 ? 8 * ((e & 7) ^ 1) + ((e >> 3) ^ 1) : 64)] = make_double2(sum.x, -sum.y);
}

// Two wavefronts spread 64 odd sites, one with the hops in x and y and one with
// those in z and t: four links a thread.  With all eight hops in a thread the
// links and vectors take over 256 VGPRs and one wavefront per SIMD is left (118
// us at 32^4 instead of 86).
constexpr int CS = PB / 2;  // sites of a block

// First half of the folded network on the odd sites y: the transported vectors
// t_p = T_p in, for every hop p' the combination u_p', and s_p' = T_p' u_p'
// delivered to the even site that reads it, through the link that t of the
// adjoint hop was formed with.  The links stay in registers, so each link of
// the lattice is read once.  C t is summed in FP64, one p at a time with t_p
// from LDS: with the eight vectors in registers the kernel takes 228 VGPRs and
// two wavefronts run on a SIMD instead of three (forward at 32^4 125 us; 118 so
// and 118 with C in FP32).  Columns col0 + nper blockIdx.y ... of the
// ncol-column field `in`, nper of them in a thread, each to s + column * 24 vh.
__global__ void __launch_bounds__(PB) spread_kernel(Geom g, const char *links, const double2 *fold, const void *in,
                                                    int ncol, int col0, int nper, int ncols, float2 *s,
                                                    const int *skip) {
    if (skip && *skip)
        return;
    __shared__ float2 lds[PB / 64][12][64];  // t_p: four of a site's in one wavefront, four in the other
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave & 1;
    const int i = site_block() * CS + (wave >> 1) * 64 + (threadIdx.x & 63);
    const bool valid = i < g.vh;
    const Site st = site_coords(g, 1, valid ? i : 0);
    Hop h[4];
    float m[4][18];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        h[l] = odd_hop(g, st, valid ? i : 0, 4 * half + l);
        load_link(links, g.vh, 2 * half + (l >> 1), h[l], m[l]);
    }
    const int j1 = min((int)(blockIdx.y + 1) * nper, ncols);
    for (int j = blockIdx.y * nper; j < j1; ++j) {
        cplx<float> t[4][3];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            cplx<float> v[3];
            FieldIO<HISQ_FP32>::template load<float>(in, g.vh, ncol, col0 + j, h[l].nb, v);
            if (l & 1)
                transport<true>(m[l], v, t[l]);
            else
                transport<false>(m[l], v, t[l]);
        }
        __syncthreads();  // the vectors of the previous column have been read
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
            for (int a = 0; a < 3; ++a)
                lds[wave][3 * l + a][threadIdx.x & 63] = make_float2(t[l][a].re, t[l][a].im);
        __syncthreads();
        if (!valid)
            continue;
        float2 *sj = s + (size_t)j * 24 * g.vh;
        cplx<double> acc[4][3];  // u of the four hops p' that go over this thread's links
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
            for (int a = 0; a < 3; ++a)
                acc[l][a].re = acc[l][a].im = 0.0;
#pragma unroll 1
        for (int p = 0; p < NHOP; ++p) {
            cplx<double> v[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float2 e = lds[(wave & ~1) + (p >> 2)][3 * (p & 3) + a][threadIdx.x & 63];
                v[a].re = e.x;
                v[a].im = e.y;
            }
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const double2 c = fold[8 * (4 * half + (l ^ 1)) + p];
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    cmac(acc[l][a], c.x, c.y, v[a]);
            }
        }
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int po = 4 * half + (l ^ 1);  // the hop p' whose vector goes over this link
            cplx<float> u[3], r[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                u[a].re = (float)acc[l][a].re;
                u[a].im = (float)acc[l][a].im;
            }
            if (l & 1)
                transport<false>(m[l], u, r);
            else
                transport<true>(m[l], u, r);
            float2 *dst = sj + (size_t)po * 3 * g.vh + h[l].nb;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                dst[(size_t)a * g.vh] = make_float2(r[a].re, r[a].im);
        }
    }
}

// c0 in + sum_p s_p of one element (FP64: the kernels wait for memory)
__device__ __forceinline__ double2 gathered(const double2 *c0, float2 in, const float2 *s, size_t stride) {
    float2 v[NHOP];
#pragma unroll
    for (int p = 0; p < NHOP; ++p)
        v[p] = s[p * stride];
    double2 r = dmul(*c0, wide(in));
#pragma unroll
    for (int p = 0; p < NHOP; ++p) {
        r.x += v[p].x;
        r.y += v[p].y;
    }
    return r;
}

// Second half: out = c0 in + sum_p' s_p' on the even sites, one thread per
// element of the one-column fields (in may be out).  keep (nullable): a copy
// of the input.
__global__ void __launch_bounds__(PB) gather_kernel(int n, const double2 *c0, const float2 *in, const float2 *s,
                                                    float2 *out, float2 *keep, const int *skip) {
    if (skip && *skip)
        return;
    const int j = blockIdx.x * PB + threadIdx.x;
    if (j >= n)
        return;
    const float2 v = in[j];
    const double2 r = gathered(c0, v, s + j, n);
    if (keep)
        keep[j] = v;
    out[j] = make_float2((float)r.x, (float)r.y);
}

// Second half in training, for column blockIdx.y of a chunk: e = N(b) - x
// (column blockIdx.y of an ne-column field) and the block partials of
// Re <x, b>, b column col0 + blockIdx.y of the ncol-column sources, x FP64.
__global__ void __launch_bounds__(PB) error_kernel(int vh, const double2 *c0, const void *b32, int ncol, int col0,
                                                   const float2 *s, const void *x64, void *e, int ne,
                                                   double *partials) {
    __shared__ double lds[PB / 64];
    const int i = blockIdx.x * PB + threadIdx.x, k = blockIdx.y;
    double part[1] = {0.0};
    if (i < vh) {
        cplx<float> b[3], d[3];
        cplx<double> x[3];
        FieldIO<HISQ_FP32>::template load<float>(b32, vh, ncol, col0 + k, i, b);
        FieldIO<HISQ_FP64>::template load<double>(x64, vh, ncol, col0 + k, i, x);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double2 y = gathered(c0, make_float2(b[a].re, b[a].im),
                                      s + (size_t)k * 24 * vh + (size_t)a * vh + i, (size_t)3 * vh);
            d[a].re = (float)(y.x - x[a].re);
            d[a].im = (float)(y.y - x[a].im);
            part[0] += x[a].re * (double)b[a].re + x[a].im * (double)b[a].im;
        }
        FieldIO<HISQ_FP32>::template store<float>(e, vh, ne, k, i, d);
    }
    block_sum<1>(part, lds);
    if (threadIdx.x == 0)
        partials[(size_t)k * gridDim.x + blockIdx.x] = part[0];
}

// Block partials of K[p'][p] and K0 for column blockIdx.y of the pair (in, g),
// both even-site fields.  A block walks groups of 64 odd sites, one wavefront
// per direction: a thread forms two t_p = T_p in and two h_q = T_q g with its
// two links, takes the eight t_p of its site through LDS and adds conj(t_p) h_q
// to 16 accumulators (q = p' ^ 1: T_p'^+ = T_q), all products and sums in FP64:
// a sum over a lattice has no bound on its length, and a product of two fields
// may lie outside FP32.  FP64 and FP32 products issue at the same rate here, so
// the kernel stays bound by its loads and their latency: with sums and chain
// rule 82 us at 32^4, 78 with products and sums in FP32, whose error grew with
// the lattice (64^3x48 3e-7 of the gradient, now 7e-8).  With two wavefronts on
// 64 sites a thread's 32 accumulators take it past 256 VGPRs; h_q goes through
// LDS as well, 162 VGPRs and three wavefronts a SIMD instead of 174 and two (90
// -> 86 us).  Slot 2 (8 p' + p) + re/im, then K0, at
// partials[(column * 130 + slot) * gridDim.x + block].
constexpr int KS = 64;  // sites of a group

__global__ void __launch_bounds__(PB, 3) correlate_kernel(Geom g, const char *links, const void *in, int nin, int cin,
                                                          const void *gr, int ngr, double *partials) {
    __shared__ float2 hops[4][6][KS], back[4][6][KS];
    __shared__ double sums[PTC_NK];
    const int k = blockIdx.y, lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double acc[32];             // re [q][p], then im
#pragma unroll
    for (int e = 0; e < 32; ++e)
        acc[e] = 0.0;
    double k0r = 0.0, k0i = 0.0;
    const int ngroups = (g.vh + KS - 1) / KS;
    for (int gi = site_block(); gi < ngroups; gi += gridDim.x) {
        const int i = gi * KS + lane;
        cplx<float> t[2][3], hf[2][3];
        if (i < g.vh) {
            const Site st = site_coords(g, 1, i);
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                const Hop h = odd_hop(g, st, i, 2 * mu + l);
                float m[18];
                cplx<float> v[3], w[3];
                load_link(links, g.vh, mu, h, m);
                FieldIO<HISQ_FP32>::template load<float>(in, g.vh, nin, cin + k, h.nb, v);
                FieldIO<HISQ_FP32>::template load<float>(gr, g.vh, ngr, k, h.nb, w);
                if (l == 0) {
                    transport<false>(m, v, t[l]);
                    transport<false>(m, w, hf[l]);
                } else {
                    transport<true>(m, v, t[l]);
                    transport<true>(m, w, hf[l]);
                }
            }
        } else {
#pragma unroll
            for (int l = 0; l < 2; ++l)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    t[l][a].re = t[l][a].im = hf[l][a].re = hf[l][a].im = 0.f;
        }
        __syncthreads();  // the vectors of the previous group have been read
#pragma unroll
        for (int l = 0; l < 2; ++l)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                hops[mu][3 * l + a][lane] = make_float2(t[l][a].re, t[l][a].im);
                back[mu][3 * l + a][lane] = make_float2(hf[l][a].re, hf[l][a].im);
            }
        __syncthreads();
        cplx<double> h[2][3];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float2 e = back[mu][3 * q + a][lane];
                h[q][a].re = e.x;
                h[q][a].im = e.y;
            }
#pragma unroll
        for (int p = 0; p < NHOP; ++p)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float2 e = hops[p >> 1][3 * (p & 1) + a][lane];
                const double tr = e.x, ti = e.y;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    double &re = acc[8 * q + p], &im = acc[16 + 8 * q + p];
                    re = fma(tr, h[q][a].re, re);
                    re = fma(ti, h[q][a].im, re);
                    im = fma(tr, h[q][a].im, im);
                    im = fma(-ti, h[q][a].re, im);
                }
            }
        if (mu == 0 && i < g.vh) {  // K0 on the even site of the same index
            cplx<double> v[3], w[3];
            FieldIO<HISQ_FP32>::template load<double>(in, g.vh, nin, cin + k, i, v);
            FieldIO<HISQ_FP32>::template load<double>(gr, g.vh, ngr, k, i, w);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                k0r = fma(v[a].re, w[a].re, fma(v[a].im, w[a].im, k0r));
                k0i = fma(v[a].re, w[a].im, fma(-v[a].im, w[a].re, k0i));
            }
        }
    }
    wave_sum_multi<32>(acc);
    // the value [re/im][q][p] of this lane goes to slot 2 (8 p' + p) + re/im, p' = (2 mu + q) ^ 1
    const int e = wave_multi_index<32>(lane), po = (2 * mu + ((e >> 3) & 1)) ^ 1;
    sums[2 * (8 * po + (e & 7)) + (e >> 4)] = acc[0];
    if (mu == 0) {
        k0r = wave_sum(k0r);
        k0i = wave_sum(k0i);
        sums[128] = k0r;
        sums[129] = k0i;
    }
    __syncthreads();
    if (threadIdx.x < PTC_NK)
        partials[((size_t)k * PTC_NK + threadIdx.x) * gridDim.x + blockIdx.x] = sums[threadIdx.x];
}

// Sum of n block partials by one wavefront, eight loads in flight a lane.
__device__ __forceinline__ double sum_blocks(const double *p, int n) {
    double v = 0.0;
    for (int b = threadIdx.x & 63; b < n; b += 512) {
        double t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            t[k] = b + 64 * k < n ? p[b + 64 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v += t[k];
    }
    return wave_sum(v);
}

// K[slot] (+)= sum over the ncols <= PTC_COLS columns of scale_k times the
// column's block partials, in a fixed order: one block per slot, one wavefront
// per column.  Training (xb given): scale_k = 2 / (B <x_k, b_k>) from the nxb
// block partials of <x, b>, and *loss (+)= sum_k <e_k, A e_k> / (B <x_k, b_k>)
// with the ndot block partials of <e, A e>; else scale_k = 1.
__global__ void __launch_bounds__(64 * PTC_COLS) correlate_sum_kernel(int ncols, int nblk, const double *partials,
                                                                      int first, double *K, const double *xb, int nxb,
                                                                      double inv_batch, const double *dot, int ndot,
                                                                      double *loss) {
    __shared__ double part[PTC_COLS], lpart[PTC_COLS];
    const int slot = blockIdx.x, k = threadIdx.x >> 6;
    double v = 0.0, l = 0.0;
    if (k < ncols) {
        v = sum_blocks(partials + ((size_t)k * PTC_NK + slot) * nblk, nblk);
        if (xb) {
            const double f = inv_batch / sum_blocks(xb + (size_t)k * nxb, nxb);
            v *= 2.0 * f;
            if (slot == 0)
                l = f * sum_blocks(dot + (size_t)k * ndot, ndot);
        }
    }
    if ((threadIdx.x & 63) == 0) {
        part[k] = v;
        lpart[k] = l;
    }
    __syncthreads();
    if (threadIdx.x != 0)
        return;
    v = first ? 0.0 : K[slot];
    for (int j = 0; j < PTC_COLS; ++j)
        v += part[j];
    K[slot] = v;
    if (xb && slot == 0) {
        l = first ? 0.0 : *loss;
        for (int j = 0; j < PTC_COLS; ++j)
            l += lpart[j];
        *loss = l;
    }
}

// dL/dw_k from K by the chain rule, sum conj(dC/dw_k) K, by one wavefront,
// lane 8 (p' - 1) + p - 1; valid in lane 0.  wf: the weights of the forward pass
// (they made the activations that multiply the gradient of a layer), wb: those
// of the backward pass (the layers above it); both in shared memory.
__device__ __forceinline__ double2 weight_gradient(const float2 *wf, const float2 *wb, const double *K, int k) {
    const int lane = threadIdx.x & 63, po = (lane >> 3) + 1, pi = (lane & 7) + 1;
    const double2 kk = make_double2(K[2 * lane], K[2 * lane + 1]), k0 = make_double2(K[128], K[129]);
    double2 f = make_double2(0.0, 0.0), f0 = f;  // dC[po][pi]/dw and dc0/dw
    if (k < PTC_W2) {
        const int c = (k - PTC_W1) / PTC_PATHS, r = (k - PTC_W1) % PTC_PATHS;
        for (int d = 0; d < PTC_CH; ++d) {
            if (r == 0) {
                dmac(f, w3_(wb, d, po), w2_(wb, d, c, pi));
                dmac(f0, w3_(wb, d, 0), w2_(wb, d, c, 0));
            } else if (r == pi) {
                dmac(f, w3_(wb, d, 0), w2_(wb, d, c, po));
                dmac(f, w3_(wb, d, po), w2_(wb, d, c, 0));
            }
        }
    } else if (k < PTC_W3) {
        const int q = (k - PTC_W2) / PTC_PATHS, r = (k - PTC_W2) % PTC_PATHS, d = q / PTC_CH, c = q % PTC_CH;
        if (r == 0) {
            f = dmul(w3_(wb, d, po), w1_(wf, c, pi));
            f0 = dmul(w3_(wb, d, 0), w1_(wf, c, 0));
        } else {
            if (r == po)
                dmac(f, w3_(wb, d, 0), w1_(wf, c, pi));
            if (r == pi)
                dmac(f, w3_(wb, d, po), w1_(wf, c, 0));
        }
    } else {
        const int d = (k - PTC_W3) / PTC_PATHS, r = (k - PTC_W3) % PTC_PATHS;
        for (int c = 0; c < PTC_CH; ++c) {
            if (r == 0) {
                dmac(f, w2_(wf, d, c, po), w1_(wf, c, pi));
                dmac(f0, w2_(wf, d, c, 0), w1_(wf, c, 0));
            } else if (r == po) {
                dmac(f, w2_(wf, d, c, 0), w1_(wf, c, pi));
                dmac(f, w2_(wf, d, c, pi), w1_(wf, c, 0));
            }
        }
    }
    double2 s = make_double2(0.0, 0.0);
    dmac(s, make_double2(f.x, -f.y), kk);
    s.x = wave_sum(s.x);
    s.y = wave_sum(s.y);
    dmac(s, make_double2(f0.x, -f0.y), k0);
    return s;
}

// grad += dL/dw, four weights a block.
__global__ void __launch_bounds__(256) chain_kernel(const float2 *fwd, const float2 *bwd, const double *K,
                                                    double2 *grad) {
    __shared__ float2 wf[PTC_NW], wb[PTC_NW];
    stage_weights<256>(fwd, wf);
    stage_weights<256>(bwd, wb);
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    const double2 s = weight_gradient(wf, wb, K, k);
    if ((threadIdx.x & 63) == 0)
        grad[k] = make_double2(grad[k].x + s.x, grad[k].y + s.y);
}

// Adam on real and imaginary parts as separate parameters; FP64 master
// weights and moments, FP32 copy for the kernels.
struct AdamArgs {
    double2 *w;
    float2 *w32;
    double2 *m, *v;
    double c1, c2;  // 1 - b1^step, 1 - b2^step
    double lr, b1, b2, eps;
};

__device__ __forceinline__ void adam(const AdamArgs &a, int k, double2 gk) {
    double2 wk = a.w[k], mk = a.m[k], vk = a.v[k];
    mk.x = a.b1 * mk.x + (1.0 - a.b1) * gk.x;
    mk.y = a.b1 * mk.y + (1.0 - a.b1) * gk.y;
    vk.x = a.b2 * vk.x + (1.0 - a.b2) * gk.x * gk.x;
    vk.y = a.b2 * vk.y + (1.0 - a.b2) * gk.y * gk.y;
    wk.x -= a.lr * (mk.x / a.c1) / (sqrt(vk.x / a.c2) + a.eps);
    wk.y -= a.lr * (mk.y / a.c1) / (sqrt(vk.y / a.c2) + a.eps);
    a.w[k] = wk;
    a.m[k] = mk;
    a.v[k] = vk;
    a.w32[k] = make_float2((float)wk.x, (float)wk.y);
}

__global__ void adam_kernel(AdamArgs a, const double2 *g) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < PTC_NW)
        adam(a, k, g[k]);
}

// The training step's gradient and Adam in one launch; weights: the copy that
// the fold kept, since w32 changes while other blocks read.
__global__ void __launch_bounds__(256) chain_adam_kernel(const float2 *weights, const double *K, AdamArgs a) {
    __shared__ float2 w[PTC_NW];
    stage_weights<256>(weights, w);
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    const double2 s = weight_gradient(w, w, K, k);
    if ((threadIdx.x & 63) == 0)
        adam(a, k, s);
}

AdamArgs adam_args(double2 *w, float2 *w32, double2 *m, double2 *v, int step, double lr, double b1, double b2,
                   double eps) {
    return AdamArgs{w, w32, m, v, 1.0 - std::pow(b1, step), 1.0 - std::pow(b2, step), lr, b1, b2, eps};
}

inline unsigned nb(int64_t n) { return (unsigned)((n + PB - 1) / PB); }

}  // namespace

// Blocks of a column in the correlation: as many as run at once over all
// columns, three on each of 256 CUs.  Limits of 512 / 768 / 1024 a column: one
// column at 32^4 87 / 82 / 86 us (sums and chain rule too), 48^4 389 / 360 / 380;
// training step on four pairs, limits of 128 / 256 / 768 a column: 32^4 1027 /
// 1034 / 1084 us, 24^3x16 279 / 288 / 306, 16^4 155 / 156 / 159.
int ptc_correlate_blocks(const Geom &g, int ncols) {
    return std::min((g.vh + KS - 1) / KS, (768 + ncols - 1) / ncols);
}

int ptc_error_blocks(const Geom &g) { return (int)nb(g.vh); }

hipError_t ptc_fold(const float2 *w, double2 *fold, float2 *keep, hipStream_t st, const int *skip) {
    fold_kernel<<<1, 576, 0, st>>>(w, fold, keep, skip);
    return hipGetLastError();
}

// From 65536 sites per parity (two wavefronts a SIMD) the columns run one after
// another in a thread, the links read once for all of them; on smaller lattices
// they are blocks of their own.  Training step of four pairs, blocks of their
// own -> one after another: 24^3x16 300 -> 278 us, 32^4 1192 -> 1058 us, 16^4
// 153 -> 156 us, 8^4 122 -> 128 us.
hipError_t ptc_spread(const Geom &g, const char *links, const double2 *fold, const void *in, int ncol, int col0,
                      int ncols, float2 *s, hipStream_t st, const int *skip) {
    const int nper = g.vh >= 65536 ? ncols : 1;
    spread_kernel<<<dim3((unsigned)((g.vh + CS - 1) / CS), (unsigned)((ncols + nper - 1) / nper)), PB, 0, st>>>(g, links, fold, in, ncol, col0,
                                                                                        nper, ncols, s, skip);
    return hipGetLastError();
}

hipError_t ptc_gather(const Geom &g, const double2 *c0, const void *in, const float2 *s, void *out, void *keep,
                      hipStream_t st, const int *skip) {
    const int n = 3 * g.vh;
    gather_kernel<<<nb(n), PB, 0, st>>>(n, c0, static_cast<const float2 *>(in), s, static_cast<float2 *>(out),
                                        static_cast<float2 *>(keep), skip);
    return hipGetLastError();
}

hipError_t ptc_error(const Geom &g, const double2 *c0, const void *b32, int ncol, int col0, int ncols, const float2 *s,
                     const void *x64, void *e, double *partials, hipStream_t st) {
    error_kernel<<<dim3(nb(g.vh), (unsigned)ncols), PB, 0, st>>>(g.vh, c0, b32, ncol, col0, s, x64, e, ncols, partials);
    return hipGetLastError();
}

hipError_t ptc_correlate(const Geom &g, const char *links, const void *in, int nin, int cin, const void *gr, int ncols,
                         double *partials, hipStream_t st) {
    const dim3 grid((unsigned)ptc_correlate_blocks(g, ncols), (unsigned)ncols);
    correlate_kernel<<<grid, PB, 0, st>>>(g, links, in, nin, cin, gr, ncols, partials);
    return hipGetLastError();
}

hipError_t ptc_correlate_sum(const Geom &g, int ncols, const double *partials, bool first, double *K, const double *xb,
                             double inv_batch, const double *dot, int ndot, double *loss, hipStream_t st) {
    correlate_sum_kernel<<<PTC_NK, 64 * PTC_COLS, 0, st>>>(ncols, ptc_correlate_blocks(g, ncols), partials,
                                                           first ? 1 : 0, K, xb, ptc_error_blocks(g), inv_batch, dot,
                                                           ndot, loss);
    return hipGetLastError();
}

hipError_t ptc_chain(const float2 *wf, const float2 *wb, const double *K, double2 *grad, hipStream_t st) {
    chain_kernel<<<PTC_NW / 4, 256, 0, st>>>(wf, wb, K, grad);
    return hipGetLastError();
}

hipError_t ptc_chain_adam(const float2 *w, const double *K, double2 *w_master, float2 *w_f32, double2 *m, double2 *v,
                          int step, double lr, double b1, double b2, double eps, hipStream_t st) {
    chain_adam_kernel<<<PTC_NW / 4, 256, 0, st>>>(w, K, adam_args(w_master, w_f32, m, v, step, lr, b1, b2, eps));
    return hipGetLastError();
}

hipError_t ptc_adam(double2 *w_master, float2 *w_f32, const double2 *grad, double2 *m, double2 *v, int step,
                    double lr, double b1, double b2, double eps, hipStream_t st) {
    adam_kernel<<<(PTC_NW + 255) / 256, 256, 0, st>>>(adam_args(w_master, w_f32, m, v, step, lr, b1, b2, eps), grad);
    return hipGetLastError();
}

}  // namespace hisq
