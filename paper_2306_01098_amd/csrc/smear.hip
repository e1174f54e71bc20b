// HISQ link smearing: thin links U -> fat links X and Naik links W, both in
// the canonical complex128 layout (4, Nt, Nz, Ny, Nx, 3, 3), ready for
// hisq_pack_links.  Two levels of smearing with a projection to U(3) between
// them (the HISQ treatment of Sec. 3.1).  FP64 throughout.
//
// One smearing level F = c1 L + c3 S3 + c5 S5 + c7 S7 + cL Lepage is built
// from nested staples in three passes, all links periodic:
//   T_{+nu}[A]_mu(x) = L_nu(x) A_mu(x+nu) L_nu(x+mu)^+
//   T_{-nu}[A]_mu(x) = L_nu(x-nu)^+ A_mu(x-nu) L_nu(x-nu+mu)
//   pass 1: Z[mu][nu] = c5 L_mu + c7 sum_s T_{s nu}[L]_mu             (12 fields)
//   pass 2: R[mu][nu] = c3 L_mu + sum_{rho not mu,nu} sum_r T_{r rho}[Z[mu][sigma]]
//           with sigma the fourth direction                          (12 fields)
//   pass 3: F_mu = c1 L_mu + sum_{nu,s} T_{s nu}[R[mu][nu] + cL T_{s nu}[L]_mu]
// which expands to the 6 three-link, 24 five-link, 48 seven-link and 6 Lepage
// paths.  The inner staple of the Lepage term is formed again in pass 3, so
// that pass 1 need not store the 24 signed staples.
//
// Bound: the matrices of neighbouring sites past the L2 and from L2 to L1, not
// the FP64 units (about 40 % busy).  At 32^4 (1M sites) one thread per matrix
// with matrices stored whole took 21.1 ms; element planes (whole-line loads),
// 12 instead of 24 fields from pass 1 and the projection and Naik links fused
// into pass 3 9.3 ms, with the block order of work_item 8.3 ms, with products
// accumulated by FMA and pass 2's three fields in a thread 7.8 ms.
// The staples run in loops that are not unrolled, so that one staple's three
// matrices are in registers at a time; forced below 256 VGPRs (three
// wavefronts per SIMD) the kernels spill and take 22 ms.
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "api_util.hpp"
#include "internal.hpp"

namespace hisq {

namespace {

constexpr int SB = 256;

struct M3 {
    double2 e[9];  // row-major, (re, im)
};

// Matrix idx of a canonical link array (matrices stored whole).
__device__ __forceinline__ void stm(double *base, size_t idx, const M3 &m) {
    double2 *p = reinterpret_cast<double2 *>(base) + idx * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        p[k] = m.e[k];
}

// Matrix of site x of field f in the workspace layout [field][element][site]:
// a wavefront reads an element of 64 neighbouring sites as one 1 KiB request.
__device__ __forceinline__ M3 ld_site(const double *base, size_t V, int f, int x) {
    const double2 *p = reinterpret_cast<const double2 *>(base) + (size_t)f * 9 * V;
    M3 m;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        m.e[k] = p[k * V + x];
    return m;
}

__device__ __forceinline__ void st_site(double *base, size_t V, int f, int x, const M3 &m) {
    double2 *p = reinterpret_cast<double2 *>(base) + (size_t)f * 9 * V;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        p[k * V + x] = m.e[k];
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cmul_conj_a(double2 a, double2 b) {  // conj(a) b
    return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

// s += a b, a conj(b), conj(a) b
__device__ __forceinline__ void mac(double2 &s, double2 a, double2 b) {
    s.x = fma(a.x, b.x, s.x);
    s.x = fma(-a.y, b.y, s.x);
    s.y = fma(a.x, b.y, s.y);
    s.y = fma(a.y, b.x, s.y);
}
__device__ __forceinline__ void mac_conj_b(double2 &s, double2 a, double2 b) {
    s.x = fma(a.x, b.x, s.x);
    s.x = fma(a.y, b.y, s.x);
    s.y = fma(-a.x, b.y, s.y);
    s.y = fma(a.y, b.x, s.y);
}

// A B, or A^+ B
template <bool ADJ = false> __device__ __forceinline__ M3 mul(const M3 &a, const M3 &b) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double2 s = ADJ ? cmul_conj_a(a.e[i], b.e[j]) : cmul(a.e[3 * i], b.e[j]);
#pragma unroll
            for (int k = 1; k < 3; ++k) {
                if (ADJ)
                    mac_conj_b(s, b.e[3 * k + j], a.e[3 * k + i]);
                else
                    mac(s, a.e[3 * i + k], b.e[3 * k + j]);
            }
            c.e[3 * i + j] = s;
        }
    return c;
}

// acc += A B D^+ (MINUS false) or A^+ B D (MINUS), one row of A B at a time.
template <bool MINUS> __device__ __forceinline__ void mac_staple(const M3 &a, const M3 &b, const M3 &d, M3 &acc) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double2 t[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            t[j] = MINUS ? cmul_conj_a(a.e[i], b.e[j]) : cmul(a.e[3 * i], b.e[j]);
#pragma unroll
            for (int k = 1; k < 3; ++k) {
                if (MINUS)
                    mac_conj_b(t[j], b.e[3 * k + j], a.e[3 * k + i]);
                else
                    mac(t[j], a.e[3 * i + k], b.e[3 * k + j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                if (MINUS)
                    mac(acc.e[3 * i + j], t[k], d.e[3 * k + j]);
                else
                    mac_conj_b(acc.e[3 * i + j], t[k], d.e[3 * j + k]);
            }
    }
}

__device__ __forceinline__ void axpy(double a, const M3 &x, M3 &y) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        y.e[k].x = fma(a, x.e[k].x, y.e[k].x);
        y.e[k].y = fma(a, x.e[k].y, y.e[k].y);
    }
}

__device__ __forceinline__ M3 zero3() {
    M3 m;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        m.e[k] = make_double2(0.0, 0.0);
    return m;
}

struct Lat {
    int n[4];  // Nx, Ny, Nz, Nt
    int V;
    int by, sz;  // rows of y and planes of z in a column of the block order (divide Ny, Nz)
};

// Coordinates of a site and its neighbours' indices (periodic).
struct Place {
    int x, c[4];
};

__device__ __forceinline__ int stride_of(const Lat &g, int d) {
    return d == 0 ? 1 : d == 1 ? g.n[0] : d == 2 ? g.n[0] * g.n[1] : g.n[0] * g.n[1] * g.n[2];
}

__device__ __forceinline__ Place place_of(const Lat &g, int x) {
    Place p;
    p.x = x;
    p.c[0] = x % g.n[0];
    x /= g.n[0];
    p.c[1] = x % g.n[1];
    x /= g.n[1];
    p.c[2] = x % g.n[2];
    p.c[3] = x / g.n[2];
    return p;
}

// p + k along d (d uniform over the block, |k| <= 2 < every extent)
__device__ __forceinline__ Place step(const Lat &g, const Place &p, int d, int k) {
    Place q = p;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j == d) {
            int v = p.c[j] + k;
            v = v >= g.n[j] ? v - g.n[j] : v < 0 ? v + g.n[j] : v;
            q.x += (v - p.c[j]) * stride_of(g, j);
            q.c[j] = v;
        }
    return q;
}

// The k-th direction (k = 0, 1, 2) other than mu.
__device__ __forceinline__ int other(int mu, int k) { return k < mu ? k : k + 1; }

// acc += T_{s nu}[A]_mu at p, A(q) the transported field's matrix at place q.
template <int S, typename F>
__device__ __forceinline__ void add_staple(const Lat &g, const double *L, const Place &p, int mu, int nu, F A,
                                           M3 &acc) {
    if constexpr (S > 0) {
        const M3 a = ld_site(L, g.V, nu, p.x);
        const M3 b = A(step(g, p, nu, 1));
        const M3 d = ld_site(L, g.V, nu, step(g, p, mu, 1).x);
        mac_staple<false>(a, b, d, acc);
    } else {
        const Place m = step(g, p, nu, -1);
        const M3 a = ld_site(L, g.V, nu, m.x);
        const M3 b = A(m);
        const M3 d = ld_site(L, g.V, nu, step(g, m, mu, 1).x);
        mac_staple<true>(a, b, d, acc);
    }
}

// Block order: workgroup b runs on XCD b mod 8, and each XCD takes one
// contiguous range of the site order (slab of sz z-planes, band of by y-rows,
// t, z, y, x), the nf fields of a block of sites side by side.  The links and
// staples of a column's neighbouring t-slices then meet in the XCD's L2: with
// by = 8, sz = 4 a slice of 32^4 is 1024 sites, and pass 2 fetches 5.6 GB past
// the L2 instead of 7.3 GB when the fields run one after another in plain
// site order (whole smearing at 32^4: 9.9 -> 8.3 ms; by, sz = 16, 4 and 8, 8
// within 2 %, 4, 4 and 8, 2 5 % slower).
__device__ __forceinline__ bool work_item(const Lat &g, int nf, int &f, int &x) {
    const int per = gridDim.x / (8 * nf);  // site blocks of an XCD
    const int j = blockIdx.x >> 3;
    f = j % nf;
    int ip = ((blockIdx.x & 7) * per + j / nf) * SB + threadIdx.x;
    if (ip >= g.V)
        return false;
    x = ip % g.n[0];
    ip /= g.n[0];
    int y = ip % g.by;
    ip /= g.by;
    int z = ip % g.sz;
    ip /= g.sz;
    const int t = ip % g.n[3];
    ip /= g.n[3];
    const int nb = g.n[1] / g.by;
    y += g.by * (ip % nb);
    z += g.sz * (ip / nb);
    x += g.n[0] * (y + g.n[1] * (z + g.n[2] * t));
    return true;
}

// canonical links -> [mu][element][site], 256 matrices of the canonical array
// through LDS so that both sides are read and written in whole lines.
__global__ void __launch_bounds__(SB) split_kernel(int64_t n, int V, const double *thin, double *L) {
    __shared__ double2 lds[9 * SB];
    const int64_t m0 = (int64_t)blockIdx.x * SB;
    const double2 *src = reinterpret_cast<const double2 *>(thin) + m0 * 9;
    const int here = (int)min((int64_t)SB, n - m0) * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        if (k * SB + (int)threadIdx.x < here)
            lds[k * SB + threadIdx.x] = src[k * SB + threadIdx.x];
    __syncthreads();
    const int64_t m = m0 + threadIdx.x;
    if (m >= n)
        return;
    const int mu = (int)(m / V), x = (int)(m - (int64_t)mu * V);
    double2 *dst = reinterpret_cast<double2 *>(L) + (size_t)mu * 9 * V + x;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        dst[(size_t)k * V] = lds[threadIdx.x * 9 + k];
}

// pass 1: field mu * 3 + k of Z, nu = nu_k
__global__ void __launch_bounds__(SB) staple1_kernel(Lat g, const double *L, double *Z, double c5, double c7) {
    int f, x;
    if (!work_item(g, 12, f, x))
        return;
    const int mu = f / 3, nu = other(mu, f % 3);
    const Place p = place_of(g, x);
    auto A = [&](const Place &q) { return ld_site(L, g.V, mu, q.x); };
    M3 acc = zero3(), z = zero3();
    add_staple<1>(g, L, p, mu, nu, A, acc);
    add_staple<-1>(g, L, p, mu, nu, A, acc);
    axpy(c5, A(p), z);
    axpy(c7, acc, z);
    st_site(Z, g.V, f, x, z);
}

// pass 2: the three fields R[mu][.] in one thread, so that the two transported
// fields of a direction rho share its links (100 matrices read per site
// instead of 156 with one field a thread).  The loop over rho rotates the
// accumulators: a0 is the one of nu = rho, which takes no staple along rho.
__global__ void __launch_bounds__(SB) staple2_kernel(Lat g, const double *L, const double *Z, double *R, double c3) {
    int mu, x;
    if (!work_item(g, 4, mu, x))
        return;
    const Place p = place_of(g, x);
    M3 a0 = zero3();
    axpy(c3, ld_site(L, g.V, mu, x), a0);
    M3 a1 = a0, a2 = a0;
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int rho = other(mu, k);
        const int j1 = k == 2 ? 0 : k + 1, j2 = k == 0 ? 2 : k - 1;
        const int xm = step(g, p, mu, 1).x - x;
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            const Place m = half ? step(g, p, rho, -1) : p;
            const Place q = half ? m : step(g, p, rho, 1);
            const M3 a = ld_site(L, g.V, rho, m.x);
            const M3 d = ld_site(L, g.V, rho, m.x + xm);
            const M3 z1 = ld_site(Z, g.V, mu * 3 + j2, q.x);
            const M3 z2 = ld_site(Z, g.V, mu * 3 + j1, q.x);
            if (half) {
                mac_staple<true>(a, z1, d, a1);
                mac_staple<true>(a, z2, d, a2);
            } else {
                mac_staple<false>(a, z1, d, a1);
                mac_staple<false>(a, z2, d, a2);
            }
        }
        const M3 t = a0;  // the next k leaves out the next accumulator
        a0 = a1;
        a1 = a2;
        a2 = t;
    }
    st_site(R, g.V, mu * 3, x, a0);
    st_site(R, g.V, mu * 3 + 1, x, a1);
    st_site(R, g.V, mu * 3 + 2, x, a2);
}

__device__ __forceinline__ M3 project(const M3 &v);

// pass 3.  Level 1 (LAST false): Y = projection of F, in the workspace layout.
// Level 2 (LAST): F with the Lepage term to the canonical fat links, and the
// Naik links W_mu(x) = cn L_mu(x) L_mu(x+mu) L_mu(x+2mu).
template <bool LAST>
__global__ void __launch_bounds__(SB) staple3_kernel(Lat g, const double *L, const double *R, double *F, double *W,
                                                      double c1, double cl, double cn) {
    int mu, x;
    if (!work_item(g, 4, mu, x))
        return;
    const Place p = place_of(g, x);
    M3 acc = zero3();
    {
        const M3 l = ld_site(L, g.V, mu, x);
        axpy(c1, l, acc);
        if constexpr (LAST) {
            const Place p1 = step(g, p, mu, 1);
            const M3 n = mul(mul(l, ld_site(L, g.V, mu, p1.x)), ld_site(L, g.V, mu, step(g, p1, mu, 1).x));
            M3 w = zero3();
            axpy(cn, n, w);
            stm(W, (size_t)mu * g.V + x, w);
        }
    }
#pragma unroll 1
    for (int j = 0; j < 6; ++j) {
        const int k = j >> 1, nu = other(mu, k);
        const bool minus = j & 1;
        const int xm = step(g, p, mu, 1).x - x;
        const Place m = minus ? step(g, p, nu, -1) : p;   // the link a, and d at m + mu
        const Place q = minus ? m : step(g, p, nu, 1);    // the transported field
        M3 b;
        if constexpr (LAST) {  // cl T[L]_mu(q) + R(q)
            const Place m2 = minus ? step(g, m, nu, -1) : q;
            const Place q2 = minus ? m2 : step(g, q, nu, 1);
            b = zero3();
            {
                const M3 a2 = ld_site(L, g.V, nu, m2.x), b2 = ld_site(L, g.V, mu, q2.x);
                const M3 d2 = ld_site(L, g.V, nu, m2.x + xm);
                if (minus)
                    mac_staple<true>(a2, b2, d2, b);
                else
                    mac_staple<false>(a2, b2, d2, b);
            }
            const M3 r = ld_site(R, g.V, mu * 3 + k, q.x);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                b.e[e].x = fma(cl, b.e[e].x, r.e[e].x);
                b.e[e].y = fma(cl, b.e[e].y, r.e[e].y);
            }
        } else {
            b = ld_site(R, g.V, mu * 3 + k, q.x);
        }
        const M3 a = ld_site(L, g.V, nu, m.x), d = ld_site(L, g.V, nu, m.x + xm);
        if (minus)
            mac_staple<true>(a, b, d, acc);
        else
            mac_staple<false>(a, b, d, acc);
    }
    if constexpr (LAST)
        stm(F, (size_t)mu * g.V + x, acc);
    else
        st_site(F, g.V, mu, x, project(acc));
}

// Y = V (V^+ V)^(-1/2).  The eigenvalues g_i of the Hermitian Q = V^+ V come
// from the trigonometric solution of its characteristic cubic; with
// s_i = sqrt(g_i), u = s0 + s1 + s2, v = s0 s1 + s0 s2 + s1 s2, w = s0 s1 s2,
// the quadratic f0 + f1 Q + f2 Q^2 that equals g^(-1/2) on the spectrum is
// f0 = (u v^2 - w (u^2 + v)) / D, f1 = (2 u v - u^3 - w) / D, f2 = u / D,
// D = w (u v - w): symmetric in the eigenvalues, so degenerate spectra are
// harmless (Hasenfratz, Hoffmann and Schaefer, JHEP 0705:029).
__device__ __forceinline__ M3 project(const M3 &v) {
    const M3 q = mul<true>(v, v);
    const double q00 = q.e[0].x, q11 = q.e[4].x, q22 = q.e[8].x;
    const double2 q01 = q.e[1], q02 = q.e[2], q12 = q.e[5];
    const double p1 = q01.x * q01.x + q01.y * q01.y + q02.x * q02.x + q02.y * q02.y + q12.x * q12.x +
                      q12.y * q12.y;
    const double tr = (q00 + q11 + q22) / 3.0;
    double g0, g1, g2;
    const double d0 = q00 - tr, d1 = q11 - tr, d2 = q22 - tr;
    const double p2 = d0 * d0 + d1 * d1 + d2 * d2 + 2.0 * p1;
    if (p2 <= 1e-30 * tr * tr) {
        g0 = g1 = g2 = tr;
    } else {
        const double p = sqrt(p2 / 6.0);
        // det(B) / 2 with B = (Q - tr 1) / p (Hermitian, so the determinant is real)
        const double b00 = d0 / p, b11 = d1 / p, b22 = d2 / p;
        const double2 b01 = make_double2(q01.x / p, q01.y / p), b02 = make_double2(q02.x / p, q02.y / p),
                      b12 = make_double2(q12.x / p, q12.y / p);
        const double n01 = b01.x * b01.x + b01.y * b01.y, n02 = b02.x * b02.x + b02.y * b02.y,
                     n12 = b12.x * b12.x + b12.y * b12.y;
        // 2 Re(b01 b12 conj(b02))
        const double2 t = cmul(b01, b12);
        const double tri = 2.0 * (t.x * b02.x + t.y * b02.y);
        double r = 0.5 * (b00 * b11 * b22 + tri - b00 * n12 - b11 * n02 - b22 * n01);
        r = fmin(1.0, fmax(-1.0, r));
        const double phi = acos(r) / 3.0;
        g0 = tr + 2.0 * p * cos(phi);
        g2 = tr + 2.0 * p * cos(phi + 2.0943951023931954923);  // + 2 pi / 3
        g1 = 3.0 * tr - g0 - g2;
    }
    const double s0 = sqrt(fmax(g0, 0.0)), s1 = sqrt(fmax(g1, 0.0)), s2 = sqrt(fmax(g2, 0.0));
    const double u = s0 + s1 + s2, vv = s0 * s1 + s0 * s2 + s1 * s2, w = s0 * s1 * s2;
    const double den = w * (u * vv - w);
    const double f0 = (u * vv * vv - w * (u * u + vv)) / den;
    const double f1 = (2.0 * u * vv - u * u * u - w) / den;
    const double f2 = u / den;
    const M3 q2 = mul(q, q);
    M3 h = zero3();
    h.e[0].x = h.e[4].x = h.e[8].x = f0;
    axpy(f1, q, h);
    axpy(f2, q2, h);
    return mul(v, h);
}

unsigned blocks(const Lat &g, int nf) { return (unsigned)((((g.V + SB - 1) / SB + 7) / 8) * 8 * nf); }

int divisor_upto(int n, int most) {
    int d = most < n ? most : n;
    while (n % d)
        --d;
    return d;
}

// 44 matrices per site, of which the passes use 32.
struct SmearLayout {
    size_t u, y, z, r, total;
};

SmearLayout smear_layout(int64_t V) {
    const size_t mat = 144;
    SmearLayout L;
    L.u = 0;
    L.y = L.u + 4 * V * mat;
    L.z = L.y + 4 * V * mat;
    L.r = L.z + 12 * V * mat;
    L.total = 44 * V * mat;  // the size callers were told before the fields were 32 matrices a site
    return L;
}

template <bool LAST>
hipError_t smear_level(const Lat &g, const double *L, double *Z, double *R, double *F, double *W, double c1, double c3,
                       double c5, double c7, double cl, double cn, hipStream_t st) {
    staple1_kernel<<<blocks(g, 12), SB, 0, st>>>(g, L, Z, c5, c7);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    staple2_kernel<<<blocks(g, 4), SB, 0, st>>>(g, L, Z, R, c3);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    staple3_kernel<LAST><<<blocks(g, 4), SB, 0, st>>>(g, L, R, F, W, c1, cl, cn);
    return hipGetLastError();
}

}  // namespace

}  // namespace hisq

using namespace hisq;

extern "C" {

size_t hisq_smear_workspace_bytes(const hisq_lattice *lat) {
    if (check_lattice(lat) != HISQ_OK)
        return 0;
    const int64_t V = (int64_t)lat->dims[0] * lat->dims[1] * lat->dims[2] * lat->dims[3];
    return smear_layout(V).total;
}

hisq_status hisq_smear_links(hisq_context *ctx, const hisq_lattice *lat, const void *thin_c128, double naik_eps,
                             void *fat_c128, void *naik_c128, void *ws, size_t ws_bytes, void *stream) {
    TRY(check_lattice(lat));
    TRY(check_ptr(thin_c128, "thin_c128"));
    TRY(check_ptr(fat_c128, "fat_c128"));
    TRY(check_ptr(naik_c128, "naik_c128"));
    TRY(check_ptr(ws, "ws"));
    if (fat_c128 == naik_c128 || fat_c128 == thin_c128 || naik_c128 == thin_c128)
        return fail(HISQ_ERR_INVALID_ARG, "thin, fat and naik buffers must be distinct");
    if (!std::isfinite(naik_eps))
        return fail(HISQ_ERR_INVALID_ARG, "naik_eps must be finite");
    Lat g;
    for (int d = 0; d < 4; ++d)
        g.n[d] = lat->dims[d];
    g.V = g.n[0] * g.n[1] * g.n[2] * g.n[3];
    g.by = divisor_upto(g.n[1], 8);
    g.sz = divisor_upto(g.n[2], 4);
    const SmearLayout L = smear_layout(g.V);
    if (ws_bytes < L.total)
        return fail(HISQ_ERR_WORKSPACE, "workspace holds %zu bytes, needs %zu", ws_bytes, L.total);
    TRY(set_device(ctx));
    const hipStream_t st = static_cast<hipStream_t>(stream);
    char *base = static_cast<char *>(ws);
    double *U = reinterpret_cast<double *>(base + L.u);
    double *Y = reinterpret_cast<double *>(base + L.y);
    double *Z = reinterpret_cast<double *>(base + L.z);
    double *R = reinterpret_cast<double *>(base + L.r);
    split_kernel<<<(unsigned)((4 * (int64_t)g.V + SB - 1) / SB), SB, 0, st>>>(4 * (int64_t)g.V, g.V, static_cast<const double *>(thin_c128), U);
    hipError_t e = hipGetLastError();
    // level 1 (fat7) and projection, level 2 (fat7 + Lepage) and Naik
    if (e == hipSuccess)
        e = smear_level<false>(g, U, Z, R, Y, nullptr, 1.0 / 8, 1.0 / 16, 1.0 / 64, 1.0 / 384, 0.0, 0.0, st);
    if (e == hipSuccess)
        e = smear_level<true>(g, Y, Z, R, static_cast<double *>(fat_c128), static_cast<double *>(naik_c128), 1.0,
                              1.0 / 16, 1.0 / 64, 1.0 / 384, -1.0 / 8, -1.0 / 24 + naik_eps / 8, st);
    return e == hipSuccess ? HISQ_OK : device_fail(e, "smear_links");
}

}  // extern "C"
