// staple.hip -- staples of the tree-level Symanzik gauge force.
//
// Paper: arXiv:1701.00426, Sec. 2.1 (tree-level Symanzik improved gauge action:
// 1x1 and 1x2 Wilson loops) and Sec. 4.3 (the gauge cycle's most expensive step:
// staples, products of 3 and 5 SU(3) links along C-shaped paths, computed per
// link with second-neighbour addressing).
//
// For the link U_mu(x) the kernel forms
//   Sigma_mu(x) = sum_{nu != mu} [ c0 (2 three-link paths) + c1 (6 five-link paths) ],
// each path a product of links leading from x + mu back to x, so U_mu(x) Sigma_mu(x)
// is the weighted sum of the closed loops through the link.
//
// One or two threads per link (with two, the paths above and below the link run
// on separate waves of the block and meet in LDS); the link's (mu, parity) is
// uniform in a block, the 8 slots of a group of sites run in adjacent blocks, and
// the sites are visited in pencil order (pencil.hpp) so that a link's radius-2
// neighbourhood is mostly in the XCD's L2.  Neighbour half indices come from
// coordinate arithmetic (no index tables).  The 8 paths of each side (above /
// below the link) share their factors:
//   above:  A = U_nu(x+mu), B = U_mu(x+nu)^dag, C = U_nu(x)^dag, X = A B,
//           Y = A U_nu(x+mu+nu) U_mu(x+2nu)^dag U_nu(x+nu)^dag,
//           Z = U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^dag B,
//           W = X U_mu(x-mu+nu)^dag U_nu(x-mu)^dag,
//   1x1: X C;  1x2: Y C (long side along nu), Z C (long side forward), W U_mu(x-mu) (long
//   side backward), so the side contributes
//           [c0 X + c1 (Y + Z)] C + c1 W U_mu(x-mu),
// 11 SU(3) products instead of 14 taken path by path; below the link likewise
// with nu -> -nu.  Products accumulate in the arithmetic type of the format
// (FP64 for complex128 links, FP32 for the 12-real FP32 / BF16 ones).
//
// The same file holds one stout-smearing step (Sec. 2.1: the fermion action is
// built on stout-smeared links; Sec. 2.3: the configurations of the stout levels
// are kept): with C_mu(x) = rho * (the six 3-link paths from x to x + mu),
// Omega = C U^dag and Q = (i/2)(Omega^dag - Omega) - (i/6) Tr(Omega^dag - Omega),
// every link becomes exp(iQ) U (Morningstar and Peardon's definition).

#include "device_common.hpp"
#include "kernels.hpp"
#include "staple.hpp"

namespace stg {

namespace {

// row 2 of an SU(3) matrix from rows 0 and 1: conj(row0 x row1), each part one chain of
// fused operations (24 instead of 30 of rebuild_row2, whose shorter chains suit the hops,
// and fewer roundings; staples at 32^4 3 % faster)
template <typename T>
__device__ __forceinline__ void finish_row2(su3<T> &u) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const cpx<T> a = u.e[0][(j + 1) % 3], b = u.e[1][(j + 2) % 3];
        const cpx<T> c = u.e[0][(j + 2) % 3], d = u.e[1][(j + 1) % 3];
        T re = a.re * b.re, im = -a.re * b.im;
        re = fmat(-a.im, b.im, re);
        im = fmat(-a.im, b.re, im);
        re = fmat(-c.re, d.re, re);
        im = fmat(c.re, d.im, im);
        re = fmat(c.im, d.im, re);
        im = fmat(c.im, d.re, im);
        u.e[2][j] = {re, im};
    }
}

// acc += a * conj(b)
template <typename T>
__device__ __forceinline__ void cfma_cb(cpx<T> &acc, cpx<T> a, cpx<T> b) {
    acc.re = fmat(a.re, b.re, acc.re);
    acc.re = fmat(a.im, b.im, acc.re);
    acc.im = fmat(a.im, b.re, acc.im);
    acc.im = fmat(-a.re, b.im, acc.im);
}

// C = A B
template <typename T>
__device__ __forceinline__ su3<T> mm(const su3<T> &a, const su3<T> &b) {
    su3<T> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<T> t = cmul(a.e[i][0], b.e[0][j]);
            cfma(t, a.e[i][1], b.e[1][j]);
            cfma(t, a.e[i][2], b.e[2][j]);
            c.e[i][j] = t;
        }
    return c;
}

// C += A B
template <typename T>
__device__ __forceinline__ void mm_acc(su3<T> &c, const su3<T> &a, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma(c.e[i][j], a.e[i][k], b.e[k][j]);
}

// C -= A B
template <typename T>
__device__ __forceinline__ void mm_sub(su3<T> &c, const su3<T> &a, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                cfma(c.e[i][j], cpx<T>{-a.e[i][k].re, -a.e[i][k].im}, b.e[k][j]);
}

// C = A B^dag
template <typename T>
__device__ __forceinline__ su3<T> mmd(const su3<T> &a, const su3<T> &b) {
    su3<T> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<T> t = {T(0), T(0)};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma_cb(t, a.e[i][k], b.e[j][k]);
            c.e[i][j] = t;
        }
    return c;
}

// C += A B^dag
template <typename T>
__device__ __forceinline__ void mmd_acc(su3<T> &c, const su3<T> &a, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma_cb(c.e[i][j], a.e[i][k], b.e[j][k]);
}

// C = A^dag B
template <typename T>
__device__ __forceinline__ su3<T> mdm(const su3<T> &a, const su3<T> &b) {
    su3<T> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<T> t = cmulc(a.e[0][i], b.e[0][j]);
            cfmac(t, a.e[1][i], b.e[1][j]);
            cfmac(t, a.e[2][i], b.e[2][j]);
            c.e[i][j] = t;
        }
    return c;
}

// C += A^dag B
template <typename T>
__device__ __forceinline__ void mdm_acc(su3<T> &c, const su3<T> &a, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) cfmac(c.e[i][j], a.e[k][i], b.e[k][j]);
}

// C = A^dag B^dag = (B A)^dag
template <typename T>
__device__ __forceinline__ su3<T> mdmd(const su3<T> &a, const su3<T> &b) {
    su3<T> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cpx<T> t = cmul(b.e[j][0], a.e[0][i]);
            cfma(t, b.e[j][1], a.e[1][i]);
            cfma(t, b.e[j][2], a.e[2][i]);
            c.e[i][j] = cconj(t);
        }
    return c;
}

// C = s C + r B
template <typename T>
__device__ __forceinline__ void axpby(su3<T> &c, T s, T r, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            c.e[i][j].re = fmat(s, c.e[i][j].re, r * b.e[i][j].re);
            c.e[i][j].im = fmat(s, c.e[i][j].im, r * b.e[i][j].im);
        }
}

// C += s B
template <typename T>
__device__ __forceinline__ void axpy(su3<T> &c, T s, const su3<T> &b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            c.e[i][j].re = fmat(s, b.e[i][j].re, c.e[i][j].re);
            c.e[i][j].im = fmat(s, b.e[i][j].im, c.e[i][j].im);
        }
}

template <typename T>
__device__ __forceinline__ void scale(su3<T> &c, T s) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            c.e[i][j].re *= s;
            c.e[i][j].im *= s;
        }
}

__device__ __forceinline__ uint32_t pick4(uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3,
                                          int i) {
    return i == 0 ? v0 : i == 1 ? v1 : i == 2 ? v2 : v3;
}

// x_d + s with periodic wrap, |s| <= 2 <= N
__device__ __forceinline__ int wrap_step(int x, int s, int n) {
    int y = x + s;
    y += (y < 0) ? n : 0;
    y -= (y >= n) ? n : 0;
    return y;
}

// Lexicographic displacement of the site x when its coordinate x_d (extent n,
// lexicographic stride st) moves by s.
__device__ __forceinline__ int lex_step(int x, int s, int n, int st) {
    return (wrap_step(x, s, n) - x) * st;
}

// Link loads through the caches: every link is read by about sixty staple
// computations of nearby links, so these loads must stay cached (the hop's loader
// streams its links past the caches instead).
template <typename T, int FMT>
struct cached_link;

template <>
struct cached_link<double, FMT_C128_18> {
    __device__ __forceinline__ static su3<double> load(const void *L, uint32_t Vh, int s,
                                                        uint32_t h) {
        const double2 *p = reinterpret_cast<const double2 *>(L) + (size_t)s * 9 * Vh + h;
        su3<double> u;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double2 v = p[(size_t)(a * 3 + b) * Vh];
                u.e[a][b] = {v.x, v.y};
            }
        return u;
    }
};

template <>
struct cached_link<double, FMT_C128_12> {
    __device__ __forceinline__ static su3<double> load(const void *L, uint32_t Vh, int s,
                                                        uint32_t h) {
        const double2 *p = reinterpret_cast<const double2 *>(L) + (size_t)s * 6 * Vh + h;
        su3<double> u;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double2 v = p[(size_t)(a * 3 + b) * Vh];
                u.e[a][b] = {v.x, v.y};
            }
        finish_row2(u);
        return u;
    }
};

template <>
struct cached_link<float, FMT_C64_12> {
    __device__ __forceinline__ static su3<float> load(const void *L, uint32_t Vh, int s,
                                                       uint32_t h) {
        const float4 *p = reinterpret_cast<const float4 *>(L) + (size_t)s * 3 * Vh + h;
        const float4 c0 = p[0], c1 = p[Vh], c2 = p[2 * (size_t)Vh];
        su3<float> u;
        u.e[0][0] = {c0.x, c0.y};
        u.e[0][1] = {c0.z, c0.w};
        u.e[0][2] = {c1.x, c1.y};
        u.e[1][0] = {c1.z, c1.w};
        u.e[1][1] = {c2.x, c2.y};
        u.e[1][2] = {c2.z, c2.w};
        finish_row2(u);
        return u;
    }
};

template <>
struct cached_link<float, FMT_BF16_12> {
    __device__ __forceinline__ static su3<float> load(const void *L, uint32_t Vh, int s,
                                                       uint32_t h) {
        const uint4 a = reinterpret_cast<const uint4 *>(L)[(size_t)s * Vh + h];
        const uint2 b = reinterpret_cast<const uint2 *>(
            reinterpret_cast<const uint4 *>(L) + (size_t)8 * Vh)[(size_t)s * Vh + h];
        su3<float> u;
        u.e[0][0] = {bf16_lo(a.x), bf16_hi(a.x)};
        u.e[0][1] = {bf16_lo(a.y), bf16_hi(a.y)};
        u.e[0][2] = {bf16_lo(a.z), bf16_hi(a.z)};
        u.e[1][0] = {bf16_lo(a.w), bf16_hi(a.w)};
        u.e[1][1] = {bf16_lo(b.x), bf16_hi(b.x)};
        u.e[1][2] = {bf16_lo(b.y), bf16_hi(b.y)};
        finish_row2(u);
        return u;
    }
};

// A 12-real link as it is stored: fetched ahead of its use and decoded (third row rebuilt)
// where it is used.
template <typename T, int FMT>
struct RawLink;

template <>
struct RawLink<double, FMT_C128_12> {
    double2 w[6];
    __device__ __forceinline__ void fetch(const void *L, uint32_t Vh, int s, uint32_t h) {
        const double2 *p = reinterpret_cast<const double2 *>(L) + (size_t)s * 6 * Vh + h;
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k] = p[(size_t)k * Vh];
    }
    __device__ __forceinline__ su3<double> link() const {
        su3<double> u;
#pragma unroll
        for (int k = 0; k < 6; ++k) u.e[k / 3][k % 3] = {w[k].x, w[k].y};
        finish_row2(u);
        return u;
    }
};

template <>
struct RawLink<float, FMT_C64_12> {
    float4 w[3];
    __device__ __forceinline__ void fetch(const void *L, uint32_t Vh, int s, uint32_t h) {
        const float4 *p = reinterpret_cast<const float4 *>(L) + (size_t)s * 3 * Vh + h;
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = p[(size_t)k * Vh];
    }
    __device__ __forceinline__ su3<float> link() const {
        su3<float> u;
        u.e[0][0] = {w[0].x, w[0].y};
        u.e[0][1] = {w[0].z, w[0].w};
        u.e[0][2] = {w[1].x, w[1].y};
        u.e[1][0] = {w[1].z, w[1].w};
        u.e[1][1] = {w[2].x, w[2].y};
        u.e[1][2] = {w[2].z, w[2].w};
        finish_row2(u);
        return u;
    }
};

template <>
struct RawLink<float, FMT_BF16_12> {
    uint4 a;
    uint2 b;
    __device__ __forceinline__ void fetch(const void *L, uint32_t Vh, int s, uint32_t h) {
        a = reinterpret_cast<const uint4 *>(L)[(size_t)s * Vh + h];
        b = reinterpret_cast<const uint2 *>(reinterpret_cast<const uint4 *>(L) +
                                            (size_t)8 * Vh)[(size_t)s * Vh + h];
    }
    __device__ __forceinline__ su3<float> link() const {
        su3<float> u;
        u.e[0][0] = {bf16_lo(a.x), bf16_hi(a.x)};
        u.e[0][1] = {bf16_lo(a.y), bf16_hi(a.y)};
        u.e[0][2] = {bf16_lo(a.z), bf16_hi(a.z)};
        u.e[1][0] = {bf16_lo(a.w), bf16_hi(a.w)};
        u.e[1][1] = {bf16_lo(b.x), bf16_hi(b.x)};
        u.e[1][2] = {bf16_lo(b.y), bf16_hi(b.y)};
        finish_row2(u);
        return u;
    }
};

// FP64-18 links have no third row to rebuild.
template <>
struct RawLink<double, FMT_C128_18> {
    su3<double> u;
    __device__ __forceinline__ void fetch(const void *L, uint32_t Vh, int s, uint32_t h) {
        u = cached_link<double, FMT_C128_18>::load(L, Vh, s, h);
    }
    __device__ __forceinline__ su3<double> link() const { return u; }
};

// Ends a group of fetches: what follows is not scheduled before it, nor the fetches after.
// Left to itself the compiler issues each link's loads where their values are needed (of
// the waits of the FP64 staple kernel 33 in 84 were for the load issued last), and two
// waves per SIMD do not hide that.
__device__ __forceinline__ void fetched() { __builtin_amdgcn_sched_barrier(0); }

// The links around one site x: lexicographic index L of x, parity P of x.
template <typename T, int FMT>
struct LinkAt {
    const void *links;
    uint32_t Vh;
    int L, P;
    // U_d(y) for y = x + (displacement dl in lexicographic units, odd-even flip par)
    __device__ __forceinline__ su3<T> operator()(int d, int dl, int flip) const {
        const int par = (P + flip) & 1;
        const uint32_t h = (uint32_t)(L + dl) >> 1;
        return cached_link<T, FMT>::load(links, Vh, 2 * d + par, h);
    }
    __device__ __forceinline__ void fetch(RawLink<T, FMT> &r, int d, int dl, int flip) const {
        const int par = (P + flip) & 1;
        r.fetch(links, Vh, 2 * d + par, (uint32_t)(L + dl) >> 1);
    }
};

template <typename T>
__device__ __forceinline__ void set_zero(su3<T> &c) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) c.e[i][j] = {T(0), T(0)};
}

template <typename T>
__device__ __forceinline__ su3<T> dagger(const su3<T> &u) {
    su3<T> r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) r.e[i][j] = cconj(u.e[j][i]);
    return r;
}

// The four paths on one side of the link (header; UP: the +nu side, else the -nu side, every
// U_nu step reversed): acc += [c0 X + c1 (Y + Z)] C, and the path whose long side
// runs backward, W U_mu(x-mu): with BACK its last factor, common to all sides, is left to
// the caller and W added to back, else c1 times the path is added to acc.  Every link is
// fetched one product or more before the one that uses it; u0 holds U_mu(x+mu) on entry
// and is fetched again for the next side.
//
// The products keep all three rows.  Two rows and their cross product would do for links in
// SU(3) (FP64-12 at 32^4 1490 us, FP32-12 752), but the links of a trajectory leave it: each
// update rounds their rows, and a product completed that way is off by their departure.
// Against 64-bit sums of the stored links, 8^3 x 16 in FP32-12 after 0 / 10 / 100 / 1000
// updates: 1.2e-7 / 2.3e-7 / 6.9e-7 / 7.7e-6 with two rows, 1.1e-7 at any number with three.
// 32^4 with every link fetched where it is used (11 products, FP64-12 on two threads) / so:
// FP64-12 1929 / 1703 us, FP32-12 1068 / 847, BF16-12 880 / 785.  In FP64 the matrices take
// 300 registers and one wave runs per SIMD; held to two, it spills 248 B per lane (2500 us),
// and with a matrix fetched twice and the last factor of every side multiplied 60 B (1815).
// The terms of the sums are products of their own, scaled and added afterwards: chained into
// the sum, each of their nine entries rounds three times at the sum's size (BF16-12 1.24e-7
// against 1.01e-7).
// mp1 .. n2: lexicographic displacements of x +- mu, x + 2mu, x +- nu, x +- 2nu (periodic).
template <typename T, int FMT, bool BACK, bool UP>
__device__ __forceinline__ void side(su3<T> &acc, su3<T> &back, RawLink<T, FMT> &u0,
                                     const LinkAt<T, FMT> &U, int mu, int nu, int mp1, int mm1,
                                     int mp2, int n1, int n2, T c0, T c1) {
    const auto mulu = [](const su3<T> &a, const su3<T> &b) {  // a step along +-nu
        return UP ? mm(a, b) : mmd(a, b);
    };
    const auto muld = [](const su3<T> &a, const su3<T> &b) {  // a step along -+nu
        return UP ? mmd(a, b) : mm(a, b);
    };
    RawLink<T, FMT> p, q;
    // Z = U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^dag B, B = U_mu(x+nu)^dag
    U.fetch(p, nu, UP ? mp2 : mp2 + n1, UP ? 0 : 1);
    U.fetch(q, mu, mp1 + n1, 0);
    fetched();
    su3<T> z = mulu(u0.link(), p.link());
    U.fetch(p, nu, UP ? mp1 : mp1 + n1, UP ? 1 : 0);
    fetched();
    z = mmd(z, q.link());
    // Y = A U_nu(x+mu+nu) U_mu(x+2nu)^dag U_nu(x+nu)^dag, A = U_nu(x+mu)
    U.fetch(q, nu, UP ? mp1 + n1 : mp1 + n2, UP ? 0 : 1);
    fetched();
    const su3<T> a = UP ? p.link() : dagger(p.link());
    U.fetch(p, mu, n2, 0);
    fetched();
    su3<T> g = mulu(a, q.link());
    U.fetch(q, nu, UP ? n1 : n2, UP ? 1 : 0);
    fetched();
    g = mmd(g, p.link());
    U.fetch(p, mu, n1, 1);
    fetched();
    g = muld(g, q.link());
    scale(g, c1);
    su3<T> x;
    {
        const su3<T> b = p.link();
        z = mmd(z, b);
        axpy(g, c1, z);
        U.fetch(q, mu, mm1 + n1, 0);
        fetched();
        x = mmd(a, b);  // X = A B
    }
    U.fetch(p, nu, UP ? mm1 : mm1 + n1, UP ? 1 : 0);
    fetched();
    axpy(g, c0, x);
    // W = X U_mu(x-mu+nu)^dag U_nu(x-mu)^dag
    x = mmd(x, q.link());
    if constexpr (!BACK) {
        U.fetch(q, mu, mm1, 1);
        fetched();
        x = muld(x, p.link());
        U.fetch(p, nu, UP ? 0 : n1, UP ? 0 : 1);
        fetched();
        axpy(acc, c1, mm(x, q.link()));
    } else {
        U.fetch(q, nu, UP ? 0 : n1, UP ? 0 : 1);
        fetched();
        if constexpr (UP)
            mmd_acc(back, x, p.link());
        else
            mm_acc(back, x, p.link());
    }
    U.fetch(u0, mu, mp1, 1);
    fetched();
    const su3<T> c = BACK ? q.link() : p.link();
    if constexpr (UP)
        mmd_acc(acc, g, c);
    else
        mm_acc(acc, g, c);
}

// The same sums for FP64-18 links, whose stored form takes half as many registers again
// (32^4: 2250 us for three-row chains against 2041 us of this form), summed as A [c0 W + c1 (U_mu(x+nu)^dag D + T U_nu(x)^dag)] + c1 E W with
//   A = U_nu(x+mu), W = U_mu(x+nu)^dag U_nu(x)^dag,
//   D = U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu),
//   T = U_nu(x+mu+nu) U_mu(x+2nu)^dag U_nu(x+nu)^dag,
//   E = U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^dag, also 11 products.
template <typename T, int FMT>
__device__ __forceinline__ void side_above_full(su3<T> &acc, const LinkAt<T, FMT> &U, int mu, int nu,
                                           int mp1, int mm1, int mp2, int np1, int np2, T c0,
                                           T c1) {
    su3<T> y = mm(mdmd(U(mu, mm1 + np1, 0), U(nu, mm1, 1)), U(mu, mm1, 1));  // D
    su3<T> x = mdm(U(mu, np1, 1), y);
    y = mmd(mmd(U(nu, mp1 + np1, 0), U(mu, np2, 0)), U(nu, np1, 1));          // T
    mmd_acc(x, y, U(nu, 0, 0));
    su3<T> w = mdmd(U(mu, np1, 1), U(nu, 0, 0));  // W = U_mu(x+nu)^dag U_nu(x)^dag
    axpby(x, c1, c0, w);                           // c0 W + c1 (...)
    mm_acc(acc, U(nu, mp1, 1), x);                 // A = U_nu(x+mu)
    y = mmd(mm(U(mu, mp1, 1), U(nu, mp2, 0)), U(mu, mp1 + np1, 0));          // E
    scale(w, c1);
    mm_acc(acc, y, w);
}

// The same on the -nu side: A' = U_nu(x+mu-nu)^dag, W' = U_mu(x-nu)^dag U_nu(x-nu),
// D' = U_mu(x-mu-nu)^dag U_nu(x-mu-nu) U_mu(x-mu), T' = U_nu(x+mu-2nu)^dag
// U_mu(x-2nu)^dag U_nu(x-2nu), E' = U_mu(x+mu) U_nu(x+2mu-nu)^dag U_mu(x+mu-nu)^dag.
template <typename T, int FMT>
__device__ __forceinline__ void side_below_full(su3<T> &acc, const LinkAt<T, FMT> &U, int mu, int nu,
                                           int mp1, int mm1, int mp2, int nm1, int nm2, T c0,
                                           T c1) {
    su3<T> y = mm(mdm(U(mu, mm1 + nm1, 0), U(nu, mm1 + nm1, 0)), U(mu, mm1, 1));  // D'
    su3<T> x = mdm(U(mu, nm1, 1), y);
    y = mm(mdmd(U(nu, mp1 + nm2, 1), U(mu, nm2, 0)), U(nu, nm2, 0));             // T'
    mm_acc(x, y, U(nu, nm1, 1));
    su3<T> w = mdm(U(mu, nm1, 1), U(nu, nm1, 1));
    axpby(x, c1, c0, w);
    mdm_acc(acc, U(nu, mp1 + nm1, 0), x);
    y = mmd(mmd(U(mu, mp1, 1), U(nu, mp2 + nm1, 1)), U(mu, mp1 + nm1, 0));     // E'
    scale(w, c1);
    mm_acc(acc, y, w);
}

// TPL threads per link (1 or 2): a block is TPL waves over the same kStapleLinks
// links; with 2, wave 0 sums the +nu sides and wave 1 the -nu sides, and wave 0
// adds wave 1's sums from LDS.  Two waves per SIMD (256 registers) are asked of the
// two-thread FP64-18 kernel only: the one-thread one would spill 248 bytes (2049 -> 3107 us
// at 32^4), the FP64-12 ones lose more than they gain (comment at side()).
// EPI 0 writes Sigma; EPI 1 (FP64 or FP32-12 links) instead adds (eps beta / 3) times the
// traceless Hermitian part of i U Sigma to the link's momentum: P -> P - eps F with the
// Symanzik gauge force F = -(beta/3) [i U Sigma]_TH, the staples never leaving the
// kernel.
template <typename T, int FMT, int TPL, int EPI>
__global__ __launch_bounds__(kStapleLinks * TPL)
__attribute__((amdgpu_waves_per_eu(FMT == FMT_C128_18 && TPL == 2 ? 2 : 1)))
void staple_kernel(StapleArgs a) {
    __shared__ cpx<T> part[9][kStapleLinks];
    const Geom &g = a.geom;
    const uint32_t blk = a.xcd_remap ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int slot = (int)(blk % 8);
    const int q = (int)threadIdx.x / kStapleLinks;  // the same in a whole wave
    const int l = (int)threadIdx.x % kStapleLinks;
    const uint32_t j = (blk / 8) * kStapleLinks + l;
    const bool valid = j < g.Vh;
    const uint32_t h = valid ? pencil_site(g, a.tile, j) : 0;
    const int mu = slot >> 1, P = slot & 1;

    // one thread per link: the last factor of the backward paths is taken once for all six
    // sides; two: a second sum of 9 entries would cost each wave more than it saves
    constexpr bool kBack = TPL == 1 && FMT != FMT_C128_18;
    su3<T> acc, back;
    set_zero(acc);
    if (kBack) set_zero(back);

    if (valid) {
        const Site s = site_coords(g, P, h);
        const int st[4] = {1, (int)g.N[0], (int)(g.N[0] * g.N[1]),
                           (int)(g.N[0] * g.N[1] * g.N[2])};
        const int L = (int)s.x[0] + st[1] * (int)s.x[1] + st[2] * (int)s.x[2] +
                      st[3] * (int)s.x[3];
        const LinkAt<T, FMT> U{a.links, g.Vh, L, P};
        const int xm = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], mu);
        const int nm = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], mu);
        const int sm = (int)pick4(st[0], st[1], st[2], st[3], mu);
        const int mp1 = lex_step(xm, 1, nm, sm), mm1 = lex_step(xm, -1, nm, sm);
        const int mp2 = lex_step(xm, 2, nm, sm);
        const T c0 = (T)a.c0, c1 = (T)a.c1;
        RawLink<T, FMT> u0;
        if constexpr (FMT != FMT_C128_18) U.fetch(u0, mu, mp1, 1);
#pragma unroll 1
        for (int k = 1; k < 4; ++k) {
            const int nu = (mu + k) & 3;
            const int xn = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], nu);
            const int nn = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], nu);
            const int sn = (int)pick4(st[0], st[1], st[2], st[3], nu);
            const int np1 = lex_step(xn, 1, nn, sn), np2 = lex_step(xn, 2, nn, sn);
            const int nm1 = lex_step(xn, -1, nn, sn), nm2 = lex_step(xn, -2, nn, sn);
            if (TPL == 1 || q == 0) {
                if constexpr (FMT == FMT_C128_18)
                    side_above_full(acc, U, mu, nu, mp1, mm1, mp2, np1, np2, c0, c1);
                else
                    side<T, FMT, kBack, true>(acc, back, u0, U, mu, nu, mp1, mm1, mp2, np1, np2,
                                              c0, c1);
            }
            if (TPL == 1 || q == 1) {
                if constexpr (FMT == FMT_C128_18)
                    side_below_full(acc, U, mu, nu, mp1, mm1, mp2, nm1, nm2, c0, c1);
                else
                    side<T, FMT, kBack, false>(acc, back, u0, U, mu, nu, mp1, mm1, mp2, nm1, nm2,
                                               c0, c1);
            }
        }
        if constexpr (kBack) axpy(acc, c1, mm(back, U(mu, mm1, 1)));
    }
    if (TPL == 2) {
        if (q == 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int k = 0; k < 3; ++k) part[i * 3 + k][l] = acc.e[i][k];
        }
        __syncthreads();
        if (q == 1) return;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cpx<T> v = part[i * 3 + k][l];
                acc.e[i][k].re += v.re;
                acc.e[i][k].im += v.im;
            }
    }
    if (!valid) return;
    const size_t base = (size_t)slot * 9 * g.Vh + h;
    if constexpr (EPI == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                st_c<T>(a.out, base + (size_t)(i * 3 + k) * g.Vh, acc.e[i][k]);
    } else {
        // M = U Sigma; [iM]_TH = i (M - M^dag) / 2 + (sum_j Im M_jj / 3) I
        const su3<T> u = cached_link<T, FMT>::load(a.links, g.Vh, slot, h);
        const su3<T> m = mm(u, acc);
        const T tr = (m.e[0][0].im + m.e[1][1].im + m.e[2][2].im) / T(3);
        const T kf = (T)a.kmom;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cpx<T> d = csub(m.e[i][k], cconj(m.e[k][i]));
                cpx<T> th = {T(-0.5) * d.im, T(0.5) * d.re};
                if (i == k) th.re += tr;
                const size_t idx = base + (size_t)(i * 3 + k) * g.Vh;
                cpx<T> pm = ld_c<T>(a.out, idx);
                pm.re = fmat(kf, th.re, pm.re);
                pm.im = fmat(kf, th.im, pm.im);
                st_c<T>(a.out, idx, pm);
            }
    }
}

// A Hermitian 3x3 matrix: the real diagonal and the entries above it.
struct herm3 {
    double d[3];
    cpx<double> o01, o02, o12;
    __device__ __forceinline__ su3<double> full() const {
        su3<double> m;
        m.e[0][0] = {d[0], 0.0};
        m.e[1][1] = {d[1], 0.0};
        m.e[2][2] = {d[2], 0.0};
        m.e[0][1] = o01;
        m.e[0][2] = o02;
        m.e[1][2] = o12;
        m.e[1][0] = cconj(o01);
        m.e[2][0] = cconj(o02);
        m.e[2][1] = cconj(o12);
        return m;
    }
};

__device__ __forceinline__ double cabs2(cpx<double> a) { return fmat(a.re, a.re, a.im * a.im); }

// Q Q of a Hermitian Q (Hermitian again)
__device__ __forceinline__ herm3 square(const herm3 &q) {
    const double n01 = cabs2(q.o01), n02 = cabs2(q.o02), n12 = cabs2(q.o12);
    herm3 s;
    s.d[0] = fmat(q.d[0], q.d[0], n01 + n02);
    s.d[1] = fmat(q.d[1], q.d[1], n01 + n12);
    s.d[2] = fmat(q.d[2], q.d[2], n02 + n12);
    s.o01 = cscale(q.d[0] + q.d[1], q.o01);
    cfma(s.o01, q.o02, cconj(q.o12));
    s.o02 = cscale(q.d[0] + q.d[2], q.o02);
    cfma(s.o02, q.o01, q.o12);
    s.o12 = cscale(q.d[1] + q.d[2], q.o12);
    cfmac(s.o12, q.o01, q.o02);
    return s;
}

// det Q = Tr(Q^3) / 3 of a traceless Hermitian Q
__device__ __forceinline__ double det(const herm3 &q) {
    cpx<double> t = cmul(q.o01, q.o12);
    const double z = fmat(t.re, q.o02.re, t.im * q.o02.im);  // Re(q01 q12 q20)
    double v = q.d[0] * fmat(q.d[1], q.d[2], -cabs2(q.o12));
    v = fmat(-q.d[1], cabs2(q.o02), v);
    v = fmat(-q.d[2], cabs2(q.o01), v);
    return fmat(2.0, z, v);
}

// exp(iQ) = f0 + f1 Q + f2 Q^2 for a traceless Hermitian Q (Cayley-Hamilton: Q^3 = c1 Q +
// c0, c0 = det Q, c1 = Tr(Q^2)/2), and with DERIV the derivatives of f0, f1, f2 by c0 and
// by c1, from which the derivative of exp(iQ) in any direction follows.
//
// The f_j are the coefficients of the exponential series reduced modulo the
// characteristic polynomial, evaluated by Horner's rule on the triple (f0, f1, f2):
// multiplying by Q maps it to (c0 f2, f0 + c1 f2, f1).  The coefficients i^n/n! are real
// or imaginary in turn, so each step is two fused operations per part and five more for
// the derivatives: about 90 (300 with the derivatives) in all, where the trigonometric
// closed form takes several times that and the series in 3x3 matrices, as the derivative
// had it before, 55 matrix products.  With c1 <= 3/4 the eigenvalues stay below 1 in
// magnitude, what the first term left out (n = 22) would add is below 4e-22 in the f_j and
// 4e-21 in their derivatives (1/22! is 8.9e-22), and no term cancels by more than a factor
// e.  Larger Q: the triple of exp(iQ/2^s), squared s times in the same ring.
struct ExpCoef {
    cpx<double> f[3], d0[3], d1[3];
};

// (f, d0, d1) of p^2 from those of p, modulo Q^3 = c1 Q + c0
template <bool DERIV>
__device__ __forceinline__ void ring_square(ExpCoef &p, double c0, double c1) {
    const cpx<double> a = p.f[0], b = p.f[1], c = p.f[2];
    const cpx<double> t3 = cscale(2.0, cmul(b, c)), t4 = cmul(c, c);  // of Q^3 and Q^4
    ExpCoef r;
    r.f[0] = cadd(cmul(a, a), cscale(c0, t3));
    r.f[1] = cadd(cscale(2.0, cmul(a, b)), cadd(cscale(c1, t3), cscale(c0, t4)));
    r.f[2] = cadd(cadd(cscale(2.0, cmul(a, c)), cmul(b, b)), cscale(c1, t4));
    if (DERIV) {
        const auto dstep = [&](const cpx<double>(&q)[3], cpx<double>(&o)[3]) {
            const cpx<double> u3 = cscale(2.0, cadd(cmul(q[1], c), cmul(b, q[2])));
            const cpx<double> u4 = cscale(2.0, cmul(c, q[2]));
            o[0] = cadd(cscale(2.0, cmul(a, q[0])), cscale(c0, u3));
            o[1] = cadd(cscale(2.0, cadd(cmul(a, q[1]), cmul(q[0], b))),
                        cadd(cscale(c1, u3), cscale(c0, u4)));
            o[2] = cadd(cscale(2.0, cadd(cadd(cmul(a, q[2]), cmul(q[0], c)), cmul(b, q[1]))),
                        cscale(c1, u4));
        };
        dstep(p.d0, r.d0);
        r.d0[0] = cadd(r.d0[0], t3);
        r.d0[1] = cadd(r.d0[1], t4);
        dstep(p.d1, r.d1);
        r.d1[1] = cadd(r.d1[1], t3);
        r.d1[2] = cadd(r.d1[2], t4);
    }
    p.f[0] = r.f[0];
    p.f[1] = r.f[1];
    p.f[2] = r.f[2];
    if (DERIV) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            p.d0[i] = r.d0[i];
            p.d1[i] = r.d1[i];
        }
    }
}

constexpr int kExpTerms = 22;

constexpr double inv_factorial(int n) {
    double v = 1.0;
    for (int i = 2; i <= n; ++i) v /= (double)i;
    return v;
}

template <int N>
struct InvFactorials {
    double v[N];
    constexpr InvFactorials() : v() {
        for (int n = 0; n < N; ++n) v[n] = inv_factorial(n);
    }
};

template <bool DERIV>
__device__ __forceinline__ ExpCoef exp_coef(double c0, double c1) {
    int sq = 0;
    while (c1 > 0.75 && sq < 40) {  // Q -> Q/2
        c1 *= 0.25;
        c0 *= 0.125;
        ++sq;
    }
    constexpr InvFactorials<kExpTerms> inv;
    // real and imaginary parts: cos and sin series, never mixed
    double f[2][3] = {}, d0[2][3] = {}, d1[2][3] = {};
#pragma unroll
    for (int n = kExpTerms - 1; n >= 0; --n) {
#pragma unroll
        for (int z = 0; z < 2; ++z) {  // 0: real, 1: imaginary
            if (DERIV) {
                const double a0 = fmat(c0, d0[z][2], f[z][2]);
                const double a1 = fmat(c1, d0[z][2], d0[z][0]);
                const double b0 = c0 * d1[z][2];
                const double b1 = fmat(c1, d1[z][2], d1[z][0]) + f[z][2];
                d0[z][2] = d0[z][1];
                d0[z][0] = a0;
                d0[z][1] = a1;
                d1[z][2] = d1[z][1];
                d1[z][0] = b0;
                d1[z][1] = b1;
            }
            const double coef = (n & 1) == z ? ((n & 2) ? -inv.v[n] : inv.v[n]) : 0.0;
            const double g0 = fmat(c0, f[z][2], coef), g1 = fmat(c1, f[z][2], f[z][0]);
            f[z][2] = f[z][1];
            f[z][0] = g0;
            f[z][1] = g1;
        }
    }
    ExpCoef e;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        e.f[i] = {f[0][i], f[1][i]};
        e.d0[i] = {d0[0][i], d0[1][i]};
        e.d1[i] = {d1[0][i], d1[1][i]};
    }
    if (sq > 0) {
        for (int r = 0; r < sq; ++r) ring_square<DERIV>(e, c0, c1);
        // from powers of Q/2^s to powers of Q
        const double h = ldexp(1.0, -sq);
        e.f[1] = cscale(h, e.f[1]);
        e.f[2] = cscale(h * h, e.f[2]);
        if (DERIV) {
            const double h2 = h * h, h3 = h2 * h;
            double w = 1.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                e.d0[i] = cscale(w * h3, e.d0[i]);
                e.d1[i] = cscale(w * h2, e.d1[i]);
                w *= h;
            }
        }
    }
    return e;
}

// f0 + f1 Q + f2 Q^2
__device__ __forceinline__ su3<double> exp_matrix(const ExpCoef &c, const herm3 &q,
                                                  const herm3 &q2) {
    const su3<double> a = q.full(), b = q2.full();
    su3<double> e;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (i == k) {
                // the largest term last (f0 of the real part, f1 Q of the imaginary one), so that
                // one addition rounds at its size
                e.e[i][k] = {c.f[0].re + fmat(c.f[2].re, b.e[i][k].re, c.f[1].re * a.e[i][k].re),
                             fmat(c.f[1].im, a.e[i][k].re, fmat(c.f[2].im, b.e[i][k].re, c.f[0].im))};
            } else {
                cpx<double> v = cmul(c.f[1], a.e[i][k]);
                cfma(v, c.f[2], b.e[i][k]);
                e.e[i][k] = v;
            }
        }
    return e;
}

// exp(iQ) for a traceless Hermitian Q
__device__ __forceinline__ su3<double> exp_iq(const herm3 &q) {
    const herm3 q2 = square(q);
    return exp_matrix(exp_coef<false>(det(q), 0.5 * (q2.d[0] + q2.d[1] + q2.d[2])), q, q2);
}

// Q = (i/2)(Omega^dag - Omega) - (i/6) Tr(Omega^dag - Omega)
__device__ __forceinline__ herm3 stout_q(const su3<double> &om) {
    const double tq = (om.e[0][0].im + om.e[1][1].im + om.e[2][2].im) / 3.0;
    herm3 q;
#pragma unroll
    for (int i = 0; i < 3; ++i) q.d[i] = om.e[i][i].im - tq;
    const auto off = [&](int i, int k) {
        const cpx<double> z = csub(cconj(om.e[k][i]), om.e[i][k]);
        return cpx<double>{-0.5 * z.im, 0.5 * z.re};
    };
    q.o01 = off(0, 1);
    q.o02 = off(0, 2);
    q.o12 = off(1, 2);
    return q;
}

// The traceless anti-Hermitian matrix G of a link between the two passes: the imaginary
// parts of G00 and G11 (G22 = -G00 - G11), then G01, G02, G12: four 16-byte words,
// [slot][word][site].
struct RawG {
    double2 w[4];
    __device__ __forceinline__ void fetch(const void *ws, uint32_t Vh, int s, uint32_t h) {
        const double2 *p = reinterpret_cast<const double2 *>(ws) + (size_t)s * 4 * Vh + h;
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = p[(size_t)k * Vh];
    }
    __device__ __forceinline__ su3<double> mat() const {
        su3<double> g;
        g.e[0][0] = {0.0, w[0].x};
        g.e[1][1] = {0.0, w[0].y};
        g.e[2][2] = {0.0, -w[0].x - w[0].y};
        g.e[0][1] = {w[1].x, w[1].y};
        g.e[0][2] = {w[2].x, w[2].y};
        g.e[1][2] = {w[3].x, w[3].y};
        g.e[1][0] = {-w[1].x, w[1].y};
        g.e[2][0] = {-w[2].x, w[2].y};
        g.e[2][1] = {-w[3].x, w[3].y};
        return g;
    }
};

__device__ __forceinline__ cpx<double> trace_mul(const su3<double> &a, const su3<double> &b) {
    cpx<double> t = {0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) cfma(t, a.e[i][k], b.e[k][i]);
    return t;
}

// Pass 1 of the force through a stout step, one thread per link l = (mu, x):
// C = rho (3-link paths from x to x+mu), Omega = C U^dag, Q, M = U Sigma'_l,
// Gamma = L(iQ, M) with L the Frechet derivative of exp; G = (Gamma - Gamma^dag)/2 +
// (conj(Tr Gamma) - Tr Gamma)/6; out_l = Sigma'_l exp(iQ) + C^dag G^dag, ws_l = G.
//
// With exp(iQ) = f0 + f1 Q + f2 Q^2 the derivative in the direction E = -iM of Q is
//   df0 + df1 Q + df2 Q^2 + f1 E + f2 (Q E + E Q),
//   df_j = (df_j/dc0) Tr(Q^2 E0) + (df_j/dc1) Tr(Q E0),  E0 = E - Tr(E)/3,
// and the part Tr(E)/3 of E along the identity adds i Tr(E)/3 exp(iQ) in place of its
// share in the terms above.  Multiples of the identity drop out of G.  (Before, L came
// from a 14-term series of 3x3 products scaled and squared back: 55 products per link of
// 75; the pass took 1209 us at 24^3 x 48 and 1752 at 32^4, now 518 and 712.)
template <int FMT>
__global__ __launch_bounds__(kStoutBlock) void stout_back1_kernel(StoutBackArgs a) {
    const Geom &g = a.geom;
    const uint32_t blk = a.xcd_remap ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int slot = (int)(blk % 8);
    const uint32_t j = (blk / 8) * kStoutBlock + threadIdx.x;
    if (j >= g.Vh) return;
    const uint32_t h = pencil_site(g, a.tile, j);
    const int mu = slot >> 1, P = slot & 1;
    const Site s = site_coords(g, P, h);
    const int st[4] = {1, (int)g.N[0], (int)(g.N[0] * g.N[1]), (int)(g.N[0] * g.N[1] * g.N[2])};
    const int L = (int)s.x[0] + st[1] * (int)s.x[1] + st[2] * (int)s.x[2] + st[3] * (int)s.x[3];
    const LinkAt<double, FMT> U{a.links, g.Vh, L, P};
    const int xm = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], mu);
    const int nm = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], mu);
    const int sm = (int)pick4(st[0], st[1], st[2], st[3], mu);
    const int mp1 = lex_step(xm, 1, nm, sm);
    su3<double> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) c.e[i][k] = {0.0, 0.0};
#pragma unroll 1
    for (int k = 1; k < 4; ++k) {
        const int nu = (mu + k) & 3;
        const int xn = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], nu);
        const int nn = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], nu);
        const int sn = (int)pick4(st[0], st[1], st[2], st[3], nu);
        const int np1 = lex_step(xn, 1, nn, sn), nm1 = lex_step(xn, -1, nn, sn);
        mmd_acc(c, mm(U(nu, 0, 0), U(mu, np1, 1)), U(nu, mp1, 1));
        mm_acc(c, mdm(U(nu, nm1, 1), U(mu, nm1, 1)), U(nu, mp1 + nm1, 0));
    }
    scale(c, a.rho);
    su3<double> m;  // E = -i U Sigma'
    herm3 q;
    {
        const su3<double> u = U(mu, 0, 0);
        q = stout_q(mmd(c, u));
        m = mm(u, cached_link<double, FMT_C128_18>::load(a.sigp, g.Vh, slot, h));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) m.e[i][k] = {m.e[i][k].im, -m.e[i][k].re};
    const herm3 q2 = square(q);
    const double c1 = 0.5 * (q2.d[0] + q2.d[1] + q2.d[2]);
    const ExpCoef f = exp_coef<true>(det(q), c1);
    const su3<double> qf = q.full(), q2f = q2.full();
    const cpx<double> t3 = cscale(1.0 / 3.0, cadd(cadd(m.e[0][0], m.e[1][1]), m.e[2][2]));
    const cpx<double> tq1 = trace_mul(qf, m);                                       // Tr(Q E0)
    const cpx<double> tq2 = csub(trace_mul(q2f, m), cscale(2.0 * c1, t3));          // Tr(Q^2 E0)
    const cpx<double> it3 = {-t3.im, t3.re};
    // of the terms al Q and be Q^2 (Hermitian matrices) only the imaginary parts of al
    // and be reach the anti-Hermitian G
    cpx<double> al = cmul(f.d0[1], tq2), be = cmul(f.d0[2], tq2);
    cfma(al, f.d1[1], tq1);
    cfma(al, it3, f.f[1]);
    cfma(al, cscale(-2.0, t3), f.f[2]);
    cfma(be, f.d1[2], tq1);
    cfma(be, it3, f.f[2]);
    su3<double> gam;
    {
        su3<double> w = mm(qf, m);
        mm_acc(w, m, qf);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                gam.e[i][k] = cmul(f.f[1], m.e[i][k]);
                cfma(gam.e[i][k], f.f[2], w.e[i][k]);
            }
    }
    su3<double> gg;
    double gd[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        gd[i] = fmat(al.im, q.d[i], fmat(be.im, q2.d[i], gam.e[i][i].im));
    const double tg = (gd[0] + gd[1] + gd[2]) / 3.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) gg.e[i][i] = {0.0, gd[i] - tg};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = i + 1; k < 3; ++k) {
            cpx<double> v = cscale(0.5, csub(gam.e[i][k], cconj(gam.e[k][i])));
            // + i (Im al Q + Im be Q^2)
            v.re = fmat(-al.im, qf.e[i][k].im, fmat(-be.im, q2f.e[i][k].im, v.re));
            v.im = fmat(al.im, qf.e[i][k].re, fmat(be.im, q2f.e[i][k].re, v.im));
            gg.e[i][k] = v;
            gg.e[k][i] = {-v.re, v.im};
        }
    double2 *gp = reinterpret_cast<double2 *>(a.ws) + (size_t)slot * 4 * g.Vh + h;
    gp[0] = make_double2(gg.e[0][0].im, gg.e[1][1].im);
    gp[g.Vh] = make_double2(gg.e[0][1].re, gg.e[0][1].im);
    gp[2 * (size_t)g.Vh] = make_double2(gg.e[0][2].re, gg.e[0][2].im);
    gp[3 * (size_t)g.Vh] = make_double2(gg.e[1][2].re, gg.e[1][2].im);
    const su3<double> gcm = mm(gg, c);  // C^dag G^dag = (G C)^dag
    const su3<double> e = exp_matrix(f, q, q2);
    const su3<double> loc = mm(cached_link<double, FMT_C128_18>::load(a.sigp, g.Vh, slot, h), e);
    const size_t base = (size_t)slot * 9 * g.Vh + h;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            st_c<double>(a.out, base + (size_t)(i * 3 + k) * g.Vh,
                         cadd(loc.e[i][k], cconj(gcm.e[k][i])));
}

// Pass 2, two threads per link l = (nu, y): add rho times every product in which l
// stands in a 3-link path of C at a neighbouring link.  For a path's own link l' the
// product ends in U_l'^dag G_l', and the G are anti-Hermitian, so for each direction
// b != nu the three paths on either side of the link share their factors.  With
// U1 = U_b(y+nu), U2 = U_nu(y+b), U3 = U_b(y), G1 = G(nu,y+b), G3 = G(b,y), G5 = G(b,y+nu)
// the side of +b adds
//   U1 U2^dag G1 U3^dag + U1 U2^dag U3^dag G3 - G5 U1 U2^dag U3^dag
//     = (P G1 - G5 P) U3^dag + (P U3^dag) G3,  P = U1 U2^dag,
// and with V1 = U_b(y-b+nu), V2 = U_nu(y-b), V3 = U_b(y-b), H1 = G(nu,y-b), H3 = G(b,y-b),
// H5 = G(b,y-b+nu) the side of -b
//   V1^dag [ V2^dag (H1 - H3) + H5 V2^dag ] V3:
// 10 matrix products and 60 16-byte loads of the 12-real links and the G per direction
// (12 and 126 when the six products were taken one by one from stored U^dag G), which is
// what bounds the pass: 1050 -> 699 us at 24^3 x 48 and 1449 -> 994 at 32^4, with every
// matrix fetched a product ahead, at two waves per SIMD.  (Both passes of 24^3 x 48 back to
// back: 1213 before the fetches ahead, 1114 with them, 1193 at three waves, which spill in
// 168 registers.)
template <int FMT>
__global__ __launch_bounds__(2 * kStapleLinks) void stout_back2_kernel(StoutBackArgs a) {
    // two waves over the same kStapleLinks links: wave 0 sums the +b sides, wave 1 the -b
    // sides; wave 1's sums meet wave 0's in LDS
    __shared__ cpx<double> part[9][kStapleLinks];
    const Geom &g = a.geom;
    const uint32_t blk = a.xcd_remap ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int slot = (int)(blk % 8);
    const int q = (int)threadIdx.x / kStapleLinks;  // the same in a whole wave
    const int l = (int)threadIdx.x % kStapleLinks;
    const uint32_t j = (blk / 8) * kStapleLinks + l;
    const bool valid = j < g.Vh;
    const uint32_t h = valid ? pencil_site(g, a.tile, j) : 0;
    const int nu = slot >> 1, P = slot & 1;
    su3<double> acc;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) acc.e[i][k] = {0.0, 0.0};
    if (valid) {
        const Site s = site_coords(g, P, h);
        const int st[4] = {1, (int)g.N[0], (int)(g.N[0] * g.N[1]),
                           (int)(g.N[0] * g.N[1] * g.N[2])};
        const int L = (int)s.x[0] + st[1] * (int)s.x[1] + st[2] * (int)s.x[2] +
                      st[3] * (int)s.x[3];
        const LinkAt<double, FMT> U{a.links, g.Vh, L, P};
        const auto fetch_g = [&](RawG &r, int d, int dl, int flip) {
            r.fetch(a.ws, g.Vh, 2 * d + ((P + flip) & 1), (uint32_t)(L + dl) >> 1);
        };
        const int xv = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], nu);
        const int nv = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], nu);
        const int sv = (int)pick4(st[0], st[1], st[2], st[3], nu);
        const int vp1 = lex_step(xv, 1, nv, sv);
#pragma unroll 1
        for (int k = 1; k < 4; ++k) {
            const int b = (nu + k) & 3;
            const int xb = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], b);
            const int nb = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], b);
            const int sb = (int)pick4(st[0], st[1], st[2], st[3], b);
            RawLink<double, FMT> u, v;
            RawG m, n;
            if (q == 0) {
                const int bp1 = lex_step(xb, 1, nb, sb);
                U.fetch(u, b, vp1, 1);
                U.fetch(v, nu, bp1, 1);
                fetch_g(m, nu, bp1, 1);
                fetched();
                const su3<double> p = mmd(u.link(), v.link());
                fetch_g(n, b, vp1, 1);
                fetched();
                su3<double> t = mm(p, m.mat());
                U.fetch(u, b, 0, 0);
                fetched();
                mm_sub(t, n.mat(), p);
                fetch_g(m, b, 0, 0);
                fetched();
                const su3<double> u3 = u.link();
                mmd_acc(acc, t, u3);
                mm_acc(acc, mmd(p, u3), m.mat());
            } else {
                const int bm1 = lex_step(xb, -1, nb, sb);
                U.fetch(v, nu, bm1, 1);
                fetch_g(m, nu, bm1, 1);
                fetch_g(n, b, bm1, 1);
                fetched();
                su3<double> d = m.mat();
                {
                    const su3<double> h3 = n.mat();
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int c = 0; c < 3; ++c) d.e[i][c] = csub(d.e[i][c], h3.e[i][c]);
                }
                const su3<double> v2 = v.link();
                fetch_g(m, b, bm1 + vp1, 0);
                fetched();
                su3<double> t = mdm(v2, d);
                U.fetch(u, b, bm1 + vp1, 0);
                fetched();
                mmd_acc(t, m.mat(), v2);
                U.fetch(v, b, bm1, 1);
                fetched();
                mm_acc(acc, mdm(u.link(), t), v.link());
            }
        }
    }
    if (q == 1) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) part[i * 3 + k][l] = acc.e[i][k];
    }
    __syncthreads();
    if (q == 1 || !valid) return;
    const size_t base = (size_t)slot * 9 * g.Vh + h;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const size_t idx = base + (size_t)(i * 3 + k) * g.Vh;
            const cpx<double> w1 = part[i * 3 + k][l];
            cpx<double> v = ld_c<double>(a.out, idx);
            v.re = fmat(a.rho, acc.e[i][k].re + w1.re, v.re);
            v.im = fmat(a.rho, acc.e[i][k].im + w1.im, v.im);
            st_c<double>(a.out, idx, v);
        }
}

// FP64-18 links: at most two waves per SIMD.  At three (136 registers) the neighbourhoods
// of the links in flight outgrow the L2 of the XCD: 857 us against 677 at 32^4.
template <int FMT>
__global__ __launch_bounds__(kStoutBlock)
__attribute__((amdgpu_waves_per_eu(1, FMT == FMT_C128_18 ? 2 : 8))) void stout_kernel(StoutArgs a) {
    const Geom &g = a.geom;
    const uint32_t blk = a.xcd_remap ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int slot = (int)(blk % 8);
    const uint32_t j = (blk / 8) * kStoutBlock + threadIdx.x;
    if (j >= g.Vh) return;
    const uint32_t h = pencil_site(g, a.tile, j);
    const int mu = slot >> 1, P = slot & 1;
    const Site s = site_coords(g, P, h);
    const int st[4] = {1, (int)g.N[0], (int)(g.N[0] * g.N[1]), (int)(g.N[0] * g.N[1] * g.N[2])};
    const int L = (int)s.x[0] + st[1] * (int)s.x[1] + st[2] * (int)s.x[2] + st[3] * (int)s.x[3];
    const LinkAt<double, FMT> U{a.links, g.Vh, L, P};
    const int xm = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], mu);
    const int nm = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], mu);
    const int sm = (int)pick4(st[0], st[1], st[2], st[3], mu);
    const int mp1 = lex_step(xm, 1, nm, sm);

    // C / rho: the 3-link paths from x to x + mu, above and below in each plane
    su3<double> c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) c.e[i][k] = {0.0, 0.0};
#pragma unroll 1
    for (int k = 1; k < 4; ++k) {
        const int nu = (mu + k) & 3;
        const int xn = (int)pick4(s.x[0], s.x[1], s.x[2], s.x[3], nu);
        const int nn = (int)pick4(g.N[0], g.N[1], g.N[2], g.N[3], nu);
        const int sn = (int)pick4(st[0], st[1], st[2], st[3], nu);
        const int np1 = lex_step(xn, 1, nn, sn), nm1 = lex_step(xn, -1, nn, sn);
        // U_nu(x) U_mu(x+nu) U_nu(x+mu)^dag
        mmd_acc(c, mm(U(nu, 0, 0), U(mu, np1, 1)), U(nu, mp1, 1));
        // U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu)
        mm_acc(c, mdm(U(nu, nm1, 1), U(mu, nm1, 1)), U(nu, mp1 + nm1, 0));
    }
    scale(c, a.rho);
    const su3<double> u = U(mu, 0, 0);
    const herm3 q = stout_q(mmd(c, u));  // of Omega = C U^dag
    const su3<double> up = mm(exp_iq(q), u);
    const size_t base = (size_t)slot * 9 * g.Vh + h;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) st_c<double>(a.out, base + (size_t)(i * 3 + k) * g.Vh, up.e[i][k]);
}

template <typename T, int FMT>
int launch_tpl(const StapleArgs &a, int threads, hipStream_t stream) {
    const dim3 grid(staple_blocks(a.geom.Vh));
    if (threads == 1) {
        staple_kernel<T, FMT, 1, 0><<<grid, kStapleLinks, 0, stream>>>(a);
        return 0;
    }
    if (threads == 2) {
        staple_kernel<T, FMT, 2, 0><<<grid, 2 * kStapleLinks, 0, stream>>>(a);
        return 0;
    }
    return -1;
}

template <typename T, int FMT>
int launch_mom(const StapleArgs &a, int threads, hipStream_t stream) {
    const dim3 grid(staple_blocks(a.geom.Vh));
    if (threads == 1) {
        staple_kernel<T, FMT, 1, 1><<<grid, kStapleLinks, 0, stream>>>(a);
        return 0;
    }
    if (threads == 2) {
        staple_kernel<T, FMT, 2, 1><<<grid, 2 * kStapleLinks, 0, stream>>>(a);
        return 0;
    }
    return -1;
}

// U -> exp(i eps P) U in place, one thread per link, in the link's own format.  Bound by
// its traffic: of the Hermitian P the diagonal and the entries above it are read (288 B
// per FP64-12 link with them, 336 with all nine; 267 -> 210 us at 32^4).  The
// exponential is formed in FP64 also for FP32 links and momenta (its cost is small
// next to the link and momentum traffic), the product with U in the format's type.
template <typename T, int FMT>
__global__ __launch_bounds__(kStoutBlock) void link_update_kernel(LinkUpdateArgs a) {
    const uint32_t Vh = a.Vh;
    const size_t n = (size_t)8 * Vh;
    const size_t t = (size_t)blockIdx.x * kStoutBlock + threadIdx.x;
    if (t >= n) return;
    const int slot = (int)(t / Vh);
    const uint32_t h = (uint32_t)(t % Vh);
    const su3<T> u = cached_link<T, FMT>::load(a.links, Vh, slot, h);
    // eps P: of a Hermitian matrix the diagonal and the entries above it are read
    const size_t base = (size_t)slot * 9 * Vh + h;
    const auto P = [&](int i, int k) {
        const cpx<T> p = ld_c<T>(a.mom, base + (size_t)(i * 3 + k) * Vh);
        return cpx<double>{a.eps * (double)p.re, a.eps * (double)p.im};
    };
    const herm3 q = {{P(0, 0).re, P(1, 1).re, P(2, 2).re}, P(0, 1), P(0, 2), P(1, 2)};
    const su3<double> e64 = exp_iq(q);
    su3<T> e;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) e.e[i][k] = {(T)e64.e[i][k].re, (T)e64.e[i][k].im};
    const su3<T> up = mm(e, u);
    if constexpr (FMT == FMT_C64_12) {
        // float4 chunks: (U00, U01), (U02, U10), (U11, U12)
        float4 *p = reinterpret_cast<float4 *>(a.links) + (size_t)slot * 3 * Vh + h;
        p[0] = make_float4(up.e[0][0].re, up.e[0][0].im, up.e[0][1].re, up.e[0][1].im);
        p[Vh] = make_float4(up.e[0][2].re, up.e[0][2].im, up.e[1][0].re, up.e[1][0].im);
        p[2 * (size_t)Vh] = make_float4(up.e[1][1].re, up.e[1][1].im, up.e[1][2].re, up.e[1][2].im);
    } else {
        constexpr int rows = FMT == FMT_C128_18 ? 3 : 2;
        const size_t lbase = (size_t)slot * rows * 3 * Vh + h;
#pragma unroll
        for (int i = 0; i < rows; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                st_c<T>(a.links, lbase + (size_t)(i * 3 + k) * Vh, up.e[i][k]);
    }
}

}  // namespace

int launch_stout_backprop(const StoutBackArgs &a, int fmt, hipStream_t stream) {
    const dim3 grid(stout_blocks(a.geom.Vh));
    const dim3 grid2(staple_blocks(a.geom.Vh));  // kStapleLinks links per block, two waves
    switch (fmt) {
        case FMT_C128_18:
            stout_back1_kernel<FMT_C128_18><<<grid, kStoutBlock, 0, stream>>>(a);
            stout_back2_kernel<FMT_C128_18><<<grid2, 2 * kStapleLinks, 0, stream>>>(a);
            return 0;
        case FMT_C128_12:
            stout_back1_kernel<FMT_C128_12><<<grid, kStoutBlock, 0, stream>>>(a);
            stout_back2_kernel<FMT_C128_12><<<grid2, 2 * kStapleLinks, 0, stream>>>(a);
            return 0;
        default: return -1;
    }
}

int launch_stout(const StoutArgs &a, int fmt, hipStream_t stream) {
    const dim3 grid(stout_blocks(a.geom.Vh));
    switch (fmt) {
        case FMT_C128_18: stout_kernel<FMT_C128_18><<<grid, kStoutBlock, 0, stream>>>(a); return 0;
        case FMT_C128_12: stout_kernel<FMT_C128_12><<<grid, kStoutBlock, 0, stream>>>(a); return 0;
        default: return -1;
    }
}

int launch_momentum(const StapleArgs &a, int fmt, int threads, hipStream_t stream) {
    switch (fmt) {
        case FMT_C128_18: return launch_mom<double, FMT_C128_18>(a, threads, stream);
        case FMT_C128_12: return launch_mom<double, FMT_C128_12>(a, threads, stream);
        case FMT_C64_12: return launch_mom<float, FMT_C64_12>(a, threads, stream);
        default: return -1;
    }
}

int launch_link_update(const LinkUpdateArgs &a, int fmt, hipStream_t stream) {
    const dim3 grid((unsigned)(((size_t)8 * a.Vh + kStoutBlock - 1) / kStoutBlock));
    switch (fmt) {
        case FMT_C128_18:
            link_update_kernel<double, FMT_C128_18><<<grid, kStoutBlock, 0, stream>>>(a);
            return 0;
        case FMT_C128_12:
            link_update_kernel<double, FMT_C128_12><<<grid, kStoutBlock, 0, stream>>>(a);
            return 0;
        case FMT_C64_12:
            link_update_kernel<float, FMT_C64_12><<<grid, kStoutBlock, 0, stream>>>(a);
            return 0;
        default: return -1;
    }
}

int launch_staples(const StapleArgs &a, int fmt, int threads, hipStream_t stream) {
    switch (fmt) {
        case FMT_C128_18: return launch_tpl<double, FMT_C128_18>(a, threads, stream);
        case FMT_C128_12: return launch_tpl<double, FMT_C128_12>(a, threads, stream);
        case FMT_C64_12: return launch_tpl<float, FMT_C64_12>(a, threads, stream);
        case FMT_BF16_12: return launch_tpl<float, FMT_BF16_12>(a, threads, stream);
        default: return -1;
    }
}

}  // namespace stg
