// HYP smearing of the gauge links (the smoothing the solver's links receive before the solve: the paper's
// quarks are HYP-smeared, Sec. 3). Three levels of staple sums restricted to the hypercubes that contain
// the link (the hypercubic blocking of Hasenfratz and Knechtli), each sum projected back to SU(3):
//
//   level 1  lv1(mu, eta):  (1 - a3) U_mu + a3/2 * staples of U_eta around U_mu        (12 fields)
//   level 2  lv2(mu, nu):   (1 - a2) U_mu + a2/4 * sum_{rho not mu, nu} staples of lv1(rho, s) around
//                           lv1(mu, s), s the direction outside {mu, nu, rho}              (12 fields)
//   level 3  V_mu:          (1 - a1) U_mu + a1/6 * sum_{nu != mu} staples of lv2(nu, mu) around lv2(mu, nu)
//
// with staples of side S around top T in direction eta at x:
//   S(x) T(x+eta) S(x+mu)^dag + S(x-eta)^dag T(x-eta) S(x-eta+mu).
//
// Proj_SU(3)(W) maximises Re tr(X^dag W) over SU(3). Where W^dag W is close to a multiple of the identity
// and the determinant phase of W is small (the usual case for smeared links) the maximiser is computed in
// closed form as a function of W^dag W (proj_direct below). Otherwise the unitary polar factor of W comes
// from scaled Newton iteration X <- (z X + X^-dag / z) / 2, z = |det X|^(-1/3), and the same closed form
// is tried from it (proj_series); failing that, the cube root of the determinant's phase (principal
// branch) is divided out and sweeps over the three SU(2) subgroups (Cabibbo-Marinari), each taking the
// subgroup element that maximises the objective, run until a sweep moves no element by more than 1e-15.
//
// One thread per (site, field). Every level is FP64. Input and output links use the natural layout [4][V][3][3]
// complex128 (a link is 9 consecutive double2); a first launch copies the input into planes, and the intermediate
// fields are planes in the caller's workspace. All directions are periodic.
//
// What bounds it. A staple pair reads six links, all of them past the 32 KB L1: measured at 20^3x64, levels 1 to 3
// drew 14.9, 12.2 and 10.9 TB/s from the L2, whatever the order of the blocks, with the FP64 units 32 to 40% busy. So the
// levels read planes (natural links of 144 bytes a lane apart cost four times the address cycles), store and read two
// rows of the projected links, and a projection takes about 500 multiply-adds where a 60-term series took 1,700:
// 3.13 -> 1.49 ms a smearing (planes 0.10, levels 0.42 + 0.64 + 0.34 ms; before 0.97 + 1.48 + 0.71 ms). Measured and
// left: one thread per run of sites along the staple direction, three loads a staple pair (2.2 ms: the runs along x
// lose their coalescing, and the carried links spill), one thread for lv1(mu, eta) and lv1(eta, mu) (1.68 ms, spills).
#include "sp_launch.h"

namespace sp {
namespace {

using C = Cx<double>;
using M3 = Su3<double>;

// Exact n / d for 0 <= n < 2^25 by one multiplication: M = ceil(2^(25 + l) / d) with 2^l >= d, so that the excess
// n (M d - 2^(25 + l)) / 2^(25 + l) stays below one.
struct Div {
    unsigned M;
    int shift;
    __device__ __forceinline__ int operator()(int n) const { return (int)(((unsigned long long)(unsigned)n * M) >> shift); }
};
Div div_by(int d) {
    int l = 0;
    while ((1L << l) < d) ++l;
    return {(unsigned)(((1ull << (25 + l)) + d - 1) / d), 25 + l};
}

struct HypGeom {
    int L[4];       // extents X, Y, Z, T
    int stride[4];  // 1, X, XY, XYZ
    Div by_L[4], by_stride[4];
    int V;
};

// Byte offsets (16 per site) of the neighbours of a site in a uniform direction mu, periodic. Hops in different
// directions commute, so the offset of n - eta + mu is that of -eta plus that of +mu.
struct Hop {
    unsigned f, b;
};
__device__ __forceinline__ Hop hop_at(const HypGeom& g, int c, int mu) {
    const int st = 16 * g.stride[mu], wrap = (g.L[mu] - 1) * st;
    return {(unsigned)(c == g.L[mu] - 1 ? -wrap : st), (unsigned)(c == 0 ? wrap : -st)};
}
__device__ __forceinline__ Hop hop(const HypGeom& g, int s, int mu) {
    const int q = g.by_stride[mu](s);
    return hop_at(g, q - g.by_L[mu](q) * g.L[mu], mu);
}

__device__ __forceinline__ C cmul(C a, C b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
// a * conj(b)
__device__ __forceinline__ C cmulc(C a, C b) { return {a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im}; }
__device__ __forceinline__ C cadd(C a, C b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ C csub(C a, C b) { return {a.re - b.re, a.im - b.im}; }

// acc + a b, acc + a conj(b), acc + conj(a) b as four fused multiply-adds
__device__ __forceinline__ C fmacc(C acc, C a, C b) {
    return {fma(-a.im, b.im, fma(a.re, b.re, acc.re)), fma(a.im, b.re, fma(a.re, b.im, acc.im))};
}
__device__ __forceinline__ C fmaccc(C acc, C a, C b) {
    return {fma(a.im, b.im, fma(a.re, b.re, acc.re)), fma(a.im, b.re, fma(-a.re, b.im, acc.im))};
}

// Row 2 of an SU(3) matrix from the other two: the conjugate of their cross product.
__device__ __forceinline__ void row2(M3& m) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const C a = m.e[0][(j + 1) % 3], b = m.e[1][(j + 2) % 3], c = m.e[0][(j + 2) % 3], d = m.e[1][(j + 1) % 3];
        m.e[2][j].re = fma(c.im, d.im, fma(-c.re, d.re, fma(-a.im, b.im, a.re * b.re)));
        m.e[2][j].im = fma(c.im, d.re, fma(c.re, d.im, fma(-a.im, b.re, -a.re * b.im)));
    }
}

// Intermediate links are stored as planes of double2, one per matrix entry, V sites each: rows 0 and 1 of the projected
// levels (ROWS = 2; row 2 of an SU(3) matrix is the conjugate cross product of the other two, formed again after a
// load: 24 multiply-adds against a third of the bytes, on a path bound by them), all three of the input links (ROWS = 3).
// A link sits at byte offset off = 16 s of its planes: a uniform plane address plus one 32-bit offset per lane (a plane
// holds less than 2^29 bytes), so that the loads of a link share their address registers.
template <int ROWS>
__device__ __forceinline__ M3 ld(const char* p, size_t plane, unsigned off) {
    M3 m;
#pragma unroll
    for (int j = 0; j < 3 * ROWS; ++j) {
        const double2 v = *(const double2*)(p + j * plane + off);
        m.e[j / 3][j % 3] = {v.x, v.y};
    }
    if constexpr (ROWS == 2) row2(m);
    return m;
}

template <int ROWS>
__device__ __forceinline__ void st(char* p, size_t plane, unsigned off, const M3& m) {
#pragma unroll
    for (int j = 0; j < 3 * ROWS; ++j)
        *(double2*)(p + j * plane + off) = make_double2(m.e[j / 3][j % 3].re, m.e[j / 3][j % 3].im);
}

__device__ __forceinline__ void scale(M3& w, double c) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            w.e[i][j].re *= c;
            w.e[i][j].im *= c;
        }
}

// Rows 0 .. ROWS-1 of a b, a b^dag and a^dag b.
template <int ROWS>
__device__ __forceinline__ M3 mul_rows(const M3& a, const M3& b) {
    M3 r;
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            r.e[i][j] = fmacc(fmacc(cmul(a.e[i][0], b.e[0][j]), a.e[i][1], b.e[1][j]), a.e[i][2], b.e[2][j]);
    return r;
}
template <int ROWS>
__device__ __forceinline__ M3 mul_nd_rows(const M3& a, const M3& b) {
    M3 r;
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            r.e[i][j] = fmaccc(fmaccc(cmulc(a.e[i][0], b.e[j][0]), a.e[i][1], b.e[j][1]), a.e[i][2], b.e[j][2]);
    return r;
}
template <int ROWS>
__device__ __forceinline__ M3 mul_dn_rows(const M3& a, const M3& b) {
    M3 r;
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            r.e[i][j] = fmaccc(fmaccc(cmulc(b.e[0][j], a.e[0][i]), b.e[1][j], a.e[1][i]), b.e[2][j], a.e[2][i]);
    return r;
}

// w += c * [S(x) T(x+eta) S(x+mu)^dag + S(x-eta)^dag T(x-eta) S(x-eta+mu)], S and T in planes. With ROWS = 2 the links
// are in SU(3), and so are the products: their third row is formed from the other two as well.
template <int ROWS>
__device__ __forceinline__ void add_staples(M3& w, double c, size_t plane, const char* S, const char* T, unsigned o,
                                            unsigned fm, Hop he) {
    const unsigned pe = o + he.f, me = o + he.b;
    auto add = [&](M3& p) {
        if constexpr (ROWS == 2) row2(p);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j)
                w.e[i][j] = {fma(c, p.e[i][j].re, w.e[i][j].re), fma(c, p.e[i][j].im, w.e[i][j].im)};
    };
    M3 a = mul_rows<ROWS>(ld<ROWS>(S, plane, o), ld<ROWS>(T, plane, pe));
    a = mul_nd_rows<ROWS>(a, ld<ROWS>(S, plane, o + fm));
    add(a);
    a = mul_dn_rows<ROWS>(ld<ROWS>(S, plane, me), ld<ROWS>(T, plane, me));
    a = mul_rows<ROWS>(a, ld<ROWS>(S, plane, me + fm));
    add(a);
}

// rows of the cofactor matrix are cross products of the other two rows
__device__ __forceinline__ void cross(const C* a, const C* b, C* out) {
    auto minor = [](C p, C q, C r, C t) { return fmacc(cmul(p, q), {-r.re, -r.im}, t); };  // p q - r t
    out[0] = minor(a[1], b[2], a[2], b[1]);
    out[1] = minor(a[2], b[0], a[0], b[2]);
    out[2] = minor(a[0], b[1], a[1], b[0]);
}

__device__ __forceinline__ C det3(const M3& x) {
    C c[3];
    cross(x.e[1], x.e[2], c);
    return fmacc(fmacc(cmul(x.e[0][0], c[0]), x.e[0][1], c[1]), x.e[0][2], c[2]);
}

// The unitary polar factor of w by Newton's iteration with determinant scaling. X^-dag = conj(cof(X)) /
// conj(det X), where the rows of cof(X) are r1 x r2, r2 x r0, r0 x r1.
__device__ __forceinline__ M3 polar_factor(const M3& w) {
    M3 x = w;
    int extra = -1;
    for (int it = 0; it < 40; ++it) {
        M3 cof;
        cross(x.e[1], x.e[2], cof.e[0]);
        cross(x.e[2], x.e[0], cof.e[1]);
        cross(x.e[0], x.e[1], cof.e[2]);
        const C d = cadd(cadd(cmul(x.e[0][0], cof.e[0][0]), cmul(x.e[0][1], cof.e[0][1])),
                         cmul(x.e[0][2], cof.e[0][2]));
        const double ad2 = d.re * d.re + d.im * d.im;
        const double z = 1.0 / cbrt(sqrt(ad2));
        const double hz = 0.5 * z, hr = 0.5 / (ad2 * z);
        // X^-dag_ij = conj(cof_ij / d) = conj(cof_ij) * d / |d|^2
        double diff = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const C q = cmulc(d, cof.e[i][j]);  // d * conj(cof_ij)
                const double nre = hz * x.e[i][j].re + hr * q.re;
                const double nim = hz * x.e[i][j].im + hr * q.im;
                diff = fmax(diff, fmax(fabs(nre - x.e[i][j].re), fabs(nim - x.e[i][j].im)));
                x.e[i][j] = {nre, nim};
            }
        // quadratic convergence: once the step is small, two more steps reach rounding level
        if (extra < 0 && diff < 1e-6) extra = 2;
        if (extra >= 0 && extra-- == 0) break;
    }
    return x;
}

__device__ __forceinline__ void su2_step(M3& x, const M3& w, int i, int j) {
    // entries (i,i), (i,j), (j,i), (j,j) of M = W X^dag
    auto m = [&](int a, int b) {
        C s = cmulc(w.e[a][0], x.e[b][0]);
        s = cadd(s, cmulc(w.e[a][1], x.e[b][1]));
        return cadd(s, cmulc(w.e[a][2], x.e[b][2]));
    };
    const C mii = m(i, i), mij = m(i, j), mji = m(j, i), mjj = m(j, j);
    // Re tr(h^dag A) over h = b0 + i b.sigma in SU(2) is 2 (b0 Re A0 + b . Re A), A = A0 + i A.sigma
    const double a0 = 0.5 * (mii.re + mjj.re);
    const double a1 = 0.5 * (mij.im + mji.im);
    const double a2 = 0.5 * (mij.re - mji.re);
    const double a3 = 0.5 * (mii.im - mjj.im);
    const double rn = 1.0 / sqrt(a0 * a0 + a1 * a1 + a2 * a2 + a3 * a3);
    const double b0 = a0 * rn, b1 = a1 * rn, b2 = a2 * rn, b3 = a3 * rn;
    const C h00 = {b0, b3}, h01 = {b2, b1}, h10 = {-b2, b1}, h11 = {b0, -b3};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const C xi = x.e[i][k], xj = x.e[j][k];
        x.e[i][k] = cadd(cmul(h00, xi), cmul(h01, xj));
        x.e[j][k] = cadd(cmul(h10, xi), cmul(h11, xj));
    }
}

// (m + m^dag) / 2
__device__ __forceinline__ void hermitize(M3& m) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        m.e[i][i].im = 0.0;
#pragma unroll
        for (int j = i + 1; j < 3; ++j) {
            const C a = m.e[i][j], b = m.e[j][i];
            m.e[i][j] = {0.5 * (a.re + b.re), 0.5 * (a.im - b.im)};
            m.e[j][i] = {m.e[i][j].re, -m.e[i][j].im};
        }
    }
}

// The maximiser of Re tr(X^dag W) over SU(3) without iterating, where it is safe. With W = up H (up the
// unitary polar factor, det up = e^{i phi}, H = up^dag W Hermitian positive definite) the maximiser is
// X = up exp(i Theta), Theta = asin(mu G) with G = H^-1: in the eigenbasis of H the problem separates into
// one phase theta_k per eigenvalue h_k, maximising sum h_k cos theta_k subject to sum theta_k = -phi, whose
// stationarity condition h_k sin theta_k = mu gives theta_k = asin(mu / h_k); mu follows from
// tr Theta = -phi. No eigenvectors are formed: the traces tr G^k come from Newton's identities, Theta from
// the arcsine series in mu G (terms to (mu G)^13) and exp(i Theta) from its Taylor series (to order 8), both
// as polynomials in G reduced to degree two by the characteristic polynomial.
// Used only when |mu| |G|_F <= 0.06, where the first omitted terms are below 1e-17 and the principal
// phases are the maximum; returns false otherwise, and the caller iterates instead.
__device__ __forceinline__ bool proj_series(const M3& w, const M3& up, M3& x) {
    constexpr double c[7] = {1.0, 1.0 / 6, 3.0 / 40, 5.0 / 112, 35.0 / 1152, 63.0 / 2816, 231.0 / 13312};
    const C du = det3(up);
    const double phi = atan2(du.im, du.re);
    M3 h = mul_dn_rows<3>(up, w);
    hermitize(h);
    M3 cof;
    cross(h.e[1], h.e[2], cof.e[0]);
    cross(h.e[2], h.e[0], cof.e[1]);
    cross(h.e[0], h.e[1], cof.e[2]);
    const double dh = h.e[0][0].re * cof.e[0][0].re - h.e[0][0].im * cof.e[0][0].im +
                      h.e[0][1].re * cof.e[0][1].re - h.e[0][1].im * cof.e[0][1].im +
                      h.e[0][2].re * cof.e[0][2].re - h.e[0][2].im * cof.e[0][2].im;  // real for Hermitian h
    if (!(dh > 0.0) || !isfinite(dh)) return false;
    const double rd = 1.0 / dh;
    M3 g;  // H^-1 = cof^T / det
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) g.e[i][j] = {cof.e[j][i].re * rd, cof.e[j][i].im * rd};
    hermitize(g);
    // power sums p_k = tr G^k: p1, p2 from the entries, then e1 p_{k-1} - e2 p_{k-2} + e3 p_{k-3}
    double p[14];
    p[1] = g.e[0][0].re + g.e[1][1].re + g.e[2][2].re;
    p[2] = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) p[2] += g.e[i][j].re * g.e[i][j].re + g.e[i][j].im * g.e[i][j].im;
    const double e1 = p[1], e2 = 0.5 * (p[1] * p[1] - p[2]), e3 = rd;
    p[3] = e1 * p[2] - e2 * p[1] + 3.0 * e3;
#pragma unroll
    for (int q = 4; q < 14; ++q) p[q] = e1 * p[q - 1] - e2 * p[q - 2] + e3 * p[q - 3];
    // tr asin(mu G) = -phi by Newton's method on the series
    double mu = -phi / p[1];
#pragma unroll
    for (int it = 0; it < 6; ++it) {
        const double m2 = mu * mu;
        double f = 0.0, df = 0.0, mp = 1.0;  // mp = mu^(2n)
#pragma unroll
        for (int n = 0; n < 7; ++n) {
            df += c[n] * (2 * n + 1) * p[2 * n + 1] * mp;
            f += c[n] * p[2 * n + 1] * mp * mu;
            mp *= m2;
        }
        mu -= (f + phi) / df;
    }
    if (!(fabs(mu) * sqrt(p[2]) <= 0.06)) return false;
    // Every power series in G reduces to a0 I + a1 G + a2 G^2 (Cayley-Hamilton: G^3 = e1 G^2 - e2 G + e3),
    // so Theta and exp(i Theta) are carried as three scalar coefficients each; G^2 is the only matrix
    // product before the last one.
    double gp[3] = {0.0, 1.0, 0.0};  // G^(2n+1)
    double th[3] = {0.0, 0.0, 0.0};  // Theta
    double mp = mu;
#pragma unroll
    for (int n = 0; n < 7; ++n) {
#pragma unroll
        for (int q = 0; q < 3; ++q) th[q] += c[n] * mp * gp[q];
#pragma unroll
        for (int rep = 0; rep < 2; ++rep) {  // times G
            const double a0 = gp[0], a1 = gp[1], a2 = gp[2];
            gp[0] = a2 * e3;
            gp[1] = a0 - a2 * e2;
            gp[2] = a1 + a2 * e1;
        }
        mp *= mu * mu;
    }
    // exp(i Theta) = 1 + i Theta (1 + i Theta / 2 (... (1 + i Theta / 8))), products reduced mod the
    // characteristic polynomial
    C ev[3] = {{1.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
    for (int q = 8; q >= 1; --q) {
        C cc[5] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {  // (i th_a) ev_b
                cc[a + b].re -= th[a] * ev[b].im;
                cc[a + b].im += th[a] * ev[b].re;
            }
#pragma unroll
        for (int kk = 4; kk >= 3; --kk) {
            cc[kk - 1] = {cc[kk - 1].re + cc[kk].re * e1, cc[kk - 1].im + cc[kk].im * e1};
            cc[kk - 2] = {cc[kk - 2].re - cc[kk].re * e2, cc[kk - 2].im - cc[kk].im * e2};
            cc[kk - 3] = {cc[kk - 3].re + cc[kk].re * e3, cc[kk - 3].im + cc[kk].im * e3};
        }
        const double rq = 1.0 / q;
#pragma unroll
        for (int a = 0; a < 3; ++a) ev[a] = {cc[a].re * rq, cc[a].im * rq};
        ev[0].re += 1.0;
    }
    const M3 g2 = mul_rows<3>(g, g);
    M3 e;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            C s = cadd(cmul(ev[1], g.e[i][j]), cmul(ev[2], g2.e[i][j]));
            if (i == j) s = cadd(s, ev[0]);
            e.e[i][j] = s;
        }
    x = mul_rows<3>(up, e);
    return true;
}

// 1 / x and 1 / sqrt(x) from the hardware estimates by two Newton steps each (within an ulp or two for normal x; zero,
// infinite, subnormal and NaN arguments give values that the caller's tests refuse).
__device__ __forceinline__ double rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double rsq(double x) {
    double r = __builtin_amdgcn_rsq(x);
    r = fma(fma(-x * r, r, 1.0), 0.5 * r, r);
    return fma(fma(-x * r, r, 1.0), 0.5 * r, r);
}

// r = a b for polynomials a0 + a1 E + a2 E^2 in a traceless 3x3 matrix E, reduced by its characteristic polynomial
// E^3 = -e2 E + e3 (e2 = -tr(E^2)/2, e3 = det E).
__device__ __forceinline__ void poly_mul(const double (&a)[3], const double (&b)[3], double e2, double e3, double (&r)[3]) {
    const double c4 = a[2] * b[2], c3 = a[1] * b[2] + a[2] * b[1];
    r[2] = a[0] * b[2] + a[1] * b[1] + a[2] * b[0] - c4 * e2;
    r[1] = a[0] * b[1] + a[1] * b[0] - c3 * e2 + c4 * e3;
    r[0] = a[0] * b[0] + c3 * e3;
}

// The same maximiser as proj_series, written entirely as a function of S = W^dag W: the polar factor is
// W S^-1/2 and H^-1 = S^-1/2, so X = W F with F = S^-1/2 exp(i Theta), sin Theta = Y = mu S^-1/2 and det W =
// |det W| e^{i phi}. With s0 = tr S / 3 and E = S / s0 - 1 (traceless) every function of S is three scalar
// coefficients of 1, E and E^2:
//   P = (1 + E)^1/2 has the symmetric functions u, v, w of its eigenvalues with w^2 = det(1 + E), u^2 = 3 + 2 v and
//   v^2 = 3 + e2 + 2 u w; u is the root next to its series start, by Newton's steps with a fixed slope (the
//   derivative 2 (u v - w) is the product of the eigenvalues' pairwise sums, so the root is well conditioned);
//   G = (1 + E)^-1/2 follows from the characteristic polynomial P^3 = u P^2 - v P + w (Hasenfratz, Hoffmann and
//   Schaefer, JHEP 0705 (2007) 029, give the coefficients of 1, P^2 and P^4): in 1, E and E^2 they are
//   [u (1 + e2) + w (2 + v)] / (w (u v - w)), -(u + w) / (w (u v - w)) and u / (w (u v - w)). u, v and w are carried as
//   their departures du, dv and k from 3, 3 and 1, and the first coefficient as its departure from 1, so that rounding
//   shrinks with E: formed from u, v and w themselves, 1 is what is left of sums of 27, and the links came out 1.6e-15
//   (rms over a link) from the maximiser in place of 2.6e-16;
//   G^2 = (1 + E)^-1 follows from the characteristic polynomial of 1 + E;
//   exp(i Theta) = (1 - Y^2)^1/2 + i Y, so only the even part needs a series.
// mu solves tr asin(mu G) = -phi, by fixed-point steps from -phi / tr G that gain a factor of about 2 / Y^2 each.
// The series run to Y^5 (Y at most 1e-3 in norm: omitted terms below 1e-19), or to Y^13 in the lanes that need it.
// Used when |E|_F <= 1/2 and |Y|_F <= 0.06 (omitted terms below 1e-17, and the principal phases are the maximum);
// returns false otherwise (x is then meaningless): the tests gather in one flag, so that nothing but the long series
// sits under a branch.
__device__ __forceinline__ bool proj_direct(const M3& w, M3& x) {
    // S = W^dag W: real diagonal, upper triangle
    double dg[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        dg[i] = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) dg[i] += w.e[k][i].re * w.e[k][i].re + w.e[k][i].im * w.e[k][i].im;
    }
    auto sij = [&](int i, int j) {
        return fmaccc(fmaccc(cmulc(w.e[0][j], w.e[0][i]), w.e[1][j], w.e[1][i]), w.e[2][j], w.e[2][i]);
    };
    C o01 = sij(0, 1), o02 = sij(0, 2), o12 = sij(1, 2);
    const double s0 = (dg[0] + dg[1] + dg[2]) * (1.0 / 3.0);
    bool ok = s0 > 0.0 && isfinite(s0);
    const double rsq0 = rsq(s0), rs0 = rsq0 * rsq0;
#pragma unroll
    for (int i = 0; i < 3; ++i) dg[i] = dg[i] * rs0 - 1.0;
    o01 = {o01.re * rs0, o01.im * rs0};
    o02 = {o02.re * rs0, o02.im * rs0};
    o12 = {o12.re * rs0, o12.im * rs0};
    const double n01 = o01.re * o01.re + o01.im * o01.im, n02 = o02.re * o02.re + o02.im * o02.im,
                 n12 = o12.re * o12.re + o12.im * o12.im;
    const double t2 = dg[0] * dg[0] + dg[1] * dg[1] + dg[2] * dg[2] + 2.0 * (n01 + n02 + n12);  // tr E^2
    ok &= t2 <= 0.25;
    const C o = cmul(o01, o12);
    const double e2 = -0.5 * t2, e3 = dg[0] * dg[1] * dg[2] + 2.0 * (o.re * o02.re + o.im * o02.im) - dg[0] * n12 -
                                      dg[1] * n02 - dg[2] * n01;
    // w = 1 + k, u = 3 + du, v = 3 + dv
    const double c = e2 + e3, c3 = 1.0 + c, rww = rsq(c3), ww = c3 * rww, rc3 = rww * rww;
    const double k = c * rcp(1.0 + ww), rhs = e2 + 6.0 * k, lin = 16.0 - 2.0 * k;
    double du = -t2 * (0.125 + t2 * (5.0 / 256.0)) + e3 * (3.0 / 16.0), dv = du * (3.0 + 0.5 * du);
    const double slope = __builtin_amdgcn_rcp(lin + 6.0 * du + 2.0 * dv * (3.0 + du));
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        du -= (du * (lin + 3.0 * du) + dv * dv - rhs) * slope;
        dv = du * (3.0 + 0.5 * du);
    }
    const double sum = du + dv, prod = du * dv, u = 3.0 + du;
    const double rden = rww * rcp(8.0 + (3.0 * sum + prod - k));  // 1 / (w (u v - w))
    const double n0 = 3.0 * e2 - 2.0 * (sum + k) + (du * e2 - prod) + k * (k - 3.0 * sum + dv - prod);
    const double h[3] = {(1.0 + e2) * rc3, -rc3, rc3};  // (1 + E)^-1
    double g0[3] = {1.0 + n0 * rden, -(u + ww) * rden, u * rden}, g1[3], g2[3];
    poly_mul(g0, h, e2, e3, g1);
    poly_mul(g1, h, e2, e3, g2);
    const C d = det3(w);
    const double q = d.im * rcp(d.re);
    // |phi| <= sqrt(3) |Y|_F or so: phases past 0.11 are refused below anyway
    ok &= d.re > 0.0 && fabs(q) <= 0.12;
    const double q2 = q * q;
    double at = -1.0 / 15.0;
#pragma unroll
    for (int k = 13; k >= 1; k -= 2) at = at * q2 + (k % 4 == 1 ? 1.0 : -1.0) / k;
    const double phi = at * q;
    auto trace = [&](const double (&a)[3]) { return 3.0 * a[0] + a[2] * t2; };
    const double rp = rcp(trace(g0)), mu0 = -phi * rp;
    const double b1 = trace(g1) * rp * (1.0 / 6.0), b2 = trace(g2) * rp * (3.0 / 40.0);
    double mu = mu0;
#pragma unroll
    for (int it = 0; it < 3; ++it) {
        const double z = mu * mu;
        mu = mu0 - mu * z * (b1 + b2 * z);
    }
    const double hn2 = trace(h);  // |G|_F^2
    double z = mu * mu;
    double a[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) a[k] = g0[k] - z * (0.5 * g1[k] + 0.125 * z * g2[k]);
    if (ok && !(z * hn2 <= 1e-6)) {
        // terms n = 3..6: G^(2n+1) from the one before
        constexpr double ca[4] = {5.0 / 112, 35.0 / 1152, 63.0 / 2816, 231.0 / 13312};
        constexpr double cs[4] = {1.0 / 16, 5.0 / 128, 7.0 / 256, 21.0 / 1024};
        double gn[4][3], bn[4];
        poly_mul(g2, h, e2, e3, gn[0]);
#pragma unroll
        for (int n = 1; n < 4; ++n) poly_mul(gn[n - 1], h, e2, e3, gn[n]);
#pragma unroll
        for (int n = 0; n < 4; ++n) bn[n] = ca[n] * trace(gn[n]) * rp;
        for (int it = 0; it < 6; ++it) {
            z = mu * mu;
            mu = mu0 - mu * z * (b1 + z * (b2 + z * (bn[0] + z * (bn[1] + z * (bn[2] + z * bn[3])))));
        }
        z = mu * mu;
        ok = z * hn2 <= 0.06 * 0.06;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            a[k] = g0[k] - z * (0.5 * g1[k] + z * (0.125 * g2[k] + z * (cs[0] * gn[0][k] + z * (cs[1] * gn[1][k] +
                   z * (cs[2] * gn[2][k] + z * cs[3] * gn[3][k])))));
    }
    // F = (a + i mu h) / sqrt(s0): the Hermitian parts P of a and Q of mu h, F = P + i Q
    double b[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a[k] *= rsq0;
        b[k] = mu * rsq0 * h[k];
    }
    // E^2
    const double q00 = dg[0] * dg[0] + n01 + n02, q11 = dg[1] * dg[1] + n01 + n12, q22 = dg[2] * dg[2] + n02 + n12;
    const C e01 = cmulc(o02, o12), e02 = o, e12 = cmulc(o02, o01);  // o02 o12*, o01 o12, o01* o02
    const C x01 = {(dg[0] + dg[1]) * o01.re + e01.re, (dg[0] + dg[1]) * o01.im + e01.im};
    const C x02 = {(dg[0] + dg[2]) * o02.re + e02.re, (dg[0] + dg[2]) * o02.im + e02.im};
    const C x12 = {(dg[1] + dg[2]) * o12.re + e12.re, (dg[1] + dg[2]) * o12.im + e12.im};
    M3 m;
    m.e[0][0] = {a[0] + a[1] * dg[0] + a[2] * q00, b[0] + b[1] * dg[0] + b[2] * q00};
    m.e[1][1] = {a[0] + a[1] * dg[1] + a[2] * q11, b[0] + b[1] * dg[1] + b[2] * q11};
    m.e[2][2] = {a[0] + a[1] * dg[2] + a[2] * q22, b[0] + b[1] * dg[2] + b[2] * q22};
    auto off = [&](C e, C ee, C& up, C& lo) {
        const C P = {a[1] * e.re + a[2] * ee.re, a[1] * e.im + a[2] * ee.im};
        const C Q = {b[1] * e.re + b[2] * ee.re, b[1] * e.im + b[2] * ee.im};
        up = {P.re - Q.im, P.im + Q.re};
        lo = {P.re + Q.im, Q.re - P.im};
    };
    off(o01, x01, m.e[0][1], m.e[1][0]);
    off(o02, x02, m.e[0][2], m.e[2][0]);
    off(o12, x12, m.e[1][2], m.e[2][1]);
    x = mul_rows<3>(w, m);
    return ok;
}

// The maximiser where proj_direct declines, out of line and through memory (m: W on entry, the maximiser on return),
// so that the level kernels hold the registers of the usual path only. WAVES per SIMD of the kernels that call it: a
// called function is allocated for the kernel with the most registers, so kernels of different budgets take their own.
template <int WAVES>
__device__ __noinline__ void proj_iterate(double2* m) {
    M3 w;
#pragma unroll
    for (int j = 0; j < 9; ++j) w.e[j / 3][j % 3] = {m[j].x, m[j].y};
    auto put = [&](const M3& r) {
#pragma unroll
        for (int j = 0; j < 9; ++j) m[j] = make_double2(r.e[j / 3][j % 3].re, r.e[j / 3][j % 3].im);
    };
    M3 x = polar_factor(w);
    M3 y;
    if (proj_series(w, x, y)) {
        put(y);
        return;
    }
    const C d = det3(x);
    const double th = -atan2(d.im, d.re) / 3.0;
    const C ph = {cos(th), sin(th)};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) x.e[i][j] = cmul(x.e[i][j], ph);
    for (int sweep = 0; sweep < 500; ++sweep) {  // nearly singular W can need hundreds
        const M3 x0 = x;
        su2_step(x, w, 0, 1);
        su2_step(x, w, 0, 2);
        su2_step(x, w, 1, 2);
        double diff2 = 0.0;  // largest |change|^2 of an element
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double dr = x.e[i][j].re - x0.e[i][j].re, di = x.e[i][j].im - x0.e[i][j].im;
                diff2 = fmax(diff2, dr * dr + di * di);
            }
        if (diff2 <= 1e-30) break;
    }
    // every sweep rounds; X (3 - X^dag X) / 2 leaves of X^dag X - 1 (1e-14 after many) its square, so that row 2 may be
    // rebuilt from the others (row2)
    M3 n = mul_dn_rows<3>(x, x);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) n.e[i][j] = {0.5 * ((i == j ? 1.0 : 0.0) - n.e[i][j].re), -0.5 * n.e[i][j].im};
    const M3 dx = mul_rows<3>(x, n);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) x.e[i][j] = cadd(x.e[i][j], dx.e[i][j]);
    put(x);
}

template <int WAVES>
__device__ __forceinline__ M3 proj_su3(const M3& w) {
    M3 x;
    if (!proj_direct(w, x)) {
        double2 m[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) m[j] = make_double2(w.e[j / 3][j % 3].re, w.e[j / 3][j % 3].im);
        proj_iterate<WAVES>(m);
#pragma unroll
        for (int j = 0; j < 9; ++j) x.e[j / 3][j % 3] = {m[j].x, m[j].y};
    }
    return x;
}

__device__ __forceinline__ int other(int a, int k) { return k < a ? k : k + 1; }  // k-th direction != a
__device__ __forceinline__ int fidx(int a, int b) { return a * 3 + (b < a ? b : b - 1); }  // field (a, b != a)

struct HypArgs {
    HypGeom g;
    const double2* U;  // natural [4][V][9] double2
    char* up;          // the links, planes [4][9][V]
    char* lv1;         // planes [12][6][V]
    char* lv2;         // planes [12][6][V]
    double2* out;      // natural [4][V][9]
    double a1, a2, a3;
    __device__ __forceinline__ size_t plane() const { return (size_t)g.V * sizeof(double2); }
    __device__ __forceinline__ char* links(int mu) const { return up + 9 * mu * plane(); }
    __device__ __forceinline__ char* level1(int a, int b) const { return lv1 + 6 * fidx(a, b) * plane(); }
    __device__ __forceinline__ char* level2(int a, int b) const { return lv2 + 6 * fidx(a, b) * plane(); }
};

constexpr int HYP_NT = 256;
// Blocks take all output fields of one run of HYP_NT sites before the next run, and each XCD gets a contiguous range
// of that order: the fields of a site share most of the links they read.
struct Work {
    int f, s, n;  // output field, first site and number of sites of the block
};
__device__ __forceinline__ Work work_of(const HypArgs& a, int nf) {
    const int l = remap_block(blockIdx.x, gridDim.x), blk = l / nf;
    return {l - blk * nf, blk * HYP_NT, min(HYP_NT, a.g.V - blk * HYP_NT)};
}

// A block's links of one direction in the natural layout [V][9], moved between memory and registers through LDS so
// that memory sees consecutive 16-byte words (a lane's own link is 144 bytes from the next lane's).
struct Stage {
    double2 w[HYP_NT * 9];
};
__device__ __forceinline__ M3 ld_nat(Stage& sm, const double2* p, const Work& wk) {
    const int n = wk.n * 9;
    const double2* src = p + (size_t)wk.s * 9;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * HYP_NT + threadIdx.x;
        if (i < n) sm.w[i] = src[i];
    }
    __syncthreads();
    M3 m;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const double2 v = sm.w[threadIdx.x * 9 + j];
        m.e[j / 3][j % 3] = {v.x, v.y};
    }
    return m;
}
__device__ __forceinline__ void st_nat(Stage& sm, double2* p, const Work& wk, const M3& m) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 9; ++j) sm.w[threadIdx.x * 9 + j] = make_double2(m.e[j / 3][j % 3].re, m.e[j / 3][j % 3].im);
    __syncthreads();
    const int n = wk.n * 9;
    double2* dst = p + (size_t)wk.s * 9;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * HYP_NT + threadIdx.x;
        if (i < n) dst[i] = sm.w[i];
    }
}

// Natural links -> planes.
__global__ __launch_bounds__(HYP_NT) void k_hyp_planes(HypArgs a) {
    __shared__ Stage sm;
    const Work wk = work_of(a, 4);
    const M3 m = ld_nat(sm, a.U + (size_t)wk.f * a.g.V * 9, wk);
    if ((int)threadIdx.x < wk.n) st<3>(a.links(wk.f), a.plane(), 16u * (wk.s + threadIdx.x), m);
}

__global__ __launch_bounds__(HYP_NT) void k_hyp_level1(HypArgs a) {
    const Work wk = work_of(a, 12);
    if ((int)threadIdx.x >= wk.n) return;
    const int s = wk.s + threadIdx.x;
    const int mu = wk.f / 3, eta = other(mu, wk.f % 3);
    M3 w = ld<3>(a.links(mu), a.plane(), 16u * s);
    scale(w, 1.0 - a.a3);
    add_staples<3>(w, 0.5 * a.a3, a.plane(), a.links(eta), a.links(mu), 16u * s,
                   hop(a.g, s, mu).f, hop(a.g, s, eta));
    st<2>(a.level1(mu, eta), a.plane(), 16u * s, proj_su3<2>(w));
}

// Levels 2 and 3 at three waves per SIMD (168 registers, none spilled); level 1 spills there and runs at two.
__global__ __launch_bounds__(HYP_NT, 3) void k_hyp_level2(HypArgs a) {
    const Work wk = work_of(a, 12);
    if ((int)threadIdx.x >= wk.n) return;
    const int s = wk.s + threadIdx.x;
    const int mu = wk.f / 3, nu = other(mu, wk.f % 3);
    M3 w = ld<3>(a.links(mu), a.plane(), 16u * s);
    const unsigned fm = hop(a.g, s, mu).f;
    scale(w, 1.0 - a.a2);
#pragma unroll 1
    for (int rho = 0; rho < 4; ++rho) {
        if (rho == mu || rho == nu) continue;
        const int sg = 6 - mu - nu - rho;
        add_staples<2>(w, 0.25 * a.a2, a.plane(), a.level1(rho, sg), a.level1(mu, sg), 16u * s, fm, hop(a.g, s, rho));
    }
    st<2>(a.level2(mu, nu), a.plane(), 16u * s, proj_su3<3>(w));
}

__global__ __launch_bounds__(HYP_NT, 3) void k_hyp_level3(HypArgs a) {
    __shared__ Stage sm;
    const Work wk = work_of(a, 4);
    const int mu = wk.f;
    const int s = wk.s + min((int)threadIdx.x, wk.n - 1);  // lanes past the end compute the last site, unstored
    M3 w = ld<3>(a.links(mu), a.plane(), 16u * s);
    const unsigned fm = hop(a.g, s, mu).f;
    scale(w, 1.0 - a.a1);
#pragma unroll 1
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == mu) continue;
        add_staples<2>(w, a.a1 / 6.0, a.plane(), a.level2(nu, mu), a.level2(mu, nu), 16u * s, fm, hop(a.g, s, nu));
    }
    st_nat(sm, a.out + (size_t)mu * a.g.V * 9, wk, proj_su3<3>(w));
}

}  // namespace

size_t hyp_workspace_bytes(const Geom& g) { return 24ull * 2 * (size_t)g.Vh * 9 * sizeof(double2); }

hipError_t launch_hyp(const Geom& g, const double* links, const double alpha[3], double* out, void* ws,
                      hipStream_t s) {
    HypArgs a;
    a.g.L[0] = g.X;
    a.g.L[1] = g.Y;
    a.g.L[2] = g.Z;
    a.g.L[3] = g.T;
    a.g.stride[0] = 1;
    a.g.stride[1] = g.X;
    a.g.stride[2] = g.X * g.Y;
    a.g.stride[3] = g.X * g.Y * g.Z;
    a.g.V = 2 * g.Vh;
    for (int mu = 0; mu < 4; ++mu) {
        a.g.by_L[mu] = div_by(a.g.L[mu]);
        a.g.by_stride[mu] = div_by(a.g.stride[mu]);
    }
    a.U = (const double2*)links;
    a.lv1 = (char*)ws;
    a.lv2 = a.lv1 + 72 * (size_t)a.g.V * sizeof(double2);
    a.up = a.lv2 + 72 * (size_t)a.g.V * sizeof(double2);  // 180 of the workspace's 216 planes in all
    a.out = (double2*)out;
    a.a1 = alpha[0];
    a.a2 = alpha[1];
    a.a3 = alpha[2];
    const int nb = blocks_for(a.g.V, HYP_NT);
    hipLaunchKernelGGL(k_hyp_planes, dim3(nb * 4), dim3(HYP_NT), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL(k_hyp_level1, dim3(nb * 12), dim3(HYP_NT), 0, s, a);
    if ((e = hipGetLastError())) return e;
    hipLaunchKernelGGL(k_hyp_level2, dim3(nb * 12), dim3(HYP_NT), 0, s, a);
    if ((e = hipGetLastError())) return e;
    hipLaunchKernelGGL(k_hyp_level3, dim3(nb * 4), dim3(HYP_NT), 0, s, a);
    return hipGetLastError();
}

}  // namespace sp
