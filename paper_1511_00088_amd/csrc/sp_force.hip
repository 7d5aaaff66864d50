// Adjoint link gradient (fermion force) and mass gradient, FP64.
//
// For a real loss l(x), x = A^-1 b, A = m^2 - D_eo D_oe, with lambda = A^-1 dl/dx, y_x = D_oe x and
// y_l = D_oe lambda, varying one link U_mu(n) changes D_eo (output at n or n+mu) and D_oe; collecting the
// two terms gives
//   n even:  Gamma_mu(n) =  1/2 eta_mu(n) s [ lambda(n) y_x(n+mu)^dag + x(n) y_l(n+mu)^dag ]
//   n odd:   Gamma_mu(n) = -1/2 eta_mu(n) s [ y_x(n) lambda(n+mu)^dag + y_l(n) x(n+mu)^dag ]
// (s: antiperiodic-time sign of the link), and F = TA(U Gamma^dag) is its projection on su(3).
//
// Bound by bytes: at 16^3x32 the links once more than the outputs, 233 MB (38 us at the copy rate), and both y. Three
// launches (4.5 + 15.5 + 41 us there; 85 us a call with its synchronisation) where there were seven (130 us; 149):
// x and lambda are packed together with the partial sums of dl/dm, one operator launch loads each link for both y, and
// Gamma and the force leave through LDS in whole cache lines.
#include "sp_launch.h"

namespace sp {

__device__ __forceinline__ void outer_acc(Cx<double> (&G)[3][3], double c, const Vec3<double>& a,
                                          const Vec3<double>& b) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            // a_i conj(b_j)
            G[i][j].re += c * (a.c[i].re * b.c[j].re + a.c[i].im * b.c[j].im);
            G[i][j].im += c * (a.c[i].im * b.c[j].re - a.c[i].re * b.c[j].im);
        }
}

// x and lambda (natural half vectors) to planes, and block partials of Re<lambda, x> for dl/dm.
__global__ __launch_bounds__(256) void k_force_pack(int Vh, const double2* __restrict__ x, const double2* __restrict__ lam,
                                                    void* xp, void* lp, double* partials) {
    using VF = VecFmt<F64>;
    const int cb = blockIdx.x * blockDim.x + threadIdx.x;
    double v[1] = {0.0};
    if (cb < Vh) {
        Vec3<double> a, b;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double2 l = lam[(size_t)cb * 3 + i], w = x[(size_t)cb * 3 + i];
            a.c[i] = {l.x, l.y};
            b.c[i] = {w.x, w.y};
        }
        VF::store(lp, Vh, cb, a);
        VF::store(xp, Vh, cb, b);
#pragma unroll
        for (int i = 0; i < 3; ++i) v[0] += a.c[i].re * b.c[i].re + a.c[i].im * b.c[i].im;
    }
    block_sum<1>(v);
    if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

// y_x = D_oe x and y_l = D_oe lambda in one launch: each link is loaded once for both.
__global__ __launch_bounds__(256) void k_force_dslash(Geom g, const void* links64, const void* x, const void* lam,
                                                      void* yx, void* yl, int remap) {
    using VF = VecFmt<F64>;
    using LF = LinkFmt<F64, 18>;
    const int cb = logical_block(remap) * blockDim.x + threadIdx.x;
    if (cb >= g.Vh) return;
    const Site s = site_of(g, 1, cb);
    Vec3<double> ax = vzero<double>(), al = vzero<double>();
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
        double sf = 0.5 * (double)eta_sign(s, mu), sb = -sf;
        if (mu == 3 && g.bc_t) {
            if (s.t == g.T - 1) sf = -sf;
            if (s.t == 0) sb = -sb;
        }
        const int nf = nbr(g, s, mu, +1), nb = nbr(g, s, mu, -1);
        const Su3<double> Uf = LF::load(link_block<LF>(links64, g.Vh, 1, mu), g.Vh, cb);
        const Vec3<double> xf = VF::load(x, g.Vh, nf), lf = VF::load(lam, g.Vh, nf);
        const Su3<double> Ub = LF::load(link_block<LF>(links64, g.Vh, 0, mu), g.Vh, nb);
        const Vec3<double> xb = VF::load(x, g.Vh, nb), lb = VF::load(lam, g.Vh, nb);
        mv_acc(ax, Uf, xf, sf);
        mv_acc(al, Uf, lf, sf);
        mdv_acc(ax, Ub, xb, sb);
        mdv_acc(al, Ub, lb, sb);
    }
    VF::store(yx, g.Vh, cb, ax);
    VF::store(yl, g.Vh, cb, al);
}

// A block's 256 consecutive links of one direction from registers to the natural layout, through LDS so that memory sees
// consecutive 16-byte words (a lane's own link is 144 bytes from the next lane's), with streaming stores: the outputs
// are most of the launch's bytes and not read again here, and ordinary stores push the links and vectors that every
// launch reads out of the caches (16^3x32: 96 us a call against 85).
struct LinkStage {
    double2 w[256 * 9];
};
__device__ __forceinline__ void store_links(LinkStage& sm, const Cx<double> (&m)[3][3], double2* dst, int n) {
    typedef double v2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < 9; ++j) sm.w[threadIdx.x * 9 + j] = make_double2(m[j / 3][j % 3].re, m[j / 3][j % 3].im);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * 256 + threadIdx.x;
        if (i < 9 * n) __builtin_nontemporal_store(v2{sm.w[i].x, sm.w[i].y}, (v2*)(dst + i));
    }
}

// Gamma, and where asked the force, of 256 consecutive links of direction blockIdx.y; the first block also finishes
// dl/dm = -2 m sum(partials), summed in block order.
__global__ __launch_bounds__(256) void k_force(Geom g, const void* links64, const void* x, const void* lam,
                                               const void* yx, const void* yl, double2* gamma, double2* force,
                                               const double* partials, int npart, double mass, double* grad_mass) {
    using VF = VecFmt<F64>;
    using LF = LinkFmt<F64, 18>;
    __shared__ LinkStage sm;
    const int mu = blockIdx.y, V = 2 * g.Vh, first = blockIdx.x * 256, n = min(256, V - first);
    if (grad_mass && blockIdx.x == 0 && mu == 0) {
        double v[1] = {0.0};
        for (int b = threadIdx.x; b < npart; b += 256) v[0] += partials[b];
        block_sum<1>(v);
        if (threadIdx.x == 0) *grad_mass = -2.0 * mass * v[0];
    }
    // lanes past the lattice compute its last link and store nothing
    const int lex = first + min((int)threadIdx.x, n - 1), cb = lex >> 1;
    const int r = divq(cb, g.Xh, g.rXh), r2 = divq(r, g.Y, g.rY), t0 = divq(r2, g.Z, g.rZ);
    const int p = (lex - r * g.X + r - r2 * g.Y + r2 - t0 * g.Z + t0) & 1;
    const Site s = site_of(g, p, cb);
    const int nf = nbr(g, s, mu, +1);
    double c = p ? -0.5 : 0.5;
    if (eta_sign(s, mu) < 0.0f) c = -c;
    if (mu == 3 && g.bc_t && s.t == g.T - 1) c = -c;
    // even: lambda(n) y_x(n+mu)^dag + x(n) y_l(n+mu)^dag; odd: y_x(n) lambda(n+mu)^dag + y_l(n) x(n+mu)^dag
    const Vec3<double> a0 = VF::load(p ? yx : lam, g.Vh, cb), a1 = VF::load(p ? yl : x, g.Vh, cb);
    const Vec3<double> b0 = VF::load(p ? lam : yx, g.Vh, nf), b1 = VF::load(p ? x : yl, g.Vh, nf);
    Cx<double> G[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) G[i][j].re = G[i][j].im = 0.0;
    outer_acc(G, c, a0, b0);
    outer_acc(G, c, a1, b1);
    store_links(sm, G, gamma + ((size_t)mu * V + first) * 9, n);
    if (force) {
        const Su3<double> U = LF::load(link_block<LF>(links64, g.Vh, p, mu), g.Vh, cb);
        // W = U Gamma^dag, W_ij = sum_k U_ik conj(G_jk)
        Cx<double> W[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double re = 0.0, im = 0.0;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    re += U.e[i][k].re * G[j][k].re + U.e[i][k].im * G[j][k].im;
                    im += U.e[i][k].im * G[j][k].re - U.e[i][k].re * G[j][k].im;
                }
                W[i][j].re = re;
                W[i][j].im = im;
            }
        // TA(W) = (W - W^dag)/2 - tr(W - W^dag)/6; tr(W - W^dag) = 2 i Im tr W
        const double imtr = W[0][0].im + W[1][1].im + W[2][2].im;
        Cx<double> F[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                F[i][j].re = 0.5 * (W[i][j].re - W[j][i].re);
                F[i][j].im = 0.5 * (W[i][j].im + W[j][i].im);
                if (i == j) F[i][j].im -= imtr / 3.0;
            }
        __syncthreads();  // gamma has left the stage
        store_links(sm, F, force + ((size_t)mu * V + first) * 9, n);
    }
}

int mass_grad_blocks(const Geom& g) { return blocks_for(g.Vh, 256); }

hipError_t launch_gradient(const Geom& g, const void* links64, const double* x, const double* lam, double mass,
                           const GradScratch& w, double* gamma, double* force, double* grad_mass, hipStream_t s) {
    const int np = mass_grad_blocks(g);
    hipLaunchKernelGGL(k_force_pack, dim3(np), dim3(256), 0, s, g.Vh, (const double2*)x, (const double2*)lam, w.x, w.lam,
                       w.partials);
    hipError_t e = hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL(k_force_dslash, dim3(blocks_for(g.Vh, 256)), dim3(256), 0, s, g, links64, w.x, w.lam, w.yx, w.yl, 1);
    if ((e = hipGetLastError())) return e;
    hipLaunchKernelGGL(k_force, dim3(blocks_for(2 * g.Vh, 256), 4), dim3(256), 0, s, g, links64, w.x, w.lam, w.yx, w.yl,
                       (double2*)gamma, (double2*)force, w.partials, np, mass, grad_mass);
    return hipGetLastError();
}

}  // namespace sp
