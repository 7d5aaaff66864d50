// Kernel templates of the even-odd staggered CG.
//
// Every solver kernel runs over a list of "groups": a group is a set of up to N systems (right-hand
// sides) that share one gauge field and geometry. A launch covers the blocks of every group; a block
// handles blockDim.x consecutive sites of one group for all of its systems, so the half operator loads
// each link once per group rather than once per system. A single solve is one group with one system,
// its descriptor passed by value (DescSingle); batches keep their descriptors in device memory
// (DescBatch; small lattices of one extent, a system per group with its own decisions: DescMany).
//
// Global dot products use a two-stage reduction: each block reduces its sites in FP64 (registers within
// a wavefront, then LDS across them) and stores one partial per system; the next launch, k_finalize (one
// block per system) or every block of it (one system, DescMany), sums the partials in a fixed order, and
// each system's device-resident state (alpha, beta, flags) advances. The kernel boundary makes the partials
// visible without any in-kernel fence, sums have a fixed order and results are bitwise reproducible.
#pragma once

#include "sp_device.h"

namespace sp {

// Vector slots of a system.
enum Slot : int { S_B64 = 0, S_X64, S_T64, S_XLO, S_P, S_R, S_T, NSLOT };

// Which systems a kernel works on.
enum Gate : int {
    G_NONE = 0,   // no state (stand-alone operator application)
    G_ITER = 1,   // CG iteration: not done, not paused for a reliable update
    G_RU = 2,     // reliable update requested by the last iteration (ST_PENDING)
    G_XPAY = 3,   // the paused iteration's p update is due after the reliable update
    G_ALIVE = 4,  // not done (set-up kernels)
};

struct SysDev {
    void* v[NSLOT];
    SolverState* st;
};

struct GroupDev {
    Geom g;
    const void* links_lo;
    const void* links64;
    double* partials;   // [nblk][2 N] block partials of the last reducing launch
    double* partials_p; // [nblk][N]   block partials of |p|^2 from the last p update
    double* partials_r; // [nblk]      block partials of |r|^2 from DS_UPDATE_FUSED
    double* rec;        // [2]         Re<p,Ap> and alpha of the last DS_UPDATE_FUSED (block 0 writes them)
    int nrhs, sys0, blk0, nblk;
    int bundle;         // groups whose blocks alternate (same links and geometry, same blk0), this one among them
};

struct DescSingle {
    GroupDev grp;
    SysDev sys;
};

struct DescBatch {
    const GroupDev* grp;
    const SysDev* sys;
    int ngroups;
};

// Several systems of one geometry that each iterate as a single system does (in-block decisions), their blocks alternating.
// The states are double-buffered as a single system's: a launch reads st[i] and writes next[i].
struct DescMany {
    const DescSingle* one;  // [n]
    SolverState *st, *next;
    int n;
};

// --- descriptor access ---------------------------------------------------------------------------------
// The group of a logical block, and the block's number in it.
struct BlockOf {
    int grp, blk;
};
__device__ __forceinline__ BlockOf block_of(const DescSingle&, int lblk) { return {0, lblk}; }
// The groups that start at or before the block, counted: lane l tests group l (then l + 64, ...), so the starts load in
// parallel instead of one after the other (starts do not decrease). The last of them closes the block's bundle, whose
// groups take the blocks in turn: neighbouring blocks then read the same links at about the same time and on one XCD, whose
// L2 serves all but the first of them. Called by whole waves at kernel entry.
__device__ __forceinline__ BlockOf block_of(const DescBatch& d, int lblk) {
    int count = 0;
    for (int g0 = 0; g0 < d.ngroups; g0 += 64) {
        const int g = g0 + (int)(threadIdx.x & 63);
        const bool started = g < d.ngroups && d.grp[g].blk0 <= lblk;
        count += __popcll(__ballot(started));
    }
    const int last = __builtin_amdgcn_readfirstlane(count - 1);
    const int k = d.grp[last].bundle, rel = lblk - d.grp[last].blk0, blk = rel / k;
    return {last - (k - 1) + (rel - blk * k), blk};
}
__device__ __forceinline__ BlockOf block_of(const DescMany& d, int lblk) {
    const int b = lblk / d.n;
    return {lblk - b * d.n, b};
}
__device__ __forceinline__ const GroupDev& grp_of(const DescSingle& d, int) { return d.grp; }
__device__ __forceinline__ const GroupDev& grp_of(const DescMany& d, int g) { return d.one[g].grp; }
__device__ __forceinline__ const GroupDev& grp_of(const DescBatch& d, int g) { return d.grp[g]; }
__device__ __forceinline__ const SysDev& sys_of(const DescSingle& d, int) { return d.sys; }
__device__ __forceinline__ const SysDev& sys_of(const DescBatch& d, int i) { return d.sys[i]; }
__device__ __forceinline__ const SysDev& sys_of(const DescMany& d, int i) { return d.one[i].sys; }
__device__ __forceinline__ SolverState* state_of(const DescSingle& d, int) { return d.sys.st; }
__device__ __forceinline__ SolverState* state_of(const DescBatch& d, int i) { return d.sys[i].st; }
__device__ __forceinline__ SolverState* state_of(const DescMany& d, int i) { return d.st + i; }
// Where a launch that takes the decisions writes the advanced state of system i (st_out: the single system's).
__device__ __forceinline__ SolverState* next_state(const DescSingle&, SolverState* st_out, int) { return st_out; }
__device__ __forceinline__ SolverState* next_state(const DescMany& d, SolverState*, int i) { return d.next + i; }

// Block order: with remap, consecutive logical blocks (neighbouring lattice slabs) go to the same XCD.
// The hardware hands block b to XCD b % 8; logical block = start of that XCD's contiguous range + b / 8.
// A bijection of [0, nb) for every nb (XCD x owns nb / 8 blocks, plus one for the first nb % 8 XCDs).
__host__ __device__ __forceinline__ int remap_block(int b, int nb) {
    const int q = nb >> 3, rem = nb & 7, x = b & 7, i = b >> 3;
    return x * q + (x < rem ? x : rem) + i;
}
__device__ __forceinline__ int logical_block(int remap) {
    return remap ? remap_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
}

// Whether a launch gated by `gate` works on a system whose state flags are f.
__device__ __forceinline__ bool gate_flags_open(int f, int gate) {
    if (gate == G_NONE) return true;
    if (f & ST_DONE) return false;
    if (gate == G_ITER) return !(f & ST_PENDING);
    if (gate == G_RU) return (f & ST_PENDING) != 0;
    if (gate == G_XPAY) return (f & ST_XPAY_DUE) != 0;
    return true;
}

// Per-launch view of the systems of this block's group.
template <int N>
struct Rhs {
    bool act[N];
    SolverState* st[N];
    bool any;
};

// The state pointers and flags of the group's systems load unconditionally (slots beyond the group's count
// repeat its first system and are marked inactive), so the loads of all systems are in flight together.
template <int N, class D>
__device__ __forceinline__ Rhs<N> rhs_of(const D& d, const GroupDev& G, int gate) {
    Rhs<N> h;
    if constexpr (N == 1) {
        h.st[0] = state_of(d, G.sys0);
        h.act[0] = G.nrhs > 0 && (gate == G_NONE || h.st[0] == nullptr || gate_flags_open(h.st[0]->flags, gate));
        h.any = h.act[0];
        return h;
    }
    h.any = false;
#pragma unroll
    for (int r = 0; r < N; ++r) h.st[r] = state_of(d, G.sys0 + (r < G.nrhs ? r : 0));
    int f[N];
#pragma unroll
    for (int r = 0; r < N; ++r) f[r] = (gate == G_NONE || h.st[r] == nullptr) ? 0 : h.st[r]->flags;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        h.act[r] = r < G.nrhs && (h.st[r] == nullptr || gate_flags_open(f[r], gate));
        h.any |= h.act[r];
    }
    return h;
}

// This thread's share of the second reduction stage over n block partials of NV arrays: acc[q] += a[q][b] for
// b = b_first, + blockDim.x, ... < n, added in increasing b (the order that makes every block of a launch
// reach the same total, bit for bit). The loads go out eight at a time: a plain loop of dependent adds waits
// for each load in turn, one memory round trip per partial.
template <int NV>
__device__ __forceinline__ void strided_sums_from(double (&acc)[NV], const double* const (&a)[NV], int n,
                                                  int b_first) {
    constexpr int K = 8;
    const int nt = blockDim.x;
    for (int b0 = b_first; b0 < n; b0 += K * nt) {
        double v[K][NV];
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int q = 0; q < NV; ++q) v[j][q] = b0 + j * nt < n ? a[q][b0 + j * nt] : 0.0;
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int q = 0; q < NV; ++q)
                if (b0 + j * nt < n) acc[q] += v[j][q];
    }
}

// The same sums split around the caller's own loads, when every thread has at most HEAD partials (up to
// HEAD x blockDim.x blocks): strided_head loads them with no branch (indices clamped to n - 1) and leaves them
// unused, so that the loads the caller issues next do not wait for them, and strided_tail adds those below n
// in the same increasing order. With more partials strided_head sums them all at once, eight loads in flight
// (moving them after the operator's gathers put two or more dependent rounds of loads after it: 2% slower
// iterations on 32^3x64), and strided_tail adds nothing.
constexpr int HEAD = 4;
template <int NV>
__device__ __forceinline__ void strided_head(double (&acc)[NV], double (&v)[HEAD][NV], const double* const (&a)[NV],
                                             int n) {
    const int nt = blockDim.x;
    if (n <= HEAD * nt) {
#pragma unroll
        for (int j = 0; j < HEAD; ++j) {
            const int b = threadIdx.x + j * nt;
            const int c = b < n ? b : n - 1;
#pragma unroll
            for (int q = 0; q < NV; ++q) v[j][q] = a[q][c];
        }
    } else {
        strided_sums_from<NV>(acc, a, n, threadIdx.x);
#pragma unroll
        for (int j = 0; j < HEAD; ++j)
#pragma unroll
            for (int q = 0; q < NV; ++q) v[j][q] = 0.0;
    }
}
template <int NV>
__device__ __forceinline__ void strided_tail(double (&acc)[NV], const double (&v)[HEAD][NV], int n) {
    if (n <= HEAD * (int)blockDim.x) {
#pragma unroll
        for (int j = 0; j < HEAD; ++j)
            if (threadIdx.x + j * blockDim.x < n) {
#pragma unroll
                for (int q = 0; q < NV; ++q) acc[q] += v[j][q];
            }
    }
}

// First reduction stage: block totals of NV values per thread, stored by thread 0 as dst[gblk][NV].
template <int NV>
__device__ __forceinline__ void block_partials(double* dst, int gblk, double (&v)[NV]) {
    __shared__ BlockSums<NV> sm;
    block_sum_all<NV>(v, sm);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) dst[(size_t)gblk * NV + k] = v[k];
    }
}

// ------------------------------------------------------------------------------------------------------
// Half operator, N right-hand sides sharing each link load. MODE:
//   DS_PLAIN : out = D_{p,1-p} in
//   DS_NORM  : t = D_oe p (out), block partials of Re<t, t_stored>; with |p|^2 from the last p update this
//              gives Re<p, A p> = m^2 |p|^2 + |D_oe p|^2 and alpha, since D_eo = -D_oe^dag for any links
//   DS_UPDATE: q = m^2 p - D_eo t (not stored); x += alpha p; r -= alpha q; block partials of |r|^2
//   DS_UPDATE_FUSED (one system, or each of DescMany): as DS_UPDATE, but every block forms alpha itself from the partials of
//              |D_oe p|^2 and |p|^2 (summed in the same order in every block, so all blocks agree bit for
//              bit); the first partials are loaded before the gathers and summed after them. Saves the
//              alpha finalize launch when the partials are few; |r|^2 partials go to partials_r, Re<p,Ap>
//              and alpha to rec for k_xpay_fused, which takes the place of the update finalize.
// POL (one system): how the operator gathers, see Policy.
// ------------------------------------------------------------------------------------------------------
enum DsMode : int { DS_PLAIN = 0, DS_NORM = 1, DS_UPDATE = 2, DS_UPDATE_FUSED = 3 };

// How a single-system operator gathers: one lane per site with cached or streaming link loads, or four lanes per site
// (cached), one direction each (dslash_quad); its blocks then cover blockDim.x / 4 sites, and lane 0 of each four does
// the rest of the site's work.
enum Policy : int { CACHED = 0, STREAM = 1, QUAD = 2 };
template <int POL>
__device__ __forceinline__ int site_index(int gblk) {
    const int i = gblk * blockDim.x + threadIdx.x;
    return POL == QUAD ? i >> 2 : i;
}
template <int POL>
__device__ __forceinline__ bool site_lead() {
    return POL != QUAD || (threadIdx.x & 3) == 0;
}

// Multi-system launches keep every load unconditional so that the compiler can keep all of them in flight:
// right-hand sides beyond the group's count read the last system's vectors and store nothing, and systems
// that are stopped or paused are computed with zero coefficients (x += 0 p, r -= 0 q, p = 0 r + 1 p leave
// their stored values unchanged). Only temporaries (t) are overwritten for them.
template <int LP, int RECON, int VP, int N, class D, int MODE, int POL = CACHED>
__global__ __launch_bounds__(256) void k_dslash(D d, int p, int in_slot, int out_slot, int gate, int use64,
                                                int remap) {
    using R = typename Real<VP>::T;
    using LF = LinkFmt<LP, RECON>;
    using VF = VecFmt<VP>;
    constexpr int XP = VP == F64 ? F64 : F32;  // x: FP64 in place for plain FP64 CG, else the FP32 x_lo
    using RX = typename Real<XP>::T;
    using XF = VecFmt<XP>;
    const int lblk = logical_block(remap);
    const BlockOf bo = block_of(d, lblk);
    const GroupDev& G = grp_of(d, bo.grp);
    const int gblk = bo.blk;
    const Rhs<N> h = rhs_of<N>(d, G, gate);
    if (!h.any) return;
    const Geom g = G.g;
    const int nr = G.nrhs;
    const void* links = use64 ? G.links64 : G.links_lo;
    const void* in[N];
#pragma unroll
    for (int r = 0; r < N; ++r) in[r] = sys_of(d, G.sys0 + (r < nr ? r : nr - 1)).v[in_slot];
    constexpr bool NT = POL == STREAM;
    static_assert(POL == CACHED || N == 1, "streaming and quad gathers are built for one system");
    const int cb = site_index<POL>(gblk);
    double dots[N];
#pragma unroll
    for (int r = 0; r < N; ++r) dots[r] = 0.0;
    constexpr bool FUSED = MODE == DS_UPDATE_FUSED;
    static_assert(!FUSED || N == 1, "alpha is formed in-block for one system only");
    double pre[2] = {0.0, 0.0};  // FUSED: this thread's share of the |D_oe p|^2 and |p|^2 partials
    double head[HEAD][2];
    const double* const psrc[2] = {G.partials, G.partials_p};
    double st_m2 = 0.0, st_rho = 0.0;
    if constexpr (FUSED) {
        strided_head<2>(pre, head, psrc, G.nblk);
        st_m2 = h.st[0]->m2;
        st_rho = h.st[0]->rho;
    }
    const bool live = cb < g.Vh;
    Vec3<R> acc[N];
#pragma unroll
    for (int r = 0; r < N; ++r) acc[r] = vzero<R>();

    if constexpr (POL == QUAD) {
        if (live) acc[0] = dslash_quad<LP, RECON, VP>(g, links, in[0], p, site_of(g, p, cb));
    } else if (live) {
        const Site s = site_of(g, p, cb);
// several systems: two directions at a time (FP32 and 16-bit vectors; 105-158 VGPRs for four systems, 1% faster
// batches than one at a time), one in FP64 (its four-system update holds 216 VGPRs already); one system: two at a time
// in FP64, where all four put 384 values in flight and leave one wave per SIMD, and for FP32 recon-12 with
// cached link loads, whose row rebuild makes four at a time cost 125-136 VGPRs (measured 3-4% slower)
        constexpr int UNROLL = N == 1 ? unroll_dirs(LP, RECON, VP, NT) : (VP == F64 ? 1 : 2);
#pragma unroll UNROLL
        for (int mu = 0; mu < 4; ++mu) {
            R e = (R)eta_sign(s, mu);
            R sf = e, sb = -e;
            if (mu == 3 && g.bc_t) {
                if (s.t == g.T - 1) sf = -sf;
                if (s.t == 0) sb = -sb;
            }
            const int nf = nbr(g, s, mu, +1);
            const int nb = nbr(g, s, mu, -1);
            const Su3<R> Uf = LF::template load<NT>(link_block<LF>(links, g.Vh, p, mu), g.Vh, cb);
            Vec3<R> v[N];
#pragma unroll
            for (int r = 0; r < N; ++r) v[r] = VF::load(in[r], g.Vh, nf);
#pragma unroll
            for (int r = 0; r < N; ++r) mv_acc(acc[r], Uf, v[r], sf);
            const Su3<R> Ub = LF::template load<NT>(link_block<LF>(links, g.Vh, 1 - p, mu), g.Vh, nb);
#pragma unroll
            for (int r = 0; r < N; ++r) v[r] = VF::load(in[r], g.Vh, nb);
#pragma unroll
            for (int r = 0; r < N; ++r) mdv_acc(acc[r], Ub, v[r], sb);
        }
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                acc[r].c[i].re *= R(0.5);
                acc[r].c[i].im *= R(0.5);
            }
    }
    R alpha_blk = R(0);
    if constexpr (FUSED) {
        __shared__ BlockSums<2> sm;
        strided_tail<2>(pre, head, G.nblk);
        block_sum_all<2>(pre, sm);
        const double pq = st_m2 * pre[1] + pre[0];
        const double a = (pq > 0.0 && isfinite(pq)) ? st_rho / pq : 0.0;  // breakdown: no update, flagged later
        if (threadIdx.x == 0 && gblk == 0) {
            G.rec[0] = pq;
            G.rec[1] = a;
        }
        alpha_blk = (R)a;
    }
    if (live && site_lead<POL>()) {
        if constexpr (MODE == DS_PLAIN) {
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (r < nr) VF::store(sys_of(d, G.sys0 + r).v[out_slot], g.Vh, cb, acc[r]);
        } else if constexpr (MODE == DS_NORM) {
#pragma unroll
            for (int r = 0; r < N; ++r) {
                if (r >= nr) continue;
                const Vec3<R> ts = VF::store_rt(sys_of(d, G.sys0 + r).v[out_slot], g.Vh, cb, acc[r]);
                double dd = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    dd += (double)acc[r].c[i].re * (double)ts.c[i].re + (double)acc[r].c[i].im * (double)ts.c[i].im;
                dots[r] = dd;
            }
        } else {
            // per group of up to four systems: loads first, then arithmetic, then stores
            constexpr int NG = N < 4 ? N : 4;
#pragma unroll
            for (int r0 = 0; r0 < N; r0 += NG) {
                Vec3<R> pc[NG], rv[NG];
                Vec3<RX> xv[NG];
#pragma unroll
                for (int j = 0; j < NG; ++j) {
                    const int r = r0 + j;
                    const SysDev& S = sys_of(d, G.sys0 + (r < nr ? r : nr - 1));
                    pc[j] = VF::load(S.v[S_P], g.Vh, cb);
                    rv[j] = VF::load(S.v[S_R], g.Vh, cb);
                    xv[j] = XF::load(S.v[XP == F64 ? S_X64 : S_XLO], g.Vh, cb);
                }
#pragma unroll
                for (int j = 0; j < NG; ++j) {
                    const int r = r0 + j;
                    const R m2 = FUSED ? (R)st_m2 : h.act[r] ? (R)h.st[r]->m2 : R(0);
                    const R a = h.act[r] ? (FUSED ? alpha_blk : (R)h.st[r]->alpha) : R(0);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const R qre = m2 * pc[j].c[i].re - acc[r].c[i].re;
                        const R qim = m2 * pc[j].c[i].im - acc[r].c[i].im;
                        xv[j].c[i].re += (RX)a * (RX)pc[j].c[i].re;
                        xv[j].c[i].im += (RX)a * (RX)pc[j].c[i].im;
                        rv[j].c[i].re -= a * qre;
                        rv[j].c[i].im -= a * qim;
                    }
                }
#pragma unroll
                for (int j = 0; j < NG; ++j) {
                    const int r = r0 + j;
                    if (r >= nr) continue;
                    const SysDev& S = sys_of(d, G.sys0 + r);
                    XF::store(S.v[XP == F64 ? S_X64 : S_XLO], g.Vh, cb, xv[j]);
                    const Vec3<R> rs = VF::store_rt(S.v[S_R], g.Vh, cb, rv[j]);
                    double dd = 0.0;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        dd += (double)rs.c[i].re * (double)rs.c[i].re + (double)rs.c[i].im * (double)rs.c[i].im;
                    dots[r] = dd;
                }
            }
        }
    }
    if constexpr (MODE == DS_UPDATE_FUSED) block_partials<N>(G.partials_r, gblk, dots);
    else if constexpr (MODE != DS_PLAIN) block_partials<N>(G.partials, gblk, dots);
}

// ------------------------------------------------------------------------------------------------------
// FP64 true residual on even sites: r = b - m^2 x + D_eo t64, t64 = D_oe x (previous launch).
// Writes R (inner precision OP); block partials of |r|^2 and Re<r, p> (p unused when init). init: 0 a reliable
// update, 1 the start of a solve from a given x0, 2 the start from x0 = 0, where r = b needs no operator (t64 is
// then neither read nor needed).
// ------------------------------------------------------------------------------------------------------
template <int OP, int N, class D, int POL = CACHED>
__global__ __launch_bounds__(256) void k_resid(D d, int init, int remap) {
    using LF = LinkFmt<F64, 18>;
    using VO = VecFmt<OP>;
    using RO = typename Real<OP>::T;
    const int lblk = logical_block(remap);
    const BlockOf bo = block_of(d, lblk);
    const GroupDev& G = grp_of(d, bo.grp);
    const int gblk = bo.blk;
    const Rhs<N> h = rhs_of<N>(d, G, init ? G_ALIVE : G_RU);
    if (!h.any) return;
    const Geom g = G.g;
    const int cb = site_index<POL>(gblk);
    double dots[2 * N];
#pragma unroll
    for (int r = 0; r < 2 * N; ++r) dots[r] = 0.0;
    const bool zero_x = init == 2;
    if (cb < g.Vh) {
        const Site s = site_of(g, 0, cb);
        Vec3<double> acc[N];
        const void* tin[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            acc[r] = vzero<double>();
            tin[r] = h.act[r] ? sys_of(d, G.sys0 + r).v[S_T64] : nullptr;
        }
        // two directions at a time for one system, as in the FP64 half operator (all four put the kernel past 256
        // registers, one wave per SIMD)
        constexpr int UNROLL = N == 1 ? 2 : 4;
        if constexpr (POL == QUAD) {
            static_assert(N == 1, "quad gathers are built for one system");
            if (!zero_x) {
                acc[0] = dslash_quad<F64, 18, F64>(g, G.links64, tin[0], 0, s);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    acc[0].c[i].re *= 2.0;
                    acc[0].c[i].im *= 2.0;
                }
            }
        }
#pragma unroll UNROLL
        for (int mu = 0; mu < (zero_x || POL == QUAD ? 0 : 4); ++mu) {
            double e = (double)eta_sign(s, mu);
            double sf = e, sb = -e;
            if (mu == 3 && g.bc_t) {
                if (s.t == g.T - 1) sf = -sf;
                if (s.t == 0) sb = -sb;
            }
            const int nf = nbr(g, s, mu, +1);
            const int nb = nbr(g, s, mu, -1);
            const Su3<double> Uf = LF::load(link_block<LF>(G.links64, g.Vh, 0, mu), g.Vh, cb);
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (h.act[r]) mv_acc(acc[r], Uf, VecFmt<F64>::load(tin[r], g.Vh, nf), sf);
            const Su3<double> Ub = LF::load(link_block<LF>(G.links64, g.Vh, 1, mu), g.Vh, nb);
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (h.act[r]) mdv_acc(acc[r], Ub, VecFmt<F64>::load(tin[r], g.Vh, nb), sb);
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
            if (!h.act[r] || !site_lead<POL>()) continue;
            const SysDev& S = sys_of(d, G.sys0 + r);
            const Vec3<double> b = VecFmt<F64>::load(S.v[S_B64], g.Vh, cb);
            const Vec3<double> x = zero_x ? vzero<double>() : VecFmt<F64>::load(S.v[S_X64], g.Vh, cb);
            const double m2 = h.st[r]->m2;
            Vec3<RO> ro, pv;
            if (!init) pv = VO::load(S.v[S_P], g.Vh, cb);
            double dd = 0.0, rp = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double re = b.c[i].re - m2 * x.c[i].re + 0.5 * acc[r].c[i].re;
                const double im = b.c[i].im - m2 * x.c[i].im + 0.5 * acc[r].c[i].im;
                dd += re * re + im * im;
                if (!init) rp += re * (double)pv.c[i].re + im * (double)pv.c[i].im;
                ro.c[i].re = (RO)re;
                ro.c[i].im = (RO)im;
            }
            dots[2 * r] = dd;
            dots[2 * r + 1] = rp;
            VO::store(S.v[S_R], g.Vh, cb, ro);
        }
    }
    block_partials<2 * N>(G.partials, gblk, dots);
}

// p = r + beta p inside an iteration (gate G_ITER); p = a r + beta p after a reliable update or at the
// start (G_XPAY). Block partials of |p|^2 (as stored) feed the next alpha.
template <int VP, int N, class D>
__global__ __launch_bounds__(256) void k_xpay(D d, int gate, int remap) {
    using R = typename Real<VP>::T;
    using VF = VecFmt<VP>;
    const int lblk = logical_block(remap);
    const BlockOf bo = block_of(d, lblk);
    const GroupDev& G = grp_of(d, bo.grp);
    const int gblk = bo.blk;
    const Rhs<N> h = rhs_of<N>(d, G, gate);
    if (!h.any) return;
    const int Vh = G.g.Vh;
    const int nr = G.nrhs;
    const int cb = gblk * blockDim.x + threadIdx.x;
    double dots[N];
#pragma unroll
    for (int r = 0; r < N; ++r) dots[r] = 0.0;
    if (cb < Vh) {
        // every load first (systems that do not update take p = 0 r + 1 p), then arithmetic, then stores
        Vec3<R> rv[N], pv[N];
        R a[N], beta[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const SysDev& S = sys_of(d, G.sys0 + (r < nr ? r : nr - 1));
            beta[r] = h.act[r] ? (R)h.st[r]->beta : R(1);
            a[r] = h.act[r] ? (gate == G_XPAY ? (R)h.st[r]->xpay_a : R(1)) : R(0);
            rv[r] = VF::load(S.v[S_R], Vh, cb);
            // beta = 0 (start of a solve, restart): p is not read, it may hold anything
            pv[r] = beta[r] != R(0) ? VF::load(S.v[S_P], Vh, cb) : vzero<R>();
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                pv[r].c[i].re = a[r] * rv[r].c[i].re + beta[r] * pv[r].c[i].re;
                pv[r].c[i].im = a[r] * rv[r].c[i].im + beta[r] * pv[r].c[i].im;
            }
        }
#pragma unroll
        for (int r = 0; r < N; ++r) {
            if (r >= nr) continue;
            const Vec3<R> ps = VF::store_rt(sys_of(d, G.sys0 + r).v[S_P], Vh, cb, pv[r]);
            double dd = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                dd += (double)ps.c[i].re * (double)ps.c[i].re + (double)ps.c[i].im * (double)ps.c[i].im;
            dots[r] = dd;
        }
    }
    block_partials<N>(G.partials_p, gblk, dots);
}

// One system (of D = DescMany: each), after DS_UPDATE_FUSED: every block of it sums the |r|^2 partials (same order in every block) and
// takes the decisions of the update finalize itself (breakdown, convergence and reliable-update triggers,
// beta), then p = r + beta p with |p|^2 partials. The state is double-buffered: all blocks read the
// descriptor's state and block 0 writes the advanced state to next_state, which the next iteration's
// launches read, so no block can see a half-written state. At a chunk end (chunk_end != 0) with a reliable
// update due, the launch instead performs the update's first step, x64 += x_lo and x_lo = 0.
template <int VP, class D>
__global__ __launch_bounds__(256) void k_xpay_fused(D d, SolverState* __restrict__ st_out, int chunk_end, int remap) {
    using R = typename Real<VP>::T;
    using VF = VecFmt<VP>;
    const BlockOf bo = block_of(d, logical_block(remap));
    const int gblk = bo.blk;
    const GroupDev& G = grp_of(d, bo.grp);
    const SysDev& S = sys_of(d, bo.grp);
    const SolverState* st = state_of(d, bo.grp);
    const StateIn si = state_in(st);
    const double pq = G.rec[0];
    const int Vh = G.g.Vh;
    const int cb = gblk * blockDim.x + threadIdx.x;
    const bool live = cb < Vh;
    // loads that do not depend on the state go first
    double part[1] = {0.0};
    double head[HEAD][1];
    const double* const src[1] = {G.partials_r};
    strided_head<1>(part, head, src, G.nblk);
    Vec3<R> rv = vzero<R>(), pv = vzero<R>();
    if (live) {
        rv = VF::load(S.v[S_R], Vh, cb);
        pv = VF::load(S.v[S_P], Vh, cb);
    }
    __shared__ BlockSums<1> sm;
    strided_tail<1>(part, head, G.nblk);
    block_sum_all<1>(part, sm);
    const bool go = goes_on(si, pq, part[0], chunk_end != 0);
    if (gblk == 0 && threadIdx.x == 0) {
        SolverState s = *st;
        if (!(s.flags & (ST_DONE | ST_PENDING))) {
            fin_alpha(&s, pq);
            if (!(s.flags & ST_DONE)) fin_update(&s, part[0], chunk_end != 0);
            if (go) s.flags |= ST_T_STALE;  // p formed here: a following k_norm_rec applies D_oe to it
        }
        *next_state(d, st_out, bo.grp) = s;
    }
    if constexpr (VP != F64) {
        // paused with nothing wrong: a reliable update is due
        const bool broken = !(pq > 0.0) || !isfinite(pq) || !isfinite(si.rho) || !isfinite(part[0]);
        const bool pending = (si.flags & ST_PENDING) || (!go && !broken);
        if (chunk_end != 0 && pending && !(si.flags & ST_DONE)) {
            // the reliable update that follows the chunk starts here: x64 += x_lo; x_lo = 0 (k_accum's step)
            if (live) {
                Vec3<double> x = VecFmt<F64>::load(S.v[S_X64], Vh, cb);
                const Vec3<float> xl = VecFmt<F32>::load(S.v[S_XLO], Vh, cb);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    x.c[i].re += (double)xl.c[i].re;
                    x.c[i].im += (double)xl.c[i].im;
                }
                VecFmt<F64>::store(S.v[S_X64], Vh, cb, x);
                VecFmt<F32>::store(S.v[S_XLO], Vh, cb, vzero<float>());
            }
            return;
        }
    }
    if (!go) return;  // paused or stopped: p and its partials stay as they are
    const R beta = (R)(part[0] / si.rho);
    double dots[1] = {0.0};
    if (live) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            pv.c[i].re = rv.c[i].re + beta * pv.c[i].re;
            pv.c[i].im = rv.c[i].im + beta * pv.c[i].im;
        }
        const Vec3<R> ps = VF::store_rt(S.v[S_P], Vh, cb, pv);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            dots[0] += (double)ps.c[i].re * (double)ps.c[i].re + (double)ps.c[i].im * (double)ps.c[i].im;
    }
    block_partials<1>(G.partials_p, gblk, dots);
}

// The first launch of an iteration of one system, or of each of D = DescMany, in FP32 or FP64 (with DS_UPDATE_FUSED
// the second). It
// replaces the p update and t = D_oe p of the three-launch iteration by the recurrence
//   p_i = r_i + beta p_{i-1},   t_i = D_oe p_i = D_oe r_i + beta t_{i-1},
// so that the operator is applied to r_i, which is complete when the launch starts, while p_i is formed in
// the same launch (each thread also updates the even site with its own index). Every block first takes the
// decisions of the last update from its |r|^2 partials (as k_xpay_fused does); block 0 writes the advanced
// state to next_state. When p was formed elsewhere (start, reliable update, end of the last chunk: ST_T_STALE)
// the launch applies D_oe to p directly and takes no decision. Partials: Re<D_oe in, t> as DS_NORM, and
// |p_i|^2 from the recurrence (the other paths leave the |p|^2 partials of the launch that formed p).
template <int LP, int RECON, int VP, int POL, class D>
__global__ __launch_bounds__(256) void k_norm_rec(D d, SolverState* __restrict__ st_out, int remap) {
    using R = typename Real<VP>::T;
    using VF = VecFmt<VP>;
    const BlockOf bo = block_of(d, logical_block(remap));
    const int gblk = bo.blk;
    const GroupDev& G = grp_of(d, bo.grp);
    const SysDev& S = sys_of(d, bo.grp);
    const SolverState* st = state_of(d, bo.grp);
    const Geom g = G.g;
    const int cb = site_index<POL>(gblk);
    const bool live = cb < g.Vh, lead = live && site_lead<POL>();
    const StateIn si = state_in(st);
    const double pq = G.rec[0];
    if (si.flags & (ST_DONE | ST_PENDING)) {
        if (gblk == 0 && threadIdx.x == 0) *next_state(d, st_out, bo.grp) = *st;
        return;
    }
    const bool direct = (si.flags & ST_T_STALE) != 0;
    double part[1] = {0.0};
    double head[HEAD][1];
    const double* const psrc[1] = {G.partials_r};
    if (!direct) strided_head<1>(part, head, psrc, G.nblk);
    Vec3<R> acc = vzero<R>(), told = vzero<R>(), rv = vzero<R>(), pv = vzero<R>();
    if (live) {
        const void* in = direct ? S.v[S_P] : S.v[S_R];
        if constexpr (POL == QUAD) acc = dslash_quad<LP, RECON, VP>(g, G.links_lo, in, 1, site_of(g, 1, cb));
        else acc = dslash_site<LP, RECON, VP, POL == STREAM>(g, G.links_lo, in, 1, site_of(g, 1, cb));
        if (!direct && lead) {
            told = VF::load(S.v[S_T], g.Vh, cb);
            rv = VF::load(S.v[S_R], g.Vh, cb);
            pv = VF::load(S.v[S_P], g.Vh, cb);
        }
    }
    if (!direct) {
        __shared__ BlockSums<1> sm;
        strided_tail<1>(part, head, G.nblk);
        block_sum_all<1>(part, sm);
    }
    if (gblk == 0 && threadIdx.x == 0) {
        SolverState s = *st;
        if (direct) {
            s.flags &= ~ST_T_STALE;
        } else {
            fin_alpha(&s, pq);
            if (!(s.flags & ST_DONE)) fin_update(&s, part[0], false);
        }
        *next_state(d, st_out, bo.grp) = s;
    }
    if (!direct && !goes_on(si, pq, part[0], false)) return;  // paused or stopped: t, p and their partials stay
    const R beta = direct ? R(0) : (R)(part[0] / si.rho);
    double dots[2] = {0.0, 0.0};
    if (lead) {
        Vec3<R> t = acc;
        if (!direct) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                t.c[i].re += beta * told.c[i].re;
                t.c[i].im += beta * told.c[i].im;
                pv.c[i].re = rv.c[i].re + beta * pv.c[i].re;
                pv.c[i].im = rv.c[i].im + beta * pv.c[i].im;
            }
            const Vec3<R> ps = VF::store_rt(S.v[S_P], g.Vh, cb, pv);
#pragma unroll
            for (int i = 0; i < 3; ++i)
                dots[1] += (double)ps.c[i].re * (double)ps.c[i].re + (double)ps.c[i].im * (double)ps.c[i].im;
        }
        const Vec3<R> ts = VF::store_rt(S.v[S_T], g.Vh, cb, t);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            dots[0] += (double)t.c[i].re * (double)ts.c[i].re + (double)t.c[i].im * (double)ts.c[i].im;
    }
    __shared__ BlockSums<2> sm2;
    block_sum_all<2>(dots, sm2);
    if (threadIdx.x == 0) {
        G.partials[gblk] = dots[0];
        if (!direct) G.partials_p[gblk] = dots[1];
    }
}

// x64 += xlo; xlo = 0 (reliable update).
template <int N, class D>
__global__ __launch_bounds__(256) void k_accum(D d, int remap) {
    const int lblk = logical_block(remap);
    const BlockOf bo = block_of(d, lblk);
    const GroupDev& G = grp_of(d, bo.grp);
    const int gblk = bo.blk;
    const Rhs<N> h = rhs_of<N>(d, G, G_RU);
    if (!h.any) return;
    const int Vh = G.g.Vh;
    const int cb = gblk * blockDim.x + threadIdx.x;
    if (cb >= Vh) return;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        if (!h.act[r]) continue;
        const SysDev& S = sys_of(d, G.sys0 + r);
        Vec3<double> x = VecFmt<F64>::load(S.v[S_X64], Vh, cb);
        const Vec3<float> xl = VecFmt<F32>::load(S.v[S_XLO], Vh, cb);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            x.c[i].re += (double)xl.c[i].re;
            x.c[i].im += (double)xl.c[i].im;
        }
        VecFmt<F64>::store(S.v[S_X64], Vh, cb, x);
        VecFmt<F32>::store(S.v[S_XLO], Vh, cb, vzero<float>());
    }
}

// Block partials of |b|^2 (-> bnorm2 and the stopping threshold tol^2 |b|^2).
template <int N, class D>
__global__ __launch_bounds__(256) void k_norm_b(D d, int remap) {
    const int lblk = logical_block(remap);
    const BlockOf bo = block_of(d, lblk);
    const GroupDev& G = grp_of(d, bo.grp);
    const int gblk = bo.blk;
    const Rhs<N> h = rhs_of<N>(d, G, G_ALIVE);
    if (!h.any) return;
    const int Vh = G.g.Vh;
    const int cb = gblk * blockDim.x + threadIdx.x;
    double dots[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
        dots[r] = 0.0;
        if (!h.act[r] || cb >= Vh) continue;
        const Vec3<double> b = VecFmt<F64>::load(sys_of(d, G.sys0 + r).v[S_B64], Vh, cb);
#pragma unroll
        for (int i = 0; i < 3; ++i) dots[r] += b.c[i].re * b.c[i].re + b.c[i].im * b.c[i].im;
    }
    block_partials<N>(G.partials, gblk, dots);
}

// ------------------------------------------------------------------------------------------------------
// Second reduction stage, one block per system: sum the partials of the previous launch in block order and
// update the state of every system that launch worked on (same gate, and no state changed in between).
// ------------------------------------------------------------------------------------------------------
enum FinKind : int {
    FIN_ALPHA = 0,
    FIN_UPDATE = 1,      // inside a chunk
    FIN_RESID = 2,
    FIN_RESID_INIT = 3,
    FIN_NORM_B = 4,
    FIN_UPDATE_END = 5,  // last iteration of a chunk: also the delta and ru_every triggers
};

// partials of FIN_ALPHA: |D_oe p|^2 (from DS_NORM) and |p|^2 (from k_xpay)
//
// The launch is latency bound: a block per system, whose 1024 threads put every partial load in flight at once (a
// few per thread) and reduce two sums; then thread 0 updates the system's state. One block per group reduced the eight sums
// of its four systems: 9.2 against 5.2 us in the 32-system workload.
template <int N, class D>
__global__ __launch_bounds__(1024) void k_finalize(D d, int kind, int gate) {
    const int grp = blockIdx.x / N, r = blockIdx.x - N * grp;
    const GroupDev& G = grp_of(d, grp);
    if (r >= G.nrhs) return;
    SolverState* const st = state_of(d, G.sys0 + r);
    if (!gate_flags_open(st->flags, gate)) return;
    // partials of a block: one value per system, two (r: 2 r and 2 r + 1) of a true residual; FIN_ALPHA takes the |p|^2
    // partials beside them
    const bool two = kind == FIN_RESID || kind == FIN_RESID_INIT;
    const double* const p0 = two ? G.partials + 2 * r : G.partials + r;
    const double* const p1 = two ? p0 + 1 : G.partials_p + r;
    const bool second = two || kind == FIN_ALPHA;
    const int step = two ? 2 * N : N;
    double s[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < G.nblk; b += blockDim.x) {
        s[0] += p0[(size_t)b * step];
        if (second) s[1] += p1[(size_t)b * step];
    }
    __shared__ BlockSums<2> sm;
    block_sum_all<2>(s, sm);
    if (threadIdx.x != 0) return;
    if (kind == FIN_ALPHA) fin_alpha(st, st->m2 * s[1] + s[0]);
    else if (kind == FIN_UPDATE || kind == FIN_UPDATE_END) fin_update(st, s[0], kind == FIN_UPDATE_END);
    else if (kind == FIN_NORM_B) {
        st->bnorm2 = s[0];
        st->stop2 = st->tol2 * s[0];
    } else fin_resid(st, s[0], s[1], kind == FIN_RESID_INIT);
}

// ------------------------------------------------------------------------------------------------------
// Packing: natural complex128 <-> planes.
// ------------------------------------------------------------------------------------------------------
// Natural links -> planes of precision P, and of FP64 as well when f64 is not null (one read of the links serves both
// packings). A block takes 256 consecutive links of direction blockIdx.y: they come in through LDS as consecutive 16-byte
// words (a lane's own link is 144 bytes from the next lane's), and each half of the block then packs the links of one
// parity, 128 consecutive sites of its planes. The links stream past the caches, and so does the FP64 packing written
// beside another: a solve's iterations read the other one. At 20^3x64 with FP32 recon 12: 125 us for both (137 without the
// streaming stores, 191 in two launches), 688 MB, 111 us at the copy rate; the FP64 packing alone 115 us.
template <int P, int RECON>
__global__ __launch_bounds__(256) void k_pack_gauge(Geom g, const double2* __restrict__ nat, void* out, void* f64) {
    using LF = LinkFmt<P, RECON>;
    __shared__ double2 sm[256 * 9];
    const int mu = blockIdx.y, V = 2 * g.Vh, first = blockIdx.x * 256, n = min(256, V - first);
    const double2* src = nat + ((size_t)mu * V + first) * 9;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int i = j * 256 + threadIdx.x;
        if (i < 9 * n) sm[i] = ldw<true>(src + i);
    }
    __syncthreads();
    const int q = threadIdx.x >> 7, k = threadIdx.x & 127;
    if (2 * k >= n) return;
    // the two sites of a pair (2 cb, 2 cb + 1) have one parity each: the even-x one has parity y + z + t
    const int cb = (first >> 1) + k;
    const int r1 = divq(cb, g.Xh, g.rXh), r2 = divq(r1, g.Y, g.rY), t = divq(r2, g.Z, g.rZ);
    const int odd = (r1 - r2 * g.Y + r2 - t * g.Z + t + q) & 1;
    const double2* w = sm + 9 * (2 * k + odd);
    double r[18];
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const double2 v = w[j];
        r[2 * j] = v.x;
        r[2 * j + 1] = v.y;
    }
    LF::store((void*)link_block<LF>(out, g.Vh, q, mu), g.Vh, cb, r);
    if constexpr (P != F64) {
        using L64 = LinkFmt<F64, 18>;
        if (f64) L64::template store<true>((void*)link_block<L64>(f64, g.Vh, q, mu), g.Vh, cb, r);
    }
}

template <int P>
__global__ __launch_bounds__(256) void k_pack_vec(int Vh, const double* __restrict__ nat, void* out) {
    using R = typename Real<P>::T;
    const int cb = blockIdx.x * blockDim.x + threadIdx.x;
    if (cb >= Vh) return;
    Vec3<R> v;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v.c[c].re = (R)nat[(size_t)cb * 6 + 2 * c];
        v.c[c].im = (R)nat[(size_t)cb * 6 + 2 * c + 1];
    }
    VecFmt<P>::store(out, Vh, cb, v);
}

template <int P>
__global__ __launch_bounds__(256) void k_unpack_vec(int Vh, const void* in, double* __restrict__ nat) {
    const int cb = blockIdx.x * blockDim.x + threadIdx.x;
    if (cb >= Vh) return;
    const auto v = VecFmt<P>::load(in, Vh, cb);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        nat[(size_t)cb * 6 + 2 * c] = (double)v.c[c].re;
        nat[(size_t)cb * 6 + 2 * c + 1] = (double)v.c[c].im;
    }
}

}  // namespace sp
