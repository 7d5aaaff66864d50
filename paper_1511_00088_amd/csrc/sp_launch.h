// Host-side launch wrappers: map runtime precision / reconstruction choices onto kernel instantiations.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "sp_kernels.h"

namespace sp {

struct LaunchCfg {
    int nt = 256;    // threads per block (64, 128 or 256)
    int remap = 1;   // XCD-aware block order
    int stream = 0;  // link loads of the single-system half operator: 0 cached, 1 streaming (non-temporal)
    int quad = 0;    // single-system half operator with four lanes per site (blocks of nt / 4 sites)
};

// Whether the single-system operator takes four lanes per site. Below about 30,000 sites per parity a lane per site
// leaves the chip a few hundred wavefronts, each walking the directions in rounds of dependent latency. Measured per
// solve (tol 1e-10, m = 0.05; four lanes against one, each with 256 threads): 2,048 sites 2.32 against 2.76 ms (FP32
// recon 12), 2.45 against 2.86 (recon 18) and 2.78 against 3.48 (FP64); 20,736 sites 3.22 against 3.59, 3.49 against
// 3.37 and 4.44 against 4.38; 32,768 sites 2.78 against 2.90 (recon 12) and 2.55 against 2.91 (fixed-point links);
// 65,536 sites 5.45 against 4.55 (recon 12), where the chip is full without it. FP32 recon 18 and FP64 move the most
// bytes a site and turn first. With the block sizes of solve_threads on both sides (tol 1e-12, m = 0.1) the line stays:
// 8,000 sites 1.79 against 2.25 (recon 12), 1.78 against 1.94 (recon 18) and 1.85 against 2.23 (FP64); 10,368 sites 1.89
// against 2.12, 1.96 against 1.86 and 2.17 against 2.09; 30,720 sites 2.54 against 2.58 (recon 12), 2.48 against 3.09
// (recon 8); 65,536 sites 4.65 against 4.30 (recon 8). FP16 and BF16 vectors keep a lane per site: the order of a site's
// eight terms decides how their last digits round, and with it, by some percent either way, where such a solve's reliable
// updates fall.
inline bool quad_lanes(int Vh, int lp, int recon, int vp) {
    if (vp != F32 && vp != F64) return false;
    const bool heavy = vp == F64 || (lp == F32 && recon == 18);
    return Vh <= (heavy ? 8192 : 32768);
}

// Maximum systems per group in batched launches.
static constexpr int NB = 4;

// Groups of one gauge field whose blocks alternate in batched launches, so that a link one of them has brought into an
// XCD's L2 serves the others. Measured (tol 1e-12, m = 0.1; bit-identical solutions; alternating 1, 2 and 4 groups): 16
// systems on 16^3x32 22.5, 19.6 and 18.7 ms, 12 on 24^3x48 79.1, 77.4 and 73.4, 16 on 20^3x64 93.9, 90.4 and 89.5; the
// 32-system workload 224, 215 and 215.
static constexpr size_t BUNDLE = 4;

// Sites per parity, summed over the systems, up to which the systems of a batch iterate as single systems in common
// launches (many_systems): two launches an iteration that take their own decisions, against five whose links a group
// loads once. Small lattices are bound by the launches, large ones by the bytes. Measured per solve (tol 1e-12, m =
// 0.1, FP32 recon 12 unless said; groups against this, ms): 3 systems on 8^4 6.75 and 2.02, 32 on 8^4 7.98 and 3.69; 3
// on 12^3x24 9.03 and 3.58, 6 (recon 18) 9.8 and 4.5, 6 (FP64, 256 threads) 12.0 and 6.2; 3 on 16^3x32 (196,608 sites)
// 11.0 and 8.5, 4 (FP64) 15.7 and 12.1, 6 (recon 18; 393,216) 13.7 and 11.8, 6 (FP16 links) 14.3 and 14.6, 16
// (1,048,576) 21.4 and 24.3; 4 on 24^3x48 (recon 18; 1,327,104) 40.1 and 54.8; 8 on 20^3x64 (2,048,000) 47.9 and 54.8.
inline long many_sites(int lp, int vp) { return lp == F32 && vp == F32 ? 400000 : 262144; }

inline int blocks_for(int n, int nt) { return (n + nt - 1) / nt; }

// The fused single-system iteration has every block sum all block partials of the previous launch (in the same
// order in every block): at most this many per thread. 32 admits 8,192 blocks of 256 threads (V/2 up to 2^21:
// the 32^3x64 control and the 28^3x96 production lattice). The partials are loaded before the gather, so their
// latency overlaps the link loads; each block reads them all (8 bytes per block of the launch) from L2.
static constexpr int FUSED_PARTIALS = 32;

// Systems per group in the launches of a descriptor.
template <class D>
struct NOf {
    static constexpr int value = 1;
};
template <>
struct NOf<DescBatch> {
    static constexpr int value = NB;
};

// Threads per block of the fused iteration, for `lanes` lanes of a system (a site has one or four): the fewest that
// keep it to one block a CU. Small lattices then spread over the chip, and a block reduces fewer wavefronts; with more
// blocks than CUs each of them sums more partials for nothing. Measured per solve (tol 1e-12, m = 0.05; ms; 64, 128 and
// 256 threads): 8^4
// FP32 recon 12 with four lanes (8,192 in all) 2.28, 2.49 and 2.68, FP64 2.31, 2.63 and 3.18, BF16 with one lane 4.67,
// 4.87 and 5.09; 16,384 lanes 2.68, 2.88 and 3.16; 20,736 (12^3x24, recon 18) 3.71, 3.52 and 3.97, FP64 4.57, 4.44 and
// 5.21, BF16 6.25, 5.94 and 6.18; 32,000 2.96, 2.69 and 2.92; 38,416 4.81, 4.40 and 4.41; 65,536 (16^3x32, recon 12)
// 6.20, 5.58 and 5.07; 82,944 (12^3x24, recon 12, four lanes) 4.51, 3.83 and 3.79; the 20^3x64 solve on FP16 links (to
// 1e-8, m = 0.01) 25.8 with 128 and 21.9 with 256. Of several systems in common launches each block sums its own system's
// partials, so the lanes of one count (m = 0.1): 3 systems on 8^4 2.01 against 2.25 with 256, 4 on 10^3x20 3.49 against
// 3.67, 4 in FP64 on 12^3x24 5.14 against 5.92.
inline int solve_threads(int lanes) { return lanes <= 64 * 256 ? 64 : lanes <= 128 * 256 ? 128 : 256; }

// Half operator (see k_dslash; mode DS_PLAIN, DS_NORM or DS_UPDATE). D = DescSingle (one system), DescBatch (up to NB
// per group) or DescMany (FP32 and FP64 vectors, cached or quad gathers, modes DS_PLAIN in FP64 and DS_UPDATE_FUSED).
template <class D>
hipError_t launch_dslash(const D& d, int nblocks, LaunchCfg c, int lp, int recon, int vp, int p, int in_slot,
                         int out_slot, int mode, int gate, int use64, hipStream_t s);
template <class D>
hipError_t launch_resid(const D& d, int nblocks, LaunchCfg c, int op, int init, hipStream_t s);
template <class D>
hipError_t launch_xpay(const D& d, int nblocks, LaunchCfg c, int vp, int gate, hipStream_t s);
template <class D>
hipError_t launch_accum(const D& d, int nblocks, LaunchCfg c, hipStream_t s);
template <class D>
hipError_t launch_norm_b(const D& d, int nblocks, LaunchCfg c, hipStream_t s);
// Fused p update of one system or of many (k_xpay_fused): reads d's state, writes the advanced state to st_out (of
// several systems: to d.next).
template <class D>
hipError_t launch_xpay_fused(const D& d, SolverState* st_out, int chunk_end, int nblocks, LaunchCfg c, int vp,
                             hipStream_t s);
hipError_t launch_state_copy(const SolverState* src, SolverState* dst, hipStream_t s);
hipError_t launch_state_publish(const SolverState* src, SolverState* dst, int n, hipStream_t s);
// First launch of the two-launch iteration of one system, or of many, in FP32 or FP64 (k_norm_rec).
template <class D>
hipError_t launch_norm_rec(const D& d, SolverState* st_out, int nblocks, LaunchCfg c, int lp, int recon, int vp,
                           hipStream_t s);
// Second reduction stage (k_finalize), one block per system.
template <class D>
hipError_t launch_finalize(const D& d, int ngroups, int kind, int gate, hipStream_t s);

hipError_t launch_pack_gauge(const Geom& g, const double* nat, int prec, int recon, void* out, void* f64, hipStream_t s);
hipError_t launch_pack_vec(int Vh, const double* nat, int prec, void* out, hipStream_t s);
hipError_t launch_unpack_vec(int Vh, const void* in, int prec, double* nat, hipStream_t s);
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);  // bytes multiple of 16

// The gradient of sp_cg_force from natural x and lambda: three launches, with packed FP64 x, lambda (even), y_x and y_l
// (odd) and mass_grad_blocks(g) partials of Re<lambda, x> as scratch. force and grad_mass may be null.
struct GradScratch {
    void *x, *lam, *yx, *yl;
    double* partials;
};
hipError_t launch_gradient(const Geom& g, const void* links64, const double* x, const double* lam, double mass,
                           const GradScratch& w, double* gamma, double* force, double* grad_mass, hipStream_t s);
int mass_grad_blocks(const Geom& g);

// Full-lattice solve helpers (sp_full.hip): split a natural full vector into packed FP64 halves, form
// b_e = m src_e - t_e in the natural half layout, merge psi_e with psi_o = (src_o - t_o) / m.
hipError_t launch_full_split(const Geom& g, const double* src, void* se, void* so, hipStream_t s);
hipError_t launch_full_source(const Geom& g, double m, const void* se, const void* te, double* be, hipStream_t s);
hipError_t launch_full_merge(const Geom& g, double m, const double* psie, const void* so, const void* to,
                             double* psi, hipStream_t s);

// HYP smearing (sp_hyp.hip): three launches, intermediate levels in ws (hyp_workspace_bytes).
size_t hyp_workspace_bytes(const Geom& g);
hipError_t launch_hyp(const Geom& g, const double* links, const double alpha[3], double* out, void* ws,
                      hipStream_t s);

// NPR contraction (sp_npr.hip): path links per hypercube, then the contraction of n field sets.
size_t npr_path_bytes(const Geom& g);
hipError_t launch_npr_paths(const Geom& g, const double* links, void* uad, hipStream_t s);
hipError_t launch_npr_contract(const Geom& g, const void* uad, int n, const double* const f[4], const int labels[4],
                               double* out, hipStream_t s);
// The same contraction from stored path links (uad, links null) or fused with their construction from the natural
// links (links non-null, uad ignored).
hipError_t launch_npr_contract_from(const Geom& g, const void* uad, const double* links, int n, const double* const f[4],
                                    const int labels[4], double* out, hipStream_t s);

}  // namespace sp
