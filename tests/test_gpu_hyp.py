"""GPU HYP smearing (sp_hyp_smear) against the FP64 oracle (oracle/hyp.py).

Small lattices are compared link by link with the oracle's full result; the 20^3x64 workload field at
sampled links against the committed oracle values (tests/golden/hyp_cfg1_samples.txt), plus properties
that hold at any size (every output link in SU(3), determinism). Both sides compute the maximiser of
Re tr(X^dag W) over SU(3): the oracle by SU(2)-subgroup sweeps from the SVD polar factor, the GPU in closed
form where that applies (every matrix of the workload field) and by sweeps from a Newton polar factor
elsewhere (most matrices of a Haar field); they agree to rounding, and the tests ask for 1e-12.
"""
import os

import numpy as np
import pytest
import torch

import lattice_inputs as li
import paper_1511_00088_amd as sp
from gpu_common import DEV, announce, to_dev, to_host
from oracle import hyp

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "hyp_cfg1_samples.txt")


def _gpu_hyp(dims, U, alpha=hyp.HYP_ALPHA):
    lat = sp.Lattice(dims)
    out = sp.hyp_smear(lat, to_dev(U), alpha)
    torch.cuda.synchronize()
    return to_host(out)


@pytest.mark.parametrize("dims,kind,alpha", [
    ((4, 4, 4, 4), "near", hyp.HYP_ALPHA),
    ((4, 6, 2, 8), "near", hyp.HYP_ALPHA),
    ((6, 4, 4, 6), "near", (0.5, 0.3, 0.9)),
    ((4, 4, 4, 4), "haar", hyp.HYP_ALPHA),
    ((8, 8, 8, 8), "near", hyp.HYP_ALPHA),
    ((4, 4, 4, 4), "near", (1.0, 1.0, 1.0)),
    ((4, 4, 4, 4), "haar", (1.0, 0.0, 1.0)),
])
def test_hyp_matches_oracle(dims, kind, alpha):
    announce(f"hyp dims={dims} {kind} alpha={alpha}")
    U = li.near_identity_links(dims, 0.5, 451) if kind == "near" else li.haar_links(dims, 452)
    V = _gpu_hyp(dims, U, alpha)
    ref = hyp.hyp_smear(dims, U, alpha)
    assert np.max(np.abs(V - ref)) <= 1e-12


@pytest.mark.parametrize("dims,eps", [((2, 2, 2, 2), 0.3), ((2, 2, 2, 34), 0.7), ((6, 2, 14, 4), 0.05),
                                      ((4, 6, 10, 2), 1.0)])
def test_hyp_blocks_and_projection_branches(dims, eps):
    """Lattices of less than a block of 256 sites, and of one block and a remainder; link fields whose projections take
    the short series (eps 0.05), the long one and the iterations (eps 1). Each projection is within a few 1e-15 of the
    oracle's and three levels of it follow one another, so 1e-12 holds with the same margin as on the other fields."""
    announce(f"hyp dims={dims} eps={eps}")
    U = li.near_identity_links(dims, eps, 454)
    assert np.max(np.abs(_gpu_hyp(dims, U) - hyp.hyp_smear(dims, U))) <= 1e-12


def _maximiser_80bit(W, start):
    """The SU(3) maximiser of Re tr(X^dag W) in 80-bit numpy: Newton-Schulz steps make the start unitary, the cube root of
    its determinant is divided out, and SU(2)-subgroup sweeps run until they move nothing that 64 bits could show."""
    X = start.astype(np.clongdouble)
    for _ in range(3):
        X = 0.5 * (3 * X - X @ hyp.dag(X) @ X)
    c = np.cross(X[..., 1, :], X[..., 2, :])
    d = np.sum(X[..., 0, :] * c, axis=-1)
    X = X * np.exp(-1j * (np.arctan2(d.imag, d.real) / 3))[..., None, None]
    for _ in range(200):
        Y = X
        for i, j in ((0, 1), (0, 2), (1, 2)):
            Y = hyp.su2_step(Y, W, i, j)
        if np.max(np.abs(Y - X)) < 1e-18:
            return Y
        X = Y
    raise AssertionError("the 80-bit sweeps did not settle")


@pytest.mark.parametrize("eps", [0.02, 0.3, 0.6])
def test_projection_is_as_exact_as_its_arithmetic(eps):
    """Weights (0.75, 0, 0): levels 1 and 2 project the links themselves, level 3 one staple sum per link, formed here in
    80 bits. Rounding alone: the sum, F of X = W F and their product round each entry some ten times by up to 2^-54 of
    values up to 1 (rms 2^-54 / sqrt(3) each, 1e-16 in all), so an rms over a link's nine entries (Frobenius) of 3 x 1e-16,
    and a little more through rows rebuilt from the others; 8e-16 is asked, and 2e-15 of the worst entry."""
    dims, a1 = (6, 4, 4, 8), 0.75
    announce(f"hyp projection error eps={eps}")
    U = li.near_identity_links(dims, eps, 457)
    V = _gpu_hyp(dims, U, (a1, 0.0, 0.0)).astype(np.clongdouble)
    # the links the levels start from: U projected (its own rounding would otherwise count as the kernel's)
    P = _maximiser_80bit(U.astype(np.clongdouble), U)
    W = [(1 - np.longdouble(a1)) * U[mu].astype(np.clongdouble) + np.longdouble(a1) / 6 *
         sum(hyp.staples(P[nu], P[mu], mu, nu, dims) for nu in range(4) if nu != mu) for mu in range(4)]
    for mu in range(4):
        err = np.abs(V[mu] - _maximiser_80bit(W[mu], hyp.polar_start(W[mu].astype(np.complex128))))
        rms = float(np.sqrt(np.mean(np.sum(err * err, axis=(-2, -1)))))
        announce(f"  mu={mu} rms={rms:.2e} max={float(err.max()):.2e}")
        assert rms <= 8e-16 and err.max() <= 2e-15, mu


@pytest.mark.parametrize("eps,alpha", [(0.05, hyp.HYP_ALPHA), (0.3, hyp.HYP_ALPHA), (1.0, hyp.HYP_ALPHA), (1.4, hyp.HYP_ALPHA),
                                       (0.3, (0.5, 0.3, 0.9))])
def test_smeared_links_are_unitary_to_rounding(eps, alpha):
    """V V^dag - 1 holds each entry's error of a link (about 3e-16, see above) twice: rms over a link below 1.5e-15, the
    worst of some 100,000 entries below 3.5e-15; with the short series, the long one and, past eps 0.7, the iterations."""
    dims = (6, 8, 6, 10)
    announce(f"hyp unitarity eps={eps} alpha={alpha}")
    V = _gpu_hyp(dims, li.near_identity_links(dims, eps, 458), alpha).astype(np.clongdouble)
    D = np.abs(V @ hyp.dag(V) - np.eye(3))
    rms = float(np.sqrt(np.mean(np.sum(D * D, axis=(-2, -1)))))
    announce(f"  rms={rms:.2e} max={float(D.max()):.2e}")
    assert rms <= 1.5e-15 and D.max() <= 3.5e-15


def test_largest_weights_on_haar_links_ill_conditioned_maximum():
    # weights (1, 1, 1) on Haar links give staple sums whose determinant phase sits at +-pi; there the
    # maximiser of Re tr(X^dag W) lies along a nearly flat direction and the SU(2)-subgroup sweeps converge
    # with a rate near 1 (the oracle needs up to its 500-sweep cap): the maximum itself is fixed to rounding,
    # the maximising link only to about 1e-6
    dims = (4, 4, 4, 4)
    announce("hyp weights (1, 1, 1) on Haar links")
    U = li.haar_links(dims, 461)
    alpha = (1.0, 1.0, 1.0)
    V = _gpu_hyp(dims, U, alpha)
    ref = hyp.hyp_smear(dims, U, alpha)
    eye = np.eye(3)
    assert np.max(np.abs(V @ np.conj(np.swapaxes(V, -1, -2)) - eye)) <= 1e-13
    assert np.max(np.abs(np.linalg.det(V) - 1.0)) <= 1e-13
    assert np.max(np.abs(V - ref)) <= 1e-5


def test_zero_weights_give_the_links_back():
    dims = (4, 4, 4, 4)
    announce("hyp zero weights")
    U = li.haar_links(dims, 453)
    assert np.max(np.abs(_gpu_hyp(dims, U, (0.0, 0.0, 0.0)) - U)) <= 1e-13


def _golden():
    rows = np.loadtxt(GOLDEN, comments="#")
    mu = rows[:, 0].astype(int)
    s = rows[:, 1].astype(int)
    m = (rows[:, 2::2] + 1j * rows[:, 3::2]).reshape(-1, 3, 3)
    return mu, s, m


def test_workload_field_sampled_vs_oracle_and_su3_everywhere():
    c = li.cfg1()
    dims = c["dims"]
    announce(f"hyp {dims} sampled")
    lat = sp.Lattice(dims)
    U = to_dev(c["links"])
    out = sp.hyp_smear(lat, U)
    out2 = sp.hyp_smear(lat, U)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)  # deterministic
    mu, s, ref = _golden()
    got = to_host(out[torch.as_tensor(mu, device=DEV), torch.as_tensor(s, device=DEV)])
    assert np.max(np.abs(got - ref)) <= 1e-12
    # every output link is in SU(3)
    eye = torch.eye(3, dtype=torch.complex128, device=DEV)
    for m in range(4):
        Vm = out[m]
        un = torch.max(torch.abs(Vm @ Vm.conj().transpose(-1, -2) - eye)).item()
        dt = torch.max(torch.abs(torch.linalg.det(Vm) - 1.0)).item()
        assert un <= 1e-13 and dt <= 1e-13, (m, un, dt)


def test_smeared_links_feed_the_solver():
    # the product of this step is a link field for the solve: smear, pack, solve, compare with the oracle
    import oracle

    dims = (4, 4, 4, 4)
    announce("hyp then solve 4^4")
    U = li.near_identity_links(dims, 0.5, 454)
    b = li.gaussian_even_source(dims, 455)
    m = 0.1
    lat = sp.Lattice(dims)
    Vs = sp.hyp_smear(lat, to_dev(U))
    G = sp.Gauge(lat, Vs, lo_prec="f32", recon=12)
    x, st = sp.cg_solve(G, m, to_dev(b), tol=1e-10, inner="f32")
    assert st.converged
    xr, status, _, _ = oracle.cg_solve(dims, hyp.hyp_smear(dims, U), m, b, tol=1e-13)
    assert status == 0
    assert np.linalg.norm(to_host(x) - xr) / np.linalg.norm(xr) <= 1e-8


def test_errors():
    dims = (4, 4, 4, 4)
    lat = sp.Lattice(dims)
    U = to_dev(li.haar_links(dims, 456))
    with pytest.raises(sp.StagError):
        sp.hyp_smear(lat, U, (0.75, 1.5, 0.3))
    with pytest.raises(sp.StagError):
        sp.hyp_smear(lat, U, out=U)
