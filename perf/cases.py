"""Timed cases of the staggered CG framework: what a lattice job has it do, through the public entry points.

`listed()` holds twelve cases, from a single half-operator call on an 8^4 lattice (a few microseconds, where launches
and latency count) to a batched solve of 32 systems. `draw(rng)` gives more cases of the same ranges: every
operation, storage precision and link packing in use, even extents from 4 upwards (the library's lattices have
even extents), ragged ones among them. Lattice sizes, masses, smearing weights and field-set counts are those of
the repository's benchmark and tests: 8^4, 12^3x24, 16^3x32, 20^3x64, one GPU's 20^3x8 share of a t-cut, and up
to 32^3x64 and 28^3x96. Links are near-identity SU(3) fields (smeared-like, as the workloads'), sources Gaussian.

Solves run to a true relative residual of 1e-12, the tolerance of the repository's reference solutions, so that
the solution is determined well below the differences between rounding orders.
"""
from __future__ import annotations

import math
import os

import torch

import paper_1511_00088_amd as sp

DEV = "cuda:0"
TOL = 1e-12
EPS = 0.3
ALPHA = (0.75, 0.6, 0.3)


def listed():
    big = dict(X=20, Y=20, Z=20, T=64, bc_t=0)
    return [
        # smallest operator call: one application on a test lattice, where the call and the launch are the cost
        dict(name="dslash_f32_8x8x8x8", op="dslash", X=8, Y=8, Z=8, T=8, bc_t=0, prec="f32", recon=12, lo="f32"),
        # the workload's operator, as an eigensolver or a smearing of sources applies it
        dict(name="dslash_f32_20x20x20x64", op="dslash", prec="f32", recon=12, lo="f32", **big),
        # FP64 operator on a ragged lattice with antiperiodic time (true residuals, the gradient's y = D x)
        dict(name="dslash_f64_14x18x22x50", op="dslash", X=14, Y=18, Z=22, T=50, bc_t=1, prec="f64", recon=18, lo="f64"),
        # a new gauge field: packed to FP64 and to FP32 recon-12 before its solves
        dict(name="pack_20x20x20x64", op="pack", recon=12, lo="f32", **big),
        # one GPU's share of a t-cut: faces packed, copied, unpacked, interior and boundary operator
        dict(name="halo_20x20x20x8", op="halo", X=20, Y=20, Z=20, T=8, bc_t=0, prec="f32", recon=12, lo="f32"),
        # smearing of a new configuration
        dict(name="hyp_20x20x20x64", op="hyp", **big),
        # NPR contraction of a few field sets on a new configuration (path links built on chip)
        dict(name="npr_fused_20x20x20x64", op="npr_fused", sets=4, **big),
        # NPR with stored path links: built once per configuration, then two operators contracted
        dict(name="npr_stored_12x12x12x24", op="npr_stored", X=12, Y=12, Z=12, T=24, bc_t=0, sets=9),
        # adjoint gradient with the su(3) force on the gradient lattice
        dict(name="force_16x16x16x32", op="force", X=16, Y=16, Z=16, T=32, bc_t=0),
        # small solve: a test lattice, hundreds of iterations of microsecond launches
        dict(name="solve_f32_8x8x8x8", op="solve", X=8, Y=8, Z=8, T=8, bc_t=0, prec="f32", recon=12, lo="f32", mass=0.05),
        # the workload: mixed-precision solve of the 20^3x64 system
        dict(name="solve_f32_20x20x20x64", op="solve", prec="f32", recon=12, lo="f32", mass=0.01, **big),
        # the batched workload: 8 right-hand sides on 20^3x64 and 8 each on three smaller lattices
        dict(name="batch_32_systems", op="batch", each=8, prec="f32", recon=12, lo="f32", mass=0.01, sizes=4, **big),
    ]


def _even(v, lo=4):
    return max(lo, 2 * int(round(v / 2)))


def _dims(rng, vmin, vmax):
    """Four even extents whose product lies roughly log-uniformly between vmin and vmax, t the longest as a rule."""
    v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
    s = (v / rng.choice((1, 2, 3))) ** 0.25
    x, y, z = (_even(s * rng.uniform(0.75, 1.25)) for _ in range(3))
    t = _even(v / (x * y * z))
    while x * y * z * t > vmax and t > 4:
        t -= 2
    return dict(X=x, Y=y, Z=z, T=t, bc_t=rng.randrange(2))


# (vector precision, link precision, recon) in use by the operator and the solver
OPERATOR_STORAGE = (("f32", "f32", 12), ("f32", "f32", 12), ("f32", "f32", 18), ("f32", "f32", 8), ("f32", "i16", 12),
                    ("f32", "f16", 18), ("f64", "f64", 18), ("bf16", "bf16", 12))
SOLVE_STORAGE = (("f32", "f32", 12), ("f32", "f32", 12), ("f32", "f32", 18), ("f32", "f32", 8), ("f32", "i16", 12),
                 ("f64", "f64", 18), ("f16", "f16", 12), ("bf16", "bf16", 12))


def draw(rng):
    op = rng.choice(("dslash", "dslash", "pack", "halo", "hyp", "npr_fused", "npr_stored", "force", "grad", "solve",
                     "solve", "solve", "batch", "full"))
    if op == "dslash":
        prec, lo, recon = rng.choice(OPERATOR_STORAGE)
        return dict(op=op, prec=prec, lo=lo, recon=recon, **_dims(rng, 2048, 2200000))
    if op == "pack":
        lo, recon = rng.choice((("f32", 12), ("f32", 18), ("f64", 18)))
        return dict(op=op, lo=lo, recon=recon, **_dims(rng, 4096, 1100000))
    if op == "halo":
        c = dict(op=op, prec="f32", lo="f32", recon=rng.choice((12, 18)), **_dims(rng, 8192, 260000))
        return dict(c, bc_t=0)
    if op == "hyp":
        return dict(op=op, **dict(_dims(rng, 4096, 520000), bc_t=0))
    if op in ("npr_fused", "npr_stored"):
        return dict(op=op, sets=rng.choice((1, 2, 3, 4, 5, 8)), **dict(_dims(rng, 4096, 520000), bc_t=0))
    if op == "force":
        return dict(op=op, **_dims(rng, 4096, 520000))
    mass = round(math.exp(rng.uniform(math.log(0.05), math.log(0.2))), 4)
    if op == "grad":
        return dict(op=op, prec="f32", lo="f32", recon=rng.choice((12, 18)), mass=mass, **_dims(rng, 4096, 135000))
    if op == "full":
        return dict(op=op, prec="f32", lo="f32", recon=12, mass=mass, **_dims(rng, 4096, 260000))
    if op == "batch":
        return dict(op=op, each=rng.choice((3, 4, 6)), sizes=1, prec="f32", lo="f32", recon=rng.choice((12, 18)),
                    mass=mass, **_dims(rng, 4096, 135000))
    prec, lo, recon = rng.choice(SOLVE_STORAGE)
    if prec == "f32" and lo == "f32" and rng.random() < 0.5:
        mass = 0.01
    return dict(op=op, prec=prec, lo=lo, recon=recon, mass=mass,
                **_dims(rng, 2048, 1000000 if prec == "f32" and lo == "f32" else 260000))


# ---------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------
_tuned = []


def _load_tuned():
    """The committed launch table, loaded once per process as a job does at its start."""
    if not _tuned:
        path = os.path.join(os.path.dirname(os.path.abspath(sp.__file__)), "tune_mi355x.json")
        if os.path.exists(path):
            sp.tune_load(path)
        _tuned.append(True)


def _shape(case):
    return (case["X"], case["Y"], case["Z"], case["T"])


def _volume(case):
    return case["X"] * case["Y"] * case["Z"] * case["T"]


def _gen(seed, stream=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (stream + 1) + seed)
    return g


def _mul3(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _su3(n, gen):
    """n near-identity SU(3) matrices: 1 + i e H - e^2 H^2 / 2 with H Gaussian in the Gell-Mann basis, then rows 0
    and 1 orthonormalised and row 2 = conj(row0 x row1)."""
    h = torch.randn(n, 8, generator=gen, device=DEV, dtype=torch.float64) * 0.5
    m = torch.zeros(n, 3, 3, dtype=torch.complex128, device=DEV)
    r3 = 1.0 / math.sqrt(3.0)
    m[:, 0, 0] = (h[:, 2] + r3 * h[:, 7]).to(m.dtype)
    m[:, 1, 1] = (r3 * h[:, 7] - h[:, 2]).to(m.dtype)
    m[:, 2, 2] = (-2 * r3 * h[:, 7]).to(m.dtype)
    for (i, j), a, b in (((0, 1), 0, 1), ((0, 2), 3, 4), ((1, 2), 5, 6)):
        m[:, i, j] = torch.complex(h[:, a], -h[:, b])
        m[:, j, i] = torch.complex(h[:, a], h[:, b])
    u = 1j * EPS * m - 0.5 * EPS * EPS * _mul3(m, m)
    r0 = u[:, 0] + torch.tensor([1.0, 0.0, 0.0], device=DEV)
    r1 = u[:, 1] + torch.tensor([0.0, 1.0, 0.0], device=DEV)
    r0 = r0 / r0.abs().square().sum(-1, keepdim=True).sqrt()
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=1)


def _links(V, gen):
    out = torch.empty(4, V, 3, 3, dtype=torch.complex128, device=DEV)
    for mu in range(4):
        for s in range(0, V, 1 << 19):
            n = min(1 << 19, V - s)
            out[mu, s:s + n] = _su3(n, gen)
    return out


def _gauss(gen, *shape):
    re = torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float64)
    im = torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float64)
    return torch.complex(re, im) / math.sqrt(2.0)


def _sets(case, seed):
    gen = _gen(seed, 3)
    V, n = _volume(case), case["sets"]
    return [_gauss(gen, n, V, 3) for _ in range(4)]


LABELS = ((15, 15, 15, 15), (6, 0, 9, 3))


def _batch_parts(case):
    """(extents, systems, mass range) of each gauge field of a batch: the case's own lattice, then, in the workload,
    the three smaller ones with masses spread over [0.01, 0.1]."""
    parts = [(_shape(case), case["each"], (case["mass"], case["mass"]))]
    if case["sizes"] == 4:
        parts += [(d, case["each"], (0.01, 0.1)) for d in ((8, 8, 8, 8), (12, 12, 12, 24), (16, 16, 16, 32))]
    return parts


def _batch_inputs(case, seed):
    out = []
    for k, (dims, n, (m0, m1)) in enumerate(_batch_parts(case)):
        V = dims[0] * dims[1] * dims[2] * dims[3]
        gen = _gen(seed, 10 + k)
        U = _links(V, gen)
        bs = [_gauss(gen, V // 2, 3) for _ in range(n)]
        out.append((dims, U, [m0 + (m1 - m0) * j / max(1, n - 1) for j in range(n)], bs))
    return out


def _inputs(case, seed):
    """Links, and the vectors an operation takes, from the seed alone."""
    V, op = _volume(case), case["op"]
    gen = _gen(seed)
    U = _links(V, gen)
    d = dict(U=U)
    if op in ("dslash", "halo", "solve"):
        d["b"] = _gauss(gen, V // 2, 3)
    elif op in ("force", "grad"):
        d["b"], d["c"] = _gauss(gen, V // 2, 3), _gauss(gen, V // 2, 3)
    elif op == "full":
        d["src"] = _gauss(gen, V, 3)
    if op == "halo":
        d["tl"] = _su3(case["X"] * case["Y"] * case["Z"], gen)
    return d


def prepare(case, seed):
    _load_tuned()
    op = case["op"]
    s = dict(op=op, case=case, ws=sp.Workspace())
    if op == "batch":
        s["systems"] = []
        for dims, U, masses, bs in _batch_inputs(case, seed):
            G = sp.Gauge(sp.Lattice(dims, case["bc_t"]), U, lo_prec=case["lo"], recon=case["recon"])
            s["systems"] += [(G, m, b) for m, b in zip(masses, bs)]
        return s
    lat = s["lat"] = sp.Lattice(_shape(case), case["bc_t"])
    d = _inputs(case, seed)
    if op in ("pack", "hyp", "npr_fused", "npr_stored"):
        s["U"] = d["U"]
        if op.startswith("npr"):
            s["f"] = _sets(case, seed)
        return s
    if op == "grad":
        s["U"] = d["U"].requires_grad_(True)
        s["m"] = torch.tensor(case["mass"], dtype=torch.float64, device=DEV, requires_grad=True)
        s["b"] = d["b"].requires_grad_(True)
        s["phi"] = d["c"]
        return s
    if op == "halo":
        # a shard of a lattice eight times as long in t, in its middle
        sh = s["sh"] = sp.Shard(_shape(case), 4 * case["T"], 8 * case["T"], case["bc_t"])
        s["G"] = sp.Gauge(sh.lat, d["U"], lo_prec=case["lo"], recon=case["recon"])
        s["ghost"] = sh.ghost_pack(d["tl"], case["lo"], case["recon"])
        s["ext"] = sh.pack_vec(d["b"], case["prec"])
        s["faces"] = [sh.face_pack(case["prec"], s["ext"], side) for side in (0, 1)]
        s["recv"] = [torch.empty_like(f) for f in s["faces"]]
        s["out"] = torch.empty(sh.lat.vec_bytes(case["prec"]), dtype=torch.uint8, device=DEV)
        return s
    if op == "force":
        s["G"] = sp.Gauge(lat, d["U"], lo_prec="f64")
        s["x"], s["lam"] = d["b"], d["c"]
        return s
    s["G"] = sp.Gauge(lat, d["U"], lo_prec=case["lo"], recon=case["recon"])
    if op == "dslash":
        s["in"] = sp.pack_vec(lat, d["b"], case["prec"])
        s["out"] = torch.empty_like(s["in"])
    elif op == "solve":
        s["b"] = d["b"]
    elif op == "full":
        s["src"] = d["src"]
    return s


PLANE = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


def run(state):
    c, op = state["case"], state["op"]
    if op == "dslash":
        # the even half of D on an odd vector
        return sp.dslash_packed(state["G"], c["prec"], state["in"], 0, out=state["out"]).view(PLANE[c["prec"]])
    if op == "pack":
        G = sp.Gauge(state["lat"], state["U"], lo_prec=c["lo"], recon=c["recon"])
        return dict(f64=G.f64.view(torch.float64), lo=G.lo.view(PLANE[c["lo"]]))
    if op == "halo":
        sh, p = state["sh"], c["prec"]
        for side in (0, 1):
            sh.face_pack(p, state["ext"], side, state["faces"][side])
            state["recv"][side].copy_(state["faces"][side])  # stands in for the transfer to the neighbour
            sh.face_unpack(p, state["recv"][side], 1 - side, state["ext"])
        sh.dslash(state["G"], state["ghost"], p, state["ext"], 1, part=1, out=state["out"])
        return sh.dslash(state["G"], state["ghost"], p, state["ext"], 1, part=2, out=state["out"]).view(PLANE[p])
    if op == "hyp":
        return sp.hyp_smear(state["lat"], state["U"], ALPHA, workspace=state["ws"])
    if op == "npr_fused":
        return sp.npr_contract_links(state["lat"], state["U"], *state["f"], LABELS[0])
    if op == "npr_stored":
        uad = sp.npr_path_links(state["lat"], state["U"])
        return [sp.npr_contract(state["lat"], uad, *state["f"], l) for l in LABELS]
    if op == "force":
        gamma, force, dm = sp.cg_force(state["G"], 0.05, state["x"], state["lam"])
        return dict(gamma=gamma, force=force, dm=dm)
    if op == "solve":
        x, _ = sp.cg_solve(state["G"], c["mass"], state["b"], tol=TOL, inner=c["prec"], workspace=state["ws"])
        return dict(x=x)
    if op == "full":
        psi, _ = sp.full_solve(state["G"], c["mass"], state["src"], tol=TOL, inner=c["prec"])
        return dict(psi=psi)
    if op == "batch":
        xs, _ = sp.cg_solve_batched(state["systems"], tol=TOL, inner=c["prec"], workspace=state["ws"])
        return dict(x=xs)
    # grad: one step of l = Re phi^dag A^-1 b
    for k in ("U", "m", "b"):
        state[k].grad = None
    x = sp.staggered_solve(state["U"], state["m"], state["b"], state["lat"], inner=c["prec"], recon=c["recon"], tol=TOL)
    torch.vdot(state["phi"].flatten(), x.flatten()).real.backward()
    return dict(x=x.detach(), dU=state["U"].grad, dm=state["m"].grad, db=state["b"].grad)


# ---------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------
def _link_bytes(lo, recon):
    return {"f64": 144, "f32": 4 * recon, "f16": 2 * recon, "bf16": 2 * recon, "i16": 2 * recon}[lo]


VEC_BYTES = {"f64": 48, "f32": 24, "f16": 16, "bf16": 12}


def _iterations(mass):
    """CG iterations to TOL on near-identity fields: a fit to 8^4, 12^3x24, 16^3x32 and 20^3x64 solves at masses from
    0.01 (659 to 808) to 0.1 (155 to 201)."""
    return min(800.0, 90.0 + 8.5 / mass)


def _cg_work(Vh, case, nrhs, mass):
    """Per iteration the links once for each half operator, and x, r, p and t read and written once."""
    lb = _link_bytes(case["lo"], case["recon"])
    it = _iterations(mass)
    vb = VEC_BYTES[case["prec"]]
    return it * Vh * (16 * lb + nrhs * 8 * vb), it * 2 * Vh * 606 * nrhs


def work(case):
    op = case["op"]
    V = _volume(case)
    Vh = V // 2
    if op == "dslash":
        return dict(bytes=Vh * (8 * _link_bytes(case["lo"], case["recon"]) + 2 * VEC_BYTES[case["prec"]]), flops=570 * Vh)
    if op == "pack":
        lb = 0 if case["lo"] == "f64" else _link_bytes(case["lo"], case["recon"])
        return dict(bytes=4 * V * (144 + 144 + lb), flops=0)
    if op == "halo":
        F = V // case["T"] // 2
        return dict(bytes=Vh * (8 * _link_bytes(case["lo"], case["recon"]) + 48) + 2 * F * 24 * 6, flops=570 * Vh)
    if op == "hyp":
        # links in and out; 192 products of 198 flop and 28 projections of about 1,000 flop a site
        return dict(bytes=2 * 4 * V * 144, flops=V * (192 * 198 + 28 * 1000))
    if op in ("npr_fused", "npr_stored"):
        nz, n = V // 16, case["sets"]
        if op == "npr_fused":
            return dict(bytes=4 * V * 144 + nz * n * 3088, flops=nz * n * 47616)
        return dict(bytes=4 * V * 144 + nz * 36864 + 2 * nz * n * 3088, flops=2 * nz * n * 47616)
    if op == "force":
        return dict(bytes=3 * 4 * V * 144 + 2 * Vh * 48, flops=V * 4 * 400 + 2 * 570 * Vh)
    if op == "batch":
        b = f = 0.0
        for dims, n, (m0, m1) in _batch_parts(case):
            vh = dims[0] * dims[1] * dims[2] * dims[3] // 2
            bb, ff = _cg_work(vh, case, n, 0.5 * (m0 + m1))
            b, f = b + bb, f + ff
        return dict(bytes=b, flops=f)
    b, f = _cg_work(Vh, case, 1, case["mass"])
    if op == "grad":
        return dict(bytes=2 * b + 4 * V * 144 * 3, flops=2 * f)
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------------------------------------------------
# the same in 64 bits with plain torch
# ---------------------------------------------------------------------------------------------------------
class _Field:
    """The full-lattice operator D on [V][3] vectors, by rolls of [T][Z][Y][X] arrays."""

    def __init__(self, U, dims, bc_t, t_below=None):
        X, Y, Z, T = dims
        self.shape, self.bc_t = (T, Z, Y, X), bc_t
        U = U.detach().reshape(4, T, Z, Y, X, 3, 3)
        ax = torch.arange
        t, z, y, x = (ax(n, device=DEV).reshape([-1 if k == j else 1 for k in range(4)])
                      for j, n in enumerate(self.shape))
        par = torch.zeros(self.shape, dtype=torch.int64, device=DEV)
        self.parity = ((par + x + y + z + t) & 1).reshape(-1)
        eta = [par, par + x, par + x + y, par + x + y + z]
        self.eta = [(1.0 - 2.0 * (e & 1).to(torch.float64)).reshape(T, Z, Y, X) for e in eta]
        self.U, self.B = [], []
        for mu in range(4):
            u = U[mu] * self.eta[mu][..., None, None]
            if mu == 3 and bc_t:
                u = u.clone()
                u[-1] = -u[-1]
            b = torch.roll(u, 1, 3 - mu)
            if mu == 3 and t_below is not None:
                b = b.clone()
                b[0] = t_below.reshape(Z, Y, X, 3, 3) * self.eta[3][-1][..., None, None]
            self.U.append(u)
            self.B.append(b.conj().transpose(-1, -2).contiguous())

    def D(self, v):
        v = v.reshape(*self.shape, 3)
        acc = torch.zeros_like(v)
        for mu in range(4):
            acc += (self.U[mu] * torch.roll(v, -1, 3 - mu)[..., None, :]).sum(-1)
            acc -= (self.B[mu] * torch.roll(v, 1, 3 - mu)[..., None, :]).sum(-1)
        return (0.5 * acc).reshape(-1, 3)

    def spread(self, h, p):
        """Half vector of parity p -> full vector, zero on the other parity."""
        full = torch.zeros(h.shape[0], 2, 3, dtype=h.dtype, device=DEV)
        q = self.parity.reshape(-1, 2)
        full[torch.arange(h.shape[0], device=DEV), (q[:, 1] == p).long()] = h
        return full.reshape(-1, 3)

    def half(self, v, p):
        return v[self.parity == p]

    def solve(self, mass, b):
        """A x = b on even sites by CG, to rounding."""
        A = lambda w: mass * mass * w - self.half(self.D(self.D(self.spread(w, 0))), 0)  # noqa: E731
        x, r = torch.zeros_like(b), b.clone()
        for _ in range(3):
            r = b - A(x)
            p, rr = r.clone(), float(r.abs().square().sum())
            stop = max(rr * 1e-20, float(b.abs().square().sum()) * 1e-29)
            for _ in range(4000):
                if rr <= stop:
                    break
                q = A(p)
                a = rr / float((p.conj() * q).sum().real)
                x, r = x + a * p, r - a * q
                new = float(r.abs().square().sum())
                p, rr = r + (new / rr) * p, new
        return x


def _planes(v, prec):
    """[n][3] complex -> the packed vector's planes, flat and in 64 bits."""
    r = torch.view_as_real(v)
    if prec == "f64":
        return r.permute(1, 0, 2).reshape(-1)
    return torch.cat([r[:, :2].reshape(-1), r[:, 2].reshape(-1)])


def _link_planes(U, dims, lo, recon):
    """Natural links -> packed planes, [parity][direction] blocks of Vh sites."""
    X, Y, Z, T = dims
    V = X * Y * Z * T
    lex = torch.arange(V, device=DEV)
    par = (lex % X + lex // X % Y + lex // (X * Y) % Z + lex // (X * Y * Z)) & 1
    out = []
    for q in (0, 1):
        for mu in range(4):
            m = torch.view_as_real(U[mu][par == q]).reshape(V // 2, 18)
            w = 2 if lo == "f64" else 4
            for k in range(0, recon, w):
                out.append(m[:, k:min(k + w, recon)].reshape(-1))
    return torch.cat(out)


def _gradient(F, U, mass, x, lam):
    """dl/dU, su(3) force and dl/dm of sp_cg_force, from x and lambda on even sites."""
    xe, le = F.spread(x, 0), F.spread(lam, 0)
    yx, yl = F.D(xe), F.D(le)
    even = (F.parity == 0).reshape(-1, 1, 1)
    gamma = []
    for mu in range(4):
        nxt = lambda v: torch.roll(v.reshape(*F.shape, 3), -1, 3 - mu).reshape(-1, 3)  # noqa: E731
        out = lambda a, b: a[:, :, None] * b.conj()[:, None, :]  # noqa: E731
        ge = out(le, nxt(yx)) + out(xe, nxt(yl))
        go = -(out(yx, nxt(le)) + out(yl, nxt(xe)))
        sign = F.eta[mu].clone()
        if mu == 3 and F.bc_t:
            sign[-1] = -sign[-1]
        gamma.append(0.5 * sign.reshape(-1, 1, 1) * torch.where(even, ge, go))
    gamma = torch.stack(gamma)
    w = _mul3(U.detach(), gamma.conj().transpose(-1, -2))
    w = 0.5 * (w - w.conj().transpose(-1, -2))
    tr = w.diagonal(dim1=-2, dim2=-1).sum(-1) / 3.0
    force = w - tr[..., None, None] * torch.eye(3, device=DEV, dtype=w.dtype)
    return gamma, force, -2.0 * mass * float((lam.conj() * x).sum().real)


def _project(w):
    """argmax Re tr(X^dag W) over SU(3) from the singular values: X = P diag(e^{i theta}) Q^dag with
    s_k sin theta_k = mu and sum theta_k = -arg det(P Q^dag)."""
    shape = w.shape
    p, s, qh = torch.linalg.svd(w.reshape(-1, 3, 3).cpu())
    phi = torch.angle(torch.linalg.det(p @ qh))
    mu = -phi / (1.0 / s).sum(-1)
    for _ in range(30):
        a = (mu[:, None] / s).clamp(-0.999999, 0.999999)
        mu = mu - (torch.asin(a).sum(-1) + phi) / (1.0 / (s * (1 - a * a).sqrt())).sum(-1)
    th = torch.asin((mu[:, None] / s).clamp(-1, 1))
    return ((p * torch.exp(1j * th)[:, None, :]) @ qh).to(DEV).reshape(shape)


def _hyp(U, dims):
    X, Y, Z, T = dims
    U = U.reshape(4, T, Z, Y, X, 3, 3)
    a1, a2, a3 = ALPHA
    dag = lambda m: m.conj().transpose(-1, -2)  # noqa: E731
    sh = lambda m, mu, d: torch.roll(m, -d, 3 - mu)  # noqa: E731

    def staples(S, Tp, mu, eta):
        up = _mul3(_mul3(S, sh(Tp, eta, 1)), dag(sh(S, mu, 1)))
        dn = _mul3(_mul3(dag(S), Tp), sh(S, mu, 1))
        return up + sh(dn, eta, -1)

    l1 = {(m, e): _project((1 - a3) * U[m] + a3 / 2 * staples(U[e], U[m], m, e))
          for m in range(4) for e in range(4) if e != m}
    l2 = {}
    for m in range(4):
        for n in range(4):
            if n != m:
                w = (1 - a2) * U[m]
                for r in set(range(4)) - {m, n}:
                    w = w + a2 / 4 * staples(l1[r, 6 - m - n - r], l1[m, 6 - m - n - r], m, r)
                l2[m, n] = _project(w)
    out = [_project((1 - a1) * U[m] + a1 / 6 * sum(staples(l2[n, m], l2[m, n], m, n) for n in range(4) if n != m))
           for m in range(4)]
    return torch.stack(out).reshape(4, -1, 3, 3)


def _npr_paths(U, dims):
    """U_AD of every hypercube, keyed by the corner pair, by the average over first steps."""
    X, Y, Z, T = dims
    U = U.reshape(4, T // 2, 2, Z // 2, 2, Y // 2, 2, X // 2, 2, 3, 3)

    def link(mu, A):
        b = [(A >> k) & 1 for k in range(4)]
        return U[mu, :, b[3], :, b[2], :, b[1], :, b[0]].reshape(-1, 3, 3)

    nz = X * Y * Z * T // 16
    P = {(A, A): torch.eye(3, dtype=U.dtype, device=DEV).expand(nz, 3, 3) for A in range(16)}
    for k in range(1, 5):
        for A in range(16):
            for D in range(16):
                steps = [m for m in range(4) if (A ^ D) >> m & 1]
                if len(steps) != k:
                    continue
                acc = 0
                for m in steps:
                    A1 = A ^ (1 << m)
                    L = link(m, A) if A1 > A else link(m, A1).conj().transpose(-1, -2)
                    acc = acc + (L if k == 1 else _mul3(L, P[A1, D]))
                P[A, D] = acc / k
    return P


def _gammas():
    s = [torch.tensor(m, dtype=torch.complex128) for m in ([[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]])]
    one = torch.eye(2, dtype=torch.complex128)
    g = [torch.kron(s[1], m) for m in s] + [torch.kron(s[0], one)]
    out = []
    for A in range(16):
        m = torch.eye(4, dtype=torch.complex128)
        for k in range(4):
            if A >> k & 1:
                m = m @ g[k]
        out.append(m)
    return out


def _npr(P, f, dims, labels):
    X, Y, Z, T = dims
    g = _gammas()
    M = [[[(torch.trace(g[A].conj().T @ g[S] @ g[B] @ g[F].conj().T) / 4).real.item() for B in range(16)]
          for A in range(16)] for S, F in (labels[:2], labels[2:])]

    def corner(v, A):
        b = [(A >> k) & 1 for k in range(4)]
        v = v.reshape(v.shape[0], T // 2, 2, Z // 2, 2, Y // 2, 2, X // 2, 2, 3)
        return v[:, :, b[3], :, b[2], :, b[1], :, b[0]].reshape(v.shape[0], -1, 3)

    c = [[corner(v, A) for A in range(16)] for v in f]
    bil = lambda i, A, j, D: (c[i][A] * (P[A, D] * c[j][D][..., None, :]).sum(-1)).sum(-1)  # noqa: E731
    out = 0
    for A in range(16):
        for B in range(16):
            if M[0][A][B]:
                for C in range(16):
                    for D in range(16):
                        if M[1][C][D]:
                            out = out + M[0][A][B] * M[1][C][D] * bil(0, A, 3, D) * bil(2, C, 1, B)
    return out


def exact(case, seed):
    op, dims, V = case["op"], _shape(case), _volume(case)
    if op == "batch" or (op == "hyp" and V > 20000) or (op == "pack" and case["recon"] == 8):
        return None
    d = _inputs(case, seed)
    U = d["U"]
    if op == "pack":
        return dict(f64=_link_planes(U, dims, "f64", 18), lo=_link_planes(U, dims, case["lo"], case["recon"]))
    if op == "hyp":
        return _hyp(U, dims)
    if op.startswith("npr"):
        P, f = _npr_paths(U, dims), _sets(case, seed)
        return _npr(P, f, dims, LABELS[0]) if op == "npr_fused" else [_npr(P, f, dims, l) for l in LABELS]
    F = _Field(U, dims, case["bc_t"], d.get("tl"))
    if op == "dslash":
        return _planes(F.half(F.D(F.spread(d["b"], 1)), 0), case["prec"])
    if op == "halo":
        return _planes(F.half(F.D(F.spread(d["b"], 0)), 1), case["prec"])
    if op == "force":
        gamma, force, dm = _gradient(F, U, 0.05, d["b"], d["c"])
        return dict(gamma=gamma, force=force, dm=torch.tensor(dm, dtype=torch.float64))
    m = case["mass"]
    if op == "solve":
        return dict(x=F.solve(m, d["b"]))
    if op == "full":
        src = d["src"]
        se, so = F.spread(F.half(src, 0), 0), F.spread(F.half(src, 1), 1)
        pe = F.spread(F.solve(m, F.half(m * se - F.D(so), 0)), 0)
        return dict(psi=pe + (so - F.D(pe)) / m)
    x, lam = F.solve(m, d["b"]), F.solve(m, d["c"])
    gamma, _, dm = _gradient(F, U, m, x, lam)
    return dict(x=x, dU=gamma, dm=torch.tensor(dm, dtype=torch.float64), db=lam)
