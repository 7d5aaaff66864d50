"""The C-ABI library loads on a machine without a GPU and exports every function include/sp_api.h
declares; host-side queries that launch nothing behave as documented."""
import ctypes
import os
import re

import pytest

import paper_1511_00088_amd as sp
from paper_1511_00088_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    txt = open(os.path.join(ROOT, "include", "sp_api.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(sp_[a-z_0-9]+)\s*\(", txt)))


def test_library_exports_every_declared_symbol():
    lib = _lib.load()
    names = _declared()
    assert len(names) >= 18
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(_lib.SIGNATURES), set(names) ^ set(_lib.SIGNATURES)


def test_host_queries():
    lib = _lib.load()
    assert lib.sp_version() == 10000
    assert lib.sp_strerror(-6) == b"CG breakdown"
    lat = sp.Lattice((20, 20, 20, 64))
    assert lat.vec_bytes("f32") == 256000 * 24
    assert lat.vec_bytes("f16") == 256000 * 16
    assert lat.vec_bytes("bf16") == 256000 * 12
    assert lat.vec_bytes("f64") == 256000 * 48
    assert lat.gauge_bytes("f32", 18) == 4 * 512000 * 72
    assert lat.gauge_bytes("f32", 12) == 4 * 512000 * 48
    assert lat.gauge_bytes("f16", 12) == 4 * 512000 * 24
    assert lat.gauge_bytes("f64", 12) == 0  # not supported
    assert lat.gauge_bytes("i16", 12) == 4 * 512000 * 24  # 16-bit fixed-point links
    assert lat.gauge_bytes("i16", 18) == 4 * 512000 * 36
    assert lat.vec_bytes("i16") == 0  # links only: no vector storage of that kind
    assert sp.Lattice((4, 4, 5, 4)).vec_bytes("f32") == 0  # odd extent
    assert sp.Lattice((256, 256, 256, 2)).vec_bytes("f32") == 0  # V/2 >= 2^24


def test_workspace_query_and_validation():
    lib = _lib.load()
    lat = sp.Lattice((8, 8, 8, 8))
    g = _lib.sp_gauge(1, 2, _lib.SP_F32, 18)
    s = _lib.sp_system(ctypes.pointer(lat.geom), ctypes.pointer(g), 0.1, 3, 4)
    prm = _lib.sp_cg_params(1e-8, 100, _lib.SP_F32, 0.1, 0, 50, 0, 1)
    n1 = lib.sp_cg_workspace_bytes(1, ctypes.byref(s), ctypes.byref(prm))
    assert n1 > 2048 * (3 * 48 + 24 + 3 * 24)
    arr = (_lib.sp_system * 3)(s, s, s)
    n3 = lib.sp_cg_workspace_bytes(3, arr, ctypes.byref(prm))
    assert 3 * (n1 - 100000) < n3 < 3 * n1 + 100000
    bad = _lib.sp_cg_params(1e-8, 100, 7, 0.1, 0, 50, 0, 1)
    assert lib.sp_cg_workspace_bytes(1, ctypes.byref(s), ctypes.byref(bad)) == 0
    # argument errors are reported before anything is launched
    st = _lib.sp_cg_stats()
    rc = lib.sp_cg_solve(ctypes.byref(lat.geom), ctypes.byref(g), 0.1, 3, 4, ctypes.byref(prm), ctypes.byref(st),
                         None, 0, None)
    assert rc == _lib.SP_ERR_WORKSPACE
    assert b"workspace" in lib.sp_last_error()
    neg = _lib.sp_cg_params(-1.0, 100, _lib.SP_F32, 0.1, 0, 50, 0, 1)
    rc = lib.sp_cg_solve(ctypes.byref(lat.geom), ctypes.byref(g), 0.1, 3, 4, ctypes.byref(neg), ctypes.byref(st),
                         None, 0, None)
    assert rc == _lib.SP_ERR_INVALID_ARG


def test_hyp_workspace_and_validation():
    # every check below fails before any device memory is touched, so fake pointers are safe
    lib = _lib.load()
    lat = sp.Lattice((20, 20, 20, 64))
    n = lib.sp_hyp_workspace_bytes(ctypes.byref(lat.geom))
    assert n == 24 * 512000 * 144
    odd = _lib.sp_geom((ctypes.c_int32 * 4)(4, 4, 3, 4), 0)
    assert lib.sp_hyp_workspace_bytes(ctypes.byref(odd)) == 0
    a = (ctypes.c_double * 3)(0.75, 0.6, 0.3)
    bad = (ctypes.c_double * 3)(0.75, -0.1, 0.3)
    L, O = 1 << 20, 1 << 40  # links and output far apart
    field = 4 * 512000 * 144
    g = ctypes.byref(lat.geom)
    assert lib.sp_hyp_smear(g, L, bad, O, 1 << 44, n, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_hyp_smear(g, None, a, O, 1 << 44, n, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_hyp_smear(g, L, a, L + field // 2, 1 << 44, n, None) == _lib.SP_ERR_INVALID_ARG  # overlap
    assert lib.sp_hyp_smear(g, L, a, O, 1 << 44, n - 16, None) == _lib.SP_ERR_WORKSPACE
    assert lib.sp_hyp_smear(g, L, a, O, None, n, None) == _lib.SP_ERR_WORKSPACE
    assert lib.sp_hyp_smear(ctypes.byref(odd), L, a, O, 1 << 44, n, None) == _lib.SP_ERR_ODD_EXTENT


def test_npr_sizes_and_validation():
    lib = _lib.load()
    lat = sp.Lattice((20, 20, 20, 64))
    assert lib.sp_npr_path_bytes(ctypes.byref(lat.geom)) == 32000 * 256 * 144
    g = ctypes.byref(lat.geom)
    ok = (ctypes.c_int32 * 4)(15, 15, 15, 15)
    bad = (ctypes.c_int32 * 4)(15, 16, 15, 15)
    F = 1 << 30  # never touched: every call below fails its checks first
    assert lib.sp_npr_contract(g, F, 1, F, F, F, F, bad, F, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_npr_contract(g, F, 0, F, F, F, F, ok, F, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_npr_contract(g, None, 1, F, F, F, F, ok, F, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_npr_path_links(g, None, F, None) == _lib.SP_ERR_INVALID_ARG


def test_geometry_limits_and_degenerate_calls():
    # all of these fail in the host-side checks, before any device memory is touched
    lib = _lib.load()
    geom = lambda d, bc=0: _lib.sp_geom((ctypes.c_int32 * 4)(*d), bc)  # noqa: E731
    for d in ((3, 4, 4, 4), (4, 4, 4, 0), (4, 4, 4, 1), (4, -2, 4, 4)):
        assert lib.sp_vec_bytes(ctypes.byref(geom(d)), _lib.SP_F32) == 0
    # the largest lattice the checkerboard index division supports is V/2 < 2^24
    big = geom((256, 256, 256, 2))  # V/2 = 2^24
    assert lib.sp_vec_bytes(ctypes.byref(big), _lib.SP_F32) == 0
    ok = geom((256, 256, 254, 2))
    assert lib.sp_vec_bytes(ctypes.byref(ok), _lib.SP_F32) == 256 * 256 * 254 * 24
    assert lib.sp_vec_bytes(ctypes.byref(geom((4, 4, 4, 4), 2)), _lib.SP_F32) == 0  # bc_t must be 0 or 1
    F = 1 << 30
    g = geom((4, 4, 4, 4))
    assert lib.sp_dslash(ctypes.byref(g), None, _lib.SP_F32, F, F + 4096, 1, None) == _lib.SP_ERR_INVALID_ARG
    gauge = _lib.sp_gauge(F, F, _lib.SP_F32, 18)
    assert lib.sp_dslash(ctypes.byref(g), ctypes.byref(gauge), _lib.SP_F32, F, F, 1, None) == _lib.SP_ERR_INVALID_ARG
    assert lib.sp_dslash(ctypes.byref(g), ctypes.byref(gauge), _lib.SP_F32, F, F + 4096, 2, None) == _lib.SP_ERR_INVALID_ARG
    prm = _lib.sp_cg_params(1e-8, 100, _lib.SP_F32, 0.1, 0, 25, 0, 1)
    st = _lib.sp_cg_stats()
    assert lib.sp_cg_solve_batched(0, None, ctypes.byref(prm), ctypes.byref(st), F, 1 << 30, None) < 0
    for bad in (_lib.sp_cg_params(0.0, 100, _lib.SP_F32, 0.1, 0, 25, 0, 1),
                _lib.sp_cg_params(1e-8, 0, _lib.SP_F32, 0.1, 0, 25, 0, 1),
                _lib.sp_cg_params(1e-8, 100, _lib.SP_F32, 1.5, 0, 25, 0, 1)):
        rc = lib.sp_cg_solve(ctypes.byref(g), ctypes.byref(gauge), 0.1, F, F + 4096, ctypes.byref(bad),
                             ctypes.byref(st), F + 8192, 1 << 30, None)
        assert rc == _lib.SP_ERR_INVALID_ARG, rc
    assert lib.sp_full_solve(ctypes.byref(g), ctypes.byref(gauge), 0.0, F, F + 4096, ctypes.byref(prm),
                             ctypes.byref(st), F + 8192, 1 << 30, None) == _lib.SP_ERR_INVALID_ARG


def test_tune_cache_roundtrip(tmp_path):
    lib = _lib.load()
    p = tmp_path / "tune.json"
    # the second entry has the form tables took before the link-load policy ("stream") existed: cached loads
    p.write_text('{\n  "20x20x20x64/l1/r18/v1": {"nt": 128, "remap": 1, "stream": 1},\n'
                 '  "20x20x20x64/l1/r18/v1/n4": {"nt": 256, "remap": 0},\n'
                 '  "20x20x20x64/l1/r18/v1/solve": {"nt": 256, "remap": 1, "stream": 1}\n}\n')
    assert lib.sp_tune_load(str(p).encode()) == 0
    q = tmp_path / "out.json"
    assert lib.sp_tune_save(str(q).encode()) == 0
    assert '"20x20x20x64/l1/r18/v1": {"nt": 128, "remap": 1, "stream": 1}' in q.read_text()
    assert '"20x20x20x64/l1/r18/v1/n4": {"nt": 256, "remap": 0, "stream": 0}' in q.read_text()
    assert '"20x20x20x64/l1/r18/v1/solve": {"nt": 256, "remap": 1, "stream": 1}' in q.read_text()
    p.write_text('{"x": {"nt": 128, "remap": 1, "strem": 1}}')
    assert lib.sp_tune_load(str(p).encode()) == _lib.SP_ERR_INVALID_ARG
    p.write_text('{"x": {"nt": 100, "remap": 1}}')
    assert lib.sp_tune_load(str(p).encode()) == _lib.SP_ERR_INVALID_ARG
    lib.sp_release_cache()


def test_shipped_tune_table_loads_and_covers_the_workloads():
    """The committed MI355X table passes the strict reader and holds, for the benchmark's lattices, the plain
    operator's entry, the batched operator's ("/n4") and the single solve's ("/solve", timed on solves)."""
    import json
    import os

    lib = _lib.load()
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1511_00088_amd",
                        "tune_mi355x.json")
    assert lib.sp_tune_load(path.encode()) == 0
    with open(path) as f:
        table = json.load(f)
    for key in ("20x20x20x64/l1/r12/v1", "20x20x20x64/l1/r12/v1/n4", "20x20x20x64/l1/r12/v1/solve",
                "20x20x20x64/l4/r12/v1/solve", "20x20x20x64/l0/r18/v0/solve", "32x32x32x64/l1/r12/v1/solve",
                "28x28x28x96/l1/r12/v1/solve", "20x20x20x64/l1/r8/v1", "20x20x20x64/l1/r8/v1/solve",
                "32x32x32x64/l1/r8/v1/solve"):
        assert key in table, key
        assert table[key]["nt"] in (64, 128, 256) and table[key]["remap"] in (0, 1)
        assert table[key].get("stream", 0) in (0, 1)
    lib.sp_release_cache()


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(_lib, "_lib", None)
    monkeypatch.setattr(_lib, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError, match="missing"):
        _lib.load()


def test_packed_buffers_checked_before_any_call():
    # a packed buffer reaches the library as a bare pointer, so the binding refuses what is not one
    import torch

    lat = sp.Lattice((4, 4, 4, 4))
    with pytest.raises(TypeError):
        sp.unpack_vec(lat, torch.zeros(4096, dtype=torch.uint8), "f32")
    with pytest.raises(TypeError):
        sp.unpack_vec(lat, torch.zeros(16, dtype=torch.float32), "f32")


def test_roofline_bytes_match_the_packed_layout():
    # the benchmark's algorithmic bytes per site come from per-link and per-vector sizes: they must be what
    # the library actually packs (host queries only), and the flop count is that of 8 complex 3x3 mat-vecs
    # (9 complex products, 6 complex sums) and 7 colour-vector sums
    import bench

    lat = sp.Lattice((4, 4, 4, 8))
    for (prec, recon), per_link in bench.LINK_BYTES.items():
        assert lat.gauge_bytes(prec, recon) == 4 * lat.V * per_link
    for prec, per_site in bench.VEC_BYTES.items():
        assert lat.vec_bytes(prec) == lat.Vh * per_site
    assert bench.FLOP_PER_SITE == 8 * (9 * 6 + 6 * 2) + 7 * 6
    assert bench.dslash_bytes_per_site("f32", 12) == 432
    assert bench.iteration_bytes_per_site("f32", 12) == 1032
    assert bench.iteration_bytes_per_site("f32", 12, "i16") == 648  # 16-bit links, FP32 vectors


def test_tune_load_rejects_truncated_and_partial_files(tmp_path):
    # an entry cut off before its closing brace once sent the reader back to the start of the file for
    # ever: run it in a child process with a time limit, then check that a file whose second entry is bad
    # changes nothing (the first entry is not applied)
    import subprocess
    import sys

    trunc = tmp_path / "trunc.json"
    trunc.write_text('{\n  "8x8x8x8/l1/r12/v1": {"nt": 128, "remap": 1')
    code = ("import sys; sys.path.insert(0, %r); from paper_1511_00088_amd import _lib; "
            "print(_lib.load().sp_tune_load(%r.encode()))" % (ROOT, str(trunc)))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and int(r.stdout.split()[-1]) == _lib.SP_ERR_INVALID_ARG

    lib = _lib.load()
    lib.sp_release_cache()
    part = tmp_path / "part.json"
    part.write_text('{\n  "6x6x6x6/l1/r12/v1": {"nt": 64, "remap": 1},\n  "6x6x6x6/l1/r18/v1": {"nt": 96, "remap": 0}\n}\n')
    assert lib.sp_tune_load(str(part).encode()) == _lib.SP_ERR_INVALID_ARG
    out = tmp_path / "out.json"
    assert lib.sp_tune_save(str(out).encode()) == 0
    assert "6x6x6x6" not in out.read_text()
    lib.sp_release_cache()


def test_product_package_never_reaches_the_oracle():
    # the oracle is test infrastructure: no source of the package (Python, HIP, headers, build) names it,
    # and importing the package does not load it
    import subprocess
    import sys

    pkg = os.path.join(ROOT, "paper_1511_00088_amd")
    for dirpath, _, files in os.walk(pkg):
        for name in files:
            if name.endswith((".py", ".hip", ".h", ".json")):
                with open(os.path.join(dirpath, name), encoding="utf-8") as fh:
                    assert "oracle" not in fh.read(), os.path.join(dirpath, name)
    code = "import sys; sys.path.insert(0, %r); import paper_1511_00088_amd; print('oracle' in sys.modules)" % ROOT
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.split()[-1] == "False"


def test_noalloc_force_refuses_lattices_beyond_its_array():
    # 28^3x96 needs 4 FP64 half vectors of 1,053,696 sites (202 MB) of scratch: refused before any launch, so
    # the placeholder pointers below are never touched
    lib = _lib.load()
    lat = sp.Lattice((28, 28, 28, 96))
    need = lib.sp_force_workspace_bytes(ctypes.byref(lat.geom))
    assert need > _lib.NOALLOC_SCRATCH_BYTES
    g = _lib.sp_gauge(256, 256, _lib.SP_F64, 18)
    rc = lib.sp_cg_force_noalloc(ctypes.byref(lat.geom), ctypes.byref(g), 0.1, ctypes.c_void_p(256),
                                 ctypes.c_void_p(256), ctypes.c_void_p(256), None, None, None)
    assert rc == _lib.SP_ERR_WORKSPACE
    assert str(need).encode() in lib.sp_last_error()
    # the 20^3x64 workload and the 16^3x32 gradient lattice fit
    for dims in ((20, 20, 20, 64), (16, 16, 16, 32)):
        assert lib.sp_force_workspace_bytes(ctypes.byref(sp.Lattice(dims).geom)) <= _lib.NOALLOC_SCRATCH_BYTES
    # null arguments are refused as by sp_cg_force
    small = sp.Lattice((4, 4, 4, 4))
    assert lib.sp_cg_force_noalloc(ctypes.byref(small.geom), None, 0.1, None, None, None, None, None,
                                   None) == _lib.SP_ERR_INVALID_ARG


@pytest.mark.parametrize("one_field", [True, False])
def test_batch_layout_grows_with_the_number_of_systems(one_field):
    """The layout of a batch (the workspace query's work, and each solve's) takes time in proportion to its systems, not
    to their square: four times the systems in less than eight times the time, best of five."""
    import time

    lib = _lib.load()
    lat = sp.Lattice((2, 2, 2, 2))
    prm = _lib.sp_cg_params(1e-8, 1000, _lib.SP_F32, 0.1, 0, 0, 0, 1)

    def query(n):
        fields = [_lib.sp_gauge(0x10000 + 0x1000 * k, 0x90000000 + 0x1000 * k, _lib.SP_F32, 12)
                  for k in range(1 if one_field else n)]
        arr = (_lib.sp_system * n)()
        for k in range(n):
            arr[k] = _lib.sp_system(ctypes.pointer(lat.geom), ctypes.pointer(fields[k % len(fields)]), 0.1, 0x1000, 0x2000)
        best = float("inf")
        for _ in range(5):
            t0 = time.perf_counter()
            assert lib.sp_cg_workspace_bytes(n, arr, ctypes.byref(prm)) > 0
            best = min(best, time.perf_counter() - t0)
        return best

    assert query(16000) < 8 * query(4000)
