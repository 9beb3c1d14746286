"""Tile heights and split tails of purifications on digit slices: S below 6 and
above 8, and S = 6, 7, 8 in the least workspace.  The plans are checked on the
host, so that a case that no longer takes the path it is here for fails."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2407_13299_amd import _lib
from paper_2407_13299_amd.workloads import spectrum_hamiltonian, tight_binding_hamiltonian

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2407_13299_amd", "csrc")
KIND, METHOD = {"int8": 1, "fp16": 2}, {"canonical": 0, "trs4": 1}
CUS = 256
STEPS = 6

HEIGHTS = [("int8", 5), ("int8", 7), ("fp16", 6), ("int8", 8)]
# more tiles than run at once (two workgroups a CU of 64 rows, one of 128), so
# that the last round is split
TAILS = [("canonical", "int8", 5, 2048), ("trs4", "int8", 5, 2048), ("canonical", "int8", 7, 2048),
         ("trs4", "int8", 7, 2048), ("canonical", "fp16", 7, 2100), ("canonical", "int8", 8, 2048),
         ("canonical", "int8", 9, 2048), ("trs4", "int8", 9, 2100)]
BATCHES = [(5, (2048, 1300)), (7, (2048, 1300)), (9, (2048, 600))]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("tails") / "tail_plan")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "tail_plan.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)

    def query(kind, s, method, forced, sizes):
        per_cu = 2 if s <= 8 and forced != 4 else 1
        text = "%d %d %d %d %d %d %s\n" % (KIND[kind], s, METHOD[method], forced, CUS * per_cu, len(sizes),
                                         " ".join(map(str, sizes)))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        groups, rb, tiles, parts = (int(x) for x in out.split())
        return groups, rb, tiles, parts
    return query


def test_the_cases_take_the_paths_they_are_for(plan):
    for kind, s in HEIGHTS:
        assert [plan(kind, s, "canonical", rb, [300])[1] for rb in (2, 4)] == [2, 4]
    for method, kind, s, n in TAILS:
        groups, rb, tiles, parts = plan(kind, s, method, 0, [n])
        assert parts > 1 and rb == (2 if s <= 8 else 4) and tiles > CUS * (2 if rb == 2 else 1)
    for s, sizes in BATCHES:
        groups, rb, tiles, parts = plan("int8", s, "canonical", 0, sizes)
        assert groups == 1 and parts > 1
    lib = _lib.load()
    lone = [(k, s, 300) for k, s in HEIGHTS] + [(k, s, n) for _, k, s, n in TAILS]
    lone += [("int8", s, n) for s, sizes in BATCHES for n in sizes]
    for kind, s, n in lone:
        least, full = (f(n, s, KIND[kind]) for f in (lib.dmp_purify_min_workspace_bytes, lib.dmp_purify_workspace_bytes))
        assert least < full if 6 <= s <= 8 else least == full
    n = (ctypes.c_int * 2)(2048, 1300)
    assert lib.dmp_purify_batched_min_workspace_bytes(2, n, 7, 1) < lib.dmp_purify_batched_workspace_bytes(2, n, 7, 1)


def gpu():
    torch = pytest.importorskip("torch")
    dmp = pytest.importorskip("paper_2407_13299_amd")
    return torch, dmp, lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def case(n):
    if n == 2048:
        return tight_binding_hamiltonian(8, 8, 8, seed=1), 512
    return spectrum_hamiltonian(n, n // 2, seed=31)[0], n // 2


def run(h, nocc, kind, s, method, max_iter=200):
    torch, dmp, dev = gpu()
    lib = _lib.load()
    nbytes = lib.dmp_purify_min_workspace_bytes(h.shape[0], s, KIND[kind]) if kind in KIND else 256
    p, e, info = dmp.purify(dev(h), nocc, tol=1e-10, slices=s, kind=kind, method=method, max_iter=max_iter,
                            workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return p.cpu().numpy(), e, info


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["canonical", "trs4"])
@pytest.mark.parametrize("kind,s", HEIGHTS)
def test_both_tile_heights(kind, s, method, monkeypatch):
    """The first STEPS iterates on 64-row and 128-row tiles, which differ in the
    order of the trace sums, against the FP64 ones: a product is off by less than e =
    sqrt(n) (2^(8 - 8 s) + 2^-52), a step has two and amplifies what it is given by
    at most 4."""
    h, nocc = case(300)
    ref, _, info = run(h, nocc, "native", s, method, STEPS)
    assert info["iters"] == STEPS
    for rows in ("64", "128"):
        monkeypatch.setenv("DMP_TILE_ROWS", rows)
        p, e, info = run(h, nocc, kind, s, method, STEPS)
        assert info["iters"] == STEPS and info["slices"] == s and np.array_equal(p, p.T)
        assert np.max(np.abs(p - ref)) < 2 * 4.0 ** STEPS * np.sqrt(300) * (2.0 ** (8 - 8 * s) + 2.0 ** -52)


@pytest.mark.gpu
@pytest.mark.parametrize("method,kind,s,n", TAILS)
def test_split_tails_are_bit_identical(method, kind, s, n, monkeypatch):
    """Split tails add integers: the bits of whole tiles (DMP_TAIL_SPLIT=0)."""
    h, nocc = case(n)
    out = []
    for split in ("1", "0"):
        monkeypatch.setenv("DMP_TAIL_SPLIT", split)
        out.append(run(h, nocc, kind, s, method))
    (p1, e1, i1), (p0, e0, i0) = out
    assert i1 == i0 and np.array_equal(p1, p0) and e1 == e0 and i1["iters"] > 0


@pytest.mark.gpu
@pytest.mark.parametrize("s,sizes", BATCHES)
def test_split_tails_in_a_batch(s, sizes, monkeypatch):
    """A batch whose tail tiles are split: the bits of its members alone on whole
    tiles."""
    torch, dmp, dev = gpu()
    lib = _lib.load()
    cases = [case(n) for n in sizes]
    hs = [dev(h) for h, _ in cases]
    n, nocc = (ctypes.c_int * 2)(*sizes), (ctypes.c_int * 2)(*[k for _, k in cases])
    ps, e, info = [torch.empty_like(h) for h in hs], (ctypes.c_double * 2)(), (_lib.DmpInfo * 2)()
    ws = torch.empty(lib.dmp_purify_batched_min_workspace_bytes(2, n, s, 1), dtype=torch.uint8, device="cuda")
    arr = lambda ts: (ctypes.c_void_p * 2)(*[t.data_ptr() for t in ts])
    monkeypatch.setenv("DMP_TAIL_SPLIT", "1")
    st = lib.dmp_purify_batched(2, arr(hs), n, nocc, 1e-10, s, 1, 200, arr(ps), e, info, ctypes.c_void_p(ws.data_ptr()),
                                ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert st >= 0
    monkeypatch.setenv("DMP_TAIL_SPLIT", "0")
    for i, (h, k) in enumerate(cases):
        lone = (ctypes.c_int * 1)(sizes[i])
        p0, e0, i0 = torch.empty_like(hs[i]), (ctypes.c_double * 1)(), (_lib.DmpInfo * 1)()
        one = lambda t: (ctypes.c_void_p * 1)(t.data_ptr())
        w = torch.empty(lib.dmp_purify_min_workspace_bytes(sizes[i], s, 1), dtype=torch.uint8, device="cuda")
        assert lib.dmp_purify_batched(1, one(hs[i]), lone, (ctypes.c_int * 1)(k), 1e-10, s, 1, 200, one(p0), e0, i0,
                                      ctypes.c_void_p(w.data_ptr()), w.numel(),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) >= 0
        torch.cuda.synchronize()
        assert torch.equal(ps[i], p0) and e[i] == e0[0] and info[i].iters == i0[0].iters
