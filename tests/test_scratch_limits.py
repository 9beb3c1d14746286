"""Purifications whose workspace is too small for residue products: digit
slices, with the result they give, and the allocation that falls back to them."""
import ctypes

import numpy as np
import pytest

from paper_2407_13299_amd import _lib
from paper_2407_13299_amd.workloads import spectrum_hamiltonian, tight_binding_hamiltonian

KIND = {"int8": 1, "fp16": 2}
STEPS = 6


def test_the_least_workspace():
    """Two n x n matrices and two operands of S digit planes, as before residue
    products came; the ordinary one where those are never used or need less."""
    lib = _lib.load()
    for n in (100, 2048, 8192):
        for kind, width in ((1, 1), (2, 2)):
            for s in (6, 7, 8):
                least, full = (f(n, s, kind) for f in (lib.dmp_purify_min_workspace_bytes,
                                                       lib.dmp_purify_workspace_bytes))
                pad = (n + 127) // 128 * 128 * ((n + 63) // 64 * 64)
                parts = 512 * 4 * s * 16 * 64 * 4 if n > 2000 else 0       # part buffer of the split tail
                fixed = 16 * n * n + 2 * s * width * pad
                # beside them vectors, descriptors and tile lists: 100 KiB and under 1 % of the matrices
                assert fixed <= least <= fixed + parts + 100 * 1024 + fixed // 100
                assert least < full
            for s in (5, 9):
                assert lib.dmp_purify_min_workspace_bytes(n, s, kind) == lib.dmp_purify_workspace_bytes(n, s, kind)
    assert lib.dmp_purify_min_workspace_bytes(512, 4, 0) == lib.dmp_purify_workspace_bytes(512, 4, 0)
    assert lib.dmp_purify_min_workspace_bytes(512, 13, 1) == 0
    n = (ctypes.c_int * 3)(128, 300, 2048)
    assert lib.dmp_purify_batched_min_workspace_bytes(3, n, 7, 1) < lib.dmp_purify_batched_workspace_bytes(3, n, 7, 1)
    assert lib.dmp_purify_batched_min_workspace_bytes(0, n, 7, 1) == 0


def test_allocation_falls_back(monkeypatch):
    torch = pytest.importorskip("torch")
    from paper_2407_13299_amd import api
    real = torch.empty

    def empty(size, **kw):
        if size > 5000:
            raise torch.OutOfMemoryError("no room")
        return real(size, **kw)
    monkeypatch.setattr(api.torch, "empty", empty)
    assert api._workspace(4000, "cpu", lambda: 1000).numel() == 4000
    assert api._workspace(6000, "cpu", lambda: 1000).numel() == 1000
    for least in (None, lambda: 6000, lambda: 5500):
        with pytest.raises(torch.OutOfMemoryError):
            api._workspace(6000, "cpu", least)


def gpu():
    torch = pytest.importorskip("torch")
    dmp = pytest.importorskip("paper_2407_13299_amd")
    return torch, dmp, lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def purify_in(nbytes, h, nocc, s, kind, method, max_iter=200):
    torch, dmp, dev = gpu()
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    p, e, info = dmp.purify(dev(h), nocc, tol=1e-10, slices=s, kind=kind, method=method, workspace=ws,
                            max_iter=max_iter)
    torch.cuda.synchronize()
    return p.cpu().numpy(), e, info


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["canonical", "trs4"])
@pytest.mark.parametrize("kind,s,n", [("int8", 7, 300), ("fp16", 7, 300), ("int8", 8, 129), ("int8", 6, 200),
                                      ("int8", 7, 2048)])
def test_least_workspace_runs_on_digit_slices(kind, s, n, method):
    """One byte short of the ordinary workspace down to the least: the same bits
    (digit slices), which are not those of the residue products; a byte less than
    the least is refused.  The first STEPS iterates against the FP64 ones: a
    product of S slices is off by less than e = sqrt(n) (2^(8 - 8 s) + 2^-52), a step
    has two and amplifies what it is given by at most 4 (the slopes of the maps on
    [0, 1])."""
    torch, dmp, dev = gpu()
    lib = _lib.load()
    if n == 2048:
        h, nocc = tight_binding_hamiltonian(8, 8, 8, seed=1), 512
    else:
        nocc = n // 2
        h, _, _ = spectrum_hamiltonian(n, nocc, seed=n)
    full, least = (f(n, s, KIND[kind]) for f in (lib.dmp_purify_workspace_bytes, lib.dmp_purify_min_workspace_bytes))
    assert least < full
    ref = purify_in(256, h, nocc, s, "native", method, STEPS)
    got = purify_in(least, h, nocc, s, kind, method, STEPS)
    assert got[2]["iters"] == ref[2]["iters"] == STEPS and got[2]["slices"] == s
    assert np.array_equal(got[0], got[0].T)
    assert np.max(np.abs(got[0] - ref[0])) < 2 * 4.0 ** STEPS * np.sqrt(n) * (2.0 ** (8 - 8 * s) + 2.0 ** -52)
    runs = [purify_in(b, h, nocc, s, kind, method) for b in (least, full - 1, full)]
    assert np.array_equal(runs[0][0], runs[1][0]) and runs[0][1] == runs[1][1]
    assert not np.array_equal(runs[0][0], runs[2][0])
    P, e, ws = torch.empty_like(dev(h)), ctypes.c_double(), torch.empty(least, dtype=torch.uint8, device="cuda")
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    assert lib.dmp_purify_ex(ptr(dev(h)), n, nocc, 1e-10, s, KIND[kind], 200, 0, 0, ptr(P), ctypes.byref(e), None,
                             ptr(ws), least - 1, None) == -4


@pytest.mark.gpu
def test_a_batch_in_the_least_workspace():
    """Every member on digit slices: the bits of the member alone in its least
    workspace."""
    torch, dmp, dev = gpu()
    lib = _lib.load()
    sizes = [64, 200, 333]
    hs = [dev(spectrum_hamiltonian(n, n // 2, seed=n)[0]) for n in sizes]
    n, nocc = (ctypes.c_int * 3)(*sizes), (ctypes.c_int * 3)(*[x // 2 for x in sizes])
    ps = [torch.empty_like(h) for h in hs]
    ws = torch.empty(lib.dmp_purify_batched_min_workspace_bytes(3, n, 7, 1), dtype=torch.uint8, device="cuda")
    e = (ctypes.c_double * 3)()
    arr = lambda ts: (ctypes.c_void_p * 3)(*[t.data_ptr() for t in ts])
    assert lib.dmp_purify_batched(3, arr(hs), n, nocc, 1e-10, 7, 1, 200, arr(ps), e, None,
                                  ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    for i, h in enumerate(hs):
        p, e1, _ = purify_in(lib.dmp_purify_min_workspace_bytes(sizes[i], 7, 1), h.cpu().numpy(), sizes[i] // 2, 7,
                             "int8", "canonical")
        assert np.array_equal(ps[i].cpu().numpy(), p) and e[i] == e1
