"""What a refused purification leaves undone."""
import ctypes

import numpy as np
import pytest

from oracle import canonical
from paper_2407_13299_amd.workloads import spectrum_hamiltonian

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
dmp = pytest.importorskip("paper_2407_13299_amd")
from paper_2407_13299_amd import _lib  # noqa: E402


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("kind,slices", [(1, 7), (1, 5), (2, 8), (0, 7)])
def test_nonfinite_member_stops_a_batch_before_its_first_iteration(kind, slices):
    """The other members of a batch with a NaN keep their initial guess: no
    iteration ran on them, whichever group of launches they are in."""
    lib = _lib.load()
    sizes, noccs = [90, 64, 130, 200], [45, 32, 5, 100]      # 200: small and thinly filled ones differ in moduli
    hs = [spectrum_hamiltonian(n, k, seed=n)[0] for n, k in zip(sizes, noccs)]
    for warm in (False, True):        # a first run of the launch sequence, and one with a known iteration count
        if warm:
            dmp.purify_batched([dev(h) for h in hs], noccs, tol=1e-9, slices=slices, kind=kind)
        bad = [h.copy() for h in hs]
        bad[1][3, 5] = bad[1][5, 3] = np.nan
        hd = [dev(h) for h in bad]
        ps = [torch.empty_like(h) for h in hd]
        n, nocc = (ctypes.c_int * 4)(*sizes), (ctypes.c_int * 4)(*noccs)
        ws = torch.empty(lib.dmp_purify_batched_workspace_bytes(4, n, slices, kind), dtype=torch.uint8, device="cuda")
        e = (ctypes.c_double * 4)()
        arr = lambda ts: (ctypes.c_void_p * 4)(*[t.data_ptr() for t in ts])
        st = lib.dmp_purify_batched_ex(4, arr(hd), n, nocc, 1e-9, slices, kind, 200, 0, 0, arr(ps), e, None,
                                       ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert st == -2 and b"non-finite" in lib.dmp_last_error()
        for i in (0, 2, 3):
            # P0 in FP64: a few roundings of values below 1
            assert np.max(np.abs(ps[i].cpu().numpy() - canonical.initial_guess(hs[i], noccs[i]))) < 1e-14
