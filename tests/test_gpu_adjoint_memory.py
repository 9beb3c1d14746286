"""Gradients of many sizes leave no device memory behind."""
import gc

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
dmp = pytest.importorskip("paper_2407_13299_amd")


def test_sizes_leave_nothing_behind():
    """A hundred sizes after the first ten: less than 1 MiB (the tile lists of a
    size, if they were kept, take about 25 KB)."""
    def gradient(n):
        g = torch.Generator(device="cuda").manual_seed(n)
        h = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g) * 0.01
        h = h + h.T + torch.diag(torch.linspace(-1.0, 1.0, n, dtype=torch.float64, device="cuda"))
        tape = dmp.PurifyTape(h, n // 2, tol=1e-8, slices=7, max_iter=2)
        tape.backward(torch.ones_like(h))

    def free():
        gc.collect()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]
    for n in range(1400, 1410):
        gradient(n)
    before = free()
    for n in range(1410, 1510):
        gradient(n)
    assert before - free() < 1 << 20
