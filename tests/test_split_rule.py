"""Where a digit split takes its own row maxima, and the same bits on both sides
of that line."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2407_13299_amd", "csrc")


def test_rule(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "split_rule"
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "split_rule.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", str(exe)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "split rule ok" in run.stdout, run.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["int8", "fp16"])
@pytest.mark.parametrize("m,n,k", [(5100, 40, 512), (5200, 40, 512), (40, 5300, 511), (9000, 33, 256)])
def test_both_sides_give_the_oracle_bits(kind, m, n, k):
    torch = pytest.importorskip("torch")
    dmp = pytest.importorskip("paper_2407_13299_amd")
    from oracle import ozaki
    rng = np.random.default_rng(m + n)
    a = rng.standard_normal((m, k)) * np.exp2(rng.integers(-9, 9, (m, 1)))
    b = rng.standard_normal((k, n)) * np.exp2(rng.integers(-9, 9, (1, n)))
    want = ozaki.ozaki_gemm(a, b, 3)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda")
    for ta, tb in ((False, False), (True, False), (False, True)):
        c = dmp.ozaki_gemm(dev(a.T) if ta else dev(a), dev(b.T) if tb else dev(b), slices=3, kind=kind, trans_a=ta,
                           trans_b=tb)
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy(), want)
