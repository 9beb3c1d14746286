"""Products through residues: the constants and tile lists on the host (no
GPU), the assembly of their GEMM, and on the GPU the purification, batches and
gradients at the sizes where tiles, widths and routes change."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2407_13299_amd.workloads import spectrum_hamiltonian

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2407_13299_amd", "csrc")


def test_constants_and_tiles(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "residue_plan"
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-ffp-contract=off", "-pthread", "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"),
                        os.path.join(HERE, "host", "residue_plan.cpp"),
                        os.path.join(CSRC, "plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "residue plan ok" in run.stdout, run.stdout


def test_m0_only_feeds_the_lds_loads(tmp_path):
    """As for the slice GEMM: m0 is only written, each time right before the
    load into LDS that reads it."""
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "modular.s"
    r = subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O3", "-S",
                        "--cuda-device-only", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-Wno-unused-command-line-argument", "-Wno-inline-asm",
                        os.path.join(CSRC, "modular.hip"), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [l.strip() for l in out.read_text().splitlines()]
    writes = 0
    for i, line in enumerate(lines):
        if line.startswith(";") or "m0" not in line.replace("m0_", ""):
            continue
        assert line.startswith("s_mov_b32 m0,"), f"other use of m0: {line}"
        assert lines[i + 1].startswith("buffer_load_dwordx4") and lines[i + 1].endswith(" lds")
        writes += 1
    assert writes > 0


def gpu():
    torch = pytest.importorskip("torch")
    dmp = pytest.importorskip("paper_2407_13299_amd")
    return torch, dmp, lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


STEPS = 6


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["canonical", "trs4"])
@pytest.mark.parametrize("n,nocc,s", [(1, 1, 7), (2, 1, 6), (33, 16, 8), (64, 20, 7), (65, 32, 7), (127, 3, 7),
                                      (129, 128, 6), (257, 1, 7), (320, 160, 8), (513, 256, 7), (1030, 515, 7)])
def test_iterates_match_fp64(method, n, nocc, s):
    """The first iterates against the FP64 ones, INT8 and FP16 bitwise equal.
    A product is off by less than e = sqrt(n) 2^(8 - 8 s) (digit slices'
    truncation, which the moduli are chosen to stay below) + sqrt(n) 2^-52; a step
    has two and amplifies what it is given by at most 4 (the slopes of the
    maps on [0, 1]), so STEPS of them stay below 2 e 4^STEPS."""
    torch, dmp, dev = gpu()
    h, _, _ = spectrum_hamiltonian(n, nocc, seed=n)
    got = {}
    for kind in ("int8", "fp16", "native"):
        p, e, info = dmp.purify(dev(h), nocc, tol=1e-13, slices=s, kind=kind, method=method, max_iter=STEPS)
        torch.cuda.synchronize()
        got[kind] = (p.cpu().numpy(), e, info["iters"])
    assert np.array_equal(got["int8"][0], got["fp16"][0]) and got["int8"][1:] == got["fp16"][1:]
    p, ref = got["int8"][0], got["native"][0]
    assert np.array_equal(p, p.T)
    if got["int8"][2] == got["native"][2]:
        bound = 2 * 4.0 ** STEPS * np.sqrt(n) * (2.0 ** (8 - 8 * s) + 2.0 ** -52)
        assert np.max(np.abs(p - ref)) < bound
    else:
        assert n <= 2     # one and two levels stop at once


@pytest.mark.gpu
@pytest.mark.parametrize("count,lo,hi", [(3, 1, 70), (40, 60, 260), (12, 500, 900)])
def test_batches_equal_single(count, lo, hi):
    """Small and wide tiles, combinations of 8 and of 4 wavefronts (from 1024
    tiles on), finished matrices beside unfinished ones: the bits of a single
    call."""
    torch, dmp, dev = gpu()
    rng = np.random.default_rng(count)
    sizes = [int(x) for x in rng.integers(lo, hi, count)]
    hs = [dev(spectrum_hamiltonian(n, max(1, n // 3), seed=i)[0]) for i, n in enumerate(sizes)]
    noccs = [max(1, n // 3) for n in sizes]
    Ps, Es, infos = dmp.purify_batched(hs, noccs, tol=1e-9, slices=7)
    for i in range(0, count, max(1, count // 6)):
        p, e, info = dmp.purify(hs[i], noccs[i], tol=1e-9, slices=7)
        torch.cuda.synchronize()
        assert torch.equal(p, Ps[i]) and e == Es[i] and info["iters"] == infos[i]["iters"]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1399, 1400])
def test_backward_routes(n):
    """Digit slices (n = 1399) and residues (n = 1400) in the backward products,
    against 9 slices, over 8 steps.  A product is off by e = sqrt(n) 2^-48 of
    its operands' scale, three a step; what a step is given it multiplies by at
    most 2 (the slope of the map), so 8 of them stay below 2^10 e."""
    torch, dmp, dev = gpu()
    h, _, _ = spectrum_hamiltonian(n, n // 2, seed=5)
    pbar = np.cos(np.arange(n * n, dtype=np.float64)).reshape(n, n) / n
    g = {}
    for s in (7, 9):
        tape = dmp.PurifyTape(dev(h), n // 2, tol=1e-13, slices=s, max_iter=8)
        g[s] = tape.backward(dev(pbar)).cpu().numpy()
    scale = np.max(np.abs(g[9]))
    assert np.max(np.abs(g[7] - g[9])) < 2.0 ** 10 * np.sqrt(n) * 2.0 ** -48 * scale


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(64, 64, 512), (65, 33, 513), (192, 130, 64), (40, 300, 2100), (130, 64, 4160)])
def test_gemm_routes_bitwise(m, n, k):
    """Splits that take their own maxima (k <= 512) and those that do not, tiles
    of 64 rows, reductions split over workgroups; transposed operands."""
    torch, dmp, dev = gpu()
    from oracle import ozaki
    rng = np.random.default_rng(m + n + k)
    a = rng.standard_normal((m, k)) * np.exp2(rng.integers(-9, 9, (m, 1)))
    b = rng.standard_normal((k, n))
    a[0, :] = 0.0
    want = ozaki.ozaki_gemm(a, b, 7)
    for ta in (False, True):
        for tb in (False, True):
            c = dmp.ozaki_gemm(dev(a.T) if ta else dev(a), dev(b.T) if tb else dev(b), slices=7, trans_a=ta, trans_b=tb)
            torch.cuda.synchronize()
            assert np.array_equal(c.cpu().numpy(), want)
