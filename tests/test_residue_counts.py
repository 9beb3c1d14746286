"""Every number of moduli the library takes: one step against extended
precision, within what the rounding of the operands to integers leaves, so that a
modulus too few or a wrong scale fails; batches whose members differ in it; the
backward products."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import canonical
from paper_2407_13299_amd.workloads import spectrum_hamiltonian

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2407_13299_amd", "csrc")
LAM, GROWTH_SQUARE = 1.0625, 1.0625     # layout.hpp

# (S, n, nocc) and the moduli they take
CASES = [(6, 100, 50, 11), (6, 127, 19, 12), (6, 200, 1, 13), (7, 127, 63, 13), (7, 127, 20, 14), (7, 200, 1, 15),
         (8, 100, 50, 15), (8, 100, 10, 16), (8, 257, 1, 16)]


@pytest.fixture(scope="module")
def limits(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("mods") / "mod_count")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "mod_count.cpp"), "-o", exe], check=True)
    text = "".join("%d %d %d 0\n" % c[:3] for c in CASES)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    return {c: (int(line.split()[0]), float(line.split()[1])) for c, line in zip(CASES, out)}


def first_step(h, nocc):
    """P0 and P1 of the canonical iteration, products in extended precision."""
    long = np.longdouble
    p = canonical.initial_guess(h, nocc).astype(long)
    p2 = p @ p
    p3 = p2 @ p
    t1, t2 = np.trace(p - p2), np.trace(p2 - p3)
    c = min(max(t2 / t1, long(0)), long(1))
    a, b, g = canonical.update_weights(c)
    return p, p2, t1, c, a * p + b * p2 + g * p3


def step_bound(p, p2, t1, c, limit):
    """(of the residues, of FP64) Frobenius norm of the error of P1.  X = p 2^-t is off
    by independent roundings of variance 1 / 12, so d, the error of p, has |d X|_F^2
    close to its mean sum_i 4^t_i / 12 |X|_F^2 (n^2 elements), and with d = e 2^t
      E1 = d P + P d^T                                of the square,
      E2 = d' P + X2 d^T + E1 P                       of the second product,
    the spectral norms of P and X2 being at most 1.  c = t2 / t1 with t1 = tr(P - X2),
    t2 = <X2, I - P>, both off by sums of |E1|_F / sqrt(n) about (four of them each),
    and dP1 / dc = -P (I - P)^2 / (1 - c)^2 or as much over c^2.  FP64 elsewhere:
    twenty roundings of the size of P."""
    n = p.shape[0]
    m = np.max(np.abs(p), axis=1).astype(float)
    nu = np.minimum(np.sqrt((n + 63) // 64 * 64.0) * m, np.sqrt(LAM * m))
    f = lambda v: float(np.linalg.norm(v.astype(float)))
    d = lambda growth: np.sqrt(np.sum(4.0 ** np.ceil(np.log2(growth * nu) - limit)) / 12.0)
    e1 = 2.0 * d(1.0) * f(p)
    e2 = d(GROWTH_SQUARE) * f(p) + d(1.0) * f(p2) + e1
    c = float(c)
    _, b, g = canonical.update_weights(c)
    dc = 8.0 * e1 / np.sqrt(n) / float(t1)
    return abs(b) * e1 + abs(g) * e2 + dc * f(p - p2) / max(c, 1.0 - c) ** 2, 20 * 2.0 ** -53 * f(p)


def test_the_bound_tells_one_modulus_from_the_next(limits):
    """The counts of the cases; and, emulated on the host, one step stays within the
    bound for its count and with one modulus fewer does not, unless FP64 rounding
    covers it."""
    from test_residue_accuracy import Residues
    told = 0
    for case, (count, limit) in limits.items():
        s, n, nocc, want = case
        assert count == want
        h, _, _ = spectrum_hamiltonian(n, nocc, seed=n)
        p, p2, t1, c, p1 = first_step(h, nocc)

        def error(limit):
            q = canonical.purify(h, nocc, tol=1e-300, max_iter=1, matmul=Residues(limit))["P"]
            return float(np.linalg.norm((q - p1).astype(float)))
        residues, fp64 = step_bound(p, p2, t1, c, limit)
        assert error(limit) < residues + fp64
        if residues > fp64 / 2:
            assert error(limit - np.log2(14.0)) > residues + fp64
            told += 1
    assert told >= 4


def gpu():
    torch = pytest.importorskip("torch")
    dmp = pytest.importorskip("paper_2407_13299_amd")
    return torch, dmp, lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["int8", "fp16"])
@pytest.mark.parametrize("case", CASES)
def test_one_step(limits, case, kind):
    torch, dmp, dev = gpu()
    s, n, nocc, _ = case
    h, _, _ = spectrum_hamiltonian(n, nocc, seed=n)
    q, _, info = dmp.purify(dev(h), nocc, tol=1e-300, slices=s, kind=kind, max_iter=1)
    torch.cuda.synchronize()
    assert info["iters"] == 1
    p, p2, t1, c, p1 = first_step(h, nocc)
    err = float(np.linalg.norm((q.cpu().numpy() - p1).astype(float)))
    assert err < sum(step_bound(p, p2, t1, c, limits[case][1]))


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["canonical", "trs4"])
@pytest.mark.parametrize("s", [6, 7, 8])
def test_a_batch_on_both_sides_of_every_line(s, method):
    """Members of 11 to 16 moduli in one call: the bits of a call of their own."""
    torch, dmp, dev = gpu()
    members = [(200, 100), (200, 80), (200, 79), (200, 99), (128, 63), (99, 50), (63, 32), (64, 32), (200, 30), (200, 29),
               (300, 2), (300, 1), (40, 20), (300, 150), (513, 1), (2, 1), (90, 0), (90, 90)]
    hs = [dev(spectrum_hamiltonian(n, k, seed=i)[0]) for i, (n, k) in enumerate(members)]
    ps, es, infos = dmp.purify_batched(hs, [k for _, k in members], tol=1e-9, slices=s, method=method, max_iter=30)
    for (n, k), h, p, e, info in zip(members, hs, ps, es, infos):
        p1, e1, i1 = dmp.purify(h, k, tol=1e-9, slices=s, method=method, max_iter=30)
        torch.cuda.synchronize()
        assert torch.equal(p, p1) and e == e1 and info == i1, (n, k)


@pytest.mark.gpu
@pytest.mark.parametrize("s", [6, 8])
def test_backward_counts(s):
    """13 and 16 moduli in the backward products (n = 1400), over 6 steps, against 11
    slices.  A product is off by e = sqrt(n) (2^(8 - 8 s) + 2^-52) of its operands'
    scale, three a step; what a step is given it multiplies by at most 2."""
    torch, dmp, dev = gpu()
    n, steps = 1400, 6
    g0 = torch.Generator(device="cuda").manual_seed(3)
    h = torch.randn((n, n), dtype=torch.float64, device="cuda", generator=g0) * 0.01
    h = h + h.T + torch.diag(torch.linspace(-1.0, 1.0, n, dtype=torch.float64, device="cuda"))
    pbar = np.cos(np.arange(n * n, dtype=np.float64)).reshape(n, n) / n
    g = {}
    for k in (s, 11):
        g[k] = dmp.PurifyTape(h, 700, tol=1e-300, slices=k, max_iter=steps).backward(dev(pbar)).cpu().numpy()
    scale = np.max(np.abs(g[11]))
    e = np.sqrt(n) * (2.0 ** (8 - 8 * s) + 2.0 ** -52)
    assert np.max(np.abs(g[s] - g[11])) < 3 * steps * 2.0 ** steps * e * scale


def test_sixteen_moduli_on_the_host(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "residue_reconstruct"
    subprocess.run([gxx, "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "host", "residue_reconstruct.cpp"), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "reconstruction ok" in run.stdout, run.stdout
