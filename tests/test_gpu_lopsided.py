"""An H whose lower half, which only the Gershgorin bounds read, differs from the
upper half, which the initial guess is made of: the spectrum of P0 may leave [0,
1], on which the scaling of residue products relies.  The FP64 kind runs the
same iteration."""
import numpy as np
import pytest

from oracle import canonical
from paper_2407_13299_amd.workloads import spectrum_hamiltonian

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
dmp = pytest.importorskip("paper_2407_13299_amd")
STEPS = 6


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def arrows(blocks, seed):
    """Upper halves of 3 x 3 arrow matrices (0 diagonal) and nothing below: the
    last row of a block has an empty disc, but eigenvalues sqrt(2) times the
    largest radius."""
    rng = np.random.default_rng(seed)
    n = 3 * blocks
    h = np.zeros((n, n))
    for b in range(blocks):
        h[3 * b:3 * b + 2, 3 * b + 2] = rng.uniform(0.99, 1.0, 2)
        h[3 * b, 3 * b] = h[3 * b + 1, 3 * b + 1] = rng.uniform(0.0, 0.02)
    return h


def close(p, ref, s, scale):
    """A product of digit slices is off by less than sqrt(n) (2^(8 - 8 s) + 2^-52)
    per squared largest entry ``scale``; a step has two and amplifies what it is
    given by at most 4 ``scale``^2."""
    n = p.shape[0]
    bound = 2 * (4.0 * scale ** 2) ** STEPS * scale ** 2 * np.sqrt(n) * (2.0 ** (8 - 8 * s) + 2.0 ** -52)
    return np.max(np.abs(p - ref)) < bound


def run(h, nocc, kind, s, method, max_iter):
    p, e, info = dmp.purify(dev(h), nocc, tol=1e-11, slices=s, kind=kind, method=method, max_iter=max_iter)
    torch.cuda.synchronize()
    return p.cpu().numpy(), e, info


@pytest.mark.parametrize("method", ["canonical", "trs4"])
@pytest.mark.parametrize("kind,s,blocks", [("int8", 7, 22), ("fp16", 7, 22), ("int8", 6, 50), ("int8", 8, 200)])
def test_spectrum_outside_the_unit_interval(kind, s, blocks, method):
    h = arrows(blocks, blocks)
    full, nocc = np.triu(h) + np.triu(h, 1).T, 3 * blocks // 2
    th, mu, lam, lo, hi, _ = canonical.initial_scalars(h, nocc)
    x0 = (hi * np.eye(len(h)) - full) / (hi - lo) if method == "trs4" else lam * (mu * np.eye(len(h)) - full) + th * np.eye(len(h))
    w = np.linalg.eigvalsh(x0)
    assert w[0] < -0.1 and w[-1] > 1.1
    ref, got = run(h, nocc, "native", s, method, STEPS), run(h, nocc, kind, s, method, STEPS)
    assert got[2]["iters"] == ref[2]["iters"] and got[2]["slices"] == s
    assert got[2]["h_max"] == ref[2]["h_max"]
    assert close(got[0], ref[0], s, max(1.0, w[-1])), np.max(np.abs(got[0] - ref[0]))


def test_a_small_difference_keeps_the_residues():
    """The rounding of an H formed as a product moves nothing: the bits of the
    symmetric H (its upper half), bounds apart."""
    h, _, _ = spectrum_hamiltonian(300, 150, seed=1)
    low = np.tril(h, -1) * (1.0 + 1e-15)
    p, e, info = run(np.triu(h) + low, 150, "int8", 7, "canonical", STEPS)
    q, e2, info2 = run(h, 150, "int8", 7, "canonical", STEPS)
    assert np.max(np.abs(p - q)) < 1e-12


def test_a_lopsided_member_of_a_batch():
    """Beside ordinary members: everyone's result is that of a call of its own."""
    hs = [spectrum_hamiltonian(100, 50, seed=1)[0], arrows(40, 3), spectrum_hamiltonian(130, 20, seed=2)[0], arrows(22, 4)]
    noccs = [50, 60, 20, 33]
    ps, es, infos = dmp.purify_batched([dev(h) for h in hs], noccs, tol=1e-11, slices=7, max_iter=40)
    torch.cuda.synchronize()
    for h, nocc, p, e, info in zip(hs, noccs, ps, es, infos):
        p1, e1, i1 = run(h, nocc, "int8", 7, "canonical", 40)
        assert np.array_equal(p.cpu().numpy(), p1) and e == e1 and info == i1


@pytest.mark.parametrize("n,stride", [(66, 1), (66, 4)])
def test_tape(n, stride):
    """The taped forward run and its gradient on digit slices, against 9 slices.
    Products of the backward pass are off by sqrt(n) 2^-48 of their operands, three
    a step, and a step multiplies what it is given by at most 4."""
    h, nocc = arrows(n // 3, 7), n // 2
    pbar = np.cos(np.arange(n * n, dtype=np.float64)).reshape(n, n) / n
    p, g = {}, {}
    for s in (7, 9):
        tape = dmp.PurifyTape(dev(h), nocc, tol=1e-11, slices=s, max_iter=STEPS, stride=stride)
        p[s], g[s] = tape.P.cpu().numpy(), tape.backward(dev(pbar)).cpu().numpy()
    assert close(p[7], p[9], 7, 1.25)
    assert np.max(np.abs(g[7] - g[9])) < 3 * STEPS * 4.0 ** (2 * STEPS) * np.sqrt(n) * 2.0 ** -48 * max(1, np.max(np.abs(g[9])))
