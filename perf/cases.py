"""Performance cases: the work a program has this package do, through its
public entry points.

Five kinds of call (the ``op`` of a case):

  gemm      C = op(A) op(B), one product (``ozaki_gemm``, or
            ``ozaki_gemm_noalloc`` where ``noalloc`` is set)
  batch     C_b = A_b B_b over a list of small products (``ozaki_gemm_batched``)
  purify    one density matrix from one Hamiltonian (``purify``)
  many      the density matrices of a list of Hamiltonians (``purify_batched``)
  grad      density matrix and dL/dH of L = tr(P W) (``Purify``)

``listed()`` holds the named cases, ``draw(rng)`` one more of the same
ranges.  ``exact`` gives what a case returns in plain FP64 torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2407_13299_amd as dmp
from paper_2407_13299_amd.workloads import symmetric_weight, tight_binding_hamiltonian

DEVICE = "cuda"


def listed():
    return [
        # the smallest product: a block of orbitals against another, where
        # launches and latency are all there is
        dict(name="gemm_64", op="gemm", m=64, n=64, k=64, slices=7, ta=False, tb=False,
             noalloc=False),
        # a serving loop's product, which cannot allocate
        dict(name="gemm_noalloc_256", op="gemm", m=256, n=256, k=256, slices=7, ta=False, tb=False,
             noalloc=True),
        # an ordinary product of odd sizes with a transposed operand
        dict(name="gemm_ragged_tn", op="gemm", m=1000, n=777, k=1301, slices=7, ta=True, tb=False,
             noalloc=False),
        # a density matrix applied to a narrow block of vectors, one slice
        # more than the default
        dict(name="gemm_skinny", op="gemm", m=4096, n=96, k=4096, slices=8, ta=False, tb=False,
             noalloc=False),
        # a large dense product
        dict(name="gemm_4096", op="gemm", m=4096, n=4096, k=4096, slices=7, ta=False, tb=False,
             noalloc=False),
        # many small products of uneven sizes in one call
        dict(name="gemm_batch_24", op="batch", count=24, lo=64, hi=512, slices=7),
        # a small molecule to a tight tolerance
        dict(name="purify_spectrum_256", op="purify", model="spectrum", n=256, nocc=128, tol=1e-12,
             slices=7, method="canonical", refine=False),
        # a mid-size lattice, canonical purification
        dict(name="purify_tb_2048", op="purify", model="tb", lx=8, ly=8, lz=8, tol=1e-8, slices=7,
             method="canonical", refine=False),
        # a lattice of odd size by the paper's own method, TRS4
        dict(name="purify_trs4_3960", op="purify", model="tb", lx=9, ly=10, lz=11, tol=1e-8,
             slices=7, method="trs4", refine=False),
        # a screening run: many Hamiltonians of uneven sizes, tuned slice counts
        dict(name="purify_many_56", op="many", count=56, lo=128, hi=1536, tol=1e-8, slices=0),
        # a density-matrix loss inside a training step: forward and backward
        dict(name="grad_tb_2048", op="grad", lx=8, ly=8, lz=8, tol=1e-8, slices=7),
        # the largest: canonical purification of the 16 x 16 x 8 lattice
        dict(name="purify_tb_8192", op="purify", model="tb", lx=16, ly=16, lz=8, tol=1e-8, slices=7,
             method="canonical", refine=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lattice(rng, top):
    """Lattice lengths >= 3 of a cell of about n orbitals, n spread over
    [108, top] by its logarithm."""
    sites = _log_int(rng, 27, top // 4)
    side = sites ** (1.0 / 3.0)
    lx = max(3, int(round(side * rng.uniform(0.75, 1.3))))
    ly = max(3, int(round(side * rng.uniform(0.75, 1.3))))
    lz = max(3, min(int(round(sites / (lx * ly))), top // (4 * lx * ly)))
    return lx, ly, lz


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm", "batch", "purify", "purify", "purify", "many", "grad"])
    if op == "gemm":
        noalloc = rng.random() < 0.2
        top = 1024 if noalloc else 4096
        return dict(op="gemm", m=_log_int(rng, 17, top), n=_log_int(rng, 17, top),
                    k=_log_int(rng, 17, top), slices=rng.choice([6, 7, 7, 7, 8]),
                    ta=rng.random() < 0.3, tb=rng.random() < 0.3, noalloc=noalloc)
    if op == "batch":
        lo = _log_int(rng, 24, 96)
        return dict(op="batch", count=rng.randint(4, 32), lo=lo, hi=_log_int(rng, 2 * lo, 700),
                    slices=rng.choice([6, 7, 7, 8]))
    if op == "purify":
        method = rng.choice(["canonical", "canonical", "trs4"])
        slices = rng.choice([7, 7, 7, 8])
        refine = rng.random() < 0.2
        if rng.random() < 0.5:
            n = _log_int(rng, 64, 2400)
            nocc = max(1, int(n * rng.uniform(0.25, 0.5)))
            return dict(op="purify", model="spectrum", n=n, nocc=nocc, tol=rng.choice([1e-8, 1e-10]),
                        slices=slices, method=method, refine=refine)
        lx, ly, lz = _lattice(rng, 5000)
        return dict(op="purify", model="tb", lx=lx, ly=ly, lz=lz, tol=1e-8, slices=slices,
                    method=method, refine=refine)
    if op == "many":
        lo = _log_int(rng, 48, 256)
        return dict(op="many", count=rng.randint(4, 48), lo=lo, hi=_log_int(rng, 2 * lo, 1200),
                    tol=1e-8, slices=rng.choice([0, 0, 7]))
    lx, ly, lz = _lattice(rng, 2048)
    return dict(op="grad", lx=lx, ly=ly, lz=lz, tol=1e-8, slices=7)


# ---- inputs -------------------------------------------------------------------


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _normal(rows, cols, gen):
    return torch.randn((rows, cols), dtype=torch.float64, device=DEVICE, generator=gen)


def _sizes(case, key):
    """Sizes of a list's members: a property of the case, not of the seed (a
    program's next inputs have the sizes of its last)."""
    rng = np.random.default_rng([case["count"], case["lo"], case["hi"]])
    return [[int(x) for x in row] for row in
            rng.integers(case["lo"], case["hi"] + 1, size=(case["count"], key))]


def _spectrum(n, nocc, gen):
    """H = Q diag(l) Q^T, Haar-like Q, nocc levels in [-1, -0.1] and the rest
    in [0.1, 1]."""
    q, _ = torch.linalg.qr(_normal(n, n, gen))
    u = torch.rand(n, dtype=torch.float64, device=DEVICE, generator=gen)
    lam = torch.where(torch.arange(n, device=DEVICE) < nocc, -1.0 + 0.9 * u, 0.1 + 0.9 * u)
    h = (q * lam) @ q.T
    return (0.5 * (h + h.T)).contiguous()


def _lattice_h(case, seed):
    h = tight_binding_hamiltonian(case["lx"], case["ly"], case["lz"], seed=int(seed))
    return torch.from_numpy(h).to(DEVICE)


def _orbitals(case):
    if case.get("model") == "spectrum":
        return case["n"], case["nocc"]
    n = 4 * case["lx"] * case["ly"] * case["lz"]
    return n, n // 4


def prepare(case, seed):
    gen = _generator(seed)
    state = dict(case=case)
    if case["op"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        state["A"] = _normal(k, m, gen) if case["ta"] else _normal(m, k, gen)
        state["B"] = _normal(n, k, gen) if case["tb"] else _normal(k, n, gen)
        state["C"] = torch.empty((m, n), dtype=torch.float64, device=DEVICE)
    elif case["op"] == "batch":
        mnk = _sizes(case, 3)
        state["A"] = [_normal(m, k, gen) for m, n, k in mnk]
        state["B"] = [_normal(k, n, gen) for m, n, k in mnk]
    elif case["op"] == "purify":
        n, nocc = _orbitals(case)
        state["nocc"] = nocc
        state["H"] = _spectrum(n, nocc, gen) if case["model"] == "spectrum" else _lattice_h(case, seed)
    elif case["op"] == "many":
        sizes = [row[0] for row in _sizes(case, 1)]
        state["nocc"] = [n // 2 for n in sizes]
        state["H"] = [_spectrum(n, n // 2, gen) for n in sizes]
    else:
        n, nocc = _orbitals(case)
        state["nocc"] = nocc
        state["H"] = _lattice_h(case, seed).requires_grad_(True)
        state["W"] = torch.from_numpy(symmetric_weight(n, int(seed) + 1)).to(DEVICE)
    return state


# ---- one pass -----------------------------------------------------------------


def run(state):
    case = state["case"]
    if case["op"] == "gemm":
        f = dmp.ozaki_gemm_noalloc if case["noalloc"] else dmp.ozaki_gemm
        return f(state["A"], state["B"], slices=case["slices"], trans_a=case["ta"],
                 trans_b=case["tb"], out=state["C"])
    if case["op"] == "batch":
        return dmp.ozaki_gemm_batched(state["A"], state["B"], slices=case["slices"])
    if case["op"] == "purify":
        p, e, _ = dmp.purify(state["H"], state["nocc"], tol=case["tol"], slices=case["slices"],
                             method=case["method"], refine=case["refine"])
        return p, e
    if case["op"] == "many":
        ps, es, _ = dmp.purify_batched(state["H"], state["nocc"], tol=case["tol"],
                                       slices=case["slices"])
        return ps, np.array(es)
    p = dmp.Purify.apply(state["H"], state["nocc"], case["tol"], case["slices"])
    (g,) = torch.autograd.grad((p * state["W"]).sum(), state["H"])
    return dict(P=p.detach(), grad=g)


# ---- what a pass cannot do without ----------------------------------------------


def _steps(model, n, method):
    """Iterations a purification of this size takes, about (measured counts:
    42, 57, 70 and 99 at n = 1024, 2048, 4096 and 8192 on the lattices)."""
    if method == "trs4":
        return 12
    return 17 if model == "spectrum" else max(20, round(57 * (n / 2048) ** 0.4))


def work(case):
    """Bytes: each input read and each output written once.  Flops: FP64
    multiply-adds of the products; a product of symmetric matrices counts one
    triangle."""
    if case["op"] == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=8 * (m * k + k * n + m * n), flops=2 * m * n * k)
    if case["op"] == "batch":
        mnk = _sizes(case, 3)
        return dict(bytes=8 * sum(m * k + k * n + m * n for m, n, k in mnk),
                    flops=2 * sum(m * n * k for m, n, k in mnk))
    if case["op"] == "purify":
        n, _ = _orbitals(case)
        products = 2 * _steps(case["model"], n, case["method"]) + (2 if case["refine"] else 0)
        return dict(bytes=16 * n * n, flops=products * n ** 3)
    if case["op"] == "many":
        sizes = [row[0] for row in _sizes(case, 1)]
        return dict(bytes=16 * sum(n * n for n in sizes),
                    flops=2 * _steps("spectrum", 0, "canonical") * sum(n ** 3 for n in sizes))
    n, _ = _orbitals(case)
    # forward: two triangles a step; backward: two full products and a triangle
    return dict(bytes=32 * n * n, flops=_steps("tb", n, "canonical") * 7 * n ** 3)


# ---- the same in plain FP64 torch -----------------------------------------------


def _gershgorin(h):
    d = torch.diagonal(h)
    rad = h.abs().sum(dim=1) - d.abs()
    return (d - rad).min(dim=0).values, (d + rad).max(dim=0).values


def _eye(h):
    return torch.eye(h.shape[0], dtype=torch.float64, device=h.device)


def _stopped(es, tol):
    """The stop rule on the energies so far: converged, or risen twice in a
    row by less than 1e-2."""
    de = es[-1] - es[-2]
    if abs(de) < tol:
        return True
    return len(es) >= 3 and 0.0 < de < 1e-2 and es[-2] - es[-3] > 0.0


def _canonical(h, nocc, tol, max_iter=200):
    """Canonical (trace-conserving) purification with plain FP64 products."""
    n = h.shape[0]
    theta = nocc / n
    lo, hi = _gershgorin(h)
    mu = torch.trace(h) / n
    lam = torch.minimum(theta / (hi - mu), (1.0 - theta) / (mu - lo))
    p = lam * (mu * _eye(h) - h) + theta * _eye(h)
    es = [float((p * h).sum())]
    for _ in range(max_iter):
        x2 = p @ p
        x3 = x2 @ p
        t1 = torch.trace(p - x2)
        t2 = (x2 * (_eye(h) - p)).sum()
        c = torch.clamp(t2 / t1, 0.0, 1.0) if float(t1) != 0.0 else t1.new_tensor(0.5)
        if float(c) >= 0.5:
            p = ((1.0 + c) * x2 - x3) / c
        else:
            p = ((1.0 - 2.0 * c) * p + (1.0 + c) * x2 - x3) / (1.0 - c)
        es.append(float((p * h).sum()))
        if _stopped(es, tol):
            break
    return p, es[-1]


def _trs4(h, nocc, tol, max_iter=200):
    """TRS4 purification with plain FP64 products."""
    lo, hi = _gershgorin(h)
    x = (hi * _eye(h) - h) / (hi - lo)
    es = [float((x * h).sum())]
    for _ in range(max_iter):
        x2 = x @ x
        tr_f = float((x2 * (4.0 * x - 3.0 * x2)).sum())
        tr_g = float(((x - x2) ** 2).sum())
        g = (nocc - tr_f) / tr_g if tr_g != 0.0 else 0.0
        if g > 6.0:
            x = 2.0 * x - x2
        elif g < 0.0:
            x = x2
        else:
            x = x2 @ ((4.0 - 2.0 * g) * x + (g - 3.0) * x2 + g * _eye(h))
            x = 0.5 * (x + x.T)
        es.append(float((x * h).sum()))
        if _stopped(es, tol):
            break
    return x, es[-1]


def exact(case, seed):
    state = prepare(case, seed)
    if case["op"] == "gemm":
        a = state["A"].T.contiguous() if case["ta"] else state["A"]
        b = state["B"].T.contiguous() if case["tb"] else state["B"]
        return a @ b
    if case["op"] == "batch":
        return [a @ b for a, b in zip(state["A"], state["B"])]
    if case["op"] == "purify":
        h, nocc = state["H"], state["nocc"]
        step = _trs4 if case["method"] == "trs4" else _canonical
        p, e = step(h, nocc, case["tol"])
        if case["refine"]:
            x2 = p @ p
            p = 3.0 * x2 - 2.0 * (x2 @ p)
            e = float((p * h).sum())
        return p, e
    if case["op"] == "many":
        out = [_canonical(h, nocc, case["tol"]) for h, nocc in zip(state["H"], state["nocc"])]
        return [p for p, _ in out], np.array([e for _, e in out])
    p, _ = _canonical(state["H"], state["nocc"], case["tol"])
    (g,) = torch.autograd.grad((p * state["W"]).sum(), state["H"])
    return dict(P=p.detach(), grad=0.5 * (g + g.T))
