"""Calls whose sums need more scratch than there is, as at the largest systems: the
third-law kernels in batches of few slots, in ordered form where not three fit, the
evaluation by the other kernels. A small system's context is told that it has only
`per` doubles a particle (its buffer stays the larger one): 18 is what a context of a
large system has where 45 do not fit, 13 and 10 hold one slot of the gradients, 39
three.

Bounds: 1e-11 of the largest component for gradients, against the autograd reference
(orders 1 and 3: against the same call with all the scratch, tested against it
elsewhere); 1e-12 for a, j, s and 1e-11 for the crackle, EX 2e-12, 4e-12, 1e-11,
against the oracle.
"""

import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import oracle.adjoint_ref as ar
from paper_1901_08532_amd import h6, ics
from _gpu import DEV, from_rows, gpu_evaluate, plummer_pred, to_rows, vec_rel_err

pytestmark = pytest.mark.gpu


def _context(n, eps, per):
    ctx = h6.Context(n, eps)
    full = 9 << 21  # doubles of a small system's scratch
    words = (C.c_int64 * 40).from_address(ctx.handle.value)
    at = [k for k in range(40) if words[k] == full]
    assert len(at) == 1  # the capacity, in the context's structure
    words[at[0]] = min(per * n, full)
    return ctx


@pytest.mark.parametrize("per", [10, 18, 30, 50])
@pytest.mark.parametrize("n", [1, 256, 1030, 2305])
def test_gradient(n, per):
    rng = np.random.Generator(np.random.PCG64(n))
    x, v, a = (rng.normal(0, 1, (n, 3)) for _ in range(3))
    m = rng.uniform(0.5, 1.5, n) / n
    cot = [rng.normal(0, 1, (n, 3)) for _ in range(3)]
    GP = torch.full((9, n), np.nan, dtype=torch.float64, device=DEV)
    gm = torch.full((n,), 0.25, dtype=torch.float64, device=DEV)
    _context(n, 1e-2, per).h6_evaluate_vjp(to_rows(x, v, a), torch.from_numpy(m).to(DEV), to_rows(*cot), GP, gm)
    if n == 1:
        assert not GP.any() and float(gm) == 0.25
        return
    ref = ar.pair_sums_vjp(x, v, m, 1e-4, cot, a=a, order=2)
    for k, name in enumerate("xva"):
        assert np.abs(from_rows(GP, k) - ref[name]).max() <= 1e-11 * np.abs(ref[name]).max(), name
    assert np.abs(gm.cpu().numpy() - 0.25 - ref["m"]).max() <= 1e-11 * np.abs(ref["m"]).max()


@pytest.mark.parametrize("per", [13, 39, 65])
@pytest.mark.parametrize("n", [256, 1030, 2305])
def test_startup_gradient(n, per):
    x, v, m = ics.plummer(n, 3)
    s = h6.System(x, v, m, 1e-2)
    s.startup()
    g = torch.Generator(device=DEV).manual_seed(n)
    cot = torch.randn((18, n), generator=g, device=DEV, dtype=torch.float64)
    got = []
    for ctx in (_context(n, 1e-2, per), h6.Context(n, 1e-2)):
        C1, gm = cot.clone(), torch.zeros(n, dtype=torch.float64, device=DEV)
        ctx.h6_init_forces_vjp(s.S, s.m, C1, gm)
        got.append((C1[0:3], C1[3:6], gm))
    for p, q in zip(*got):
        assert float((p - q).abs().max()) <= 1e-11 * float(q.abs().max())


@pytest.mark.parametrize("per", [9, 18, 27, 45])
@pytest.mark.parametrize("n", [5001, 5633])
def test_evaluation(n, per):
    eps = 1e-2
    x, v, a, m = plummer_pred(n, n, eps * eps)
    want = oracle.forces(x, v, m, eps * eps, a=a, order=2)[:3]
    ctx = _context(n, eps, per)
    for prec, tol in ((h6.H6_FP64, (1e-12,) * 3), (h6.H6_EX, (2e-12, 4e-12, 1e-11))):
        for g, w, t in zip(gpu_evaluate(ctx, x, v, a, m, precision=prec), want, tol):
            assert vec_rel_err(g, w).max() <= t


@pytest.mark.parametrize("per", [18, 45])
def test_startup_and_steps(per):
    n, eps = 5633, 1e-2
    x, v, m = ics.plummer(n, 7)
    s = h6.System(x, v, m, eps, ctx=_context(n, eps, per))
    s.startup()
    want = oracle.startup(x, v, m, eps * eps)
    for name, w in zip("ajsc", want):
        assert vec_rel_err(s.field(name), w).max() <= (1e-11 if name == "c" else 1e-12), name
    ref = h6.System(x, v, m, eps)
    ref.startup()
    for t in (s, ref):
        t.shared_steps(1.0 / 1024, 3)
    for k in range(5):  # x, v, a, j, s
        w = ref.S[3 * k:3 * k + 3]
        assert float((s.S[3 * k:3 * k + 3] - w).abs().max()) <= 1e-11 * float(w.abs().max()), k


@pytest.mark.parametrize("per", [18, 45])
@pytest.mark.parametrize("n", [500, 6145])
def test_energy_gradient_and_active_gradient(n, per):
    x, v, m = ics.plummer(n, 9)
    s, ref = h6.System(x, v, m, 1e-2, ctx=_context(n, 1e-2, per)), h6.System(x, v, m, 1e-2)
    got = []
    g = torch.Generator(device=DEV).manual_seed(n)
    P, CF = (torch.randn((9, n), generator=g, device=DEV, dtype=torch.float64) for _ in range(2))
    act = torch.randperm(n, generator=g, device=DEV).to(torch.int32)
    for t in (s, ref):
        G, gm = torch.zeros((18, n), dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
        t.ctx.h6_energy_vjp(t.S, t.m, None, G, gm)
        GP, gp = torch.zeros_like(P), torch.zeros_like(gm)
        t.ctx.h6_evaluate_vjp_active(P, t.m, act, n, CF, GP, gp)
        got.append((G[0:3], G[3:6], gm, GP[0:3], GP[3:6], GP[6:9], gp))
    for p, q in zip(*got):
        assert float((p - q).abs().max()) <= 1e-11 * float(q.abs().max())


def test_ordered_gradient_in_batches():
    # more than 1024 superblocks of 256: the ordered form in two batches of offsets
    n = 270_001
    g = torch.Generator(device=DEV).manual_seed(n)
    P, CF = (torch.randn((9, n), generator=g, device=DEV, dtype=torch.float64) for _ in range(2))
    m = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) / n
    got = []
    for ctx in (_context(n, 1e-2, 10), h6.Context(n, 1e-2)):
        GP, gm = torch.full_like(P, float("nan")), torch.zeros_like(m)
        ctx.h6_evaluate_vjp(P, m, CF, GP, gm)
        got.append((GP[0:3], GP[3:6], GP[6:9], gm))
    for p, q in zip(*got):
        assert float((p - q).abs().max()) <= 1e-11 * float(q.abs().max())
