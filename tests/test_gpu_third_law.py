"""All particles by the third law at the edges of its work split: one more and
one less than a superblock (512), odd and even numbers of superblocks, runs
that cut a superblock, several batches of offsets, with the self mask.

Bounds: 1e-12 relative to the oracle for a, j, s and 1e-11 for the start-up's
crackle, as for the other evaluation kernels; the gradient 1e-11 of its largest
component relative to the autograd reference, as in the other adjoint tests.
"""

import numpy as np
import pytest
import torch

import oracle
import oracle.adjoint_ref as ar
from paper_1901_08532_amd import h6, ics
from _gpu import DEV, from_rows, gpu_evaluate, plummer_pred, to_rows, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eps", [(5000, 1e-4), (5119, 1e-4), (5120, 0.0), (5121, 1e-4), (5633, 0.0),
                                   (8192, 1e-4)])
def test_evaluation(n, eps):
    x, v, a, m = plummer_pred(n, 900 + n, eps * eps)
    m = ics.salpeter_masses(n, 901)
    ctx = h6.Context(n, eps)
    got = gpu_evaluate(ctx, x, v, a, m)
    again = gpu_evaluate(ctx, x, v, a, m)
    want = oracle.forces(x, v, m, eps * eps, a=a, order=2)[:3]
    for g, g2, w in zip(got, again, want):
        assert np.array_equal(g, g2)
        assert vec_rel_err(g, w).max() <= 1e-12


def test_evaluation_in_batches():
    n, eps = 70001, 1e-4
    x, v, m = ics.plummer(n, 902)
    a = np.ascontiguousarray(-x / ((x * x).sum(axis=1, keepdims=True) + 0.35) ** 1.5)
    got = gpu_evaluate(h6.Context(n, eps), x, v, a, m)
    idx = np.concatenate([np.arange(0, n, 521), [511, 512, 34999, 35000, 69631, 69632, n - 1]])
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=idx, order=2)[:3]
    for g, w in zip(got, want):
        assert vec_rel_err(g[idx], w).max() <= 1e-12


@pytest.mark.parametrize("n,eps", [(5001, 1e-4), (5632, 0.0)])
def test_startup(n, eps):
    x, v, m = ics.plummer(n, 910 + n)
    s = h6.System(x, v, m, eps)
    s.startup()
    want = oracle.startup(x, v, m, eps * eps)
    for name, w in zip("ajsc", want):
        assert vec_rel_err(s.field(name), w).max() <= (1e-11 if name == "c" else 1e-12), name


@pytest.mark.parametrize("n,eps", [(1, 1e-2), (2, 0.0), (64, 1e-2), (255, 1e-2), (257, 1e-2), (512, 0.0),
                                   (769, 1e-2), (1030, 1e-2)])
def test_gradient(n, eps):
    rng = np.random.Generator(np.random.PCG64(920 + n))
    x, v, a = (rng.normal(0, 1, (n, 3)) for _ in range(3))
    m = rng.uniform(0.5, 1.5, n) / n
    cot = [rng.normal(0, 1, (n, 3)) for _ in range(3)]
    GP = torch.full((9, n), np.nan, dtype=torch.float64, device=DEV)
    gm = torch.full((n,), 0.25, dtype=torch.float64, device=DEV)  # accumulated into
    h6.Context(n, eps).h6_evaluate_vjp(to_rows(x, v, a), torch.from_numpy(m).to(DEV), to_rows(*cot), GP, gm)
    if n == 1:  # no pair
        assert not GP.any() and float(gm) == 0.25
        return
    ref = ar.pair_sums_vjp(x, v, m, eps * eps, cot, a=a, order=2)
    for k, name in enumerate("xva"):
        assert np.abs(from_rows(GP, k) - ref[name]).max() <= 1e-11 * np.abs(ref[name]).max(), name
    assert np.abs(gm.cpu().numpy() - 0.25 - ref["m"]).max() <= 1e-11 * np.abs(ref["m"]).max()


@pytest.mark.parametrize("eps", [1e-2, 0.0])
@pytest.mark.parametrize("n,n_act", [(2, 1), (300, 33), (513, 513), (2199, 2199), (2200, 2200), (2305, 2305)])
def test_double_single(n, n_act, eps):
    # the bounds of the EX tests: 2e-12, 4e-12, 1e-11 for a, j, s
    x, v, m = ics.plummer(n, 930 + n)
    a = np.ascontiguousarray(-x / ((x * x).sum(axis=1, keepdims=True) + 0.35) ** 1.5)
    act = np.arange(n - n_act, n, dtype=np.int32) if n_act < n else None
    got = gpu_evaluate(h6.Context(n, eps), x, v, a, m, active=act, precision=h6.H6_EX)
    idx = None if act is None else act.astype(np.int64)
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=idx, order=2)[:3]
    for g, w, tol in zip(got, want, (2e-12, 4e-12, 1e-11)):
        assert vec_rel_err(g, w).max() <= tol
