"""All particles by the third law at the edges of its work split: one more and
one less than a superblock (512), odd and even numbers of superblocks, runs
that cut a superblock, several batches of offsets, with the self mask.

Bounds: 1e-12 relative to the oracle for a, j, s and 1e-11 for the start-up's
crackle, as for the other evaluation kernels.
"""

import numpy as np
import pytest

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

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
