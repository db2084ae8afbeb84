"""The whole-workgroup evaluation at the edges of its
shapes: tile (512 sources), slice (64) and target-group remainders,
one target to a part-filled last group, with and without the self mask.

Evaluation bound: 1e-12 relative to the oracle, as for the other kernels.
"""

import numpy as np
import pytest

import oracle
from paper_1901_08532_amd import h6
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-4, 0.0])
@pytest.mark.parametrize("n,n_act", [(2, 1), (65, 33), (511, 2), (512, 257), (513, 513), (1025, 31),
                                     (2049, 1000), (4097, 129), (20001, 5), (9001, 3000)])
def test_evaluation_edges(n, n_act, eps):
    x, v, a, m = plummer_pred(n, 500 + n + n_act, eps * eps)
    rng = np.random.Generator(np.random.PCG64(n_act))
    act = rng.choice(n, n_act, replace=False).astype(np.int32)
    ctx = h6.Context(n, eps)
    got = gpu_evaluate(ctx, x, v, a, m, active=act)
    again = gpu_evaluate(ctx, x, v, a, m, active=act)
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=act.astype(np.int64), order=2)[:3]
    for g, g2, w in zip(got, again, want):
        assert np.array_equal(g, g2)
        assert vec_rel_err(g, w).max() <= 1e-12
