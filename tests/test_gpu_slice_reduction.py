"""The reductions of slice sums at the edges of their choice: below and from 16
slices, at most 2048 outputs (a wave each) and more, whole and part rounds of a
wave's 8 x 64 loads.

Bound: 1e-12 relative to the oracle, as for the evaluation itself.
"""

import numpy as np
import pytest

import oracle
from paper_1901_08532_amd import h6
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_act", [1, 227, 228])
@pytest.mark.parametrize("n,n_split", [(2000, 15), (2000, 16), (4097, 64), (4161, 65), (32768, 512),
                                       (33000, 516)])
def test_split_sums(n, n_split, n_act):
    eps = 1e-3
    x, v, a, m = plummer_pred(n, 900 + n + n_act, eps * eps)
    act = np.random.Generator(np.random.PCG64(n_act)).choice(n, n_act, replace=False).astype(np.int32)
    ctx = h6.Context(n, eps)
    ctx.set_eval_config(block=64, ipl=1, n_split=n_split, small_max=0)
    got = gpu_evaluate(ctx, x, v, a, m, active=act)
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=act.astype(np.int64), order=2)[:3]
    for g, w in zip(got, want):
        assert vec_rel_err(g, w).max() <= 1e-12
