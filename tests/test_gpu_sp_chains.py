"""Single-precision chains by two waves (up to 1536 chains of 64 targets on 256
CUs) and by one: batches of 8 sources, tiles and slices of 64, part-filled last
ones, the smallest sets and the sizes on both sides of the choice.

Bounds: those of the single-precision evaluation, 1e-4 (a), 2e-4 (j), 5e-4 (s)
relative to the oracle, at a softening of 1e-2.
"""

import numpy as np
import pytest

import oracle
from paper_1901_08532_amd import h6
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_act", [(1, 1), (2, 2), (7, 3), (63, 63), (64, 1), (65, 65), (129, 64),
                                     (1000, 7), (4097, 4097), (20001, 65), (98304, 98304),
                                     (98305, 98305)])
def test_against_oracle(n, n_act):
    eps = 1e-2
    x, v, a, m = plummer_pred(min(n, 20001), 70 + n, eps * eps)
    if n > 20001:  # five copies of the sphere, apart
        rng = np.random.Generator(np.random.PCG64(n))
        pick = rng.integers(0, 20001, n)
        x, v, a, m = x[pick] + 0.5 * rng.standard_normal((n, 3)), v[pick], a[pick], m[pick] / 5
    act = np.random.Generator(np.random.PCG64(n_act)).permutation(n)[:n_act].astype(np.int32)
    got = gpu_evaluate(h6.Context(n, eps), x, v, a, m, active=act, precision=h6.H6_SP)
    some = np.unique(np.linspace(0, n_act - 1, 60).astype(np.int64))
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=act[some].astype(np.int64), order=2)[:3]
    if n == 1:
        assert all(np.all(g == 0.0) for g in got)
        return
    for g, w, bound in zip(got, want, (1e-4, 2e-4, 5e-4)):
        assert vec_rel_err(g[some], w).max() <= bound
