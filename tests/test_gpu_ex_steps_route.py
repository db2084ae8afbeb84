"""Which evaluation double-single shared steps take, on both sides of its limits:
chains below 3000 particles, the third law from there on, in one batch of slots
(with the corrector on the slots) or in several (large systems, separate kernels).

Bounds: those of the EX tests, 2e-12, 4e-12, 1e-11 for a, j, s, on sampled targets
against the oracle at the step's predicted state.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import from_rows, vec_rel_err

pytestmark = pytest.mark.gpu

CHAINS, THIRD_LAW = 0, 3  # kinds of the measurement hook


@pytest.mark.parametrize("n,kind", [(2999, CHAINS), (3000, THIRD_LAW), (30001, THIRD_LAW), (33001, THIRD_LAW),
                                    (40001, THIRD_LAW)])
def test_route(n, kind):
    eps = 1e-2
    x, v, m = ics.plummer(n, 40 + n)
    s = h6.System(x, v, m, eps)
    s.startup()
    s.ctx.h6_profile_enable(1)
    s.shared_steps(1.0 / 4096, 1, h6.H6_EX)
    recs = s.ctx.h6_profile_read()
    assert [(r["order"], r["precision"], r["kind"]) for r in recs] == [(2, h6.H6_EX, kind)]
    xp, vp, ap = (from_rows(s.P, k) for k in range(3))
    idx = np.unique(np.linspace(0, n - 1, 60).astype(np.int64))
    want = oracle.forces(xp, vp, m, eps * eps, a=ap, idx=idx, order=2)[:3]
    for name, w, tol in zip("ajs", want, (2e-12, 4e-12, 1e-11)):
        assert vec_rel_err(s.field(name)[idx], w).max() <= tol, name
