"""Double-single shared steps at the edges of their two forms: chains below 3000
particles (64 targets and sources a tile, batches of 8, part-filled last ones),
the third law from there on.

Bound: the double-single evaluation's largest, 1e-11 (the snap), of the largest
component against FP64 steps by the separate kernels.
"""

import pytest
import torch

from paper_1901_08532_amd import h6, ics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1.0 / 64, 0.0])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 71, 700, 1025, 2999, 3000])
def test_one_step(n, eps):
    x, v, m = ics.plummer(n, 50 + n)
    runs = []
    for prec in (h6.H6_EX, h6.H6_FP64):
        s = h6.System(x, v, m, eps)
        s.startup()
        if prec == h6.H6_FP64:
            s.ctx.set_eval_config(block=64)
        s.shared_steps(1.0 / 4096, 1, prec)
        torch.cuda.synchronize()
        assert s.ctx.h6_check_status() == h6.H6_OK
        runs.append(s)
    ex, ref = runs
    for k in range(5):  # x, v, a, j, s
        w = ref.S[3 * k:3 * k + 3]
        assert float((ex.S[3 * k:3 * k + 3] - w).abs().max()) <= 1e-11 * float(w.abs().max()), k
