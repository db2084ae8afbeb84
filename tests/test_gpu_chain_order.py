"""What the serial chains of the FP32-based evaluations keep.

Single precision: the two-wave kernel takes a target's additions in the order of the
one-wave kernel, so the sums are the same bits. More than 1536 chains of 64 targets
(on 256 CUs) take the one-wave kernel, fewer the two-wave one; with 1024 or more
both take each target's sources in one slice.

Double-single shared steps: the crackle, a difference of accelerations over h^3, with
the error that the evaluation's bounds allow it: a, j, s of the step's end off by
2e-12, 4e-12, 1e-11 of their size move it by (60 da + 36 h dj + 9 h^2 ds) / h^3.
"""

import numpy as np
import pytest
import torch

from paper_1901_08532_amd import h6, ics
from _gpu import DEV, to_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-2, 0.0])
@pytest.mark.parametrize("n", [3, 64, 71, 1000, 2085])
def test_single_precision_bits(n, eps):
    x, v, m = ics.plummer(n, 20 + n)
    P, mt = to_rows(x, v, -x), torch.from_numpy(m).to(DEV)
    one_wave, two_waves = 64 * 1537, 64 * 1100
    ctx = h6.Context(one_wave, eps)
    act = torch.arange(one_wave, device=DEV).remainder(n).to(torch.int32)
    F1 = torch.full((9, one_wave), float("nan"), dtype=torch.float64, device=DEV)
    F2 = torch.full((9, two_waves), float("nan"), dtype=torch.float64, device=DEV)
    ctx.h6_evaluate(P, mt, act, one_wave, h6.H6_SP, F1)
    ctx.h6_evaluate(P, mt, act, two_waves, h6.H6_SP, F2)
    assert torch.isfinite(F1).all()
    assert torch.equal(F1[:, :two_waves], F2)


@pytest.mark.parametrize("n", [64, 200, 700, 2999, 3000])
def test_crackle_of_double_single_steps(n):
    h, eps = 1.0 / 256, 1.0 / 64
    x, v, m = ics.plummer(n, 30 + n)
    runs = []
    for prec in (h6.H6_EX, h6.H6_FP64):
        s = h6.System(x, v, m, eps)
        s.startup()
        s.shared_steps(h, 1, prec)
        torch.cuda.synchronize()
        runs.append(s)
    size = {k: np.linalg.norm(runs[1].field(k), axis=1) for k in "ajs"}
    bound = (60 * 2e-12 * size["a"] + 36 * h * 4e-12 * size["j"] + 9 * h * h * 1e-11 * size["s"]) / h ** 3
    off = np.linalg.norm(runs[0].field("c") - runs[1].field("c"), axis=1)
    assert (off <= bound).all(), float((off / bound).max())
