"""The mixed whole-workgroup evaluation and one-kernel shared step at the edges
of their shapes: runs of 8 sources, slices (64), tiles (512) and target groups
(16, 32), the smallest (33) and largest sets, with and without the self mask.

Both kernels and the tiled one (a forced launch shape) add the same FP32 sums of
8 consecutive sources in FP64, in another order: n / 8 roundings of 1.1e-16 of
a sum that cancels at most a thousandfold, 1e-11 relative. Other FP32 sums
would differ by 1e-7.
"""

import numpy as np
import pytest
import torch

from paper_1901_08532_amd import h6, ics
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-4, 0.0])
@pytest.mark.parametrize("n,n_act", [(33, 33), (65, 34), (257, 48), (511, 100), (513, 513),
                                     (1031, 49), (4097, 1000), (20001, 33), (10007, 10007),
                                     (20001, 6249), (20001, 6250)])
def test_evaluation_edges(n, n_act, eps):
    x, v, a, m = plummer_pred(n, 300 + n + n_act, eps * eps)
    act = np.random.Generator(np.random.PCG64(n_act)).choice(n, n_act, replace=False).astype(np.int32)
    got = []
    for block in (0, 64):
        ctx = h6.Context(n, eps)
        if block:
            ctx.set_eval_config(block=block)
        got.append(gpu_evaluate(ctx, x, v, a, m, active=act, precision=h6.H6_MIXED))
    for g, w in zip(*got):
        assert vec_rel_err(g, w).max() <= 1e-11


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 513, 2049, 4096, 4097])
def test_shared_step(n):
    x, v, m = ics.plummer(n, 700 + n)
    runs = []
    for forced in (False, True):
        s = h6.System(x, v, m, 1.0 / 64)
        s.startup()
        if forced:
            s.ctx.set_eval_config(block=64, small_max=32)
        s.shared_steps(1.0 / 1024, 1, h6.H6_MIXED)
        torch.cuda.synchronize()
        assert s.ctx.h6_check_status() == h6.H6_OK
        runs.append(s)
    one, sep = runs
    for k in range(5):  # x, v, a, j, s
        w = sep.S[3 * k:3 * k + 3]
        assert float((one.S[3 * k:3 * k + 3] - w).abs().max()) <= 1e-11 * float(w.abs().max()), k
