"""The whole-workgroup evaluation and the one-kernel shared step at the edges
of their shapes: tile (512 sources), slice (64) and target-group remainders,
one target to a part-filled last group, with and without the self mask.

Evaluation bound: 1e-12 relative to the oracle, as for the other kernels.
Shared steps: the one-kernel steps (and from 4097 particles on the two-kernel
ones) and the separate kernels (a forced launch
shape) do the same arithmetic but for the order of the pair sums, which
differ by about 1e-15 relative; over the 3 steps of 1/1024 of a Plummer
sphere at softening 1/64 that stays below 1e-12 of the largest component.
The interpolated crackle divides such a difference of a by h^3 / 60, 6e10,
so it is compared at 1e-12 x 60 / h^3 of the acceleration.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import gpu_evaluate, plummer_pred, vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-4, 0.0])
@pytest.mark.parametrize("n,n_act", [(2, 1), (65, 33), (511, 2), (512, 257), (513, 513), (1025, 31),
                                     (2049, 1000), (4097, 129), (20001, 5), (9001, 3000),
                                     (12500, 9999), (12500, 10001)])
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


@pytest.mark.parametrize("n", [1, 2, 255, 257, 513, 2049, 4096, 4097])
@pytest.mark.parametrize("nsteps", [1, 3])
def test_shared_steps_one_kernel(n, nsteps):
    h, eps = 1.0 / 1024, 1.0 / 64
    x, v, m = ics.plummer(n, 700 + n)
    runs = []
    for forced in (False, True):
        s = h6.System(x, v, m, eps)
        s.startup()
        if forced:
            s.ctx.set_eval_config(block=64)
        s.shared_steps(h, nsteps)
        torch.cuda.synchronize()
        assert s.ctx.h6_check_status() == h6.H6_OK
        runs.append(s)
    one, sep = runs
    big = float(sep.S[6:9].abs().max())
    for k in range(5):  # x, v, a, j, s
        w = sep.S[3 * k:3 * k + 3]
        assert float((one.S[3 * k:3 * k + 3] - w).abs().max()) <= 1e-12 * float(w.abs().max()), k
    assert float((one.S[15:18] - sep.S[15:18]).abs().max()) <= 1e-12 * 60 / h ** 3 * max(big, 1e-300)
    # the work arrays end as with separate kernels: the last step's
    for w, g in ((sep.P, one.P), (sep.F, one.F)):
        assert float((g - w).abs().max()) <= 1e-11 * float(w.abs().max())


@pytest.mark.parametrize("n", [777, 6001])
def test_shared_steps_at_once_or_one_by_one(n):
    # the backward pass replays single steps and relies on the same values
    runs = []
    for counts in ([5], [1] * 5, [2, 3]):
        s = h6.System(*ics.plummer(n, 4), 1e-3)
        s.startup()
        for c in counts:
            s.shared_steps(1.0 / 256, c)
        runs.append((s.S, s.P, s.F))
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert torch.equal(a, b)
