"""Double-single evaluation away from Henon units: coordinates in metres with G m
as masses, where R^-3 alone leaves the single-precision exponent range and m R^-3
does not. Every form of it: active sets, all particles (whole workgroups and the
third law), shared steps (chains and the third law).

Bounds: those of the EX tests, 2e-12, 4e-12, 1e-11 for a, j, s (nothing in them
depends on the units); of the largest component for shared steps, against FP64.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import gpu_evaluate, vec_rel_err

pytestmark = pytest.mark.gpu

GM = 1.3e20  # total G m, m^3 / s^2


def _metres(n, seed, length):
    x, v, m = ics.plummer(n, seed)
    return x * length, v * np.sqrt(GM / length), m * GM


@pytest.mark.parametrize("length", [1.5e11, 1.5e13])
@pytest.mark.parametrize("n,n_act", [(300, 33), (700, 700), (2305, 2305)])
def test_evaluation_in_metres(n, n_act, length):
    x, v, m = _metres(n, 80 + n, length)
    eps = 1e-2 * length
    a = oracle.forces(x, v, m, eps * eps, order=1)[0]
    act = np.arange(n - n_act, n, dtype=np.int32) if n_act < n else None
    got = gpu_evaluate(h6.Context(n, eps), x, v, a, m, active=act, precision=h6.H6_EX)
    idx = None if act is None else act.astype(np.int64)
    want = oracle.forces(x, v, m, eps * eps, a=a, idx=idx, order=2)[:3]
    for g, w, tol in zip(got, want, (2e-12, 4e-12, 1e-11)):
        assert vec_rel_err(g, w).max() <= tol


@pytest.mark.parametrize("n", [700, 3000])
def test_shared_step_in_metres(n):
    length = 1.5e13
    x, v, m = _metres(n, 90 + n, length)
    dt = np.sqrt(length ** 3 / GM) / 4096
    runs = []
    for prec in (h6.H6_EX, h6.H6_FP64):
        s = h6.System(x, v, m, 1e-2 * length)
        s.startup()
        s.shared_steps(dt, 1, prec)
        torch.cuda.synchronize()
        assert s.ctx.h6_check_status() == h6.H6_OK
        runs.append(s)
    ex, ref = runs
    for k in range(5):  # x, v, a, j, s
        w = ref.S[3 * k:3 * k + 3]
        assert float((ex.S[3 * k:3 * k + 3] - w).abs().max()) <= 1e-11 * float(w.abs().max()), k
