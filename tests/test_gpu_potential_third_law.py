"""Potential and energy gradient with each pair taken once, at the edges of that
form: from 6000 particles on, superblocks of 512 and 1024, 64-source chunks, even
and odd superblock counts, part-filled last ones.

Bounds as for the ordered form: 1e-13 relative to the oracle for the potential
and the mass gradient (terms of one sign), 1e-12 per particle for the position
gradient.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-3, 0.0])
@pytest.mark.parametrize("n", [5999, 6000, 6145, 7168, 8192, 12289])
def test_edges(n, eps):
    x, v, _ = ics.plummer(n, 60 + n)
    m = ics.salpeter_masses(n, 61)
    s = h6.System(x, v, m, eps)
    phi = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    s.ctx.h6_potential(s.S, s.m, phi)
    want = oracle.potential(x, m, eps * eps)
    assert np.abs(phi.cpu().numpy() / want - 1).max() <= 1e-13
    G = torch.full((18, n), np.nan, dtype=torch.float64, device="cuda")
    gm = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    cot = torch.tensor([-0.75], dtype=torch.float64, device="cuda")
    s.ctx.h6_energy_vjp(s.S, s.m, cot, G, gm)
    a = oracle.forces(x, v, m, eps * eps, order=1)[0]
    assert vec_rel_err(G[0:3].T.cpu().numpy(), 0.75 * m[:, None] * a).max() <= 1e-12
    assert np.array_equal(G[3:6].T.cpu().numpy(), -0.75 * (m[:, None] * v))
    half = 0.5 * (v * v).sum(axis=1)
    err = np.abs(gm.cpu().numpy() + 0.75 * (half + want)) / (half + np.abs(want))
    assert err.max() <= 1e-13
