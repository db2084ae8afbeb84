"""Potential, energy and the energy gradient at the edges of their launch
shapes: one to 64 targets a workgroup, 512-source tiles, 64-source slice
units, a middle block alone, part-filled last groups.

Bounds: the potential and the energies sum terms of one sign, so they hold
1e-13 relative to the oracle, as in the other tests of these calls; so does
the mass gradient |v|^2 / 2 + phi relative to |v|^2 / 2 + |phi|. The position
gradient -m a holds the evaluation's 1e-12 per particle.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import vec_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-3, 0.0])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 513, 1024, 1025, 1537, 2050, 4099, 9001])
def test_edges(n, eps):
    x, v, _ = ics.plummer(n, 800 + n)
    m = ics.salpeter_masses(n, 801)
    s = h6.System(x, v, m, eps)
    phi = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    s.ctx.h6_potential(s.S, s.m, phi)
    want = oracle.potential(x, m, eps * eps)
    assert np.abs(phi.cpu().numpy() / want - 1).max() <= 1e-13
    ek, ep, _ = s.energy()
    wk, wp, _ = oracle.energy(x, v, m, eps * eps)
    assert abs(ek - wk) <= 1e-13 * wk and abs(ep - wp) <= 1e-13 * abs(wp)
    G = torch.full((18, n), np.nan, dtype=torch.float64, device="cuda")
    gm = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    s.ctx.h6_energy_vjp(s.S, s.m, None, G, gm)
    a = oracle.forces(x, v, m, eps * eps, order=1)[0]
    assert vec_rel_err(G[0:3].T.cpu().numpy(), -m[:, None] * a).max() <= 1e-12
    half = 0.5 * (v * v).sum(axis=1)
    assert (np.abs(gm.cpu().numpy() - (half + want)) / (half + np.abs(want))).max() <= 1e-13
