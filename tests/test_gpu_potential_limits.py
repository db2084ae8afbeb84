"""Potential and energy gradient on both sides of the largest system that takes each
pair once (one batch of slots: 137728 particles for the potential, 91136 for the
gradient on 256 CUs). Bounds as at the other sizes: 1e-13 for the potential and the
mass gradient, 1e-12 for the position gradient, on sampled particles."""

import numpy as np
import pytest
import torch

import oracle
from paper_1901_08532_amd import h6, ics
from _gpu import vec_rel_err

pytestmark = pytest.mark.gpu


def _potential(x, m, eps, idx):
    out = np.empty(len(idx))
    for q, i in enumerate(idx):
        r2 = ((x - x[i]) ** 2).sum(axis=1) + eps * eps
        t = m / np.sqrt(r2)
        t[i] = 0.0
        out[q] = -t.sum()
    return out


@pytest.mark.parametrize("n", [91136, 91137, 137728, 137729])
def test_both_sides(n):
    eps = 1e-3
    x, v, m = ics.plummer(n, n)
    s = h6.System(x, v, m, eps)
    idx = np.unique(np.linspace(0, n - 1, 40).astype(np.int64))
    want = _potential(x, m, eps, idx)
    phi = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    s.ctx.h6_potential(s.S, s.m, phi)
    assert np.abs(phi.cpu().numpy()[idx] / want - 1).max() <= 1e-13
    G = torch.full((18, n), np.nan, dtype=torch.float64, device="cuda")
    gm = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    s.ctx.h6_energy_vjp(s.S, s.m, None, G, gm)
    a = oracle.forces(x, v, m, eps * eps, idx=idx, order=1)[0]
    assert vec_rel_err(G[0:3].T.cpu().numpy()[idx], -m[idx, None] * a).max() <= 1e-12
    half = 0.5 * (v[idx] ** 2).sum(axis=1)
    assert (np.abs(gm.cpu().numpy()[idx] - (half + want)) / (half + np.abs(want))).max() <= 1e-13
