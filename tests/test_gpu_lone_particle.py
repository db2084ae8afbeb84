"""Potential and energy gradient of one particle: no pairs, so potential 0, mass
gradient |v|^2 / 2 and no force, wherever it is, at infinity too (where only the
force's component along the infinite coordinate, infinity times zero, is undefined)."""

import pytest
import torch

from paper_1901_08532_amd import h6

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-2, 0.0])
@pytest.mark.parametrize("x", [0.25, 1e18, -1e18, float("inf"), float("-inf")])
def test_one_particle(x, eps):
    S = torch.zeros((18, 1), dtype=torch.float64, device="cuda")
    S[0], S[1], S[2], S[3], S[4], S[5] = x, 0.5, -2.0, 1.0, 2.0, 3.0
    m = torch.tensor([0.75], dtype=torch.float64, device="cuda")
    phi, G, gm = torch.full_like(m, float("nan")), torch.full_like(S, float("nan")), torch.full_like(m, float("nan"))
    ctx = h6.Context(1, eps)
    ctx.h6_potential(S, m, phi)
    ctx.h6_energy_vjp(S, m, None, G, gm)
    assert float(phi) == 0.0
    assert float(gm) == 7.0
    assert G[3:6, 0].tolist() == [0.75, 1.5, 2.25]
    assert G[1:3, 0].abs().tolist() == [0.0, 0.0]
    assert not torch.isfinite(S[0]).all() or float(G[0]) == 0.0
