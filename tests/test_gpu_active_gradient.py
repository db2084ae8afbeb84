"""The gradient of an active set's evaluation at the edges of its launch shapes:
rings of 4, 16 and 64 sources and their remainders, one tile of particles per
workgroup or four, chunks in parts, tile groups in batches, unsorted lists.

Bound: 1e-11 of the largest component, as in the other adjoint tests; against
the autograd reference for small systems, against the all-pairs gradient
(tested against it elsewhere) with zero cotangents off the set for large ones.
"""

import numpy as np
import pytest
import torch

import oracle.adjoint_ref as ar
from paper_1901_08532_amd import h6
from _gpu import DEV, from_rows, to_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-2, 0.0])
@pytest.mark.parametrize("n,n_act", [(2, 1), (65, 4), (64, 5), (130, 16), (257, 17), (300, 48), (300, 49),
                                     (511, 65), (700, 700)])
def test_against_the_reference(n, n_act, eps):
    rng = np.random.Generator(np.random.PCG64(n + n_act))
    x, v, a = (rng.normal(0, 1, (n, 3)) for _ in range(3))
    m = rng.uniform(0.5, 1.5, n) / n
    act = rng.permutation(n)[:n_act].astype(np.int32)
    cot = [rng.normal(0, 1, (n_act, 3)) for _ in range(3)]
    full = [np.zeros((n, 3)) for _ in range(3)]
    for f, c in zip(full, cot):
        f[act] = c
    ref = ar.pair_sums_vjp(x, v, m, eps * eps, full, a=a, order=2)
    GP = torch.full((9, n), 0.5, dtype=torch.float64, device=DEV)  # accumulated into
    gm = torch.full((n,), 0.25, dtype=torch.float64, device=DEV)
    h6.Context(n, eps).h6_evaluate_vjp_active(to_rows(x, v, a), torch.from_numpy(m).to(DEV),
                                              torch.from_numpy(act).to(DEV), n_act, to_rows(*cot), GP, gm)
    for k, name in enumerate("xva"):
        tol = 1e-11 * max(np.abs(ref[name]).max(), 0.5)
        assert np.abs(from_rows(GP, k) - 0.5 - ref[name]).max() <= tol, name
    assert np.abs(gm.cpu().numpy() - 0.25 - ref["m"]).max() <= 1e-11 * max(np.abs(ref["m"]).max(), 0.25)


@pytest.mark.parametrize("n,n_act", [(20001, 1000), (40000, 30001)])
def test_against_all_pairs(n, n_act):
    g = torch.Generator(device=DEV).manual_seed(n)

    def rand(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)

    P, CF, m = rand(9, n), rand(9, n_act), rand(n).abs() / n
    act = torch.randperm(n, generator=g, device=DEV)[:n_act]
    full = torch.zeros((9, n), dtype=torch.float64, device=DEV)
    full[:, act] = CF
    ctx = h6.Context(n, 1e-2)
    G1, G2 = torch.zeros_like(P), torch.zeros_like(P)
    m1, m2 = torch.zeros_like(m), torch.zeros_like(m)
    ctx.h6_evaluate_vjp_active(P, m, act.to(torch.int32), n_act, CF, G1, m1)
    ctx.h6_evaluate_vjp(P, m, full, G2, m2)
    for k in range(3):
        w = G2[3 * k:3 * k + 3]
        assert float((G1[3 * k:3 * k + 3] - w).abs().max()) <= 1e-11 * float(w.abs().max())
    assert float((m1 - m2).abs().max()) <= 1e-11 * float(m2.abs().max())
