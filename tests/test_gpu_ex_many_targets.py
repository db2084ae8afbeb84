"""Double-single evaluation of more targets than one launch holds (2^28 of them: a
list may name a particle any number of times). Each target's sums are those of the
same particle in a short list, to the bound of the EX tests' a: the first and last
entries, those at the launches' limits, and all of the first 2^28."""

import pytest
import torch

from paper_1901_08532_amd import h6, ics
from _gpu import DEV, to_rows

pytestmark = pytest.mark.gpu


def test_many_targets():
    n, n_act, eps = 64, (1 << 28) + 100, 1e-2
    if torch.cuda.mem_get_info()[0] < 128 << 30:
        pytest.skip("needs 105 GB of device memory")
    x, v, m = ics.plummer(n, 5)
    P, mt = to_rows(x, v, -x), torch.from_numpy(m).to(DEV)
    ctx = h6.Context(n_act, eps)
    short = torch.arange(n, dtype=torch.int32, device=DEV).repeat(4096)
    want = torch.empty((9, len(short)), dtype=torch.float64, device=DEV)
    ctx.h6_evaluate(P, mt, short, len(short), h6.H6_EX, want)
    act = torch.arange(n, dtype=torch.int32, device=DEV).repeat((n_act + n - 1) // n)[:n_act].contiguous()
    F = torch.empty((9, n_act), dtype=torch.float64, device=DEV)
    ctx.h6_evaluate(P, mt, act, n_act, h6.H6_EX, F)
    for k in (0, 1 << 27, 1 << 28, n_act - 64):  # 64 targets from here on
        ids = act[k:k + 64].long()
        got, ref = F[:, k:k + 64], want[:, ids]
        assert float((got - ref).abs().max()) <= 2e-12 * float(ref.abs().max()), k
    whole = (1 << 28) // n
    sums = F[:, :1 << 28].view(9, whole, n)
    assert float((sums - want[:, None, :n]).abs().amax()) <= 2e-12 * float(want.abs().max())
    ctx.close()
