"""Device memory a context takes: 18 doubles a particle of partial sums for the
largest systems (45 up to 2^23 particles), energy partials of 5 bytes a particle,
scheduler arrays of less than 1, rounded up by the allocator (64 MiB allowed)."""

import pytest
import torch

from paper_1901_08532_amd import h6

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,doubles", [((1 << 23) + 1, 18), (20_000_000, 18), (1 << 23, 45)])
def test_context_memory(n, doubles):
    h6.Context(1000, 1e-2).close()  # the library's code and fixed scratch are loaded by the first one
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    ctx = h6.Context(n, 1e-2)
    taken = free0 - torch.cuda.mem_get_info()[0]
    ctx.close()
    assert taken <= (8 * doubles + 6) * n + (64 << 20), taken / n
