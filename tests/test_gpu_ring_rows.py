"""GPU parity, ring batches of any N on the 16-bit matrix in LDS (sixteen lanes per order): step and row remainders, the
largest N, every rank type, entries below and above 2^16, batches that end inside a workgroup's pass."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]

CALLS = {np.int32: cc.cc_ring_cost_batch, np.uint8: cc.cc_ring_cost_batch_u8, np.int16: cc.cc_ring_cost_batch_u16}


def _check(c, perms, rank, offset=0):
    n, b = perms.shape[1], perms.shape[0]
    room = torch.empty(b * n + offset, dtype=getattr(torch, np.dtype(rank).name), device="cuda")
    view = room[offset:].view(b, n)
    view.copy_(dev(perms.astype(rank)))
    for objective, name in ((cc.CC_RING_SUM, oracle.SUM), (cc.CC_RING_MAX, oracle.MAX)):
        got = CALLS[rank](dev(c), view, objective)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.ring_cost_batch(c, perms, name))


@pytest.mark.parametrize("rank", [np.int32, np.uint8, np.int16])
@pytest.mark.parametrize("n", [2, 7, 15, 17, 31, 33, 100, 127, 129, 130, 200, 201, 255, 256, 279, 280, 281])
def test_ring_batch_rows(n, rank):
    if rank is np.uint8 and n > 256:
        pytest.skip("one byte per rank holds N <= 256")
    first = max((96 if n == 256 else 64) * n, -(-(1 << 20) // n))             # the smallest batch that takes this kernel
    perms = random_perms(n, first + 67, seed=n)
    for top in ((1 << 16) - 1, COST_MAX):
        c = random_matrix(n, n + top % 5, symmetric=False, lo=0, hi=top)
        c[0, n - 1] = top
        for b in (first - 1, first, first + 67):
            say(f"ring batch rows N={n} B={b} {np.dtype(rank).name} largest entry {top}")
            _check(c, perms[:b], rank)


@pytest.mark.parametrize("n", [8, 16, 64, 128])
def test_ring_batch_rows_serves_unaligned_streams(n):
    say(f"ring batch rows N={n}, orders off 16-byte alignment")
    c = random_matrix(n, n, symmetric=False, lo=0, hi=60000)
    for rank in CALLS:
        _check(c, random_perms(n, (1 << 20) // n + 1, seed=n), rank, offset=1)
