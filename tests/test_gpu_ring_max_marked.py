"""GPU parity, max-hop ring batches at 280 < N <= 1024 (marked hops): row and word remainders, matrices whose marks are
many, few or none, orders all of whose hops are small, batches that end inside a workgroup's pass."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


def _matrices(n):
    yield "spread", random_matrix(n, n, symmetric=False, lo=0, hi=COST_MAX)
    yield "zeros", np.zeros((n, n), dtype=np.int32)
    rng = np.random.default_rng(n)
    levels = np.array([5, 40, 41], dtype=np.int32)[rng.choice(3, size=(n, n), p=[0.05, 0.05, 0.9])]
    np.fill_diagonal(levels, 0)
    yield "three levels, most at the top", levels
    rare = random_matrix(n, n + 1, symmetric=False, lo=1, hi=9)
    rare[n - 1, 0] = COST_MAX
    yield "one large entry", rare
    near = np.abs(np.subtract.outer(np.arange(n), np.arange(n))).astype(np.int32)      # the identity's hops are 1, but one
    yield "distance on a line", near


@pytest.mark.parametrize("n", [281, 319, 320, 321, 500, 512, 1000, 1023, 1024])
def test_ring_batch_max_marked(n):
    b = 28672 + 5                                      # just above the smallest batch that takes this kernel
    perms = random_perms(n, b, seed=n)
    perms[0] = np.arange(n)
    perms[1] = np.roll(np.arange(n), 3)[::-1]
    for name, c in _matrices(n):
        say(f"max-hop ring batch, marked hops, N={n} B={b}, {name}")
        want = oracle.ring_cost_batch(c, perms, oracle.MAX)
        for call, rank in ((cc.cc_ring_cost_batch, np.int32), (cc.cc_ring_cost_batch_u16, np.int16)):
            room = torch.empty(b * n + 1, dtype=getattr(torch, np.dtype(rank).name), device="cuda")
            view = room[1:].view(b, n)                 # off 16-byte alignment
            view.copy_(dev(perms.astype(rank)))
            got = call(dev(c), view, cc.CC_RING_MAX)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want)

