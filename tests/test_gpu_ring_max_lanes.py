"""GPU parity, max-hop ring batches by marked hops: both sides of every number of ranks per lane, the smallest batch of the kernel, one order
more than a pass, matrices whose marks are few, all the largest entry, or many beside a rare largest one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [281, 320, 321, 384, 385, 448, 449, 512, 513, 576, 577, 640, 641, 704, 705, 768, 769, 896, 897, 960, 961, 1024])
def test_every_number_of_ranks_per_lane(n):
    rng = np.random.default_rng(n)
    b = 24577
    perms = random_perms(n, b, seed=n)
    perms[-1] = np.arange(n)[::-1]
    two = rng.integers(0, 2, size=(n, n)).astype(np.int32) * 7 + 2
    rare = np.where(rng.random((n, n)) < 1.0 / n, 3, rng.integers(1, 3, size=(n, n))).astype(np.int32)
    for name, c in (("spread", random_matrix(n, n, symmetric=False, lo=0, hi=1 << 20)), ("two values", two), ("rare largest", rare)):
        say(f"max-hop ring batch, ranks per lane, N={n} B={b}, {name}")
        want = oracle.ring_cost_batch(c, perms, oracle.MAX)
        for call, rank in ((cc.cc_ring_cost_batch, np.int32), (cc.cc_ring_cost_batch_u16, np.int16)):
            got = call(dev(c), dev(perms.astype(rank)), cc.CC_RING_MAX)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want)
