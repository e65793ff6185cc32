"""GPU parity, halving-doubling and base-4 BCube batches at N = 4 .. 32 (one order per lane): batches around a wavefront and
beyond one pass of the grid, weighted rounds, order streams off 16-byte alignment."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n,base", [(4, 2), (8, 2), (16, 2), (32, 2), (4, 4), (16, 4)])
def test_rounds_batch_small(n, base):
    c = random_matrix(n, n + base, symmetric=False, lo=0, hi=COST_MAX)
    rounds = {2: {4: 2, 8: 3, 16: 4, 32: 5}, 4: {4: 1, 16: 2}}[base][n]
    w = np.array([3, 0, 1 << 30, 7, 1][:rounds], dtype=np.int32)
    b_all = 256 * 2048 + 5                                  # one order more than a full grid takes in a pass, and some
    perms = random_perms(n, b_all, seed=n)
    want = oracle.bcube_cost_batch(c, base, perms)
    weighted = oracle.bcube_cost_weighted_batch(c, base, w, perms[:333])
    for offset in (0, 1):
        room = torch.empty(b_all * n + offset, dtype=torch.int32, device="cuda")
        view = room[offset:].view(b_all, n)
        view.copy_(dev(perms))
        for b in (1, 63, 65, 257, b_all):
            say(f"rounds batch N={n} base={base} B={b} offset={offset}")
            got = cc.cc_bcube_cost_batch(dev(c), base, view[:b])
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want[:b])
        got = cc.cc_bcube_cost_batch_weighted(dev(c), base, dev(w), view[:333])
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), weighted)
