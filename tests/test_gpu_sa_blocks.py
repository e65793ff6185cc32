"""GPU parity, annealing over the ring: chains around the blocks of 64 drawn steps, at the edges of the kernels' ranges of N, from
cold (whole blocks rejected) to hot (nearly every step accepted), and the largest step count the acceptance bound is computed for."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [4, 7, 31, 62, 63, 64, 65, 127, 128, 129, 256, 257])
def test_steps_around_the_blocks(n):
    c = random_matrix(n, 900 + n, symmetric=True, lo=1, hi=2000)
    d = dev(c)
    for steps in (1, 63, 64, 65, 127, 128, 129, 191, 193, 500):
        for ts, te in ((0, 0), (30, 0), (500, 500), (COST_MAX, COST_MAX)):
            say(f"sa blocks N={n} steps={steps} T={ts}->{te}")
            got = cc.cc_sa_search_ex(d, 5, steps, ts, te, 41 + n)
            torch.cuda.synchronize()
            want = oracle.sa_search(c, 5, steps, ts, te, 41 + n)
            assert np.array_equal(got.restart_costs.cpu().numpy(), want["costs"])
            assert np.array_equal(got.restart_moves.cpu().numpy(), want["accepted"])
            assert np.array_equal(got.restart_tours.cpu().numpy(), want["tours"])


def test_cold_order_stays_cold_over_many_blocks():
    """A chain started at its own result: nearly all rounds reject everything, at every offset into the block."""
    n = 20
    c = random_matrix(n, 5, symmetric=True, lo=1, hi=100000)
    init = oracle.sa_search(c, 6, 20000, 20000, 0, 3)["tours"]
    say("sa blocks cold start")
    got = cc.cc_sa_search_ex(dev(c), 6, 6000, 300, 0, 9, init_tours=dev(init))
    torch.cuda.synchronize()
    want = oracle.sa_search(c, 6, 6000, 300, 0, 9, init)
    assert np.array_equal(got.restart_moves.cpu().numpy(), want["accepted"]) and want["accepted"].max() < 300
    assert np.array_equal(got.restart_tours.cpu().numpy(), want["tours"])


def test_largest_step_count():
    """2^24 steps, the temperature at its limit: the products of the acceptance bound at their largest."""
    n = 4
    c = random_matrix(n, 6, symmetric=True, lo=1, hi=COST_MAX)
    say("sa blocks 2^24 steps")
    got = cc.cc_sa_search_ex(dev(c), 1, 1 << 24, COST_MAX, 0, 12)
    torch.cuda.synchronize()
    want = oracle.sa_search(c, 1, 1 << 24, COST_MAX, 0, 12)
    assert np.array_equal(got.restart_moves.cpu().numpy(), want["accepted"])
    assert np.array_equal(got.restart_costs.cpu().numpy(), want["costs"])
