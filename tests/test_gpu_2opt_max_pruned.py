"""GPU parity of the pruned max-hop descents at the edges of their launch shapes (ranks per thread, waves per restart),
directed with and without the orientation flip and undirected, on matrices with distinct entries up to the ceiling
and with many ties."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix
from gpu_util import assert_search_equal, dev, gpu_search, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [4, 5, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("directed", [False, True])
def test_pruned_max_hop_equals_the_exhaustive_sweep(n, directed):
    restarts = 12 if n <= 129 else 4 if n <= 257 else 2
    for hi in (COST_MAX, 5, 1):
        say(f"pruned max-hop N={n} directed={directed} entries<={hi} R={restarts}")
        c = random_matrix(n, 600 + n + hi % 89, symmetric=not directed, lo=0, hi=hi)
        obj = oracle.MAX_DIRECTED if directed else oracle.MAX
        assert_search_equal(gpu_search(c, obj, restarts, n), oracle.search(c, obj, restarts, n))


@pytest.mark.parametrize("n", [5, 70, 200, 300])
def test_pruned_max_hop_with_the_flip(n):
    for hi in (COST_MAX, 9):
        say(f"pruned max-hop + flip N={n} entries<={hi}")
        c = random_matrix(n, 77 + n, symmetric=False, lo=0, hi=hi)
        classes = cc.CC_MOVES_2OPT | cc.CC_MOVES_FLIP
        b = cc.cc_local_search_ex(dev(c), cc.CC_RING_MAX_DIRECTED, classes, 5, 3)
        torch.cuda.synchronize()
        costs, tours, moves = oracle.local_restarts(c, oracle.MAX_DIRECTED, classes, 3, 0, 5)
        assert np.array_equal(b.restart_costs.cpu().numpy(), costs)
        assert np.array_equal(b.restart_tours.cpu().numpy(), tours)
        assert np.array_equal(b.restart_moves.cpu().numpy(), moves)
