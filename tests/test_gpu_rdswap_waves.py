"""GPU parity of the pair-swap descents on both sides of every restart count at which their wavefronts per restart change."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import hierarchical_matrix, random_matrix
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n,restarts", [(8, 3072), (8, 3073), (16, 1536), (16, 1537), (16, 3073), (32, 768), (32, 769), (32, 3073), (64, 768),
                                        (64, 769), (64, 1281), (128, 257), (256, 257), (512, 2), (512, 257), (1024, 1), (1024, 257),
                                        (8, 2304), (8, 2305), (32, 2560), (32, 2561), (64, 512), (64, 513)])
def test_every_number_of_wavefronts(n, restarts):
    matrices = [(hierarchical_matrix(n, (4, 8), ((50, 100), (200, 400), (800, 2000)), 0.3, False, n), "racks")]
    if n < 512:
        matrices += [(random_matrix(n, n, symmetric=False, lo=0, hi=6), "ties"),
                     (random_matrix(n, n, symmetric=False, lo=0, hi=1 << 20), "beyond 2^16")]
    for c, tag in matrices:
        say(f"pair swaps, wavefronts per restart N={n} R={restarts} {tag}")
        b = cc.cc_rd_swap_search_ex(dev(c), restarts, 5)
        torch.cuda.synchronize()
        costs, tours, moves = b.restart_costs.cpu().numpy(), b.restart_tours.cpu().numpy(), b.restart_moves.cpu().numpy()
        for r in {0, restarts - 1} if n <= 512 else {restarts - 1}:
            oc, ot, om = oracle.rd_swap_restarts(c, 5, r, r + 1)
            assert costs[r] == oc[0] and moves[r] == om[0] and np.array_equal(tours[r], ot[0])
        k = int(np.argmin(costs))
        assert int(b.best_restart.item()) == k and int(b.best_cost.item()) == costs[k]


@pytest.mark.parametrize("n,restarts", [(512, 128), (512, 129), (512, 257), (1024, 32), (1024, 33), (1024, 257)])
def test_pairs_beside_and_after_the_scans(n, restarts):
    """Equal values, and entries from 2^16 up, where the pairs come beside the scans or after them by the number of restarts; above
    256 restarts no wavefronts are there for them."""
    ties = random_matrix(n, n, symmetric=True, lo=0, hi=400)
    for c, tag in [(ties, "ties"), (ties * 4000, "ties beyond 2^16")] + \
                  ([(random_matrix(n, n, symmetric=False, lo=0, hi=1 << 20), "beyond 2^16")] if n == 512 else []):
        say(f"pair swaps, pairs beside or after the scans N={n} R={restarts} {tag}")
        b = cc.cc_rd_swap_search_ex(dev(c), restarts, 9)
        torch.cuda.synchronize()
        r = restarts - 1
        oc, ot, om = oracle.rd_swap_restarts(c, 9, r, r + 1)
        assert int(b.restart_costs[r].item()) == oc[0] and int(b.restart_moves[r].item()) == om[0]
        assert np.array_equal(b.restart_tours[r].cpu().numpy(), ot[0])
