"""GPU parity of the ring-sum descents with several wavefronts per restart: every number of wavefronts the launches choose, of the kernel
that keeps pairs and of the pruned one that goes on with what it leaves, entries on both sides of 2^16, ties, costs of two values."""
import numpy as np
import pytest

import oracle
from gen import hierarchical_matrix, random_matrix
from gpu_util import gpu_search, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n,restarts", [(129, 3), (129, 300), (192, 256), (192, 257), (193, 3), (256, 256), (257, 3), (257, 257), (257, 513),
                                        (448, 257), (512, 513), (513, 257), (768, 2), (769, 2)])
def test_every_number_of_wavefronts(n, restarts):
    zones = np.where(np.random.default_rng(n).integers(0, 2, n)[:, None] == np.random.default_rng(n).integers(0, 2, n)[None, :], 100, 1000)
    np.fill_diagonal(zones, 0)
    for c, tag in ((hierarchical_matrix(n, (4, 8), ((50, 100), (200, 400), (800, 2000)), 0.3, True, n), "racks"),
                   (random_matrix(n, n, symmetric=True, lo=0, hi=4), "ties"), (zones.astype(np.int32), "two zones"),
                   (random_matrix(n, n, symmetric=True, lo=1, hi=1 << 20), "beyond 2^16")):
        say(f"pruned ring sum groups N={n} R={restarts} {tag}")
        got = gpu_search(c, oracle.SUM, restarts, 21)
        k = int(np.argmin(got["costs"]))
        assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]
        for r in {0, restarts // 2, restarts - 1}:
            costs, tours, moves = oracle.restarts(c, oracle.SUM, 21, r, r + 1)
            assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0]
            assert np.array_equal(got["tours"][r], tours[0])


@pytest.mark.parametrize("n,restarts", [(200, 300), (208, 257), (209, 257), (225, 512), (246, 300), (255, 257), (256, 300)])
def test_two_restarts_per_unit_with_short_lists(n, restarts):
    """Passed candidates by entry and by place, lists so short that many nodes are scanned against every node."""
    test_every_number_of_wavefronts(n, restarts)


@pytest.mark.parametrize("n,restarts", [(300, 513), (320, 600), (384, 513), (448, 513), (449, 513), (512, 257), (512, 513), (513, 2), (640, 257),
                                        (768, 2), (768, 257), (769, 257), (1024, 2)])
def test_every_number_of_wavefronts_of_what_is_left(n, restarts):
    """Two zones of equal costs: about an eighth of all N^2 pairs stand for the first moves, 11000 at N = 300 and 33000 at N = 513, more
    than there is room for (2000 to 4500 with several restarts per unit, 17000 with one), so every descent is left at once."""
    say(f"pruned ring sum groups N={n} R={restarts}: descents that are left")
    zone = np.random.default_rng(n).permutation(n) * 2 // n
    for near, far in ((100, 1000), (1 << 16, 1 << 20)):
        c = np.where(zone[:, None] == zone[None, :], near, far).astype(np.int32)
        np.fill_diagonal(c, 0)
        got = gpu_search(c, oracle.SUM, restarts, 22)
        k = int(np.argmin(got["costs"]))
        assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]
        for r in (0, restarts - 1):
            costs, tours, moves = oracle.restarts(c, oracle.SUM, 22, r, r + 1)
            assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0] and np.array_equal(got["tours"][r], tours[0])
