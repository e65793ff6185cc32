"""GPU parity of the pruned insertion descents, with and without 2-opt, at the edges of their launch shapes: every restart
with several wavefronts, with one, and a workgroup per restart; ties, entries beyond 2^16, orders that are no
permutation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, hierarchical_matrix, random_matrix
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]
BOTH, INSERTION = cc.CC_MOVES_2OPT | cc.CC_MOVES_OROPT, cc.CC_MOVES_OROPT


def check(c, classes, restarts, seed, sample):
    b = cc.cc_local_search_ex(dev(c), cc.CC_RING_SUM, classes, restarts, seed)
    torch.cuda.synchronize()
    costs, tours, moves = b.restart_costs.cpu().numpy(), b.restart_tours.cpu().numpy(), b.restart_moves.cpu().numpy()
    for r in sample:
        oc, ot, om = oracle.local_restarts(c, oracle.SUM, classes, seed, r, r + 1)
        assert costs[r] == oc[0] and moves[r] == om[0] and np.array_equal(tours[r], ot[0])
    k = int(np.argmin(costs))
    assert int(b.best_restart.item()) == k and int(b.best_cost.item()) == costs[k]
    assert np.array_equal(b.best_perm.cpu().numpy(), tours[k])


@pytest.mark.parametrize("n", [9, 10, 63, 65, 127, 129, 193, 255, 256, 257, 321, 385])
@pytest.mark.parametrize("classes", [BOTH, INSERTION])
def test_pruned_insertion_equals_the_exhaustive_sweep(n, classes):
    restarts = 20 if n < 64 else 4 if n < 200 else 2
    for hi in (COST_MAX, 65535, 3) if n < 256 else (70000, 3):
        say(f"pruned insertion N={n} classes={classes} entries<={hi} R={restarts}")
        check(random_matrix(n, 30 + n + hi % 79, symmetric=True, lo=0, hi=hi), classes, restarts, n, range(restarts))


@pytest.mark.parametrize("n,restarts", [(33, 3000), (80, 1100), (150, 520), (130, 400)])
def test_restarts_that_share_a_workgroup(n, restarts):
    say(f"pruned insertion N={n} R={restarts}: nine restarts and the winner compared")
    check(random_matrix(n, n, symmetric=True, lo=1, hi=4000), BOTH, restarts, 5, np.linspace(0, restarts - 1, 9).astype(int))


@pytest.mark.parametrize("n", [40, 150, 300])
def test_orders_that_are_no_permutation_end(n):
    say(f"pruned insertion N={n}: orders that are no permutation")
    init = np.random.default_rng(6).integers(-5, n + 5, size=(3, n)).astype(np.int32)
    c = random_matrix(n, 18, symmetric=True, lo=0, hi=30)
    b = cc.cc_local_search_ex(dev(c), cc.CC_RING_SUM, BOTH, 3, 1, init_tours=dev(init))
    torch.cuda.synchronize()
    clamped = np.clip(init, 0, n - 1)
    assert (b.restart_costs.cpu().numpy() <= [oracle.ring_cost(c, t) for t in clamped]).all()


@pytest.mark.parametrize("n", [150, 256, 400])
def test_a_node_twice_in_one_wavefronts_ranks_leaves_the_order_alone(n):
    """Only one wavefront of the restart sees the repeated node; all of them have to stop, while the next restart's search."""
    restarts = min((n + 63) // 64, 6) + 1
    init = np.stack([np.random.default_rng(r).permutation(n) for r in range(restarts)]).astype(np.int32)
    for r in range(restarts - 1):
        init[r, 64 * r] = init[r, min(64 * (r + 1), n) - 1]        # both are ranks of wavefront r
    say(f"pruned insertion N={n}: a node twice among one wavefront's ranks")
    c = random_matrix(n, 19, symmetric=True, lo=0, hi=3000)
    b = cc.cc_local_search_ex(dev(c), cc.CC_RING_SUM, BOTH, restarts, 1, init_tours=dev(init))
    torch.cuda.synchronize()
    costs, tours, moves = b.restart_costs.cpu().numpy(), b.restart_tours.cpu().numpy(), b.restart_moves.cpu().numpy()
    assert np.array_equal(tours[:-1], init[:-1]) and not moves[:-1].any()
    assert np.array_equal(costs[:-1], [oracle.ring_cost(c, t) for t in init[:-1]])
    oc, ot, om = oracle.local_restarts(c, oracle.SUM, BOTH, 1, 0, 1, init=init[-1:])
    assert costs[-1] == oc[0] and moves[-1] == om[0] and np.array_equal(tours[-1], ot[0])


def _zones(n, count, near=1, far=10):
    """Equal costs inside a zone, equal ones across."""
    zone = np.random.default_rng(n).permutation(n) * count // n
    c = np.where(zone[:, None] == zone[None, :], near, far)
    return np.where(np.eye(n, dtype=bool), 0, c).astype(np.int32)


@pytest.mark.parametrize("n", [64, 65, 96, 128, 150, 192, 256, 257, 400])
@pytest.mark.parametrize("classes", [BOTH, INSERTION])
def test_few_values_go_to_the_exhaustive_kernel(n, classes):
    """Either side of the lines: one zone of equal costs to thirty, with entries below 2^16 and beyond."""
    restarts = 3 if n < 200 else 2
    for count, near, far in ((1, 5, 5), (2, 1, 10), (2, 9000, 90000), (3, 1, 10), (4, 2, 3), (8, 1, 10), (30, 0, 10)):
        say(f"insertion N={n} classes={classes} {count} zones {near}/{far} R={restarts}")
        check(_zones(n, count, near, far), classes, restarts, n, range(restarts))


def test_ties_do_not_score_every_pair():
    """Two zones of equal costs take less time than costs that all differ (2.7 times as long in the pruned kernel)."""
    n, restarts = 192, 256
    say(f"insertion N={n} R={restarts}: time with two zones of equal costs")
    buffers = cc.SearchBuffers(n, oracle.SUM, restarts, "cuda")

    def seconds(c):
        c, best = dev(c), float("inf")
        for _ in range(3):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            cc.cc_local_search_ex(c, oracle.SUM, BOTH, restarts, 5, buffers=buffers)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end))
        return best

    assert seconds(_zones(n, 2)) < 1.3 * seconds(hierarchical_matrix(n, (4, 32), ((50, 100), (200, 400), (800, 2000)), 0.3, True, n))
