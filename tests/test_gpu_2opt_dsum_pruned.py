"""GPU parity of the pruned directed ring-sum descents: every number of wavefronts the launch chooses on both sides of its lines (48, 64, 65 and 96
with 513 restarts are beyond them, other kernels'), ties, costs that hardly differ by direction, entries beyond 2^16, a zero in every row and
column, the orientation flip, orders that are no permutation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix
from gpu_util import dev, gpu_search, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


def _matrices(n):
    yield "spread", random_matrix(n, n, symmetric=False, lo=1, hi=5000)
    yield "ties", random_matrix(n, n + 1, symmetric=False, lo=0, hi=4)
    yield "symmetric", random_matrix(n, n + 2, symmetric=True, lo=1, hi=3000)
    yield "beyond 2^16", random_matrix(n, n + 3, symmetric=False, lo=0, hi=(1 << 21) - 1)
    zero = random_matrix(n, n + 4, symmetric=False, lo=1, hi=5000)
    ring = np.random.default_rng(n).permutation(n)
    zero[ring, np.roll(ring, 1)] = 0
    yield "a zero in every row and column", zero


@pytest.mark.parametrize("n,restarts", [(48, 3), (64, 5), (65, 256), (65, 257), (65, 513), (96, 512), (96, 513), (97, 513), (128, 3), (129, 3), (129, 300),
                                        (192, 2), (255, 257), (256, 2), (257, 2), (257, 257), (512, 1)])
def test_every_launch(n, restarts):
    for name, c in _matrices(n):
        say(f"directed sum N={n} R={restarts} {name}")
        got = gpu_search(c, oracle.SUM_DIRECTED, restarts, 31)
        k = int(np.argmin(got["costs"]))
        assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]
        for r in sorted({0, restarts - 1}):
            costs, tours, moves = oracle.restarts(c, oracle.SUM_DIRECTED, 31, r, r + 1)
            assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0] and np.array_equal(got["tours"][r], tours[0])


@pytest.mark.parametrize("n", [65, 100, 130, 513])
def test_flip_and_orders_that_are_no_permutation(n, monkeypatch):
    """Against the general kernel, which scores every move."""
    init = np.random.default_rng(n).integers(0, n, size=(4, n)).astype(np.int32)
    init[3] = np.random.default_rng(n + 1).permutation(n)
    for name, c in _matrices(n):
        if n > 500 and name != "spread":
            continue
        for classes in (cc.CC_MOVES_2OPT, cc.CC_MOVES_2OPT | cc.CC_MOVES_FLIP):
            say(f"directed sum N={n} {name} classes={classes}: orders that are no permutation")
            runs = []
            for path in ("", "general"):
                monkeypatch.setenv("CC_FORCE_PATH", path)
                b = cc.cc_local_search_ex(dev(c), cc.CC_RING_SUM_DIRECTED, classes, 4, 1, dev(init))
                torch.cuda.synchronize()
                runs.append([x.cpu().numpy() for x in (b.restart_costs, b.restart_tours, b.restart_moves)])
            assert all(np.array_equal(x, y) for x, y in zip(*runs))


def _one_way(n):
    """Every hop of the ascending order costs the most there is, the descending one hardly anything: prefix sums close to 2^31."""
    c = np.where(np.arange(n)[:, None] > np.arange(n)[None, :], COST_MAX, np.random.default_rng(n).integers(0, 4, (n, n))).astype(np.int32)
    c[0, n - 1] = COST_MAX
    np.fill_diagonal(c, 0)
    return c


@pytest.mark.parametrize("n", [513, 1023, 1024])
def test_the_largest_costs_one_way(n):
    init = np.stack([np.arange(n), np.arange(n)[::-1], np.random.default_rng(1).permutation(n)]).astype(np.int32)
    for c, tag in ((_one_way(n), "as walked"), (np.ascontiguousarray(_one_way(n).T), "the other way"),
                   (random_matrix(n, n, symmetric=False, lo=0, hi=COST_MAX), "spread")):
        say(f"directed sum N={n}: the largest costs, {tag}")
        got = gpu_search(c, oracle.SUM_DIRECTED, 3, 1, init)
        costs, tours, moves = oracle.restarts(c, oracle.SUM_DIRECTED, 1, 0, 3, init=init)
        assert np.array_equal(got["costs"], costs) and np.array_equal(got["moves"], moves) and np.array_equal(got["tours"], tours)
