"""GPU parity of the pruned max-hop descents on both sides of every size and restart count at which their workgroups change."""
import numpy as np
import pytest

import oracle
from gen import random_matrix
from gpu_util import gpu_search, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n,restarts", [(129, 1024), (129, 1025), (256, 3), (257, 512), (257, 513), (512, 3), (513, 512), (513, 513), (1024, 2)])
@pytest.mark.parametrize("objective", [oracle.MAX, oracle.MAX_DIRECTED])
def test_every_workgroup(n, restarts, objective):
    for hi in (5000, 6, 1 << 20):
        say(f"pruned max-hop workgroups N={n} R={restarts} objective={objective} entries<={hi}")
        c = random_matrix(n, n + hi, symmetric=objective == oracle.MAX, lo=1, hi=hi)
        got = gpu_search(c, objective, restarts, 3)
        k = int(np.argmin(got["costs"]))
        assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]
        for r in {0, restarts - 1} if n < 512 else {restarts - 1}:
            costs, tours, moves = oracle.restarts(c, objective, 3, r, r + 1)
            assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0] and np.array_equal(got["tours"][r], tours[0])
