"""GPU parity of the pruned pair-swap descent at the edges of its dispatch: every power of two, entries around 2^16
(N >= 256 changes where it reads the matrix), ties among the largest links, and orders that are no permutation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix
from gpu_util import assert_search_equal, dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [2, 4, 16, 64, 128, 256, 512])
@pytest.mark.parametrize("hi", [2, 65535, 65536, COST_MAX])
def test_pruned_swaps_equal_the_exhaustive_sweep(n, hi):
    restarts = {2: 3, 4: 9, 16: 40, 64: 20, 128: 6, 256: 3, 512: 1}[n]
    say(f"pruned pair swaps N={n} entries<={hi} R={restarts}")
    if n == 512 and hi > 2:          # few distinct large entries: short descents that the oracle replays quickly
        c = np.where(np.random.default_rng(7).random((n, n)) < 0.98, 1, random_matrix(n, 91, symmetric=False, lo=1, hi=hi))
        c = c.astype(np.int32)
        np.fill_diagonal(c, 0)
        c[1, 2] = hi
    else:
        c = random_matrix(n, 8000 + n + hi % 97, symmetric=False, lo=0, hi=hi)
        c[0, 1] = hi
    want = oracle.rd_swap_search(c, restarts, seed=n)
    b = cc.cc_rd_swap_search_ex(dev(c), restarts, n)
    torch.cuda.synchronize()
    assert_search_equal(dict(best_perm=b.best_perm.cpu().numpy(), best_cost=int(b.best_cost.item()),
                             best_restart=int(b.best_restart.item()), costs=b.restart_costs.cpu().numpy(),
                             tours=b.restart_tours.cpu().numpy(), moves=b.restart_moves.cpu().numpy()), want)


@pytest.mark.parametrize("n", [64, 512])
def test_orders_that_are_no_permutation_end(n):
    """Repeated and out-of-range nodes: results are unspecified, the call ends and its costs do not grow."""
    say(f"pruned pair swaps N={n}: orders that are no permutation")
    rng = np.random.default_rng(3)
    init = rng.integers(-5, n + 5, size=(4, n)).astype(np.int32)
    c = random_matrix(n, 17, symmetric=True, lo=0, hi=3)
    b = cc.cc_rd_swap_search_ex(dev(c), 4, 1, init_tours=dev(init))
    torch.cuda.synchronize()
    clamped = np.clip(init, 0, n - 1)
    assert (b.restart_costs.cpu().numpy() <= [oracle.rd_cost(c, t) for t in clamped]).all()
