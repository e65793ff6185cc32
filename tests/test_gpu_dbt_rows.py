"""GPU parity, double binary tree batches on the 16-bit matrix in LDS (sixteen lanes per order): the smallest trees, full and
nearly empty last levels, the largest N served, entries below and above 2^16, batches that end inside a workgroup's pass."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [2, 3, 4, 7, 8, 15, 16, 17, 31, 32, 33, 63, 65, 100, 127, 128, 129, 200, 230, 255, 256])
def test_dbt_batch_rows(n):
    first = -(-(1 << 20) // n)                         # the smallest batch that takes this kernel
    perms = random_perms(n, first + 3, seed=n)
    for top in ((1 << 16) - 1, COST_MAX):
        c = random_matrix(n, n + top % 5, symmetric=False, lo=0, hi=top)
        c[0, n - 1] = top
        for b in (first - 1, first, first + 3):
            say(f"tree batch rows N={n} B={b} largest entry {top}")
            got = cc.cc_dbt_cost_batch(dev(c), dev(perms[:b]))
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), oracle.dbt_cost_batch(c, perms[:b]))
