"""GPU parity, cost matrix from probes with the bracket from a pilot: both sides of every register form, and samples for which
the pilot says nothing (drift, steps, ties, blocks), so that the bracket is missed or overflows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]

EDGES = [511, 512, 513, 1024, 1025, 1026, 1027, 2048, 2049, 3072, 3073, 4097, 6144, 6145, 8192, 8193, 8195, 10240, 10241, 12288, 12289, 16383]


def traces(n, k, seed):
    """One kind of sample sequence per ordered pair."""
    rng = np.random.default_rng(seed)
    i = np.arange(k)
    kinds = [
        lambda: 900 * (1 + rng.exponential(3.0, k)),                                        # queueing
        lambda: i * 3 + rng.integers(0, 5, k),                                              # drift
        lambda: np.where(i < k // 2, 500, 90000) + rng.integers(0, 50, k),                  # a step half way
        lambda: rng.integers(0, 3, k) * 1000,                                               # three values
        lambda: np.full(k, 4242),
        lambda: np.where(rng.random(k) < 0.1, 10, 11),                                      # ties on both sides of the 10th
        lambda: np.where((i // 4) % 2 == 0, 5, COST_MAX - rng.integers(0, 9, k)),           # blocks of a lane's four
        lambda: np.where(i % 4 == (i // 256) % 4, 100000 + rng.integers(0, 99, k), rng.integers(0, 99, k)),   # the pilot's own
        lambda: rng.integers(-(1 << 31), 1 << 31, k),                                       # out of range on both sides
        lambda: np.where(rng.random(k) < 0.5, 0, COST_MAX),
        lambda: (1 << rng.integers(0, 21, k)) + rng.integers(-1, 2, k),                     # edges of the bits
        lambda: np.where(i % 256 < 4, rng.integers(50, 60, k), 70000),                      # all inside in one lane
    ]
    s = np.stack([kinds[p % len(kinds)]() for p in range(n * n)]).reshape(n, n, k)
    return np.clip(s, -(1 << 31), (1 << 31) - 1).astype(np.int32)


@pytest.mark.parametrize("k", EDGES)
def test_forms_and_sequences_a_pilot_does_not_describe(k):
    s = traces(5, k, k)
    d = dev(s)
    for q in (0, 1, 10, 50, 90, 99, 100):
        for sym in (True, False):
            say(f"probes bracket K={k} percentile={q} symmetrize={sym}")
            out = cc.cc_cost_matrix_from_probes(d, q, sym)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), oracle.cost_matrix_from_probes(s, q, sym))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 9, 16, 31])
def test_every_pair_of_odd_and_even_n_is_written(n):
    say(f"probes bracket N={n} K=1100")
    s = np.random.default_rng(n).integers(1, 30000, size=(n, n, 1100)).astype(np.int32)
    for symmetrize in (False, True):
        out = torch.full((n, n), -1, dtype=torch.int32, device="cuda")
        got = cc.cc_cost_matrix_from_probes(dev(s), 25, symmetrize, out=out)
        torch.cuda.synchronize()
        assert got is out
        assert np.array_equal(out.cpu().numpy(), oracle.cost_matrix_from_probes(s, 25, symmetrize))
