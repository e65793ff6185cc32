"""GPU parity of the ring-sum descents above N = 96: with many restarts the exhaustive kernels and the pruned one with a wavefront per
restart; with fewer the kernel that keeps pairs and, for what that leaves, the pruned one with several.  Edges of their sizes, entries on
both sides of 2^16 (16-bit matrix in LDS or not), ties, rows whose partners outgrow the lists, and orders that are no permutation."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, hierarchical_matrix, random_matrix
from gpu_util import assert_search_equal, dev, gpu_search, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


@pytest.mark.parametrize("n", [129, 192, 193, 255, 256, 257, 320, 321, 449, 513, 641, 769])
def test_pruned_ring_sum_equals_the_exhaustive_sweep(n):
    restarts = 5 if n <= 321 else 2
    for hi, tag in ((COST_MAX, "entries up to COST_MAX"), (65535, "16-bit entries"), (4, "ties")):
        say(f"pruned ring sum N={n} {tag} R={restarts}")
        c = random_matrix(n, 40 + n + hi % 83, symmetric=True, lo=0, hi=hi)
        assert_search_equal(gpu_search(c, oracle.SUM, restarts, n), oracle.search(c, oracle.SUM, restarts, n))


@pytest.mark.parametrize("n,restarts", [(98, 1600), (127, 1601), (130, 700), (192, 1100), (98, 2050), (127, 2049), (130, 2049), (192, 3080),
                                        (200, 2100), (255, 2049), (256, 2050)])
def test_one_wavefront_per_restart(n, restarts):
    """From 2049 restarts on (192: 3073); the first four sizes are below the line, a workgroup per restart."""
    for c, tag in ((random_matrix(n, n, symmetric=True, lo=1, hi=70000), "uniform, beyond 2^16"),
                   (hierarchical_matrix(n, (4, 8), ((50, 100), (200, 400), (800, 2000)), 0.3, True, n), "racks")):
        say(f"pruned ring sum N={n} R={restarts} {tag} (every 50th restart and the winner compared)")
        got = gpu_search(c, oracle.SUM, restarts, 9)
        for r in range(0, restarts, 50):
            costs, tours, moves = oracle.restarts(c, oracle.SUM, 9, r, r + 1)
            assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0]
            assert np.array_equal(got["tours"][r], tours[0])
        k = int(np.argmin(got["costs"]))
        assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]


@pytest.mark.parametrize("n", [150, 400])
def test_orders_that_are_no_permutation_end(n):
    say(f"pruned ring sum N={n}: orders that are no permutation")
    rng = np.random.default_rng(5)
    init = rng.integers(-5, n + 5, size=(3, n)).astype(np.int32)
    c = random_matrix(n, 18, symmetric=True, lo=0, hi=30)
    got = gpu_search(c, oracle.SUM, 3, 1, init)
    clamped = np.clip(init, 0, n - 1)
    assert (got["costs"] <= [oracle.ring_cost(c, t) for t in clamped]).all()


@pytest.mark.parametrize("n", [130, 192, 256, 400, 1024])
def test_a_node_twice_in_one_wavefronts_ranks_leaves_the_order_alone(n):
    """Only one wavefront of the restart sees the repeated node; all of them have to stop, while the next restart's search."""
    restarts = min((n + 63) // 64, 6) + 1
    init = np.stack([np.random.default_rng(r).permutation(n) for r in range(restarts)]).astype(np.int32)
    for r in range(restarts - 1):
        last = min(64 * (r + 1), n) - 1
        init[r, 64 * r] = init[r, last]              # 64 r and last are ranks of wavefront r
    say(f"pruned ring sum N={n}: a node twice among one wavefront's ranks")
    c = random_matrix(n, 19, symmetric=True, lo=0, hi=3000)
    got = gpu_search(c, oracle.SUM, restarts, 1, init)
    assert np.array_equal(got["tours"][:-1], init[:-1]) and not got["moves"][:-1].any()
    assert np.array_equal(got["costs"][:-1], [oracle.ring_cost(c, t) for t in init[:-1]])
    costs, tours, moves = oracle.restarts(c, oracle.SUM, 1, 0, 1, init=init[-1:])
    assert got["costs"][-1] == costs[0] and got["moves"][-1] == moves[0] and np.array_equal(got["tours"][-1], tours[0])


def _seconds(c, restarts, buffers):
    best = float("inf")
    for _ in range(3):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        cc.cc_2opt_search_ex(c, oracle.SUM, restarts, 5, buffers=buffers)
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end))
    return best


def _racks(n):
    return hierarchical_matrix(n, (4, 32), ((50, 100), (200, 400), (800, 2000)), 0.3, True, n)


def _one_zero_each(n):
    c, a = _racks(n), np.random.default_rng(n).permutation(n)
    c[a[0:n - 1:2], a[1::2]] = c[a[1::2], a[0:n - 1:2]] = 0
    return c


def _wide(n):
    u = np.triu(np.exp(np.random.default_rng(n).uniform(0, 14.5, (n, n))).astype(np.int32), 1)
    u = np.where(u < 3, 0, u)
    return (u + u.T).astype(np.int32)


def _zones(n, count=2, near=1, far=10):
    """Equal costs inside a zone, equal ones across."""
    zone = np.random.default_rng(n).permutation(n) * count // n
    c = np.where(zone[:, None] == zone[None, :], near, far)
    return np.where(np.eye(n, dtype=bool), 0, c).astype(np.int32)


@pytest.mark.parametrize("n,restarts", [(130, 3), (191, 700), (256, 3), (300, 2)])
@pytest.mark.parametrize("make", [_one_zero_each, lambda n: _racks(n) // 100, _wide, _zones, lambda n: _zones(n, 5, 2, 5),
                                  lambda n: _zones(n, 16, 3, 4), lambda n: _zones(n, 1, 7)],
                         ids=["one zero each", "coarse", "wide", "two zones", "five zones", "sixteen zones", "all equal"])
def test_zeros_and_wide_spreads_and_ties(n, restarts, make):
    say(f"pruned ring sum N={n} R={restarts}: zeros, spreads, ties")
    c = make(n).astype(np.int32)
    got = gpu_search(c, oracle.SUM, restarts, 3)
    for r in range(0, restarts, 100):
        costs, tours, moves = oracle.restarts(c, oracle.SUM, 3, r, r + 1)
        assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0] and np.array_equal(got["tours"][r], tours[0])
    if restarts < 10:
        assert_search_equal(got, oracle.search(c, oracle.SUM, restarts, 3))


def test_a_partner_at_cost_zero_does_not_switch_the_lists_off():
    """With one partner at cost 0 per node the search takes about the time it takes without (12 times while the buckets of
    cost covered 8 octaves from the smallest one on)."""
    n, restarts = 512, 32
    say(f"pruned ring sum N={n} R={restarts}: time with a zero per node")
    buffers = cc.SearchBuffers(n, oracle.SUM, restarts, "cuda")
    plain, zeros = (dev(c) for c in (_racks(n), _one_zero_each(n)))
    assert _seconds(zeros, restarts, buffers) < 3 * _seconds(plain, restarts, buffers)


def test_ties_do_not_bring_all_moves_back():
    """Two zones of equal costs take less time than racks of costs that all differ (6 times as long while every node looked
    for the moves that only equal the known one)."""
    n, restarts = 512, 768
    say(f"pruned ring sum N={n} R={restarts}: time with two zones of equal costs")
    buffers = cc.SearchBuffers(n, oracle.SUM, restarts, "cuda")
    plain, zones = (dev(c) for c in (_racks(n), _zones(n)))
    assert _seconds(zones, restarts, buffers) < 1.5 * _seconds(plain, restarts, buffers)


@pytest.mark.parametrize("n,restarts", [(97, 3), (99, 2047), (100, 1537), (128, 2), (128, 300), (192, 257), (192, 3073), (256, 257), (256, 1537),
                                        (65, 513), (79, 520), (96, 1025), (97, 2049), (127, 2049), (128, 1025), (128, 1500), (192, 1537),
                                        (192, 3072), (256, 2049)])
@pytest.mark.parametrize("hi", [65535, 65536])
def test_sizes_with_an_exhaustive_kernel_of_16_bit_entries(n, restarts, hi):
    """Either side of 2^16 and of the lines between the kernels.  The two that are enqueued take turns at 65 .. 79 from 513 restarts on, at
    80 .. 96 and 128 from 1025 on and at 192 with 1537 to 3072; fewer are the kernel's that keeps pairs, more the pruned one's."""
    say(f"ring sum N={n} R={restarts} entries<={hi}")
    c = random_matrix(n, n, symmetric=True, lo=0, hi=hi)
    c[0, n - 1] = c[n - 1, 0] = hi
    got = gpu_search(c, oracle.SUM, restarts, 9)
    for r in np.linspace(0, restarts - 1, 5).astype(int):
        costs, tours, moves = oracle.restarts(c, oracle.SUM, 9, int(r), int(r) + 1)
        assert got["costs"][r] == costs[0] and got["moves"][r] == moves[0] and np.array_equal(got["tours"][r], tours[0])
    k = int(np.argmin(got["costs"]))
    assert got["best_restart"] == k and got["best_cost"] == got["costs"][k]
