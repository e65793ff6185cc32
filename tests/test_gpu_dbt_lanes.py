"""GPU parity, double binary tree batches: the one-order-per-lane kernel at the edges of its trees (two or three ranks at the bottom,
full and nearly empty last levels), orders that do not begin at 16 bytes, batches that end inside a tile, matrices of small,
some large and only large entries; the wave-per-order kernel at the edges of its subtree depths; the register kernel below 8."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


def matrices(n):
    yield "small", random_matrix(n, n, symmetric=False, lo=0, hi=60000)
    c = random_matrix(n, n + 1, symmetric=False, lo=0, hi=60000)
    c[np.random.default_rng(n).random((n, n)) < 0.1] = 65534
    c[0, n - 1] = 65535
    yield "around 2^16", c
    yield "large", random_matrix(n, n + 2, symmetric=False, lo=65535, hi=COST_MAX)


@pytest.mark.parametrize("n", [8, 9, 11, 12, 15, 16, 23, 24, 31, 32, 47, 48, 63, 64, 65, 95, 96, 127, 128, 185, 186, 191, 192, 193, 254, 255])
def test_dbt_lanes(n):
    perms = random_perms(n, 40001, seed=n)
    padded = torch.empty(perms.size + 4, dtype=torch.int32, device="cuda")
    for name, c in matrices(n):
        d = dev(c)
        want = oracle.dbt_cost_batch(c, perms)
        for b, shift in ((40000, 0), (40001, 0), (40001, 1), (40001, 3)):
            say(f"tree batch lanes N={n} B={b} {name} entries, {shift} words from alignment")
            orders = padded[shift:shift + b * n].view(b, n)
            orders.copy_(dev(perms[:b]))
            got = cc.cc_dbt_cost_batch(d, orders)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want[:b])


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 8, 20, 31, 32, 62, 63, 65, 100, 127, 128, 255, 256, 257, 511, 512, 513, 1023, 1024])
def test_dbt_small_batches(n):
    for b in (1, 5, 300):
        perms = random_perms(n, b, seed=n + b)
        for name, c in matrices(n):
            say(f"tree batch small N={n} B={b} {name} entries")
            got = cc.cc_dbt_cost_batch(dev(c), dev(perms))
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), oracle.dbt_cost_batch(c, perms))


def test_ranks_out_of_range_are_clamped():
    """Bad data: unspecified results in general, here those of the clamped orders."""
    n = 100
    c = random_matrix(n, 4, symmetric=False, lo=0, hi=60000)
    perms = np.random.default_rng(5).integers(-(1 << 31), 1 << 31, size=(40001, n)).astype(np.int32)
    clamped = np.clip(perms, 0, n - 1).astype(np.int32)
    for b in (7, 40001):
        say(f"tree batch clamped ranks B={b}")
        got = cc.cc_dbt_cost_batch(dev(c), dev(perms[:b]))
        same = cc.cc_dbt_cost_batch(dev(c), dev(clamped[:b]))
        torch.cuda.synchronize()
        assert torch.equal(got, same)


@pytest.mark.parametrize("n", [186, 191, 192, 193, 255])
@pytest.mark.parametrize("first", ["large", "mostly large", "small"])
def test_dbt_where_the_first_entries_decide(n, first):
    """The first entries of the matrix say whether it is staged: nearly all from 65535 up and the others small, fifteen of sixteen, or
    small ones before a large half."""
    c = random_matrix(n, n, symmetric=False, lo=0, hi=60000)
    large = random_matrix(n, n + 1, symmetric=False, lo=65535, hi=COST_MAX)
    flat, other = c.reshape(-1), large.reshape(-1)
    if first == "small":
        flat[17000:] = other[17000:]
    else:
        flat[:16384] = other[:16384]
    if first == "mostly large":
        flat[:16384:16] = 5
    b = 7000
    perms = random_perms(n, b, seed=n)
    say(f"tree batch, first entries {first} N={n} B={b}")
    got = cc.cc_dbt_cost_batch(dev(c), dev(perms))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.dbt_cost_batch(c, perms))
