"""GPU parity, halving-doubling batch at N = 512 and 1024 with a workspace (marked links): matrices whose marks are many,
few or none, orders all of whose links are small, and batches that end inside a workgroup's pass."""
import numpy as np
import pytest
import torch

import oracle
import paper_2105_14088_amd as cc
from gen import COST_MAX, random_matrix, random_perms
from gpu_util import dev, gpu_rd, say

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]


def _matrices(n):
    rng = np.random.default_rng(n)
    yield "spread", random_matrix(n, n, symmetric=False, lo=0, hi=COST_MAX)
    yield "one value", np.where(np.eye(n, dtype=bool), 0, 7).astype(np.int32)
    yield "zeros", np.zeros((n, n), dtype=np.int32)
    levels = np.array([5, 40, 41], dtype=np.int32)[rng.choice(3, size=(n, n), p=[0.05, 0.05, 0.9])]
    np.fill_diagonal(levels, 0)
    yield "three levels, most at the top", levels
    rare = random_matrix(n, n + 1, symmetric=True, lo=1, hi=9)
    rare[3, n - 1] = COST_MAX
    yield "one large entry, one direction", rare
    # dear links only between the halves of the nodes: most rounds of the identity order have no marked link
    half = random_matrix(n, n + 2, symmetric=False, lo=1, hi=500)
    half[: n // 2, n // 2:] += 10000
    yield "two islands", half
    side = np.arange(n) >= n // 2
    yield "two islands, two values", np.where(side[:, None] == side[None, :], 3, 9).astype(np.int32)


@pytest.mark.parametrize("n", [512, 1024])
def test_rd_batch_marked_links(n):
    for name, c in _matrices(n):
        for b in (1, 16, 241):
            say(f"rd batch, marked links, N={n} B={b}, {name}")
            perms = random_perms(n, b, seed=n + b)
            perms[0] = np.arange(n)
            assert np.array_equal(gpu_rd(c, perms), oracle.rd_cost_batch(c, perms))


@pytest.mark.parametrize("n", [512, 1024])
def test_rd_batch_marked_links_several_passes_weights_and_unaligned_orders(n):
    say(f"rd batch, marked links, N={n}: 4111 orders, weighted rounds, order stream 4 bytes off")
    c = random_matrix(n, 3 * n, symmetric=False, lo=0, hi=COST_MAX)
    perms = random_perms(n, 4111, seed=n)
    assert np.array_equal(gpu_rd(c, perms), oracle.rd_cost_batch(c, perms))
    rounds = n.bit_length() - 1
    w = np.array([1 << 30, 0] + list(range(3, rounds + 1)), dtype=np.int32)
    room = torch.empty(200 * n + 1, dtype=torch.int32, device="cuda")
    view = room[1:].view(200, n)
    view.copy_(dev(perms[:200]))
    got = cc.cc_bcube_cost_batch_weighted(dev(c), 2, dev(w), view)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.bcube_cost_weighted_batch(c, 2, w, perms[:200]))


def test_bcube_base_4_marked_links():
    n = 1024
    for name, c in _matrices(n):
        for b in (1, 16, 241):
            say(f"bcube base 4, marked links, N={n} B={b}, {name}")
            perms = random_perms(n, b, seed=n + b)
            perms[0] = np.arange(n)
            got = cc.cc_bcube_cost_batch(dev(c), 4, dev(perms))
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), oracle.bcube_cost_batch(c, 4, perms))


def test_bcube_base_4_marked_links_several_passes_weights_and_unaligned_orders():
    n = 1024
    say("bcube base 4, marked links: 4111 orders, weighted rounds, order stream 4 bytes off")
    c = random_matrix(n, 3 * n, symmetric=False, lo=0, hi=COST_MAX)
    perms = random_perms(n, 4111, seed=n)
    got = cc.cc_bcube_cost_batch(dev(c), 4, dev(perms))
    w = np.array([1 << 30, 0, 3, 4, 5], dtype=np.int32)
    room = torch.empty(200 * n + 1, dtype=torch.int32, device="cuda")
    view = room[1:].view(200, n)
    view.copy_(dev(perms[:200]))
    weighted = cc.cc_bcube_cost_batch_weighted(dev(c), 4, dev(w), view)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.bcube_cost_batch(c, 4, perms))
    assert np.array_equal(weighted.cpu().numpy(), oracle.bcube_cost_weighted_batch(c, 4, w, perms[:200]))


@pytest.mark.parametrize("n,wanted", [(512, 0.02), (1024, 0.01)])
@pytest.mark.parametrize("noise", [0.0, 0.05])
@pytest.mark.parametrize("group", [4, 32])
def test_rd_batch_marks_do_not_follow_how_nodes_are_numbered(n, wanted, noise, group):
    """Nodes numbered by host (4) or rack (32) and pairs that cost what these do: about as many links are marked as where the
    numbers are in no order.  2048 samples in quadruples that may hold one value put the share within a factor of 1.7 of
    what is wanted (three standard deviations of the third of 32); 16 equal samples put it beyond a factor of 2.3."""
    say(f"rd batch, share of marked links, N={n}, groups of {group}, noise {noise}")
    rng = np.random.default_rng(n + group)
    of = np.arange(n) // group
    base = rng.integers(800, 2000, size=(n // group, n // group))
    c = base[of][:, of] * np.exp(noise * rng.standard_normal((n, n)))
    c = np.triu(np.rint(c), 1).astype(np.int32)
    c = c + c.T
    for numbering in (np.arange(n), rng.permutation(n)):
        m = np.ascontiguousarray(c[numbering][:, numbering])
        perms = random_perms(n, 16, seed=n)
        room = torch.zeros(cc.cc_rd_batch_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        got = cc.cc_rd_cost_batch(dev(m), dev(perms), workspace=room)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.rd_cost_batch(m, perms))
        share = np.unpackbits(room[: n * n // 8].cpu().numpy()).mean()
        assert wanted / 3 < share < wanted * 1.9, share
