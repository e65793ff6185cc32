"""The work that users of the rank-order library have it do, as cases whose time is worth watching.

A user holds a measured cost matrix of N nodes on the GPU.  They score batches of candidate orders under the model of
their collective (ring, halving-doubling, BCube, double binary tree), search for a good order (2-opt, wider move sets,
pair swaps, annealing), and before all that turn latency probes into the matrix.  N is however many machines they
rent: 8 to 1024, often no round number; only the models with rounds ask for a power of their base.

listed() names the cases, draw() gives others of the same ranges, prepare() makes what the program has in hand, run()
is one pass through the public calls.
"""
import math

import torch

import paper_2105_14088_amd as cc

OBJECTIVES = ("sum", "max", "sum_directed", "max_directed")


def listed():
    return [
        # Scoring all rings of a handful of machines: one short call, its latency is all there is.
        {"name": "ring-n8-small", "kind": "ring", "n": 8, "batch": 4096, "objective": "sum", "ranks": "i32"},
        # The headline batch: a million orders of 64 machines.
        {"name": "ring-n64-million", "kind": "ring", "n": 64, "batch": 1 << 20, "objective": "sum", "ranks": "i32"},
        # Bottleneck hop of compactly stored orders, a cluster that is no power of two.
        {"name": "ring-n500-compact", "kind": "ring", "n": 500, "batch": 65000, "objective": "max", "ranks": "u16"},
        # Halving-doubling over the largest cluster.
        {"name": "halving-n1024", "kind": "rounds", "n": 1024, "base": 2, "batch": 65536},
        # Double binary tree, the model that takes any N, on a ragged one.
        {"name": "tree-n100", "kind": "tree", "n": 100, "batch": 100000},
        # The usual search: a ring for 64 machines, a thousand restarts.
        {"name": "search-n64", "kind": "search", "n": 64, "restarts": 1024, "objective": "sum", "keep": True},
        # Bottleneck search on bandwidths that differ by direction, called once without kept buffers.
        {"name": "search-n100-bottleneck", "kind": "search", "n": 100, "restarts": 1000, "objective": "max_directed", "keep": False},
        # A ring for a large, ragged cluster.
        {"name": "search-n1000", "kind": "search", "n": 1000, "restarts": 128, "objective": "sum", "keep": True},
        # 2-opt with segment insertion on a middling cluster.
        {"name": "insertion-n150", "kind": "local", "n": 150, "restarts": 512, "classes": 3, "keep": True},
        # Pair swaps under halving-doubling.
        {"name": "swap-n256", "kind": "swap", "n": 256, "restarts": 256, "keep": True},
        # Annealing over the ring.
        {"name": "anneal-n64", "kind": "anneal", "n": 64, "chains": 1024, "steps": 20000, "model": "ring", "keep": True},
        # Ten thousand probes of every ordered pair of 64 machines, 10th percentile.
        {"name": "probes-n64", "kind": "probes", "n": 64, "probes": 10000, "percentile": 10, "symmetrize": True},
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ring", "ring", "rounds", "tree", "search", "search", "search", "local", "swap", "anneal", "probes"])
    if kind == "probes":
        n = _log_between(rng, 8, 256)
        probes = _log_between(rng, 100, min(16384, 40_000_000 // (n * n)))
        return {"kind": kind, "n": n, "probes": probes, "percentile": rng.choice([10, 50]), "symmetrize": rng.random() < 0.75}
    if kind in ("ring", "tree"):
        n = _log_between(rng, 8, 1024)
        batch = _log_between(rng, 1000, min(1 << 20, (1 << 26) // n))
        if kind == "tree":
            return {"kind": kind, "n": n, "batch": batch}
        ranks = rng.choice(["i32", "i32", "u16", "u8" if n <= 256 else "u16"])
        return {"kind": kind, "n": n, "batch": batch, "objective": rng.choice(["sum", "max"]), "ranks": ranks}
    if kind == "rounds":
        base = rng.choice([2, 2, 4])
        n = base ** rng.randint(3, 10) if base == 2 else base ** rng.randint(2, 5)
        return {"kind": kind, "n": n, "base": base, "batch": _log_between(rng, 1000, min(1 << 20, (1 << 26) // n))}
    keep = rng.random() < 0.75
    if kind == "search":
        objective = rng.choice(["sum", "sum", "max", "sum_directed", "max_directed"])
        n = _log_between(rng, 8, 512 if objective == "sum_directed" else 1024)
        most = 25_000_000_000 if objective == "sum_directed" else 100_000_000_000
        return {"kind": kind, "n": n, "restarts": _log_between(rng, 32, min(4096, most // n**3)), "objective": objective, "keep": keep}
    if kind == "local":
        n = _log_between(rng, 8, 400)
        return {"kind": kind, "n": n, "restarts": _log_between(rng, 32, min(2048, 6_000_000_000 // n**3)), "classes": rng.choice([3, 3, 2]), "keep": keep}
    if kind == "swap":
        n = 2 ** rng.randint(3, 9)
        return {"kind": kind, "n": n, "restarts": _log_between(rng, 16, 1024 if n <= 256 else 256), "keep": keep}
    model = rng.choice(["ring", "ring", "rd"])
    n = _log_between(rng, 8, 1024) if model == "ring" else 2 ** rng.randint(3, 10)
    most = 40_000_000 if model == "ring" else 10_000_000
    chains = _log_between(rng, 64, 2048)
    return {"kind": kind, "n": n, "chains": chains, "steps": _log_between(rng, 1000, min(50000, most // chains)), "model": model, "keep": keep}


def _matrix(n, directed, seed):
    """A datacentre's cost matrix: nodes in hosts and racks, a base cost per pair from its level's range, lognormal
    tenant noise, node names in no order.  Latencies in 0.1 us, symmetric; or, directed, inverse bandwidths whose two
    directions differ."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def rand():
        return torch.rand(n, n, generator=g, device="cuda", dtype=torch.float64)

    def noise(sigma):
        return torch.exp(sigma * torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))

    where = torch.randperm(n, generator=g, device="cuda")
    same_host = (where[:, None] // 4) == (where[None, :] // 4)
    rack = 8 if n <= 64 else 32
    same_rack = (where[:, None] // rack) == (where[None, :] // rack)
    u = torch.triu(rand(), 1)
    u = u + u.T
    if directed:
        far = 4000 + 6000 * u
        c = torch.where(same_rack, far / 8, far) * noise(0.25)
    else:
        c = torch.where(same_rack, 200 + 200 * u, 800 + 1200 * u)
        if n > 64:
            c = torch.where(same_host, 50 + 50 * u, c)
        c = torch.triu(c * noise(0.3 if n > 64 else 0.25), 1)
        c = c + c.T
    c = torch.clamp(torch.round(c), min=1).to(torch.int32)
    return c.fill_diagonal_(0).contiguous()


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    state = {"case": case, "seed": 0xC0FFEE00 + seed}
    if kind == "probes":
        # round-trip times: the pair's base, queueing on top of it
        base = _matrix(n, False, seed).to(torch.float32)
        g = torch.Generator(device="cuda").manual_seed(seed + 1)
        s = torch.empty(n, n, case["probes"], device="cuda", dtype=torch.float32).exponential_(3.0, generator=g)
        state["samples"] = s.add_(1.0).mul_(base[:, :, None]).to(torch.int32)
        return state
    directed = "directed" in case.get("objective", "")
    state["matrix"] = _matrix(n, directed, seed)
    if "batch" in case:
        orders = cc.cc_init_tours(n, case["batch"], state["seed"])
        narrow = {"u8": torch.uint8, "u16": torch.int16}.get(case.get("ranks"))
        state["orders"] = orders.to(narrow) if narrow else orders
    elif case["keep"]:
        objective = OBJECTIVES.index(case.get("objective", "sum"))
        state["buffers"] = cc.SearchBuffers(n, objective, case["restarts" if "restarts" in case else "chains"], "cuda")
    return state


def _outputs(buffers):
    return [buffers.best_perm, buffers.best_cost, buffers.best_restart, buffers.restart_costs, buffers.restart_tours, buffers.restart_moves]


def run(state):
    case, kind, seed, c = state["case"], state["case"]["kind"], state["seed"], state.get("matrix")
    if kind == "probes":
        return cc.cc_cost_matrix_from_probes(state["samples"], case["percentile"], case["symmetrize"])
    if kind == "ring":
        call = {"i32": cc.cc_ring_cost_batch, "u8": cc.cc_ring_cost_batch_u8, "u16": cc.cc_ring_cost_batch_u16}[case["ranks"]]
        return call(c, state["orders"], OBJECTIVES.index(case["objective"]))
    if kind == "rounds":
        if case["base"] == 2:
            return cc.cc_rd_cost_batch(c, state["orders"])
        return cc.cc_bcube_cost_batch(c, case["base"], state["orders"])
    if kind == "tree":
        return cc.cc_dbt_cost_batch(c, state["orders"])
    if kind == "search":
        args = (c, OBJECTIVES.index(case["objective"]), case["restarts"], seed)
        calls = (cc.cc_2opt_search, cc.cc_2opt_search_ex)
    elif kind == "local":
        args = (c, cc.CC_RING_SUM, case["classes"], case["restarts"], seed)
        calls = (cc.cc_local_search, cc.cc_local_search_ex)
    elif kind == "swap":
        args = (c, case["restarts"], seed)
        calls = (cc.cc_rd_swap_search, cc.cc_rd_swap_search_ex)
    else:
        # temperature from a typical cost difference down to zero
        args = (c, case["chains"], case["steps"], 300, 0, seed)
        calls = (cc.cc_sa_search, cc.cc_sa_search_ex) if case["model"] == "ring" else (cc.cc_sa_rd_search, cc.cc_sa_rd_search_ex)
    if case["keep"]:
        return _outputs(calls[1](*args, buffers=state["buffers"]))
    return list(calls[0](*args))


def work(case):
    """Bytes: inputs once, outputs once.  Operations: an order's hops; a search's applied moves, each of which has to
    look at all N ranks at least once (about one applied move per node, a fifth of that under the bottleneck); a
    proposal of annealing draws, looks up four costs and decides."""
    kind, n = case["kind"], case["n"]
    matrix = 4 * n * n
    if kind == "probes":
        samples = n * (n - 1) * case["probes"]
        return {"bytes": 4 * samples + matrix, "flops": samples}
    if "batch" in case:
        b = case["batch"]
        wide = {"u8": 1, "u16": 2}.get(case.get("ranks"), 4)
        if kind == "rounds":
            rounds = round(math.log(n, case["base"]))
            flops = b * n * (case["base"] - 1) * rounds
        else:
            flops = b * n * (4 if kind == "tree" else 1)
        return {"bytes": matrix + b * (wide * n + 8), "flops": flops}
    r = case["restarts" if "restarts" in case else "chains"]
    out = 4 * n + 8 + (r * (4 * n + 12) + 4 if case["keep"] else 0)
    if kind == "anneal":
        return {"bytes": matrix + out, "flops": 16 * r * case["steps"]}
    moves = n / 5 if kind == "swap" or "max" in case.get("objective", "") else n
    return {"bytes": matrix + out, "flops": r * moves * n}


def tolerance(case):
    return "exact"  # every result is an integer
