"""Timing cases: the work that users of this library have it do, from a few
thousand contact records counted at order 3 to hypergraphs of millions of
hyperedges counted, sampled and trained on at order 4.

The inputs follow the three shapes that the repository's workloads follow
(``workloads/synth.py``), generated on the GPU from the seed:

- ``ranked``: a small population whose members are active by rank (weights
  r^-0.8), hyperedges of 2, 3 or 4 nodes;
- ``contact``: face-to-face proximity, communities of 40, hyperedges of 2 to 5
  nodes, a share of them recorded more than once;
- ``coauthorship`` and ``communication``: Pareto-distributed activity,
  hyperedges of up to 25 or 50 nodes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2209_10241_amd as hm

# (largest size, exponent of P(size) ~ size^-exponent, Pareto exponent of the activity)
HEAVY = {"coauthorship": (25, 2.5, 1.2), "communication": (50, 2.0, 1.0)}
ORDER3_CLASSES, ORDER4_CLASSES = 6, 171
ORDER5_ROWS = 1 << 16
MLP_MACS = 16 * 64 + 64 * 64 + 64


def _case(name, path, recipe, nodes, edges, k, **options):
    return {"name": name, "path": path, "recipe": recipe, "nodes": nodes, "edges": edges, "k": k, **options}


def listed():
    return [
        # A small contact study read from a file: numpy arrays in, order 3.
        # The smallest call that is made; its time is launches and one wait.
        _case("exact3_small", "exact", "ranked", 200, 2000, 3, host=True, repeats=0.0),
        # One face-to-face network (the benchmark's workload) built and counted.
        _case("exact4_contact", "exact", "contact", 400, 30000, 4, host=False, repeats=0.0),
        # A study of many networks (days, classes, subjects), each of its own
        # size, counted in one call as the benchmark's throughput does.
        _case("exact4_many", "many", "contact", 400, 30000, 4, graphs=48, workers=8),
        # The two large shapes, built and counted exactly: no bit rows.
        _case("exact4_coauthorship", "exact", "coauthorship", 1_000_000, 2_000_000, 4, host=False, repeats=0.0),
        _case("exact4_communication", "exact", "communication", 50_000, 5_000_000, 4, host=False, repeats=0.0),
        # Estimates on a hypergraph that is kept: the face-to-face network at
        # the fraction that reaches 2% error, and the communication network.
        _case("sampled4_contact", "sampled", "contact", 400, 30000, 4, fraction=0.03),
        _case("sampled4_communication", "sampled", "communication", 50_000, 5_000_000, 4, fraction=0.02),
        # One estimate of a large hypergraph seen for the first time.
        _case("sampled4_new_coauthorship", "sampled_new", "coauthorship", 1_000_000, 2_000_000, 4, fraction=0.01),
        # Over- and under-expression against 64 stub-matched copies, on a kept
        # network whose pipeline has been planned ...
        _case("nulls4_contact", "nulls", "contact", 400, 30000, 4, copies=64),
        # ... and against the configuration model on a network seen for the
        # first time, an odd number of copies, order 3.
        _case("nulls3_new_small", "nulls_new", "ranked", 200, 2000, 3, copies=33, sweeps=10),
        # Order 5 by sampling (the paper's reach beyond exact counting).
        _case("order5_communication", "order5", "communication", 200, 20000, 5, fraction=0.05),
        # The learned proposal trained on a 5% subsample of the co-authorship
        # network: features, exact contributions, and the training steps.
        _case("train_coauthorship", "train", "coauthorship", 1_000_000, 100_000, 4, epochs=30, batch=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    path = rng.choice(["exact_contact", "exact_heavy", "many", "sampled_contact", "sampled_heavy", "sampled_new", "nulls",
                       "nulls_new", "order5", "train"])
    shape = rng.choice(sorted(HEAVY))
    # contact networks: from a class of a few dozen to a site of about two thousand
    nodes = _log_int(rng, 60, 2000)
    edges = _log_int(rng, 5 * nodes, min(75 * nodes, 60_000))
    # heavy-tailed networks at any scale up to the full one
    scale = math.exp(rng.uniform(math.log(0.01), 0.0))
    big = (_log_int(rng, 900_000 * scale, 1_000_000 * scale), int(2_000_000 * scale)) if shape == "coauthorship" else \
        (_log_int(rng, 45_000 * scale, 50_000 * scale), int(5_000_000 * scale))
    k = rng.choice([3, 4, 4])
    if path == "exact_contact":
        c = _case("", "exact", "contact", nodes, edges, k, host=rng.random() < 0.5, repeats=rng.choice([0.0, 0.3]))
    elif path == "exact_heavy":
        c = _case("", "exact", shape, *big, k, host=rng.random() < 0.3, repeats=rng.choice([0.0, 0.1]))
    elif path == "many":
        nodes = min(nodes, 500)
        c = _case("", "many", "contact", nodes, min(edges, 75 * nodes, 30_000), k, graphs=rng.randint(2, 48),
                  workers=rng.choice([1, 3, 8]))
    elif path == "sampled_contact":
        c = _case("", "sampled", "contact", nodes, edges, k, fraction=math.exp(rng.uniform(math.log(0.005), math.log(0.1))))
    elif path == "sampled_heavy":
        c = _case("", "sampled", shape, *big, k, fraction=math.exp(rng.uniform(math.log(0.0005), math.log(0.02))))
    elif path == "sampled_new":
        c = _case("", "sampled_new", shape, *big, k, fraction=math.exp(rng.uniform(math.log(0.0005), math.log(0.02))))
    elif path == "nulls":
        nodes = min(nodes, 1000)
        c = _case("", "nulls", "contact", nodes, min(edges, 30_000), k, copies=rng.randint(5, 64))
    elif path == "nulls_new":
        nodes = min(nodes, 400)
        c = _case("", "nulls_new", rng.choice(["ranked", "contact"]), nodes, min(edges, 10_000), k,
                  copies=rng.randint(5, 64), sweeps=rng.randint(1, 10))
    elif path == "order5":
        nodes = rng.randint(120, 200)
        c = _case("", "order5", "communication", nodes, 100 * nodes, 5, fraction=rng.uniform(0.01, 0.05))
    else:
        scale = math.exp(rng.uniform(math.log(0.05), 0.0))
        c = _case("", "train", "coauthorship", int(1_000_000 * scale), int(100_000 * scale), k,
                  epochs=rng.randint(5, 30), batch=rng.choice([1024, 4096]))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs
def _sizes(recipe):
    """(sizes, probabilities) of a hyperedge."""
    if recipe == "ranked":
        return np.array([2, 3, 4]), np.array([0.70, 0.25, 0.05])
    if recipe == "contact":
        s = np.arange(2, 6)
        p = 0.4 ** (s - 2.0)
    else:
        smax, exponent, _ = HEAVY[recipe]
        s = np.arange(2, smax + 1)
        p = s.astype(np.float64) ** -exponent
    return s, p / p.sum()


def _mean_size(recipe):
    s, p = _sizes(recipe)
    return float((s * p).sum())


def _pick(cdf, gen, count):
    u = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64)
    return torch.searchsorted(cdf, u, right=True).clamp_(max=cdf.numel() - 1)


def _hypergraph(recipe, nodes, edges, repeats, seed):
    """(members int32, offsets int64) on the GPU; members of a hyperedge are distinct."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s, p = _sizes(recipe)
    size = torch.as_tensor(s, device="cuda")[_pick(torch.as_tensor(np.cumsum(p), device="cuda"), gen, edges)]
    size = size.clamp_(max=nodes)
    seg = torch.repeat_interleave(torch.arange(edges, device="cuda"), size)
    if recipe == "contact":
        groups = max(1, nodes // 40)
        group = torch.randint(groups, (edges,), generator=gen, device="cuda")

        def members_at(where):
            n = where.numel()
            low = group[where] * nodes // groups
            width = (group[where] + 1) * nodes // groups - low
            local = low + (torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * width).long()
            anywhere = torch.randint(nodes, (n,), generator=gen, device="cuda")
            inside = torch.rand(n, generator=gen, device="cuda") < 0.9
            return torch.where(inside, local, anywhere)
    else:
        # the quantiles of the activity distribution, so that hypergraphs of
        # different seeds have like tails, over ids in random order
        rank = np.arange(1, nodes + 1, dtype=np.float64)
        weight = rank ** -0.8 if recipe == "ranked" else (rank / nodes) ** (-1.0 / HEAVY[recipe][2])
        if recipe != "ranked":
            weight = weight[np.random.Generator(np.random.PCG64(seed)).permutation(nodes)]
        cdf = np.cumsum(weight)
        cdf = torch.as_tensor(cdf / cdf[-1], device="cuda")

        def members_at(where):
            return _pick(cdf, gen, where.numel())
    members = members_at(seg)
    active = torch.arange(members.numel(), device="cuda")
    while active.numel():
        key, order = torch.sort(seg[active] * nodes + members[active], stable=True)
        again = active[order[1:][key[1:] == key[:-1]]]
        if again.numel() == 0:
            break
        members[again] = members_at(seg[again])
        bad = torch.zeros(edges, dtype=torch.bool, device="cuda")
        bad[seg[again]] = True
        active = active[bad[seg[active]]]
    offsets = torch.zeros(edges + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(size, 0, out=offsets[1:])
    if repeats:
        # the same hyperedges recorded again, at random places of the list
        extra = torch.randint(edges, (int(repeats * edges),), generator=gen, device="cuda")
        take = torch.cat([torch.arange(edges, device="cuda"), extra])
        take = take[torch.randperm(take.numel(), generator=gen, device="cuda")]
        size = size[take]
        start = torch.repeat_interleave(offsets[take], size)
        new = torch.zeros(take.numel() + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(size, 0, out=new[1:])
        within = torch.arange(int(new[-1]), device="cuda") - torch.repeat_interleave(new[:-1], size)
        members, offsets = members[start + within], new
    return members.to(torch.int32), offsets


def _many_shapes(case):
    """(nodes, edges) of each hypergraph of a study: full size down to a third."""
    n = case["graphs"]
    return [(max(50, case["nodes"] * (3 * n - 2 * g) // (3 * n)), max(50, case["edges"] * (3 * n - 2 * g) // (3 * n)))
            for g in range(n)]


def prepare(case, seed):
    path = case["path"]
    if path == "many":
        graphs = []
        for g, (nodes, edges) in enumerate(_many_shapes(case)):
            graphs.append((*_hypergraph(case["recipe"], nodes, edges, 0.0, seed * 1009 + g), nodes))
        return {"case": case, "graphs": graphs}
    members, offsets = _hypergraph(case["recipe"], case["nodes"], case["edges"], case.get("repeats", 0.0), seed)
    if case.get("host"):
        members, offsets = members.cpu().numpy().view(np.uint32), offsets.cpu().numpy().astype(np.uint64)
    state = {"case": case, "members": members, "offsets": offsets, "seed": seed % 1_000_003}
    if path in ("sampled", "nulls", "order5", "train"):
        state["graph"] = hm.hm_graph_create(members, offsets, case["nodes"])
        # what the handle keeps from its first call on (indices of the
        # adjacency, the planned pipeline of the null copies, the 5-node set)
        if path == "sampled":
            hm.count_sampled(state["graph"], case["k"], case["fraction"], state["seed"] + 1)
        elif path == "nulls":
            hm.count_nulls(state["graph"], case["k"], case["copies"], state["seed"] + 1)
        elif path == "order5":
            hm.hm_order5_sizes(state["graph"])
    return state


def run(state):
    case, seed = state["case"], state.get("seed", 0)
    path, k = case["path"], case["k"]
    if path == "exact":
        with hm.hm_graph_create(state["members"], state["offsets"], case["nodes"]) as graph:
            return hm.count_exact(graph, k)
    if path == "many":
        return hm.count_exact_many(state["graphs"], k, workers=case["workers"])
    if path == "sampled":
        return hm.count_sampled(state["graph"], k, case["fraction"], seed)
    if path == "sampled_new":
        with hm.hm_graph_create(state["members"], state["offsets"], case["nodes"]) as graph:
            return hm.count_sampled(graph, k, case["fraction"], seed)
    if path == "nulls":
        return hm.count_nulls(state["graph"], k, case["copies"], seed)
    if path == "nulls_new":
        with hm.hm_graph_create(state["members"], state["offsets"], case["nodes"]) as graph:
            return hm.count_nulls_model(graph, k, case["copies"], hm.HM_NULL_CONFIG, case["sweeps"], seed)
    if path == "order5":
        # the classes found, in a table of fixed size (their number differs from draw to draw)
        found = hm.count_sampled5(state["graph"], case["fraction"], seed)
        table = tuple(np.zeros(ORDER5_ROWS, dtype=column.dtype) for column in found)
        for rows, column in zip(table, found):
            rows[:len(column)] = column
        return table
    with hm.hm_model_train(state["graph"], k, epochs=case["epochs"], batch=case["batch"], seed=seed) as model:
        return model.params(), model.loss()


def work(case):
    """The hyperedge list read once (4 bytes a member, 8 an offset) and the
    results written once.  The counts' integer work has no lower bound that
    holds for every algorithm and is not counted; the training steps'
    products are."""
    classes = ORDER3_CLASSES if case["k"] == 3 else ORDER4_CLASSES

    def listed_bytes(edges):
        return edges * (4.0 * _mean_size(case["recipe"]) + 8.0)
    path = case["path"]
    if path == "many":
        return {"bytes": sum(listed_bytes(e) for _, e in _many_shapes(case)) + 8.0 * classes * case["graphs"], "flops": 0.0}
    bytes_in = listed_bytes(case["edges"] * (1.0 + case.get("repeats", 0.0)))
    if path == "exact":
        return {"bytes": bytes_in + 8.0 * classes, "flops": 0.0}
    if path in ("sampled", "sampled_new"):
        return {"bytes": bytes_in + 12.0 * classes, "flops": 0.0}
    if path in ("nulls", "nulls_new"):
        return {"bytes": bytes_in + classes * (8.0 * case["copies"] + 12.0), "flops": 0.0}
    if path == "order5":
        return {"bytes": bytes_in, "flops": 0.0}
    s, p = _sizes(case["recipe"])
    rows = case["edges"] * float(p[s <= case["k"]].sum())
    return {"bytes": bytes_in + 4.0 * 5313, "flops": 6.0 * MLP_MACS * rows * case["epochs"]}


def exact(case, seed):
    """None throughout: the counts are whole numbers, the estimates, z-scores
    and order-5 classes are those of pseudo-random draws, each one formula of
    whole numbers formed in 64 bits and rounded once, and the trained weights
    are the end of a chain of bf16 products, which no 64-bit run follows."""
    return None
