"""Performance cases: the calls that a user of the partitioner makes, over the range of sizes they are made at.

Graphs are drawn on the GPU from the seed alone and are of the three families
the benchmark and the tests use: R-MAT (0.57, 0.19, 0.19, 0.05) without id
permutation (web and social graphs), Barabasi-Albert (power-law, connected) and
2-D random geometric graphs with the radius 0.55 sqrt(ln n / n) (meshes).
"""
import math
import random

import numpy as np
import torch

import paper_1404_4797_amd as sc

DEVICE = "cuda"


def listed():
    return [
        # The smallest graph of the benchmark: one level, then refinement. Latency and launches count.
        {"name": "ba14_k2", "op": "partition", "family": "ba", "n": 1 << 14, "deg": 8, "k": 2, "eps": 0.03,
         "weighted": False, "max_levels": 1},
        # A first call from a script: numpy arrays in and out, the graph copied to the device inside the call.
        {"name": "rmat16_host_k8", "op": "partition_host", "family": "rmat", "n": 1 << 16, "deg": 16, "k": 8,
         "eps": 0.03, "weighted": False},
        # A small mesh of odd size into few blocks, tight balance, initial partition on the device.
        {"name": "rgg50001_k7_device_initial", "op": "partition", "family": "rgg", "n": 50001, "deg": 0, "k": 7,
         "eps": 0.01, "weighted": True, "initial_partitioner": 1},
        # The quality setting on a mid-sized weighted graph: two V-cycles, clustering by increasing degree.
        {"name": "rmat300k_k32_vcycles", "op": "partition", "family": "rmat", "n": 300007, "deg": 12, "k": 32,
         "eps": 0.05, "weighted": True, "vcycles": 2, "degree_order": 1},
        # A mesh at the size the benchmark partitions.
        {"name": "rgg20_k64", "op": "partition", "family": "rgg", "n": 1 << 20, "deg": 0, "k": 64, "eps": 0.03,
         "weighted": False},
        # A social network of a million nodes, an ordinary single call.
        {"name": "rmat20_k16", "op": "partition", "family": "rmat", "n": 1 << 20, "deg": 16, "k": 16, "eps": 0.03,
         "weighted": False},
        # The benchmark's headline graph, the largest: half a billion adjacency slots.
        {"name": "rmat24_k64", "op": "partition", "family": "rmat", "n": 1 << 24, "deg": 16, "k": 64, "eps": 0.03,
         "weighted": False},
        # What the serving loop packs into one batch: 64 weighted graphs of all three families, 2^10 to 2^18 nodes.
        {"name": "batch64_mix", "op": "batch", "family": "mix", "n": 1 << 18, "deg": 0, "k": 64, "eps": 0.03,
         "weighted": True, "count": 64},
        # Single steps for programs that drive their own multilevel loop: clustering a weighted graph,
        {"name": "cluster_rmat22w", "op": "cluster", "family": "rmat", "n": 1 << 22, "deg": 16, "k": 64, "eps": 0.03,
         "weighted": True},
        # contracting that clustering,
        {"name": "contract_rmat22", "op": "contract", "family": "rmat", "n": 1 << 22, "deg": 16, "k": 64,
         "eps": 0.03, "weighted": False},
        # improving a partition of a graph whose nodes have changed since,
        {"name": "refine_rmat21_k100", "op": "refine", "family": "rmat", "n": (1 << 21) - 77, "deg": 16, "k": 100,
         "eps": 0.03, "weighted": True},
        # and carrying a coarse partition up to the finer graph and weighing it there.
        {"name": "project_cut_ba20", "op": "project_cut", "family": "ba", "n": 1 << 20, "deg": 8, "k": 64,
         "eps": 0.03, "weighted": True},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["partition"] * 5 + ["partition_host", "batch", "cluster", "cluster", "contract", "refine",
                                         "refine", "project_cut"])
    family = "mix" if op == "batch" else rng.choice(["rmat", "rmat", "ba", "rgg"])
    # the launches of a call on a few nodes cost what they cost on a few thousand, so the range begins there
    n = _log_uniform(rng, 1000, {"batch": 1 << 18, "partition_host": 1 << 20}.get(op, 1 << 22))
    case = {"op": op, "family": family, "n": n, "deg": 0, "k": _log_uniform(rng, 2, 300),
            "eps": rng.choice([0.01, 0.03, 0.05]), "weighted": rng.random() < 0.5}
    if family == "rmat":
        case["deg"] = rng.randint(8, 16)
    elif family == "ba":
        case["deg"] = rng.choice([4, 8, 16]) if n <= 1 << 20 else rng.choice([4, 8])
    if op == "batch":
        case["count"] = _log_uniform(rng, 4, 64)
        case["weighted"] = True
    if op == "partition" and rng.random() < 0.4:
        case.update(rng.choice([{"vcycles": 2}, {"degree_order": 1}, {"initial_partitioner": 1}]))
    return case


# ------------------------------------------------------------------- graphs

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _csr(n, u, v, weighted, gen):
    """Symmetric CSR of the distinct pairs among (u, v), rows sorted; weights in [1, 4] if asked for."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    u, v = key // n, key % n
    del key
    both = torch.cat([u * n + v, v * n + u])
    if weighted:
        w = torch.randint(1, 5, (u.numel(),), generator=gen, device=DEVICE, dtype=torch.int32)
        del u, v
        both, at = torch.sort(both)
        adjwgt = torch.cat([w, w])[at]
        del at, w
    else:
        del u, v
        both = torch.sort(both)[0]
        adjwgt = torch.ones(both.numel(), dtype=torch.int32, device=DEVICE)
    xadj = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    xadj[1:] = torch.cumsum(torch.bincount(both // n, minlength=n), 0)
    return {"n": n, "xadj": xadj, "adjncy": (both % n).to(torch.int32), "adjwgt": adjwgt,
            "vwgt": torch.ones(n, dtype=torch.int32, device=DEVICE)}


def _rmat(n, edge_factor, weighted, gen):
    """edge_factor * 2^scale draws at the smallest scale that holds n; draws touching ids >= n are dropped."""
    scale = max(1, (n - 1).bit_length())
    m = edge_factor << scale
    u = torch.zeros(m, dtype=torch.int32, device=DEVICE)
    v = torch.zeros(m, dtype=torch.int32, device=DEVICE)
    for _ in range(scale):
        r = torch.rand(m, generator=gen, device=DEVICE)
        u.mul_(2).add_(r >= 0.76)
        v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    if n < 1 << scale:
        keep = (u < n) & (v < n)
        u, v = u[keep], v[keep]
    return _csr(n, u.to(torch.int64), v.to(torch.int64), weighted, gen)


def _ba(n, m, weighted, gen):
    """Every new node draws m endpoints of earlier edges uniformly: edge e's target is the source or the target
    of an earlier edge, found by following the draws back until one names a source."""
    e = torch.arange((n - m) * m, device=DEVICE)
    source = e // m + m
    earlier = (source - m) * m * 2  # endpoints that exist when the node arrives
    r = (torch.rand(e.numel(), generator=gen, device=DEVICE, dtype=torch.float64) * earlier).to(torch.int64)
    target = torch.where(earlier == 0, e, -1)  # the first node joins nodes 0..m-1
    while True:
        first = r % 2 == 0
        found = torch.where(first, source[r // 2], target[r // 2])
        target = torch.where(target < 0, found, target)
        if bool((target >= 0).all()):
            break
        # those still open point one draw further back
        r = torch.where(target < 0, r[r // 2], r)
    return _csr(n, source, target, weighted, gen)


def _rgg(n, weighted, gen):
    radius = 0.55 * math.sqrt(math.log(max(n, 2)) / n)
    p = torch.rand(n, 2, generator=gen, device=DEVICE, dtype=torch.float64)
    side = max(1, int(1 / radius))
    at = torch.clamp((p * side).to(torch.int64), max=side - 1)
    cell = at[:, 1] * side + at[:, 0]
    members = torch.argsort(cell, stable=True)
    start = torch.zeros(side * side + 1, dtype=torch.int64, device=DEVICE)
    start[1:] = torch.cumsum(torch.bincount(cell, minlength=side * side), 0)
    us, vs = [], []
    for dx, dy in ((0, 0), (1, 0), (-1, 1), (0, 1), (1, 1)):  # each pair of cells once
        x, y = at[:, 0] + dx, at[:, 1] + dy
        u = torch.nonzero((x >= 0) & (x < side) & (y < side))[:, 0]
        c = y[u] * side + x[u]
        count = start[c + 1] - start[c]
        rep = torch.repeat_interleave(torch.arange(u.numel(), device=DEVICE), count)
        first = torch.cumsum(count, 0) - count
        v = members[start[c][rep] + torch.arange(rep.numel(), device=DEVICE) - first[rep]]
        u = u[rep]
        near = ((p[u] - p[v]) ** 2).sum(1) < radius * radius
        us.append(u[near])
        vs.append(v[near])
    return _csr(n, torch.cat(us), torch.cat(vs), weighted, gen)


def _graph(family, n, deg, weighted, gen):
    if family == "rmat":
        return _rmat(n, deg, weighted, gen)
    return _ba(n, deg, weighted, gen) if family == "ba" else _rgg(n, weighted, gen)


def _batch(case, seed):
    """A third of each family, n log-uniform up to case["n"], k a power of two up to case["k"]; the mix is the case's."""
    rng, gen = random.Random(case["n"] * 64 + case["count"]), _generator(seed)
    graphs, k, eps = [], [], []
    for i in range(case["count"]):
        n = _log_uniform(rng, min(1 << 10, case["n"]), case["n"])
        family = ("ba", "rmat", "rgg")[i % 3]
        deg = {"ba": rng.choice([4, 8, 16]), "rmat": rng.randint(8, 16), "rgg": 0}[family]
        graphs.append(_graph(family, n, deg, case["weighted"], gen))
        k.append(2 << rng.randrange(max(1, int(math.log2(case["k"])))))
        eps.append(rng.choice([0.01, 0.03, 0.05]))
    base = np.concatenate([[0], np.cumsum([g["n"] for g in graphs])])
    slots = np.concatenate([[0], np.cumsum([g["adjncy"].numel() for g in graphs])])
    d = {"n": int(base[-1]),
         "xadj": torch.cat([graphs[0]["xadj"][:1]] + [g["xadj"][1:] + int(s) for g, s in zip(graphs, slots)]),
         "adjncy": torch.cat([g["adjncy"] + int(b) for g, b in zip(graphs, base)]),
         "adjwgt": torch.cat([g["adjwgt"] for g in graphs]), "vwgt": torch.cat([g["vwgt"] for g in graphs])}
    return d, base.astype(np.int32), np.array(k), np.array(eps), seed + np.arange(case["count"])


# ---------------------------------------------------------------- the calls

def _options(case):
    return {key: case[key] for key in ("max_levels", "vcycles", "degree_order", "initial_partitioner")
            if key in case}


def _cluster_bound(case):
    return max(1, case["n"] // (18 * case["k"]))  # unit node weights


def _most_slots(case):
    """More adjacency slots than any graph of the case has."""
    n, deg = case["n"], case["deg"]
    return {"rmat": 2 * deg << max(1, (n - 1).bit_length()), "ba": 2 * deg * n, "rgg": 2 * n * int(math.log(n) + 1)}[
        case["family"]]


def prepare(case, seed):
    op, k = case["op"], case["k"]
    s = {"case": case, "seed": seed}
    if op == "batch":
        s["graph"], s["base"], s["k"], s["eps"], s["seeds"] = _batch(case, seed)
        return s
    gen = _generator(seed)
    g = s["graph"] = _graph(case["family"], case["n"], case["deg"], case["weighted"], gen)
    if op == "partition_host":
        s["graph"] = {key: v if key == "n" else v.cpu().numpy() for key, v in g.items()}
    elif op == "contract":
        s["labels"] = sc.cluster_dev(g, _cluster_bound(case), seed=seed)[0]
        # a level's buffers, sized once for any graph of this kind
        n, cap = case["n"], _most_slots(case)
        s["level"] = {key: torch.zeros(size, dtype=kind, device=DEVICE) for key, size, kind in (
            ("xadj", n + 1, torch.int64), ("adjncy", cap, torch.int32), ("adjwgt", cap, torch.int32),
            ("vwgt", n, torch.int32))}
    elif op == "refine":
        # a partition of the graph, a tenth of whose nodes have been placed anew since
        s["part"] = sc.partition_dev(g, k, case["eps"], seed)["part"]
        moved = torch.rand(case["n"], generator=gen, device=DEVICE) < 0.1
        anew = torch.randint(0, k, (case["n"],), generator=gen, device=DEVICE, dtype=torch.int32)
        s["part"] = torch.where(moved, anew, s["part"])
        s["lmax"] = sc.lmax(case["n"], k, case["eps"])
    elif op == "project_cut":
        s["C"], coarse = sc.contract_dev(g, sc.cluster_dev(g, _cluster_bound(case), seed=seed)[0])
        s["coarse_part"] = torch.randint(0, k, (coarse["n"],), generator=gen, device=DEVICE, dtype=torch.int32)
    torch.cuda.synchronize()
    return s


def run(state):
    case, seed, g = state["case"], state["seed"], state["graph"]
    op, k, eps = case["op"], case["k"], case["eps"]
    if op == "partition" or op == "partition_host":
        call = sc.partition if op == "partition_host" else sc.partition_dev
        r = call(g, k, eps, seed, **_options(case))
        return {key: r[key] for key in ("part", "cut", "block_weights", "status")}
    if op == "batch":
        r = sc.partition_batch_dev(g, state["base"], state["k"], state["eps"], state["seeds"])
        return {key: r[key] for key in ("part", "cut", "block_weights", "levels", "status")}
    if op == "cluster":
        return sc.cluster_dev(g, _cluster_bound(case), seed=seed)
    if op == "contract":
        C, coarse = sc.contract_dev(g, state["labels"])
        for key, to in state["level"].items():
            to[:coarse[key].numel()].copy_(coarse[key])
        return C, coarse["n"], coarse["adjncy"].numel(), state["level"]
    if op == "refine":
        return sc.refine_dev(g, k, state["lmax"], state["part"].clone(), seed=seed)
    part = sc.project_dev(state["C"], state["coarse_part"])
    return (part,) + sc.cut_dev(g, part, k)


def work(case):
    """The graph read once and the outputs written once; rows by the families' mean degrees."""
    n = case["n"]
    slots = {"rmat": 1.9 * case["deg"], "ba": 2.0 * case["deg"], "rgg": 0.95 * math.log(max(n, 2)),
             "mix": 17.0}[case["family"]] * n
    if case["op"] == "batch":  # the mean of a log-uniform size
        lo = min(1 << 10, n)
        scale = case["count"] * ((n - lo) / math.log(n / lo) if n > lo else n) / n
        n, slots = n * scale, slots * scale
    graph = 8 * (n + 1) + 4 * n + 8 * slots
    more = 4 * n  # the part or the labels
    if case["op"] == "contract":
        more += 4 * n + graph / 4  # labels read; the coarse graph
    elif case["op"] in ("refine", "project_cut"):
        more += 4 * n  # the part before; the coarse ids
    return {"bytes": graph + more, "flops": 0}


def exact(case, seed):
    """Partitions and clusterings are the method's own; projection, cut and block weights have plain values."""
    if case["op"] != "project_cut":
        return None
    s = prepare(case, seed)
    g, part = s["graph"], s["coarse_part"][s["C"].long()]
    rows = torch.repeat_interleave(torch.arange(case["n"], device=DEVICE), g["xadj"].diff())
    crossing = part[rows] != part[g["adjncy"].long()]
    cut = int(g["adjwgt"].long()[crossing].sum()) // 2
    return part, cut, torch.bincount(part, minlength=case["k"]).cpu().numpy()
