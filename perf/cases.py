"""Performance cases of the batched max-flow library: what a schedule generator asks of it, at the sizes it does.

A generator run has four stages, and every stage is here.  The optimality search asks for verdicts on one fabric, many
(sink, candidate) max-flows at a time (`batch`, `feasible`, `floor`), or runs as a whole from the link list to (U, k)
(`search`).  Edge splitting asks how much each pair of links through a switch can give (`gamma`) and removes the
switches (`remove`).  Tree construction packs the trees on what is left (`trees`).

The fabrics are the ones of this repository's benchmark configurations, redrawn for every seed: boxes of compute nodes
around a box switch whose network cards go to one spine or to rails; a two-level fat tree; directly connected boxes; a
random fabric of given out-degree.  A seed draws what differs between two real clusters of one kind: box generations,
links that run at half their rate, random wiring.  Everything is an integer, so results have to be equal.
"""
import itertools
import random

import numpy as np
import torch

import paper_2402_06787_amd as fc

DEV = "cuda"


# ------------------------------------------------------------------------------------------------------------ cases

def listed():
    return [
        # Two boxes of eight nodes, one candidate, every node as sink: the smallest question, asked while a fabric is
        # explored interactively.  One launch; latency is all there is.
        {"name": "batch_two_boxes", "op": "batch", "fabric": "boxes", "boxes": 2, "per_box": 8, "rails": 1, "nic": 8,
         "candidates": 1, "k": 4, "bounded": False},
        # Two directly connected boxes of 16, eight candidates: a node pair as sold, one round of a search.
        {"name": "batch_direct_2x16", "op": "batch", "fabric": "direct", "boxes": 2, "per_box": 16, "candidates": 8, "k": 4,
         "bounded": True},
        # 16 boxes of eight nodes around one spine, 32 candidates: verdicts and witnesses of a common cluster.
        {"name": "feasible_boxes_16x8", "op": "feasible", "fabric": "boxes", "boxes": 16, "per_box": 8, "rails": 1, "nic": 2,
         "candidates": 32, "k": 8, "bounded": True, "flows": False},
        # A fat tree of 64 boxes with leaves and spines, 16 candidates.
        {"name": "batch_fat_tree_64x8", "op": "batch", "fabric": "fat_tree", "boxes": 64, "per_box": 8, "candidates": 16, "k": 4,
         "bounded": True},
        # The largest list: a heterogeneous fabric of 1024 nodes and 128 switches, 16 candidates.
        {"name": "batch_random_1024", "op": "batch", "fabric": "random", "nodes": 1024, "switches": 128, "degree": 8,
         "candidates": 16, "k": 16, "bounded": True},
        # A ragged fabric and an odd number of candidates, default options, all flow values wanted.
        {"name": "feasible_random_523", "op": "feasible", "fabric": "random", "nodes": 523, "switches": 61, "degree": 7,
         "candidates": 11, "k": 9, "bounded": False, "flows": True},
        # A fixed number of trees per node: rational multipliers and rounded-down capacities.
        {"name": "floor_random_777", "op": "floor", "fabric": "random", "nodes": 777, "switches": 95, "degree": 8,
         "candidates": 16, "k": 2, "bounded": True, "flows": False},
        # From the link list of a new fabric to its optimal throughput: ingest, per-sink tables, every round of the
        # search, and which nodes limit it.
        {"name": "search_random_1024", "op": "search", "fabric": "random", "nodes": 1024, "switches": 128, "degree": 8,
         "candidates": 16},
        # 256 link pairs through the switches of a cluster, 2N max-flows each, only gamma wanted.
        {"name": "gamma_boxes_16x8", "op": "gamma", "fabric": "boxes", "boxes": 16, "per_box": 8, "rails": 1, "nic": 2,
         "pairs": 256, "flows": False},
        # All switches of that cluster removed.
        {"name": "remove_boxes_16x8", "op": "remove", "fabric": "boxes", "boxes": 16, "per_box": 8, "rails": 1, "nic": 2},
        # The spanning trees of that cluster.
        {"name": "trees_boxes_16x8", "op": "trees", "fabric": "boxes", "boxes": 16, "per_box": 8, "rails": 1, "nic": 2},
        # The spanning trees of a rail-optimised cluster of 256 nodes.
        {"name": "trees_rails_32x8", "op": "trees", "fabric": "boxes", "boxes": 32, "per_box": 8, "rails": 8, "nic": 2},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges: every kind of question, on every kind of fabric that it is asked of."""
    op = rng.choice(["batch", "batch", "feasible", "feasible", "floor", "search", "gamma", "remove", "trees"])
    c = {"op": op}
    # the back end (and gamma) needs as much bandwidth into every vertex as out of it, and is asked of switched clusters
    fabric = "boxes" if op in ("gamma", "remove", "trees") else "random" if op == "search" else rng.choice(["boxes", "fat_tree", "direct", "random", "random"])
    c["fabric"] = fabric
    if fabric == "random":
        nodes = _log_uniform(rng, 128 if op == "search" else 24, 1024)
        c.update(nodes=nodes, switches=max(2, nodes // rng.randint(6, 12)), degree=rng.randint(6, 8))
        size = nodes
    elif fabric == "fat_tree":
        c.update(boxes=4 * rng.randint(2, 16), per_box=rng.choice([4, 8]))
        size = c["boxes"] * c["per_box"]
    elif fabric == "direct":
        c.update(boxes=rng.randint(2, 8), per_box=rng.choice([8, 12, 16]))
        size = c["boxes"] * c["per_box"]
    else:
        per_box = rng.choice([4, 6, 8])
        c.update(boxes=_log_uniform(rng, 6, 16 if op == "gamma" else 24 if op in ("remove", "trees") else 128), per_box=per_box,
                 rails=rng.choice([1, per_box]), nic=2)
        size = c["boxes"] * c["per_box"]
    if op in ("batch", "feasible", "floor"):
        most = max(1, min(32, 16384 // size))
        c.update(candidates=_log_uniform(rng, 1, most), k=rng.randint(1, 16) if op != "floor" else rng.randint(1, 4), bounded=rng.random() < 0.5)
    if op in ("feasible", "floor"):
        c["flows"] = c["candidates"] < 4 or rng.random() < 0.5
    if op == "search":
        c["candidates"] = rng.choice([8, 16, 32])
    if op == "gamma":
        c.update(pairs=_log_uniform(rng, 16, 256), flows=rng.random() < 0.3)
    return c


# ---------------------------------------------------------------------------------------------------------- fabrics

class _Links:
    def __init__(self, n, n_compute):
        self.n, self.n_compute = n, n_compute
        self.t, self.h, self.b = [], [], []

    def arc(self, u, v, bw):
        self.t.append(u), self.h.append(v), self.b.append(bw)

    def link(self, u, v, bw):
        self.arc(u, v, bw), self.arc(v, u, bw)

    def arrays(self):
        is_compute = np.zeros(self.n, dtype=np.uint8)
        is_compute[: self.n_compute] = 1
        return self.n, np.array(self.t, np.int32), np.array(self.h, np.int32), np.array(self.b, np.int32), is_compute


def _boxes(c, rng):
    """Boxes of compute nodes around a box switch; node j of a box has a network card to rail j (or to the one spine).
    Box generations differ in the bandwidth inside, and every fourth box has cards of twice the rate; where verdicts are
    asked for, one card in fifty runs at half its rate.  (Two boxes: the box switches themselves go to the spine, as in
    the smallest configuration, and every node has a bandwidth of its own.)"""
    boxes, per_box, rails, nic = c["boxes"], c["per_box"], c["rails"], c["nic"]
    n_compute = boxes * per_box
    f = _Links(n_compute + boxes + rails, n_compute)
    if boxes == 2:
        for u in range(n_compute):
            f.link(u, n_compute + u // per_box, rng.randint(8, 16))
        for box in range(2):
            f.link(n_compute + box, n_compute + 2, nic - rng.randint(0, nic // 4))
        return f.arrays()
    slow = set()
    if c["op"] in ("batch", "feasible", "floor"):
        slow = set(rng.sample(range(n_compute), max(1, n_compute // 50)))
    newer = set(rng.sample(range(boxes), boxes // 4))
    for box in range(boxes):
        inside = 2 * rng.randint(10, 16)
        card = 2 * nic if box in newer else nic
        for j in range(per_box):
            u = box * per_box + j
            f.link(u, n_compute + box, inside)
            f.link(u, n_compute + boxes + j % rails, card // 2 if u in slow else card)
    return f.arrays()


def _fat_tree(c, rng):
    """Boxes with a switch inside, four boxes to a leaf, every leaf to four spines; one uplink in fifty at half its rate."""
    boxes, per_box = c["boxes"], c["per_box"]
    n_compute, leaves = boxes * per_box, boxes // 4
    f = _Links(n_compute + boxes + leaves + 4, n_compute)
    slow = set(rng.sample(range(n_compute), max(1, n_compute // 50)))
    for u in range(n_compute):
        box = u // per_box
        f.link(u, n_compute + box, 32)
        f.link(u, n_compute + boxes + box // 4, 2 if u in slow else 4)
    for leaf in range(leaves):
        for spine in range(4):
            f.link(n_compute + boxes + leaf, n_compute + boxes + leaves + spine, 8 * per_box)
    return f.arrays()


def _direct(c, rng):
    """Boxes whose nodes are joined directly, by up to four parallel links of bandwidth 2 a pair and eight a node, and
    four network cards a box to one switch."""
    boxes, per_box = c["boxes"], c["per_box"]
    n_compute = boxes * per_box
    f = _Links(n_compute + 1, n_compute)
    for box in range(boxes):
        base = box * per_box
        free = [8] * per_box
        for j in range(per_box):               # a ring first: a box hangs together
            f.link(base + j, base + (j + 1) % per_box, 2)
            free[j] -= 1
            free[(j + 1) % per_box] -= 1
        pairs = list(itertools.combinations(range(per_box), 2))
        rng.shuffle(pairs)
        for i, j in pairs:
            for _ in range(min(rng.randint(0, 4), free[i], free[j])):
                f.link(base + i, base + j, 2)
                free[i] -= 1
                free[j] -= 1
        for j in range(0, per_box, per_box // 4):
            f.link(base + j, n_compute, rng.randint(1, 2))
    return f.arrays()


def _random(c, rng):
    """A ring through all vertices and random arcs up to the out-degree, bandwidths 1 to 100."""
    n, degree = c["nodes"] + c["switches"], c["degree"]
    f = _Links(n, c["nodes"])
    for u in range(n):
        heads = [(u + 1) % n]
        while len(heads) < degree:
            v = rng.randrange(n)
            if v != u and v not in heads:
                heads.append(v)
        for v in heads:
            f.arc(u, v, rng.randint(1, 100))
    return f.arrays()


_FABRICS = {"boxes": _boxes, "fat_tree": _fat_tree, "direct": _direct, "random": _random}


def _device(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


# -------------------------------------------------------------------------------------------------- states and passes

def prepare(case, seed):
    rng = random.Random(seed)
    n, tail, head, bw, is_compute = _FABRICS[case["fabric"]](case, rng)
    op = case["op"]
    s = {"case": case, "fabric": (n, tail, head, bw, is_compute)}
    if op == "search":
        return s                               # the whole path starts from the link list
    g = fc.fc_graph_upload(n, tail, head, bw, is_compute)
    compute = np.flatnonzero(is_compute)
    if op in ("batch", "feasible", "floor"):
        # candidates around the optimum of this fabric, half of them below it, as a search's rounds have them (a single one
        # lies a quarter below it)
        C, k = case["candidates"], case["k"]
        if op == "floor":
            best = fc.fc_fixed_k_search(g, k, 16)["U_star"]
            base = best.numerator
            s["den"] = _device(np.full(C, best.denominator))
        else:
            best = fc.fc_opt_throughput_search(g, 16)["inv_xstar"]
            base = -((-k * best.numerator) // best.denominator)
        mult = np.maximum(1, base - (C // 2 if C > 1 else -(-base // 4)) + np.arange(C))
        cap = np.full(C, k)
        s["options"] = {"src_cap_bound": k} if case["bounded"] else None
        if op == "batch":
            s["sink"] = _device(np.tile(compute, C))
            mult, cap = np.repeat(mult, len(compute)), np.repeat(cap, len(compute))
            room = fc.fc_maxflow_batch_workspace_bytes(g, len(mult))
        else:
            room = fc.fc_feasible_workspace_bytes(g, C)
        s.update(g=g, mult=_device(mult), cap=_device(cap), ws=torch.empty(max(room, 256), dtype=torch.uint8, device=DEV))
        return s
    # the stages after the search work on the integer capacities U * b with k trees per node
    found = fc.fc_opt_throughput_search(g, 16)
    U, k = found["U"].numerator, found["k"] * found["U"].denominator
    if op == "gamma":
        into = np.flatnonzero(is_compute[head] == 0)
        pairs = []
        for _ in range(case["pairs"]):
            e = int(into[rng.randrange(len(into))])
            out = np.flatnonzero(tail == head[e])
            pairs.append((tail[e], head[e], head[out[rng.randrange(len(out))]]))
        room = fc.fc_split_gamma_workspace_bytes(g, len(pairs))
        s.update(g=g, U=U, k=k, pairs=[_device(x) for x in zip(*pairs)], ws=torch.empty(room, dtype=torch.uint8, device=DEV))
        return s
    g.close()
    capacity = (bw.astype(np.int64) * U).astype(np.int32)
    s.update(capacity=capacity, k=k)
    if op == "trees":
        star = fc.fc_remove_switches(n, tail, head, capacity, is_compute, k)["links"]     # compute nodes come first: ids stay
        s.update(n_compute=len(compute), links=star)
    return s


def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "batch":
        # a caller that keeps its workspace, or one that leaves it to the call
        return fc.fc_maxflow_batch(s["g"], s["sink"], s["mult"], s["cap"], d_workspace=s["ws"] if case["bounded"] else None, options=s["options"])[0]
    if op in ("feasible", "floor"):
        kw = dict(want_flows=case["flows"], d_workspace=s["ws"] if case["bounded"] else None, options=s["options"])
        if op == "feasible":
            r = fc.fc_feasible(s["g"], s["mult"], s["cap"], **kw)
        else:
            r = fc.fc_feasible_floor(s["g"], s["mult"], s["den"], s["cap"], **kw)
        return [r["feasible"], r["witness"]] + ([r["flows"]] if case["flows"] else [])
    if op == "search":
        with fc.fc_graph_upload(*s["fabric"]) as g:
            r = fc.fc_opt_throughput_search(g, case["candidates"])
            # and what every node gets just below the optimum: which ones limit the fabric
            p, q = r["inv_xstar"].numerator, r["inv_xstar"].denominator
            below = fc.fc_feasible(g, _device([max(1, p - 1)]), _device([q]), want_flows=True)["flows"]
        return [p, q, r["U"].numerator, r["U"].denominator, r["k"], below]
    if op == "gamma":
        r = fc.fc_split_gamma_batch(s["g"], s["U"], s["k"], *s["pairs"], want_flows=case["flows"], d_workspace=s["ws"])
        return [r["gamma"]] + ([r["flows"]] if case["flows"] else [])
    n, tail, head, _, is_compute = s["fabric"]
    if op == "remove":
        r = fc.fc_remove_switches(n, tail, head, s["capacity"], is_compute, s["k"])
        # the link matrix of the digraph that is left, and how much of a link each switch carries
        N = int(is_compute.sum())
        left, routed = np.zeros((N, N), dtype=np.int32), np.zeros((n - N, N, N), dtype=np.int32)
        for (u, t), c in r["links"].items():
            left[u, t] = c
        for (u, t), row in r["table"].items():
            for w, c in row.items():
                routed[w - N, u, t] = c
        return [left, routed]
    # every node's k trees in the order they were made, each as its edges in the order they were added
    N, k = s["n_compute"], s["k"]
    trees = fc.fc_construct_trees(N, s["links"], k)["trees"]
    edges = itertools.chain.from_iterable(itertools.chain.from_iterable(e for _, _, e in trees))
    edges = np.fromiter(edges, dtype=np.int32, count=2 * len(trees) * (N - 1)).reshape(len(trees), N - 1, 2)
    times = [mult for _, mult, _ in trees]
    return [np.repeat(np.array([root for root, _, _ in trees], dtype=np.int32), times), np.repeat(edges, times, axis=0)]


def _sizes(case):
    """Vertices, compute nodes and arcs."""
    f = case["fabric"]
    if f == "random":
        n = case["nodes"] + case["switches"]
        return n, case["nodes"], n * case["degree"]
    n_compute = case["boxes"] * case["per_box"]
    if f == "direct":
        return n_compute + 1, n_compute, case["boxes"] * (8 * case["per_box"] + 8)
    if f == "fat_tree":
        return n_compute + case["boxes"] * 5 // 4 + 4, n_compute, 4 * n_compute + 2 * case["boxes"]
    return n_compute + case["boxes"] + case["rails"], n_compute, 4 * n_compute


def work(case):
    """Bytes: the fabric (tail, head, bandwidth of every arc) and the questions read once, the answers written once.
    Operations: one addition for every compute node of every max-flow that has to be known (its units leave it along at
    least one arc); for the searches and loops, the max-flows of one round or of one step of every tree."""
    n, N, m = _sizes(case)
    op, fabric = case["op"], 12 * m + n
    if op in ("batch", "feasible", "floor"):
        C = case["candidates"]
        asked = 12 * C * N if op == "batch" else 12 * C
        told = 4 * C * N if op == "batch" or case["flows"] else 0
        return {"bytes": fabric + asked + told + (5 * C if op != "batch" else 0), "flops": C * N * N}
    if op == "search":
        return {"bytes": fabric + 48 + 4 * N, "flops": case["candidates"] * N * N}
    if op == "gamma":
        return {"bytes": fabric + 16 * case["pairs"] + (8 * N * case["pairs"] if case["flows"] else 0), "flops": 2 * case["pairs"] * N * N}
    if op == "remove":
        return {"bytes": fabric + 4 * N * N * (n - N + 1), "flops": 4 * N * N * (n - N)}
    return {"bytes": fabric + 8 * N * (N - 1), "flops": N * N * (N - 1)}


def tolerance(case):
    return "exact"                             # integers, and the same choice of links and trees every time
