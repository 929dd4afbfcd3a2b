"""GPU tests of the per-sink solver (batches that ask about every compute node): what one max-flow settles for the other
candidates of its sink, in every order and with every kind of candidate, against the oracle and against the solver that takes one
problem at a time."""
import numpy as np
import pytest

import oracle as o
import workloads as w

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():          # selected explicitly on a machine without a GPU
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2402_06787_amd as fc   # noqa: E402

DEV = torch.device("cuda:0")
ALONE = {"global_relabel_steps": 32}       # (its default: an option that only the other solver knows takes the call there)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _random(n, degree, seed, hub=False, halves=False):
    """A ring through all vertices (two rings that nothing joins with `halves`) and random arcs, some with the link back."""
    rng = np.random.default_rng(seed)
    t, h = [], []
    for u in range(n):
        lo, hi = (0, n) if not halves else ((0, n // 2) if u < n // 2 else (n // 2, n))
        heads = {lo + (u - lo + 1) % (hi - lo)} | set(rng.integers(lo, hi, degree).tolist())
        if hub and u == 3:
            heads |= set(range(n))
        for v in sorted(heads - {u}):
            t.append(u); h.append(v)
            if rng.random() < 0.2:
                t.append(v); h.append(u)
    isc = np.ones(n, np.uint8)
    isc[rng.permutation(n)[: n // 10]] = 0
    return w.Topology(f"r{n}", n, np.array(t, np.int32), np.array(h, np.int32), rng.integers(1, 60, len(t)).astype(np.int32), isc)


def _spine(boxes, per_box, seed):
    """Boxes around a switch, every node with a card to one spine; some cards at half their rate."""
    rng = np.random.default_rng(seed)
    N = boxes * per_box
    t, h, b = [], [], []
    for u in range(N):
        for x, bw in ((N + u // per_box, 24), (N + boxes, 1 if rng.random() < 0.05 else 2)):
            t += [u, x]; h += [x, u]; b += [bw, bw]
    isc = np.zeros(N + boxes + 1, np.uint8)
    isc[:N] = 1
    return w.Topology("spine", N + boxes + 1, np.array(t, np.int32), np.array(h, np.int32), np.array(b, np.int32), isc)


TOPOLOGIES = {
    "few links": lambda: _random(300, 6, 1),                  # heights are searched by links
    "many links": lambda: _random(620, 8, 2),                 # ... by a queue
    "257 vertices": lambda: _random(257, 4, 3, hub=True),     # the first size beyond the bit rows; a row longer than any chunk
    "two halves": lambda: _random(266, 5, 4, halves=True),    # half of the nodes cannot reach a sink: a cut without bandwidth
    "long rows": lambda: _random(280, 24, 6),                 # first arcs are chosen one vertex at a time
    "rails": lambda: w.rail_fabric(36, 8),
    "spine": lambda: _spine(34, 8, 5),
}


def _merged(topo):
    tail, head, bw = o.links(topo)
    return w.Topology(topo.name, topo.n_vertices, tail, head, bw, topo.is_compute)


def _in_bw(topo):
    into = np.zeros(topo.n_vertices, np.int64)
    np.add.at(into, topo.head, topo.bandwidth)
    return into[topo.compute_nodes]


def _candidates(topo, C, seed, wide=False):
    """C candidates around the sink cuts' optimum: mixed and equal k, in no order, some twice, some far off, some invalid."""
    rng = np.random.default_rng(seed)
    N = topo.n_compute
    base = N / max(1, int(np.median(_in_bw(topo))))
    k = np.where(rng.random(C) < 0.5, 6, rng.integers(1, 30, C))
    if wide:
        k = k * (70000 // N)                                  # demands on both sides of 65535
    U = np.maximum(1, (k * base * rng.choice([0.05, 0.5, 0.8, 0.95, 1.0, 1.05, 1.3, 2.0, 6.0], C) * rng.uniform(0.97, 1.03, C)).astype(np.int64))
    if C >= 9:
        U[3], k[3] = U[7], k[7]
        U[5] = 0
        k[6] = 0
    return U.astype(np.int32), k.astype(np.int32)


def _want(topo, U, k):
    """[C, N] values, FC_FLOW_INVALID where the candidate is."""
    comp = topo.compute_nodes
    ok = (U >= 1) & (k >= 1)
    want = np.full((len(U), len(comp)), fc.FC_FLOW_INVALID, np.int64)
    C = int(ok.sum())
    want[ok] = o.aux_maxflow_batch(topo, np.tile(comp, C).astype(np.int32), np.repeat(U[ok], len(comp)), np.repeat(k[ok], len(comp)), threads=16).reshape(C, len(comp))
    return want


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("C", [1, 9, 66])
@pytest.mark.parametrize("name", TOPOLOGIES)
def test_values_in_every_order(name, C, wide):
    topo = TOPOLOGIES[name]()
    comp, N = topo.compute_nodes, topo.n_compute
    U, k = _candidates(topo, C, 17 * C + wide, wide)
    want = _want(topo, U, k).reshape(-1)
    sink, Us, ks = np.tile(comp, C), np.repeat(U, N), np.repeat(k, N)
    rng = np.random.default_rng(C)
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        alone, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks), options=ALONE)
        assert (alone.cpu().numpy() == want).all()
        orders = {"over and over": np.arange(C * N), "in a row": np.arange(C * N).reshape(C, N).T.reshape(-1), "mixed": rng.permutation(C * N)}
        for order, perm in orders.items():
            got, _ = fc.fc_maxflow_batch(g, _dev(sink[perm]), _dev(Us[perm]), _dev(ks[perm]))
            assert (got.cpu().numpy() == want[perm]).all(), order
        if not wide:                                          # the caller's bound leaves out the 32-bit state
            got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks), options={"src_cap_bound": int(k.max()), "tree_certificate": 1})
            assert (got.cpu().numpy() == want).all()
        else:                                                 # and refuses what breaks the promise
            got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks), options={"src_cap_bound": 1})
            over = ks.astype(np.int64) * N > 65535
            assert (got.cpu().numpy() == np.where(over & (Us >= 1), fc.FC_FLOW_UNSUPPORTED, want)).all()
        need = k.astype(np.int64) * N
        for flows in (True, False):
            r = fc.fc_feasible(g, _dev(U), _dev(k), want_flows=flows)
            low = want.reshape(C, N) < need[:, None]
            ok = (U >= 1) & (k >= 1)
            assert (r["feasible"].cpu().numpy().astype(bool) == (ok & ~low.any(axis=1))).all(), flows
            assert (r["witness"].cpu().numpy() == np.where(ok & low.any(axis=1), comp[low.argmax(axis=1)], -1)).all(), flows
            if flows:
                assert (r["flows"].cpu().numpy().reshape(-1) == want).all()


@pytest.mark.parametrize("C", [1, 3, 21])
@pytest.mark.parametrize("name", TOPOLOGIES)
def test_rounded_down_capacities(name, C):
    topo = TOPOLOGIES[name]()
    comp, N = topo.compute_nodes, topo.n_compute
    rng = np.random.default_rng(C + 5)
    base = N / max(1, int(np.median(_in_bw(topo))))
    den = rng.integers(1, 60, C)
    k = np.where(rng.random(C) < 0.7, 3, rng.integers(1, 9, C))
    num = np.maximum(1, (k * den * base * rng.choice([0.3, 0.9, 1.0, 1.1, 1.5, 3.0], C)).astype(np.int64))
    want = o.aux_maxflow_batch_floor(topo, np.tile(comp, C), np.repeat(num, N), np.repeat(den, N), np.repeat(k, N), threads=16).reshape(C, N)
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        low = want < (k * N)[:, None]
        for flows in (False, True):
            r = fc.fc_feasible_floor(g, _dev(num), _dev(den), _dev(k), want_flows=flows)
            assert (r["feasible"].cpu().numpy().astype(bool) == ~low.any(axis=1)).all(), flows
            assert (r["witness"].cpu().numpy() == np.where(low.any(axis=1), comp[low.argmax(axis=1)], -1)).all(), flows
        assert (r["flows"].cpu().numpy() == want).all()
        got, _ = fc.fc_maxflow_batch_floor(g, _dev(np.tile(comp, C)), _dev(np.repeat(num, N)), _dev(np.repeat(den, N)), _dev(np.repeat(k, N)))
        assert (got.cpu().numpy().reshape(C, N) == want).all()


def test_weights_and_updated_bandwidths():
    topo = _random(290, 6, 8)
    comp, N, C = topo.compute_nodes, topo.n_compute, 12
    rng = np.random.default_rng(9)
    weights = np.zeros(topo.n_vertices, np.int32)
    weights[comp] = rng.integers(0, 4, N)
    U, k = rng.integers(1, 40, C).astype(np.int32), np.full(C, 3, np.int32)
    sink, Us, ks = np.tile(comp, C), np.repeat(U, N), np.repeat(k, N)
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        # links in both directions at a fraction of their bandwidth, tables rebuilt: what a search by links reads has to follow
        caps = o.link_capacities(topo)
        some = sorted(caps)[:: 7]
        now = {**caps, **{key: max(1, caps[key] // 5) for key in some}}
        fc.fc_graph_update_arcs(g, [a for a, _ in some], [b for _, b in some], [now[key] for key in some], refresh_tables=True)
        keys = sorted(now)
        changed = w.Topology("changed", topo.n_vertices, np.array([a for a, _ in keys], np.int32), np.array([b for _, b in keys], np.int32),
                             np.array([now[key] for key in keys], np.int32), topo.is_compute)
        want = o.aux_maxflow_batch(changed, sink, Us, ks, threads=16)
        got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks))
        assert (got.cpu().numpy() == want).all()
        fc.fc_graph_set_source_weights(g, weights)
        some_p = np.concatenate([np.arange(c * N, c * N + N, 17) for c in range(C)])
        got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks))
        alone, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(Us), _dev(ks), options=ALONE)
        assert torch.equal(got, alone)
        assert (got.cpu().numpy()[some_p] == o.weighted_aux_maxflow_batch(changed, sink[some_p], Us[some_p], ks[some_p], weights)).all()
        # verdicts of rounded-down capacities: what a cut forbids counts the weights on the sink's side
        total = int(weights.sum())
        kk = np.array([1, 2, 2, 2, 2, 2, 2, 2, 3, 3, 3, 2], np.int32)
        num = np.maximum(1, (kk * 7 * total / _in_bw(changed).min() * np.linspace(0.2, 4.0, C)).astype(np.int64))
        args = _dev(num), _dev(np.full(C, 7)), _dev(kk)
        r, single = fc.fc_feasible_floor(g, *args), fc.fc_feasible_floor(g, *args, want_flows=True, options=ALONE)
        assert torch.equal(r["feasible"], single["feasible"]) and torch.equal(r["witness"], single["witness"])
        assert (single["flows"].cpu().numpy() < (kk.astype(np.int64) * total)[:, None]).any(axis=1).any() and single["feasible"].any()
        some_n = np.arange(0, N, 29)
        ref = o.weighted_aux_maxflow_batch(_merged(changed), np.tile(comp[some_n], C), np.repeat(num, len(some_n)), np.repeat(kk, len(some_n)), weights, U_den=np.full(C * len(some_n), 7))
        assert (single["flows"].cpu().numpy()[:, some_n].reshape(-1) == ref).all()


def test_a_cut_too_wide_for_its_product_forbids_nothing():
    """A minimum cut of 2.1e11 units of bandwidth, none of which carries anything at the smallest multiplier: its bandwidth times the others'
    numerator is beyond 2^63, and all of them are feasible."""
    N, S, W = 256, 255, 1 << 23
    t, h, b = [], [], []

    def link(x, y, bw):
        t.append(x); h.append(y); b.append(bw)
    for s in range(S):
        link(N + s, 0, W)                                     # 255 links that just carry a unit at 1 / 2^23 ...
        for j in range(100):
            link(1 + (s + j) % (N - 1), N + s, W - 1)         # ... behind 25 500 that do not
    for v in range(2, N):                                     # the other nodes are a binary tree
        link(v, v // 2, W); link(v // 2, v, W)
    link(0, 1, W)
    isc = np.zeros(N + S, np.uint8)
    isc[:N] = 1
    topo = w.Topology("wide cut", N + S, np.array(t, np.int32), np.array(h, np.int32), np.array(b, np.int32), isc)
    num, den, k = np.array([1] + [1 << 26] * 7), np.array([W] + [1] * 7), np.ones(8, np.int64)
    want = o.aux_maxflow_batch_floor(topo, np.tile(topo.compute_nodes, 2), np.repeat(num[:2], N), np.repeat(den[:2], N), np.ones(2 * N, np.int64), threads=16).reshape(2, N)
    assert want[0, 0] == 1 and (want[1] == N).all()
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for flows in (False, True):
            r = fc.fc_feasible_floor(g, _dev(num), _dev(den), _dev(k), want_flows=flows)
            assert r["feasible"].cpu().tolist() == [0] + [1] * 7, flows
            assert r["witness"].cpu().tolist() == [int(topo.compute_nodes[(want[0] < N).argmax()])] + [-1] * 7, flows
        assert (r["flows"].cpu().numpy() == want[[0] + [1] * 7]).all()


@pytest.mark.parametrize("N", [300, 620])                     # heights searched by links, by a queue
def test_nearly_all_vertices_stuck_on_one_level(N):
    """Every node is joined to all three switches and to nothing else: all other nodes lie two levels above a sink, and at a small multiplier
    none of them gets rid of its units by its first arc, or at all.  (The values were right too when the list of the level's vertices could be
    written over by the vertices left with excess.)"""
    rng = np.random.default_rng(N)
    S = 3
    t, h, b = [], [], []
    for u in range(N):
        for x in range(S):
            t += [u, N + x]; h += [N + x, u]; b += rng.integers(1, 4, 2).tolist()
    for x in range(S):
        t.append(N + x); h.append(N + (x + 1) % S); b.append(5)
    isc = np.zeros(N + S, np.uint8)
    isc[:N] = 1
    topo = w.Topology("one level", N + S, np.array(t, np.int32), np.array(h, np.int32), np.array(b, np.int32), isc)
    comp = topo.compute_nodes
    U = np.array([1, 2, 9, N // 9, N // 6, N // 5, N // 4, N // 3, N], np.int32)
    k = np.array([3, 7, 30, 1, 1, 1, 1, 1, 1], np.int32)
    want = _want(topo, U, k)
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        got, _ = fc.fc_maxflow_batch(g, _dev(np.tile(comp, len(U))), _dev(np.repeat(U, N)), _dev(np.repeat(k, N)))
        assert (got.cpu().numpy() == want.reshape(-1)).all()
        for c in range(len(U)):                               # each candidate by itself: no other settles it
            got, _ = fc.fc_maxflow_batch(g, _dev(comp), _dev(np.repeat(U[c:c + 1], N)), _dev(np.repeat(k[c:c + 1], N)))
            assert (got.cpu().numpy() == want[c]).all(), c
        r = fc.fc_feasible(g, _dev(U), _dev(k))
        assert (r["feasible"].cpu().numpy().astype(bool) == (want == (k.astype(np.int64) * N)[:, None]).all(axis=1)).all()


@pytest.mark.parametrize("C", [2, 5, 9, 130])
@pytest.mark.parametrize("name", ["few links", "many links", "spine"])
def test_lists_in_no_order(name, C):
    """Lists that are neither the same sinks over and over nor each sink's problems in a row, of sinks that come unequally often: one of them
    half of the time (more often than a wavefront has lanes), switches, vertices that do not exist; and lists that look ordered but for a few places."""
    topo = TOPOLOGIES[name]()
    comp, N, n = topo.compute_nodes, topo.n_compute, topo.n_vertices
    rng = np.random.default_rng(C)
    U, k = _candidates(topo, max(C, 3), 5 * C)
    U, k = U[:C], k[:C]
    P = C * N
    sink = rng.integers(0, n, P)                              # any vertex, switches among them
    sink[rng.random(P) < 0.5] = comp[N // 3]
    strange = rng.choice(P, 7, replace=False)
    sink[strange] = [-1, n, n + 5, -2 ** 31, 2 ** 31 - 1, -7, n]
    nearly = np.tile(comp, C)                                 # over and over, but for a few
    places = rng.choice(P, 9, replace=False)
    nearly[places] = rng.integers(-1, n + 1, 9)
    tail = np.tile(comp, C)                                   # ordered, then not
    tail[P // 2:] = rng.permutation(tail[P // 2:])
    rows = np.repeat(comp, C)
    rows[places] = comp[0]
    known = {}

    def values(sinks, c):
        todo = sorted({(int(t), int(x)) for t, x in zip(sinks, c)} - set(known))
        ok = [(t, x) for t, x in todo if 0 <= t < n and U[x] >= 1 and k[x] >= 1]
        known.update({q: fc.FC_FLOW_INVALID for q in todo})
        if ok:
            got = o.aux_maxflow_batch(topo, np.array([t for t, _ in ok], np.int32), U[[x for _, x in ok]], k[[x for _, x in ok]], threads=16)
            known.update(zip(ok, got.tolist()))
        return np.array([known[(int(t), int(x))] for t, x in zip(sinks, c)])

    c = np.repeat(np.arange(C), N)
    with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for sinks, cand in ((sink, c), (nearly, c), (tail, c), (rows, np.tile(np.arange(C), N)), (sink, rng.integers(0, C, P))):
            got, _ = fc.fc_maxflow_batch(g, _dev(sinks), _dev(U[cand]), _dev(k[cand]))
            assert (got.cpu().numpy() == values(sinks, cand)).all()


@pytest.mark.parametrize("bounded", [True, False])            # with the caller's bound one size of flows, without it both
@pytest.mark.parametrize("C,kinds", [(8, 8), (16, 16), (17, 5), (17, 17), (40, 9), (70, 3), (70, 70), (130, 12)])
@pytest.mark.parametrize("name", ["few links", "spine", "many links"])
def test_verdicts_of_rounded_down_capacities_and_many_k(name, C, kinds, bounded):
    """One or many different k among the candidates: problems of one k share a workgroup, blocks of 64 candidates with more than eight go to the
    other solver; one block may be of either kind."""
    topo = TOPOLOGIES[name]()
    comp, N = topo.compute_nodes, topo.n_compute
    rng = np.random.default_rng(C + kinds)
    base = N / max(1, int(np.median(_in_bw(topo))))
    k = rng.permutation(np.arange(C) % kinds + 1)
    if C > 64:
        k[64:] = np.sort(k[64:]) // 4 + 1                     # fewer in the second block
    if not bounded:
        k *= 1 + 70000 // (N * kinds)                         # demands on both sides of 65535
    den = rng.integers(1, 50, C)
    num = np.maximum(1, (k * den * base * rng.choice([0.4, 0.9, 0.97, 1.0, 1.03, 1.1, 1.6], C)).astype(np.int64))
    num[C // 2] = 0
    ok = num >= 1
    some = np.sort(rng.choice(N, 40, replace=False)) if C > 20 else np.arange(N)      # (the oracle solves one by one)
    want = o.aux_maxflow_batch_floor(topo, np.tile(comp[some], int(ok.sum())), np.repeat(num[ok], len(some)), np.repeat(den[ok], len(some)),
                                     np.repeat(k[ok], len(some)), threads=16).reshape(-1, len(some))
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        opts = {"src_cap_bound": int(k.max())} if bounded else {}
        alone = fc.fc_feasible_floor(g, _dev(num), _dev(den), _dev(k), want_flows=True, options=dict(opts, **ALONE))
        flows = alone["flows"].cpu().numpy()
        assert (flows[ok][:, some] == want).all() and (flows[~ok] == fc.FC_FLOW_INVALID).all()
        for _ in range(2):
            r = fc.fc_feasible_floor(g, _dev(num), _dev(den), _dev(k), options=opts)
            assert torch.equal(r["feasible"], alone["feasible"]) and torch.equal(r["witness"], alone["witness"])


@pytest.mark.parametrize("n,degree,back", [(1400, 2, 0.0), (1300, 6, 0.2), (3000, 5, 0.2)])
def test_more_vertices_than_the_registers_hold(n, degree, back):
    """Set-up keeps 1024 labels and 1280 first-pass entries a problem in registers and takes the rest one by one; 2800 links are searched link by
    link, the others by a queue."""
    rng = np.random.default_rng(n)
    t, h = [], []
    for u in range(n):
        for v in sorted(({(u + 1) % n} | set(rng.integers(0, n, degree - 1).tolist())) - {u}):
            t.append(u); h.append(v)
            if rng.random() < back:
                t.append(v); h.append(u)
    isc = np.zeros(n, np.uint8)
    isc[rng.permutation(n)[:130]] = 1
    topo = w.Topology(f"large{n}", n, np.array(t, np.int32), np.array(h, np.int32), rng.integers(1, 60, len(t)).astype(np.int32), isc)
    comp, N, C = topo.compute_nodes, topo.n_compute, 5
    U, k = _candidates(topo, C, n)
    k[C - 1] = 70000 // N                                     # one demand beyond 65535
    U[C - 1] = U[C - 1] * 50
    want = _want(topo, U, k)
    perm = rng.permutation(C * N)
    sink, Us, ks = np.tile(comp, C), np.repeat(U, N), np.repeat(k, N)
    with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for p in (np.arange(C * N), perm):
            got, _ = fc.fc_maxflow_batch(g, _dev(sink[p]), _dev(Us[p]), _dev(ks[p]))
            assert (got.cpu().numpy() == want.reshape(-1)[p]).all()
        r = fc.fc_feasible(g, _dev(U), _dev(k))
        assert (r["feasible"].cpu().numpy().astype(bool) == (want == (k.astype(np.int64) * N)[:, None]).all(axis=1)).all()


def test_demands_of_both_sizes_in_two_launches():
    """10 500 links: the state with 32-bit flows fits a CU three times and the one with 16-bit flows four times, and 450 sinks need more places
    than that, so each size of demand has a launch of its own.  Candidates of one sink lie on both sides of 65535."""
    topo = _random(500, 17, 12)
    comp, N, C = topo.compute_nodes, topo.n_compute, 12
    assert N == 450 and 9000 < topo.n_arcs < 11000
    rng = np.random.default_rng(31)
    base = N / max(1, int(np.median(_in_bw(topo))))
    k = rng.permutation(np.array([1, 3, 20, 144, 145, 146, 147, 160, 200, 400, 145, 146]))      # 145 * 450 = 65250, 146 * 450 = 65700
    U = np.maximum(1, (k * base * rng.choice([0.6, 0.95, 1.0, 1.05, 1.4], C)).astype(np.int64)).astype(np.int32)
    k = k.astype(np.int32)
    want = _want(topo, U, k)
    need = k.astype(np.int64) * N
    assert (need <= 65535).sum() >= 4 and (need > 65535).sum() >= 4
    sink, Us, ks = np.tile(comp, C), np.repeat(U, N), np.repeat(k, N)
    low = want < need[:, None]
    with fc.fc_graph_upload(topo.n_vertices, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for p in (np.arange(C * N), np.arange(C * N).reshape(C, N).T.reshape(-1), rng.permutation(C * N)):
            got, _ = fc.fc_maxflow_batch(g, _dev(sink[p]), _dev(Us[p]), _dev(ks[p]))
            assert (got.cpu().numpy() == want.reshape(-1)[p]).all()
        for flows in (True, False):
            r = fc.fc_feasible(g, _dev(U), _dev(k), want_flows=flows)
            assert (r["feasible"].cpu().numpy().astype(bool) == ~low.any(axis=1)).all(), flows
            assert (r["witness"].cpu().numpy() == np.where(low.any(axis=1), comp[low.argmax(axis=1)], -1)).all(), flows
            if flows:
                assert (r["flows"].cpu().numpy() == want).all()
        # the same capacities as rational multipliers
        r = fc.fc_feasible_floor(g, _dev(U.astype(np.int64) * 3), _dev(np.full(C, 3)), _dev(k))
        assert (r["feasible"].cpu().numpy().astype(bool) == ~low.any(axis=1)).all()
        assert (r["witness"].cpu().numpy() == np.where(low.any(axis=1), comp[low.argmax(axis=1)], -1)).all()
