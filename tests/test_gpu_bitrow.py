"""GPU tests of the bit-row solver (graphs of at most 256 vertices): every number of words per row and the edges between
them, one vertex beyond, both kinds of multiplier, weights, in-place updates, and the other solver on the same graphs."""
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


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _random_topology(rng, n, degree):
    """A ring and random arcs, about a third of them with the link back; one vertex joined to everybody (rows longer than a
    wavefront on the larger graphs)."""
    t, h = [], []
    for u in range(n):
        heads = {(u + 1) % n} | set(rng.integers(0, n, degree).tolist())
        if u == 0:
            heads |= set(range(n))
        for v in sorted(heads - {u}):
            t.append(u); h.append(v)
            if rng.random() < 0.35:
                t.append(v); h.append(u)
    isc = np.zeros(n, np.uint8)
    isc[rng.permutation(n)[:max(2, int(n * rng.uniform(0.5, 1.0)))]] = 1
    return w.Topology(f"r{n}", n, np.array(t, np.int32), np.array(h, np.int32), rng.integers(1, 30, len(t)).astype(np.int32), isc)


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257])
def test_values_match_the_oracle_at_the_edges_of_the_row_words(n):
    rng = np.random.default_rng(1000 + n)
    for degree in (1, 6):
        topo = _random_topology(rng, n, degree)
        P, N = 120, topo.n_compute
        sink = rng.integers(0, n, P).astype(np.int32)
        k = rng.integers(1, 9, P).astype(np.int32)
        k[::5] = (2 ** 31 - 1) // N                       # the largest flows there are: sums of two residuals pass 2^31
        U = np.maximum(1, k.astype(np.int64) * N // 40 * rng.integers(1, 80, P) // 30).clip(1, 2 ** 30).astype(np.int32)
        den = rng.integers(1, 90, P).astype(np.int32)     # many capacities round down to nothing
        want = o.aux_maxflow_batch(topo, sink, U, k, threads=16)
        with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
            for stats in (False, True):
                got, st = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k), want_stats=stats)
                assert (got.cpu().numpy().astype(np.int64) == want).all(), (n, degree, stats)
            assert st["not_converged"] == 0
            other, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k), options={"force_wide": 1})
            assert (other.cpu().numpy() == want).all(), (n, degree)
            small = k < 1000                              # (the product num * b stays within the entry point's bounds)
            got, _ = fc.fc_maxflow_batch_floor(g, _dev(sink[small]), _dev(U[small]), _dev(den[small]), _dev(k[small]))
            ref = o.aux_maxflow_batch_floor(_merge(topo), sink[small], U[small], den[small], k[small], threads=16)
            assert (got.cpu().numpy().astype(np.int64) == ref).all(), (n, degree)


@pytest.mark.parametrize("n", [40, 150])
def test_a_broken_source_bound_is_refused(n):
    # N * bound fits 16 bits: a problem within the bound, one above it that still fits, and demands beyond 16 bits
    topo = _random_topology(np.random.default_rng(n), n, 3)
    N = topo.n_compute
    k = np.array([1, 2, 65535 // N, 65535 // N + 1, 10 * (65535 // N)], np.int32)
    sink, U = np.full(5, topo.compute_nodes[0], np.int32), np.full(5, 7, np.int32)
    want = o.aux_maxflow_batch(topo, sink, U, k, threads=4).tolist()[:3] + [fc.FC_FLOW_UNSUPPORTED] * 2
    with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for solver in ({}, {"global_relabel_steps": 32}):
            for stats in (False, True):
                got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k), options={"src_cap_bound": 1, **solver}, want_stats=stats)
                assert got.cpu().tolist() == want, (solver, stats)
            r = fc.fc_feasible(g, _dev(U), _dev(k), want_flows=True, options={"src_cap_bound": 1, **solver})
            assert (r["flows"].cpu().numpy()[3:] == fc.FC_FLOW_UNSUPPORTED).all() and r["feasible"].cpu().tolist()[3:] == [0, 0]
            assert (r["flows"].cpu().numpy()[:3] > 0).all()


def _merge(topo):
    acc = {}
    for a, b, c in zip(topo.tail.tolist(), topo.head.tolist(), topo.bandwidth.tolist()):
        acc[(a, b)] = acc.get((a, b), 0) + c
    keys = sorted(acc)
    return w.Topology(topo.name, topo.n_vertices, np.array([a for a, _ in keys], np.int32), np.array([b for _, b in keys], np.int32),
                      np.array([acc[x] for x in keys], np.int32), topo.is_compute)


@pytest.mark.parametrize("n", [40, 150])
def test_updated_links_and_weights_reach_the_bit_rows(n):
    rng = np.random.default_rng(n)
    topo = _merge(_random_topology(rng, n, 3))
    P = 100
    sink = rng.integers(0, n, P).astype(np.int32); k = rng.integers(1, 6, P).astype(np.int32); U = rng.integers(1, 12, P).astype(np.int32)
    with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        hit = rng.permutation(len(topo.tail))[: len(topo.tail) // 4]
        bw = topo.bandwidth.copy(); bw[hit] = rng.integers(0, 40, len(hit))
        fc.fc_graph_update_arcs(g, topo.tail[hit], topo.head[hit], bw[hit], refresh_tables=False)
        after = w.Topology("after", n, topo.tail, topo.head, bw, topo.is_compute)
        got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k))
        assert (got.cpu().numpy() == o.aux_maxflow_batch(after, sink, U, k, threads=16)).all()
        wts = rng.integers(0, 4, n).astype(np.int32); wts[np.flatnonzero(topo.is_compute)[0]] = 2
        fc.fc_graph_set_source_weights(g, wts)
        got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k))
        assert (got.cpu().numpy() == o.weighted_aux_maxflow_batch(after, sink, U, k, wts)).all()


@pytest.mark.parametrize("n", [2, 64, 65, 129, 256])
def test_updates_in_place_leave_the_tables_of_a_fresh_upload(n):
    # all links of one vertex down (bits of one word together) and up again, spare links and single directions of a pair brought
    # to life, a link listed twice, an update that changes nothing
    rng = np.random.default_rng(7000 + n)
    topo = _merge(_random_topology(rng, n, 4))
    have = set(zip(topo.tail.tolist(), topo.head.tolist()))
    spares = [(a, b) for a, b in rng.integers(0, n, (2 * n, 2)).tolist() if a != b and (a, b) not in have]
    cap = dict(zip(zip(topo.tail.tolist(), topo.head.tolist()), topo.bandwidth.tolist()))
    cap.update({key: 0 for key in spares})
    keys = sorted(cap)
    P = 64
    sink = rng.integers(0, n, P).astype(np.int32); k = rng.integers(1, 6, P).astype(np.int32); U = rng.integers(1, 12, P).astype(np.int32)
    t, h = ([x[i] for x in keys] for i in (0, 1))
    with fc.fc_graph_upload_with_spares(n, t, h, [cap[x] for x in keys], topo.is_compute) as g:
        for change in ([(x, 0) for x in keys if x[0] == 0 or x[1] == n - 1], [(x, 3 + x[1]) for x in keys if x[0] == 0], [(x, 5) for x in spares],
                       [(keys[0], 9), (keys[0], 2), (keys[-1], cap[keys[-1]])], [(x, int(rng.integers(0, 30))) for x in keys]):
            if not change:
                continue
            fc.fc_graph_update_arcs(g, [x[0] for x, _ in change], [x[1] for x, _ in change], [b for _, b in change], refresh_tables=False)
            cap.update(dict(change))
            after = w.Topology("after", n, np.array(t, np.int32), np.array(h, np.int32), np.array([cap[x] for x in keys], np.int32), topo.is_compute)
            want = o.aux_maxflow_batch(after, sink, U, k, threads=16)
            for options in (None, {"global_relabel_steps": 32}):
                got, _ = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k), options=options)
                assert (got.cpu().numpy() == want).all(), (n, options)


def _spine(boxes, per_box):
    """Boxes around a box switch, every node on one spine."""
    n = boxes * per_box
    t = [c for c in range(n) for _ in (0, 1)]; h = [x for c in range(n) for x in (n + c // per_box, n + boxes)]
    isc = np.zeros(n + boxes + 1, np.uint8); isc[:n] = 1
    return w.Topology("spine", len(isc), np.array(t + h, np.int32), np.array(h + t, np.int32), np.tile([9, 2], 2 * n).astype(np.int32), isc)


def _regular(n, degree):
    t = np.repeat(np.arange(n, dtype=np.int32), degree); h = (t + np.tile(np.cumsum(np.arange(1, degree + 1, dtype=np.int32)), n)) % n
    keep = t != h
    isc = np.ones(n, np.uint8)
    return _merge(w.Topology("regular", n, t[keep], h[keep].astype(np.int32), (1 + (t[keep] * 7 + h[keep] * 3) % 50).astype(np.int32), isc))


# (fabric, problems that still take the bit rows, problems that are too many for them)
@pytest.mark.parametrize("name,topo,few,many", [("one word", lambda: _regular(60, 4), 3000, 40000), ("two words", lambda: _regular(120, 6), 2000, 40000),
                                                ("short rows", lambda: _regular(250, 4), 500, 4000), ("three words", lambda: _regular(180, 4), 1500, 12000),
                                                ("longer rows", lambda: _regular(180, 7), 5000, 20000), ("long rows", lambda: _regular(250, 14), 1500, 12000),
                                                ("a spine", lambda: _spine(27, 8), 5000, 60000), ("dense", lambda: _regular(128, 110), 0, 100)])
def test_the_bit_rows_take_a_batch_where_they_are_ahead(name, topo, few, many):
    topo = topo()
    n, comp = topo.n_vertices, np.array(topo.compute_nodes, np.int32)
    with fc.fc_graph_upload(n, topo.tail, topo.head, topo.bandwidth, topo.is_compute) as g:
        for P, bit_rows in ((few, True), (many, False)):
            if P == 0:
                continue
            sink = comp[np.arange(P) % len(comp)]
            U = np.full(P, 2, np.int32); k = (1 + np.arange(P) // len(comp) % 4).astype(np.int32)
            flows, st = fc.fc_maxflow_batch(g, _dev(sink), _dev(U), _dev(k), want_stats=True)
            # (on bit rows every problem searches for heights at least once and nothing is relabeled one by one)
            assert (st["relabels"] == 0 and st["global_relabels"] >= P) == bit_rows, (name, P, st)
            one = min(P, 4 * len(comp))                      # the problems repeat from here on
            assert (flows[:one].cpu().numpy() == o.aux_maxflow_batch(topo, sink[:one], U[:one], k[:one], threads=16)).all()
            assert torch.equal(flows[:one].repeat(-(-P // one))[:P], flows)


def _scaled_rail_fabric(boxes, per_box, caps, U):
    """An Eulerian cluster (boxes around a switch, one rail per place in a box) with one bandwidth inside per box, times U."""
    n_compute = boxes * per_box
    t, h, b = [], [], []
    for c in range(n_compute):
        for a, v, x in ((c, n_compute + c // per_box, caps[c // per_box]), (c, n_compute + boxes + c % per_box, 2)):
            t += [a, v]; h += [v, a]; b += [x * U, x * U]
    isc = np.zeros(n_compute + boxes + per_box, np.uint8); isc[:n_compute] = 1
    return w.Topology("rails", len(isc), np.array(t, np.int32), np.array(h, np.int32), np.array(b, np.int32), isc)


@pytest.mark.parametrize("boxes,per_box", [(3, 2), (12, 4), (16, 7), (22, 8)])     # 1, 2, 3 and 4 words per row
def test_edge_splitting_on_bit_rows_agrees_with_the_other_solver(boxes, per_box):
    rng = np.random.default_rng(boxes)
    k = 2
    D = _scaled_rail_fabric(boxes, per_box, 2 * rng.integers(10, 17, boxes), boxes - 1)     # optimum (boxes - 1) / 2
    n, isc = D.n_vertices, D.is_compute
    into = np.flatnonzero(isc[D.head] == 0)
    pairs = []
    for _ in range(24):
        e = int(rng.choice(into)); out = np.flatnonzero(D.tail == D.head[e])
        pairs.append((D.tail[e], D.head[e], D.head[int(rng.choice(out))]))
    pairs += [(0, 1, 2), (0, n - 1, n), (0, n - 1, n - 1)]                                  # no pair of links through a switch
    d = [_dev(x) for x in zip(*pairs)]
    with fc.fc_graph_upload(n, D.tail, D.head, D.bandwidth, isc) as g:
        for flows in (False, True):
            here = fc.fc_split_gamma_batch(g, 1, k, *d, want_flows=flows, want_stats=True)
            there = fc.fc_split_gamma_batch(g, 1, k, *d, want_flows=flows, options={"split_two_launches": 2})
            assert torch.equal(here["gamma"], there["gamma"]), (here["gamma"], there["gamma"])
            assert here["stats"]["not_converged"] == 0 and int((here["gamma"] > 0).sum()) > 0
            if flows:
                assert torch.equal(here["flows"], there["flows"])
    if boxes <= 16:
        here = fc.fc_remove_switches(n, D.tail, D.head, D.bandwidth, isc, k)
        there = fc.fc_remove_switches(n, D.tail, D.head, D.bandwidth, isc, k, options={"split_two_launches": 1})
        assert here["links"] == there["links"] and here["table"] == there["table"]


@pytest.mark.parametrize("boxes,per_box", [(10, 5), (42, 2), (12, 9), (31, 7)])    # 65, 128, 129 and 255 vertices
def test_switch_removal_by_cuts_agrees_with_the_other_solver(boxes, per_box):
    k = 2
    D = _scaled_rail_fabric(boxes, per_box, 2 * np.random.default_rng(boxes).integers(10, 17, boxes), boxes - 1)
    args = (D.n_vertices, D.tail, D.head, D.bandwidth, D.is_compute)
    here = fc.fc_remove_switches(*args, k)
    there = fc.fc_remove_switches(*args, k, options={"split_two_launches": 2})
    assert here["links"] == there["links"] and here["table"] == there["table"]
    assert 1 < here["batches"] < there["batches"] // 2, (here["batches"], there["batches"])     # by cuts to the end
    for options in (None, {"split_two_launches": 2}):                                       # more than the fabric carries
        with pytest.raises(fc.FcError) as err:
            fc.fc_remove_switches(*args, k + 1, options=options)
        assert err.value.code == fc.FC_ENOCONVERGE


def test_a_digraph_too_dense_for_the_chip_goes_to_the_other_solver():
    # 142 nodes linked to all but one of the others, in a ring by one unit each, the missing unit through a switch: records of 160 KB
    n = 142
    t = np.repeat(np.arange(n, dtype=np.int32), n - 2); h = (t + np.tile(np.arange(1, n - 1, dtype=np.int32), n)) % n
    u = np.arange(n, dtype=np.int32); sw = np.full(n, n, np.int32)
    isc = np.ones(n + 1, np.uint8); isc[n] = 0
    args = (n + 1, np.concatenate([t, u, sw]), np.concatenate([h.astype(np.int32), sw, u]), np.ones(len(t) + 2 * n, np.int32), isc, 1)
    here = fc.fc_remove_switches(*args)
    there = fc.fc_remove_switches(*args, options={"split_two_launches": 1})
    assert here["links"] == there["links"] and here["table"] == there["table"] and len(here["table"]) == n
    assert here["batches"] == there["batches"] >= n


def test_a_switch_without_links_is_removed_whatever_the_others_carry():
    isc = np.array([1, 1, 1, 0], np.uint8)
    got = fc.fc_remove_switches(4, [0, 1, 2], [1, 2, 0], [1, 1, 1], isc, 5)
    assert got["links"] == {(0, 1): 1, (1, 2): 1, (2, 0): 1} and got["table"] == {}


def _ring_with_chords(n, k):
    """A ring in both directions that carries k out-trees per root (two links into every interval), and some chords."""
    rng = np.random.default_rng(n)
    links = {(u, (u + d) % n): -(-(n - 1) * k // 2) for u in range(n) for d in (1, n - 1)}
    for u, v in rng.integers(0, n, (n, 2)).tolist():
        if u != v:
            links[(u, v)] = links.get((u, v), 0) + int(rng.integers(1, 4))
    return links


@pytest.mark.parametrize("n,k", [(2, 1), (3, 1), (33, 1), (40, 2), (24, 3)])
def test_trees_by_cuts_use_every_unit_and_agree_with_the_other_solver(n, k):
    # one tree per root: never a copy; more than one: copies, and the construction changes over to the other solver
    links = w.superposed_out_trees(n, k, 100 + n)
    here = fc.fc_construct_trees(n, links, k)
    there = fc.fc_construct_trees(n, links, k, options={"threads_per_problem": 64})
    assert here["trees"] == there["trees"] and there["batches"] >= n - 1
    if all(m == k for _, m, _ in here["trees"]):                                            # no copy: by cuts to the end
        assert here["batches"] < max(2, n // 4), (here["batches"], there["batches"])
    short = dict(links)
    short[max(short, key=lambda e: (short[e], e))] -= 1                                     # every unit was needed
    for options in (None, {"threads_per_problem": 64}):
        with pytest.raises(fc.FcError) as err:
            fc.fc_construct_trees(n, short, k, options=options)
        assert err.value.code == fc.FC_ENOCONVERGE


@pytest.mark.parametrize("n,k", [(63, 1), (64, 2), (65, 1), (128, 1), (129, 1), (193, 1), (256, 1)])
def test_trees_by_cuts_agree_with_the_other_solver_at_the_edges_of_the_row_words(n, k):
    links = _ring_with_chords(n, k)
    here = fc.fc_construct_trees(n, links, k)
    there = fc.fc_construct_trees(n, links, k, options={"threads_per_problem": 64})
    assert here["trees"] == there["trees"]
    if all(m == k for _, m, _ in here["trees"]):                                            # no copy: by cuts to the end
        assert here["batches"] < n // 4 <= there["batches"], (here["batches"], there["batches"])


def test_tree_options_take_the_loop_that_knows_them():
    n, k = 24, 1
    links = _ring_with_chords(n, k)
    by_cuts = fc.fc_construct_trees(n, links, k)
    assert all(m == k for _, m, _ in by_cuts["trees"]) and by_cuts["batches"] < n // 2       # no copy
    runs = {c: fc.fc_construct_trees(n, links, k, options={"tree_chain_states": c}) for c in (1, 4)}
    runs.update({-v: fc.fc_construct_trees(n, links, k, options={"tree_warm_start": v}) for v in (1, 2)})
    assert all(r["trees"] == by_cuts["trees"] for r in runs.values())
    assert runs[1]["batches"] == n * (n - 1) > runs[4]["batches"] > runs[-1]["batches"] == runs[-2]["batches"] >= n
