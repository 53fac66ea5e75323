"""Parity of the waypoint and forbidden-switch checks (pc_trace_flows_watch,
pc_masked_reach_via, pc_report_paths) with the CPU oracle, bit-exact, on
seeded inputs: the tiny end-to-end case, small combined workloads, fat-trees
with long and full watch lists, the bitset and the map search, and malformed
lists."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_run
    return gpu_run


@pytest.fixture(params=["buckets", "default", "walk"])
def trace_path(request, monkeypatch):
    if request.param == "buckets":
        monkeypatch.setenv("PC_TRACE_WALK_MAX", "0")
    elif request.param == "walk":
        monkeypatch.setenv("PC_TRACE_WALK_MAX", str(10**9))
    return request.param


def _same(a, b, what):
    a, b = np.asarray(a), np.asarray(b)
    assert a.shape == b.shape, (what, a.shape, b.shape)
    bad = np.argwhere(a != b)
    assert bad.size == 0, f"{what}: first mismatch at {tuple(bad[0])}: gpu {a[tuple(bad[0])]} oracle {b[tuple(bad[0])]}"


def _same_traces(a, b):
    for f in ("jmask", "last_switch", "last_port", "hops", "state"):
        _same(a[f], b[f], f)


def _oracle_paths(orc, wl):
    oo = orc.run_workload(wl)
    tr, visit, terr = orc.trace(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"],
                                wl["hdr"], wl["ingress"], wl["ttl"], watch=wl["watch"])
    d, rerr = orc.reach_via(wl["V"], wl["adj_off"], wl["adj"], wl["region"], wl["src"], wl["allowed"],
                            wl["target"], wl["via"], wl["forbid"])
    pss, reason, summ, perr = orc.report(wl["intents"], oo["feasible"], oo["popcnt"], wl["N"], tr, wl["expect"], d,
                                         visit, wl["pexp"])
    return dict(feasible=oo["feasible"], popcnt=oo["popcnt"], traces=tr, visit=visit, reach=d, pass_=pss,
                reason=reason, summary=summ, flags=oo["sel_err"] | terr | rerr | perr)


def _check_paths(g, orc, wl):
    gp = g.run_paths_workload(wl)
    oo = _oracle_paths(orc, wl)
    _same(gp["feasible"], oo["feasible"], "feasible")
    _same(gp["popcnt"], oo["popcnt"], "popcnt")
    _same_traces(gp["traces"], oo["traces"])
    _same(gp["visit"], oo["visit"], "visit")
    _same(gp["reach"], oo["reach"], "reach_via")
    _same(gp["reason"], oo["reason"], "reason")
    _same(gp["pass"], oo["pass_"], "pass")
    for f in ("counts", "no_path"):
        _same(gp["summary"][f], oo["summary"][f], f)
    assert gp["flags"] == oo["flags"]
    return gp, oo


@pytest.mark.parametrize("variant", ["rpath", "literal", "dense"])
def test_paths_cfg1(g, orc, variant, trace_path):
    _check_paths(g, orc, synth.cfg1(0, variant, paths=True))


@pytest.mark.parametrize("seed", [1, 2])
def test_paths_combined_small(g, orc, seed):
    wl = synth.combined_workload(seed, 3000 + 37, 16, 8, 4, 700, 3001, paths=True)
    gp, oo = _check_paths(g, orc, wl)
    r = oo["reason"] & 0x7F
    assert (r == 0).sum() > 0 and (r == 8).sum() > 0 and (r == 9).sum() > 0


def _watch_lists(rng, T, K, S, ingress):
    w = rng.integers(-1, S, size=(T, K)).astype(np.int32)
    w[::5, 0] = ingress[::5]
    return w


@pytest.mark.parametrize("K", [1, 7, 32])
def test_trace_watch_fat_tree(g, orc, K, trace_path):
    wl = synth.trace_workload(3, 8, 4, 512, 20000, 24, 3000, variant="rpath")
    rng = np.random.default_rng(K)
    watch = _watch_lists(rng, wl["hdr"].shape[0], K, wl["S"], wl["ingress"])
    tg, vg = g.trace_watch(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"],
                           wl["hdr"], wl["ingress"], wl["ttl"], watch)
    to, vo, err = orc.trace(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"],
                            wl["hdr"], wl["ingress"], wl["ttl"], watch=watch)
    _same_traces(tg, to)
    _same(vg, vo, "visit")
    assert (vo != 0).sum() > 1000


def test_trace_watch_dense_loops(g, orc, trace_path):
    """Random walks with loops and TTL ends; slot k watches switch k, so the
    visit word is the whole visited set."""
    rng = np.random.default_rng(3)
    topo = synth.random_graph(rng, 9, 14, 2, 4)
    rule_off, rules, _ = synth.build_tables(rng, topo, 40, 0.03, prio="small", prio_range=3)
    T = 3000
    hdr = synth.random_keys(rng, T)
    ingress = rng.integers(0, 9, size=T).astype(np.int32)
    watch = np.tile(np.arange(9, dtype=np.int32), (T, 1))
    for ttl in (0, 1, 7, 255):
        tg, vg = g.trace_watch(9, topo["port_off"], topo["port_peer"], topo["jur"], rule_off, rules, hdr, ingress,
                               ttl, watch)
        to, vo, _ = orc.trace(9, topo["port_off"], topo["port_peer"], topo["jur"], rule_off, rules, hdr, ingress,
                              ttl, watch=watch)
        _same_traces(tg, to)
        _same(vg, vo, "visit")


def test_trace_watch_malformed(g, orc):
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(6, 4, 2, 64, 500, 8, 100)
    rng = np.random.default_rng(6)
    watch = _watch_lists(rng, wl["hdr"].shape[0], 3, wl["S"], wl["ingress"])
    watch[7, 1] = wl["S"] + 5
    watch[9, 2] = -4
    ingress = wl["ingress"].copy()
    ingress[4] = -3
    ctx = pc.context()
    ctx.data_errors(clear=True)
    tg, vg = g.trace_watch(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"],
                           wl["hdr"], ingress, wl["ttl"], watch)
    flags = ctx.data_errors(clear=True)
    to, vo, err = orc.trace(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"],
                            wl["hdr"], ingress, wl["ttl"], watch=watch)
    _same_traces(tg, to)
    _same(vg, vo, "visit")
    assert flags == err == orc.F_SWITCH


def _via_lists(rng, Q, V, Kv, Kf, src, target):
    via = rng.integers(0, V, size=(Q, Kv)).astype(np.int32)
    m = rng.integers(0, Kv + 1, size=Q)
    for q in range(Q):
        via[q, m[q]:] = -1
    if Kv >= 2:
        via[::9, 1] = via[::9, 0]
    forbid = rng.integers(-1, V, size=(Q, Kf)).astype(np.int32)
    if Kf:
        forbid[::11, 0] = src[::11]       # forbidden source
        forbid[5::11, 0] = target[5::11]  # forbidden target
        if Kv:
            forbid[7::13, -1] = via[7::13, 0]  # forbidden waypoint (or -1)
    return via, forbid


@pytest.mark.parametrize("Kv,Kf", [(0, 0), (0, 3), (1, 2), (3, 5)])
@pytest.mark.parametrize("V", [1500, 40000])
def test_reach_via_rgg(g, orc, V, Kv, Kf):
    """The bitset search (1,500 vertices) and the map search (40,000)."""
    Q = 1100 if V <= 6016 else 40
    wl = synth.rgg_workload(V + Kv + Kf, V, 8, Q, mean_degree=7.0, full_rows=False)
    rng = np.random.default_rng(V + 10 * Kv + Kf)
    via, forbid = _via_lists(rng, Q, V, Kv, Kf, wl["src"], wl["target"])
    if V <= 6016 and Kv:
        # waypoints near the source, so that many walks exist
        near = wl["adj"][wl["adj_off"][wl["src"]]]
        via[::2, 0] = near[::2]
    dg, used = g.kernels(lambda: g.reach_via(wl["V"], wl["adj_off"], wl["adj"], wl["region"], wl["src"], wl["allowed"],
                                             wl["target"], via, forbid))
    do, _ = orc.reach_via(wl["V"], wl["adj_off"], wl["adj"], wl["region"], wl["src"], wl["allowed"], wl["target"],
                          via, forbid)
    _same(dg, do, "reach_via")
    assert ("k_rc_bitset" if V <= 6016 else "k_rc_map") in used
    if V <= 6016:
        assert (do >= 0).sum() > 10 and (do == -1).sum() > 10


def test_reach_via_fat_tree(g, orc):
    k = 16
    topo = synth.fat_tree(k, 6)
    S = topo["S"]
    rng = np.random.default_rng(4)
    Q = 2000
    src = rng.integers(0, k * k, size=Q).astype(np.int32)
    tgt = rng.integers(0, k * k, size=Q).astype(np.int32)
    allowed = rng.integers(0, 64, size=Q).astype(np.uint32)
    allowed[::3] = 63
    via = rng.integers(k * k, S, size=(Q, 2)).astype(np.int32)  # cores
    via[::2, 1] = -1
    forbid = rng.integers(0, S, size=(Q, 2)).astype(np.int32)
    dg = g.reach_via(S, topo["adj_off"], topo["adj"], topo["jur"], src, allowed, tgt, via, forbid)
    do, _ = orc.reach_via(S, topo["adj_off"], topo["adj"], topo["jur"], src, allowed, tgt, via, forbid)
    _same(dg, do, "reach_via")
    assert (do >= 0).sum() > 100 and (do == -1).sum() > 100


def test_reach_via_malformed(g, orc):
    import paper_2602_16100_amd as pc
    wl = synth.rgg_workload(2, 800, 4, 70, mean_degree=6.0, full_rows=False)
    rng = np.random.default_rng(2)
    via, forbid = _via_lists(rng, 70, 800, 2, 2, wl["src"], wl["target"])
    via[3, 0] = 5000
    forbid[4, 1] = -9
    ctx = pc.context()
    ctx.data_errors(clear=True)
    dg = g.reach_via(wl["V"], wl["adj_off"], wl["adj"], wl["region"], wl["src"], wl["allowed"], wl["target"], via,
                     forbid)
    flags = ctx.data_errors(clear=True)
    do, err = orc.reach_via(wl["V"], wl["adj_off"], wl["adj"], wl["region"], wl["src"], wl["allowed"],
                            wl["target"], via, forbid)
    _same(dg, do, "reach_via")
    assert flags == err == orc.F_SWITCH


def test_report_paths_cfg1_visit_patterns(g, orc):
    """Every combination of must / forbid masks and visit words on the tiny
    case's traces."""
    wl = synth.cfg1(0, paths=True)
    oo = orc.run_workload(wl)
    rng = np.random.default_rng(8)
    T = wl["hdr"].shape[0]
    visit = rng.integers(0, 8, size=T).astype(np.uint32)
    pexp = np.zeros(wl["intents"].shape[0], synth.PATH_EXPECT_DT)
    pexp["must"] = rng.integers(0, 8, size=pexp.shape[0])
    pexp["forbid"] = rng.integers(0, 8, size=pexp.shape[0]) & ~pexp["must"]
    pg, rg, sg = g.report_paths(wl["intents"], oo["feasible"], oo["popcnt"], wl["N"], oo["traces"], wl["expect"],
                                oo["reach"], visit, pexp)
    po, ro, so, _ = orc.report(wl["intents"], oo["feasible"], oo["popcnt"], wl["N"], oo["traces"], wl["expect"],
                               oo["reach"], visit, pexp)
    _same(rg, ro, "reason")
    _same(pg, po, "pass")
    _same(sg["counts"], so["counts"], "counts")
    _same(sg["no_path"], so["no_path"], "no_path")


# legs of the map search, of the bitset search, and of the bitset search in source order
@pytest.mark.parametrize("Q", [80, 130, 500, 4700])
@pytest.mark.parametrize("kind", ["symmetric", "asymmetric", "unsorted", "bad_offsets"])
def test_reach_via_leg_direction(g, orc, kind, Q):
    """Legs are searched from their far end only on symmetric graphs with
    sorted lists; one-way entries, unsorted lists, or a vertex whose offsets
    are invalid (push never expands it, yet a neighbour's list names it) must
    give the forward results."""
    wl = synth.rgg_workload(11, 1200, 4, Q, mean_degree=9.0, full_rows=False)
    adj_off, adj = wl["adj_off"].copy(), wl["adj"].copy()
    rng = np.random.default_rng(1)
    if kind == "asymmetric":
        for p in rng.choice(adj.shape[0], size=40, replace=False):
            adj[p] = int(rng.integers(0, wl["V"]))
        for u in range(wl["V"]):  # keep each list sorted
            adj[adj_off[u]:adj_off[u + 1]] = np.sort(adj[adj_off[u]:adj_off[u + 1]])
    elif kind == "unsorted":
        for u in range(wl["V"]):
            adj[adj_off[u]:adj_off[u + 1]] = adj[adj_off[u]:adj_off[u + 1]][::-1]
    elif kind == "bad_offsets":
        hub = int(np.argmax(np.diff(adj_off)))
        adj_off[hub + 1] = adj_off[hub] - 1 if adj_off[hub] > 0 else adj.shape[0] + 5
    near = adj[np.clip(adj_off[wl["src"]], 0, adj.shape[0] - 1)]
    via = np.stack([near, rng.integers(0, wl["V"], size=Q)], axis=1).astype(np.int32)
    via[::3, 1] = -1
    forbid = rng.integers(-1, wl["V"], size=(Q, 2)).astype(np.int32)
    dg, used = g.kernels(lambda: g.reach_via(wl["V"], adj_off, adj, wl["region"], wl["src"], wl["allowed"], wl["target"],
                                             via, forbid))
    assert ("k_rc_map" if Q == 80 else "k_rc_bitset") in used and ("k_rc_legs" in used) == (Q in (80, 4700))
    do, _ = orc.reach_via(wl["V"], adj_off, adj, wl["region"], wl["src"], wl["allowed"], wl["target"], via, forbid)
    _same(dg, do, "reach_via")
    assert (do >= 0).sum() > 5


@pytest.mark.parametrize("ttl", [0, 1, 2, 7, 8, 9, 31, 64, 254, 255])
def test_trace_loops_of_every_length(g, orc, ttl):
    """Rings of 1 to 13 switches (a switch may forward to itself), entered through lines of 0 to 6 switches:
    records, visit words, visited-switch summaries and walk records of traces that loop until their TTL."""
    import torch
    import paper_2602_16100_amd as pc
    peer, start = [], []
    for ring in range(1, 14):
        for line in range(7):
            first = len(peer)
            start.append(first)
            peer += [first + i + 1 for i in range(line)]
            peer += [first + line + (i + 1) % ring for i in range(ring)]
    S = len(peer)
    port_off = np.arange(S + 1, dtype=np.int32)
    jur = (np.arange(S) % 31).astype(np.uint8)
    rules = np.zeros(S, synth.RULE_DT)  # one rule a switch: every header, out of its only port
    T = 3 * len(start)
    ingress = np.repeat(start, 3).astype(np.int32) + np.tile([0, 1, 2], len(start)).astype(np.int32)
    ingress = np.minimum(ingress, S - 1)
    hdr = synth.random_keys(np.random.default_rng(1), T)
    watch = (ingress[:, None] + np.arange(8)[None, :] * 2 - 2).astype(np.int32)
    watch[(watch < 0) | (watch >= S)] = -1
    args = (S, port_off, np.array(peer, np.int32), jur, port_off, rules, hdr, ingress, ttl)
    to, vo, so, wo, _ = orc.trace(*args, watch=watch, summary=True)
    tg, vg = g.trace_watch(*args, watch)
    assert np.array_equal(tg, to) and np.array_equal(vg, vo)
    d = lambda a: pc.to_device(a, "cuda")  # noqa: E731
    out = torch.zeros((T, 12), dtype=torch.uint8, device="cuda")
    vsum = torch.zeros(T, dtype=torch.int64, device="cuda")
    walk = torch.full((T, 8), -5, dtype=torch.int32, device="cuda")
    pc.pc_trace_flows_delta(S, d(port_off), d(args[2]), d(jur), d(port_off), d(rules), d(hdr), d(ingress), ttl, out,
                            vsum, walk=walk, ctx=pc.Context(0))
    torch.cuda.synchronize()
    assert np.array_equal(pc.records(out, pc.TRACE_OUT_DT), to)
    assert np.array_equal(vsum.cpu().numpy().view(np.uint64), so) and np.array_equal(walk.cpu().numpy(), wo)


def test_walks_from_a_long_list(g, orc, monkeypatch):
    """The walk takes over after a level whose list is many times longer than its grid, most of its slots ended."""
    monkeypatch.setenv("PC_TRACE_WALK_MAX", "70000")
    wl = synth.trace_workload(7, 8, 4, 256, 600_000, 16, 20_000)
    a = (wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"], wl["hdr"], wl["ingress"], 16)
    assert np.array_equal(g.trace(*a), orc.trace(*a)[0])


@pytest.mark.parametrize("R,T", [(1, 1), (63, 500), (256, 3000), (1024, 3276), (1024, 3277), (1025, 300)])
@pytest.mark.parametrize("bad", [False, True])
def test_trace_small_tables(g, orc, R, T, bad):
    """Tables matched rule by rule and, past 1,024 rules per switch or 2^26 matches, through chunk sets: skewed and
    shared rule ranges, more than 64 ports on a switch, and malformed ingress, actions, peers, watch and offsets."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(R * 7 + T)
    wl = synth.trace_workload(R + T, 4, 4, R, T, 16, max(T // 4, 1))
    S, off, rules, peer = wl["S"], wl["rule_off"].copy(), wl["rules"].copy(), wl["port_peer"].copy()
    port_off, ingress = wl["port_off"].copy(), wl["ingress"].copy()
    assert S == 20
    port_off[3:] += 70  # switch 2 takes 70 more ports, all to its neighbours
    peer = np.insert(peer, wl["port_off"][3], rng.choice(peer[peer >= 0], 70))
    lo, hi = off[2], off[3]
    rules["action"][lo:hi][rng.random(hi - lo) < 0.5] = 68
    off[10] = off[11] if R > 1 else off[10]  # one empty table, one of double length
    watch = rng.integers(-1, S, size=(T, 5)).astype(np.int32)
    if bad:
        ingress[::7] = S
        ingress[3::11] = -4
        rules["action"][::5] = 3000
        peer[5] = S + 9
        watch[::9, 2] = S
        off[15] = off[14] - 1 if R > 1 else -1
    a = (S, port_off, peer, wl["jur"], off, rules, wl["hdr"], ingress, 16)
    ctx = pc.context()
    ctx.data_errors(clear=True)
    tg, vg = g.trace_watch(*a, watch)
    flags = ctx.data_errors(clear=True)
    to, vo, err = orc.trace(*a, watch=watch)
    _same_traces(tg, to)
    _same(vg, vo, "visit")
    assert flags == err


@pytest.mark.parametrize("T", [4000, 4200])
def test_trace_many_switches(g, orc, T):
    """A ring of more switches than one workgroup lays out, rule by rule and through chunk sets (T above 2^26 / S)."""
    S = 16390
    off = np.arange(S + 1, dtype=np.int32)
    peer = np.roll(np.arange(S, dtype=np.int32), -1)
    peer[100::1000] = -1
    rules = np.zeros(S, synth.RULE_DT)
    rng = np.random.default_rng(T)
    a = (S, off, peer, (np.arange(S) % 31).astype(np.uint8), off, rules, synth.random_keys(rng, T),
         rng.integers(0, S, size=T).astype(np.int32), 200)
    assert np.array_equal(g.trace(*a), orc.trace(*a)[0])


@pytest.mark.parametrize("k,Q,Kv", [(6, 65, 0), (6, 33, 1), (6, 43, 2), (8, 200, 20), (8, 70, 31), (8, 61, 32),
                                    (32, 6553, 1), (32, 6554, 1), (32, 4400, 2), (32, 26300, 0)])
def test_reach_bitset_orders(g, orc, k, Q, Kv):
    """Legs searched and summed by their workgroup, and in source order past 2^24 legs x vertices (2^25 targets without
    legs): whole-query remainders, lists cut at every length, forbidden vertices, and on one context a graph that is
    symmetric, one that is not, and the first again, with invalid lists in between."""
    import paper_2602_16100_amd as pc
    topo = synth.fat_tree(k, 4)
    S, off, adj = topo["S"], topo["adj_off"], topo["adj"].copy()
    rng = np.random.default_rng(k * Q + Kv)
    src, target = (rng.integers(0, S, size=Q).astype(np.int32) for _ in range(2))
    allowed = rng.integers(0, 16, size=Q).astype(np.uint32)
    allowed[::2] = 15
    via, forbid = _via_lists(rng, Q, S, Kv, 3, src, target)
    oneway = adj.copy()
    for u in (1, S // 2):  # this vertex's list names others that do not name it
        oneway[off[u]:off[u + 1]] = np.sort(rng.integers(0, S, off[u + 1] - off[u]))
    bad_via, bad_adj = via.copy(), adj.copy()
    if Kv:
        bad_via[Q // 2, 0] = S + 3
    bad_adj[off[3]] = -7
    ctx = pc.context()
    some = 0
    for a, v in ((adj, via), (oneway, via), (adj, via), (bad_adj, bad_via), (adj, via)):
        ctx.data_errors(clear=True)
        dg = g.reach_via(S, off, a, topo["jur"], src, allowed, target, v, forbid)
        flags = ctx.data_errors(clear=True)
        do, err = orc.reach_via(S, off, a, topo["jur"], src, allowed, target, v, forbid)
        _same(dg, do, "reach_via")
        assert flags == err
        some += (do >= 0).sum()
        if k == 32 and a is oneway:
            break
    assert some > 0


@pytest.mark.parametrize("variant", ["rpath", "prefix", "dense"])
@pytest.mark.parametrize("R,T", [(1, 4100), (33, 2559), (33, 2560), (128, 9000), (257, 4100), (1500, 5000), (4096, 4100),
                                 (4097, 12900), (8300, 19300)])
def test_match_forms(g, orc, monkeypatch, variant, R, T):
    """Levels matched with the table's sets in LDS (one to three slices, one to thirty-two lanes a lookup) and, as they
    shrink or for few lookups a table, in registers: one and many matching rules per header, ties of priority."""
    monkeypatch.setenv("PC_TRACE_WALK_MAX", "0")
    wl = synth.trace_workload(R + T, 4, 4, R, T, 16, 40, variant=variant)
    a = (wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"], wl["hdr"], wl["ingress"], 16)
    _same_traces(g.trace(*a), orc.trace(*a)[0])


def test_match_failing_candidates(g, orc, monkeypatch):
    """Rules of the highest priorities that pass the chunk filter and fail in full: the first two survivors of every
    lookup fail, up to twenty more do before the one that matches, which some switches lack; two match at a tie."""
    monkeypatch.setenv("PC_TRACE_WALK_MAX", "0")
    rng = np.random.default_rng(5)
    wl = synth.trace_workload(9, 4, 4, 200, 6000, 16, 40)
    S, off, rules = wl["S"], wl["rule_off"], wl["rules"].copy()
    key = synth.random_keys(rng, 1)[0]
    hdr = np.repeat(key[None], 6000, 0).astype(np.uint32)
    for s in range(S):
        n = off[s + 1] - off[s]
        r = rules[off[s]:off[s + 1]]
        r["value"], r["mask"] = key[None], np.array([~np.uint32(0)] * 3 + [np.uint32(255)], np.uint32)
        at = rng.integers(0, 26, n)
        r["value"][np.arange(n), at // 8] ^= (np.uint32(5) << (4 * (at % 8)).astype(np.uint32))
        r["priority"] = rng.integers(100, 65536, n)
        r["action"] = rng.integers(0, 4, n)
        if s % 5:
            for x in rng.integers(0, n, 2):
                r["mask"][x], r["priority"][x] = 0, 50
    a = (S, wl["port_off"], wl["port_peer"], wl["jur"], off, rules, hdr, wl["ingress"], 16)
    _same_traces(g.trace(*a), orc.trace(*a)[0])


@pytest.mark.parametrize("I", [1, 63, 256, 257, 1024, 1025, 2500])
def test_report_sizes(g, orc, I):
    """One workgroup that writes the summary (up to 1,024 intents) and several that add to it."""
    wl = synth.cfg1(0, "rpath")
    oo = orc.run_workload(wl)
    rng = np.random.default_rng(I)
    pick = rng.integers(0, wl["intents"].shape[0], I)
    intents, expect = wl["intents"][pick].copy(), wl["expect"][pick].copy()
    intents["trace_end"][::17] = 1 << 30
    T = wl["hdr"].shape[0]
    visit = rng.integers(0, 8, size=T).astype(np.uint32)
    pexp = np.zeros(I, synth.PATH_EXPECT_DT)
    pexp["must"] = rng.integers(0, 2, size=I)
    for _ in range(2):
        pg, rg, sg = g.report_paths(intents, oo["feasible"], oo["popcnt"], wl["N"], oo["traces"], expect, oo["reach"],
                                    visit, pexp)
        po, ro, so, _ = orc.report(intents, oo["feasible"], oo["popcnt"], wl["N"], oo["traces"], expect, oo["reach"],
                                   visit, pexp)
        _same(rg, ro, "reason")
        _same(pg, po, "pass")
        _same(sg["counts"], so["counts"], "counts")
        _same(sg["no_path"], so["no_path"], "no_path")


@pytest.mark.parametrize("deg", [1, 15, 16, 17, 31, 32, 33, 80])
def test_reach_target_degrees(g, orc, deg):
    """Targets of every number of neighbours around the look-ahead's two registers per lane, some reached through one
    of them only, most of them forbidden on the way."""
    rng = np.random.default_rng(deg)
    hubs, ring = 40, 300  # hub h: deg neighbours on a ring
    pairs = [(v, hubs + (v - hubs + 1) % ring) for v in range(hubs, hubs + ring)]
    pairs += [(h, hubs + int(x)) for h in range(hubs) for x in rng.choice(ring, deg, replace=False)]
    pairs = np.array(pairs, np.int32)
    pairs = np.unique(np.concatenate([pairs, pairs[:, ::-1]]), axis=0)
    V = hubs + ring
    off = np.zeros(V + 1, np.int32)
    off[1:] = np.cumsum(np.bincount(pairs[:, 0], minlength=V))
    adj = pairs[:, 1].astype(np.int32)
    Q = 130
    target = rng.integers(0, hubs, Q).astype(np.int32)
    src = rng.integers(hubs, V, Q).astype(np.int32)
    region = (rng.random(V) < 0.2).astype(np.uint8)
    region[:hubs] = 0
    allowed = rng.integers(0, 2, Q).astype(np.uint32) * 2 + 1
    forbid = np.stack([adj[off[target] + np.minimum(k, off[target + 1] - off[target] - 1)] for k in range(6)], 1).astype(np.int32)
    none = np.full((Q, 0), -1, np.int32)
    dg = g.reach_via(V, off, adj, region, src, allowed, target, none, forbid)
    do, _ = orc.reach_via(V, off, adj, region, src, allowed, target, none, forbid)
    _same(dg, do, "reach_via")


def _with_hub(wl, rules, n, rng):
    """wl with n rules at its switch 0: its own first, then exact ones that match no header drawn."""
    off = wl["rule_off"].astype(np.int64)
    more = np.zeros(n - (off[1] - off[0]), synth.RULE_DT)
    more["value"] = synth.random_keys(rng, more.shape[0])
    more["mask"] = np.array([0xFFFFFFFF] * 3 + [0xFF], np.uint32)
    more["priority"] = rng.integers(0, 65536, more.shape[0])
    off[1:] += more.shape[0]
    return off.astype(np.int32), np.concatenate([rules[:wl["rule_off"][1]], more, rules[wl["rule_off"][1]:]])


@pytest.mark.parametrize("total,T,indexed", [(16_384, 100, False), (30_269, 1000, False), (30_270, 1000, True), (46_064, 1, False),
                                             (46_065, 1, True), (200_001, 1, True), (262_144, 100, True)])
@pytest.mark.parametrize("bad", [False, True])
def test_trace_one_long_table(g, orc, total, T, indexed, bad):
    """Nearly all rules on the switch where every trace enters (16 on each of the 319 others).  Rule by rule, a wavefront
    takes 2 ms for the sweep and one hop through 262,144 of them: past 40,960 rules in a table, or 25 million by traces, the
    call forms chunk sets after all."""
    import torch
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(total)
    wl = synth.trace_workload(3, 16, 4, 16, T, 16, 50)
    S = wl["S"]
    off, rules = _with_hub(wl, wl["rules"], total - 16 * (S - 1), rng)
    ingress = np.zeros(T, np.int32)
    watch = rng.integers(-1, S, (T, 32)).astype(np.int32)
    if bad:
        rules["action"][off[1] - 5] = 3000
        watch[-1, -1] = S
    assert rules.shape[0] == total
    a = (S, wl["port_off"], wl["port_peer"], wl["jur"], off, rules, wl["hdr"], ingress, 16)
    d = [x if isinstance(x, int) else g.dev(np.ascontiguousarray(x)) for x in a]
    ctx = pc.context()
    ctx.data_errors(clear=True)
    for timed in (False, True):
        ctx.profile(True)
        out, visit = pc.pc_trace_flows_watch(*d, g.dev(watch))
        torch.cuda.synchronize()
        used = ctx.profile_read()
    ctx.profile(False)
    flags = ctx.data_errors(clear=True)
    to, vo, err = orc.trace(*a, watch=watch)
    _same_traces(pc.records(out, pc.TRACE_OUT_DT), to)
    _same(visit.cpu().numpy().view(np.uint32), vo, "visit")
    assert flags == err
    assert "k_tr_direct" in used and ("k_tr_prep" in used) == indexed
    assert sum(ms for _, ms in used.values()) < 0.5, used


@pytest.mark.parametrize("S,total,T,indexed", [(16_390, 57_349, 600, False), (16_390, 57_350, 600, True),
                                               (16_384, 57_343, 0, True), (16_384, 40_960, 0, False)])
def test_trace_one_long_table_of_many_switches(g, orc, S, total, T, indexed):
    """A rule a switch and one long table, on a ring of more switches than one workgroup looks over; and only the
    sweeps (no traces)."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(total)
    off = np.arange(S + 1, dtype=np.int32)
    peer = np.roll(np.arange(S, dtype=np.int32), -1)
    peer[100::1000] = -1
    more_off, rules = _with_hub(dict(rule_off=off), np.zeros(S, synth.RULE_DT), total - S + 1, rng)
    rules["action"][-3] = 7
    ingress = np.minimum(rng.integers(0, 2 * S, T), S - 1).astype(np.int32)
    ingress[::2] = 0
    a = (S, off, peer, (np.arange(S) % 31).astype(np.uint8), more_off, rules, synth.random_keys(rng, T), ingress, 60)
    ctx = pc.context()
    for _ in range(3):
        ctx.data_errors(clear=True)
        ctx.profile(True)
        got = g.trace(*a)
        used = ctx.profile_read()
        ctx.profile(False)
        assert ("k_tr_prep" in used) == indexed
        to, err = orc.trace(*a)
        _same_traces(got, to)
        assert ctx.data_errors(clear=True) == err


@pytest.mark.parametrize("k,R,T", [(24, 200, 400), (32, 100, 500)])
def test_trace_many_small_tables(g, orc, k, R, T):
    """As many rules in all, but none of the tables long: rule by rule, no chunk sets."""
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(R, k, 4, R, T, 16, 50)
    a = (wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"], wl["hdr"], wl["ingress"], 16)
    ctx = pc.context()
    ctx.profile(True)
    got = g.trace(*a)
    used = ctx.profile_read()
    ctx.profile(False)
    assert set(used) == {"k_tr_direct", "k_tr_walk"}, used
    _same_traces(got, orc.trace(*a)[0])


@pytest.mark.parametrize("bad", [False, True])
def test_trace_long_watch_lists(g, orc, bad):
    """Two million watched ids over 20 switches of small tables: the sweep has workgroups of its own."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(2)
    wl = synth.trace_workload(4, 4, 4, 16, 60_000, 16, 500)
    watch = rng.integers(-1, wl["S"], (60_000, 32)).astype(np.int32)
    if bad:
        watch[-1, -1] = wl["S"]
    a = (wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"], wl["hdr"], wl["ingress"], 16)
    ctx = pc.context()
    g.trace_watch(*a, watch)
    ctx.data_errors(clear=True)
    ctx.profile(True)
    tg, vg = g.trace_watch(*a, watch)
    used = ctx.profile_read()
    ctx.profile(False)
    flags = ctx.data_errors(clear=True)
    to, vo, err = orc.trace(*a, watch=watch)
    _same_traces(tg, to)
    _same(vg, vo, "visit")
    assert flags == err
    assert used["k_tr_direct"][1] < 0.1, used


def test_priorities_refused(g, orc, monkeypatch):
    """Where the auxiliary buffer holds the chunk sets but not the rules' priorities, levels of many lookups are
    matched in registers."""
    import paper_2602_16100_amd as pc
    T, part = 100_000, np.arange(0, 100_000, 5000)
    wl = synth.trace_workload(3, 24, 4, 3000, T, 12, 2000)
    small = synth.trace_workload(3, 24, 4, 16, 8, 12, 8)
    d = {k: g.dev(wl[k]) for k in ("port_off", "port_peer", "jur", "rule_off", "rules", "hdr", "ingress")}
    ctx = pc.Context(0)

    def run(n, rule_off, rules):
        ctx.profile(True)
        out = pc.records(pc.pc_trace_flows(wl["S"], d["port_off"], d["port_peer"], d["jur"], rule_off, rules, d["hdr"][:n],
                                           d["ingress"][:n], 12, ctx=ctx), pc.TRACE_OUT_DT)
        used = ctx.profile_read()
        ctx.profile(False)
        return out, used

    run(T, g.dev(small["rule_off"]), g.dev(small["rules"]))  # the arena
    run(8000, d["rule_off"], d["rules"])                     # the chunk sets, by walks
    monkeypatch.setenv("PC_FAIL_ALLOC", "1")
    refused, used = run(T, d["rule_off"], d["rules"])
    assert "k_tr_match_wide" in used and "k_tr_match" not in used
    monkeypatch.delenv("PC_FAIL_ALLOC")
    normal, used = run(T, d["rule_off"], d["rules"])
    assert "k_tr_match" in used
    _same_traces(refused, normal)
    to, _ = orc.trace(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], wl["rule_off"], wl["rules"], wl["hdr"],
                      wl["ingress"], 12, idx=part)
    _same_traces(refused[part], to)


def test_trace_many_rules_captured(g, orc):
    """A call that would ask for its tables' lengths waits for nothing while its stream is captured: the graph's replays
    trace the headers of the moment."""
    import torch
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(5, 16, 4, 100, 1000, 16, 50)
    names = ("port_off", "port_peer", "jur", "rule_off", "rules", "hdr", "ingress")
    d = {k: g.dev(wl[k]) for k in names}
    ctx = pc.Context(0)

    def call():
        return pc.pc_trace_flows(wl["S"], *(d[k] for k in names), 16, ctx=ctx)

    call()  # the scratch
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    first, hdr = d["hdr"].clone(), wl["hdr"]
    for turn in (0, 17, 500):
        d["hdr"].copy_(first.roll(turn, 0))
        graph.replay()
        torch.cuda.synchronize()
        got = pc.records(out, pc.TRACE_OUT_DT)
        to, _ = orc.trace(wl["S"], *(wl[k] for k in names[:5]), np.roll(hdr, turn, 0), wl["ingress"], 16)
        _same_traces(got, to)
        _same_traces(pc.records(call(), pc.TRACE_OUT_DT), to)


def test_trace_one_long_table_refused(g, orc, monkeypatch):
    """Where the chunk sets of a call with one long table are refused, its rules are matched one by one all the same."""
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(3, 16, 4, 16, 100, 16, 50)
    off, rules = _with_hub(wl, wl["rules"], 50_000, np.random.default_rng(1))
    rules["action"][off[1] - 5] = 3000
    a = (wl["S"], wl["port_off"], wl["port_peer"], wl["jur"])
    hdr, ingress = wl["hdr"], np.zeros(100, np.int32)
    ctx = pc.Context(0)

    def run(off, rules):
        ctx.profile(True)
        out = pc.pc_trace_flows(a[0], *(g.dev(x) for x in (*a[1:], off, rules, hdr, ingress)), 16, ctx=ctx)
        used = ctx.profile_read()
        ctx.profile(False)
        return pc.records(out, pc.TRACE_OUT_DT), ctx.data_errors(clear=True), used

    run(wl["rule_off"], wl["rules"])  # the arena
    monkeypatch.setenv("PC_FAIL_ALLOC", "1")
    got, flags, used = run(off, rules)
    monkeypatch.delenv("PC_FAIL_ALLOC")
    to, err = orc.trace(*a, off, rules, hdr, ingress, 16)
    _same_traces(got, to)
    assert flags == err and used["k_tr_walk"][0] == 2 and "k_tr_prep" not in used
    got, flags, used = run(off, rules)
    _same_traces(got, to)
    assert flags == err and "k_tr_prep" in used


def test_trace_levels_refused(g, orc, monkeypatch):
    """60,000 traces are walked unless a table is large, and need no room for levels: they are where that is refused."""
    import paper_2602_16100_amd as pc
    T, part = 60_000, np.arange(0, 60_000, 3000)
    wl = synth.trace_workload(3, 24, 4, 300, T, 12, 2000)
    names = ("port_off", "port_peer", "jur", "rule_off", "rules", "hdr", "ingress")
    d = {k: g.dev(wl[k]) for k in names}
    ctx = pc.Context(0)

    def run(n):
        ctx.profile(True)
        out = pc.pc_trace_flows(wl["S"], *(d[k] for k in names[:5]), d["hdr"][:n], d["ingress"][:n], 12, ctx=ctx)
        used = ctx.profile_read()
        ctx.profile(False)
        return pc.records(out, pc.TRACE_OUT_DT), used

    run(8000)  # the chunk sets, and an arena without levels
    monkeypatch.setenv("PC_FAIL_ALLOC", "1")
    got, used = run(T)
    assert "k_tr_prep" in used and "k_tr_plan" not in used
    to, _ = orc.trace(wl["S"], *(wl[k] for k in names), 12, idx=part)
    _same_traces(got[part], to)
    monkeypatch.delenv("PC_FAIL_ALLOC")
    _same_traces(got, run(T)[0])
