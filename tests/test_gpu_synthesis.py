"""Parity of pc_synthesize_paths (through the C ABI) with the CPU oracle:
hop counts, walks and the 40-byte compiled rules, bit-exact, plus the
data-error word; on random graphs and fat-trees, BFS and weighted, with
waypoints, forbidden switches and every failure case.  End to end: the
synthesized rules of simple walks, installed as flow tables, are traced by
pc_trace_flows to EGRESS along exactly the synthesized walks."""
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


def _same(a, b, what):
    a, b = np.asarray(a), np.asarray(b)
    assert a.shape == b.shape, (what, a.shape, b.shape)
    bad = np.argwhere(a != b)
    assert bad.size == 0, f"{what}: first mismatch at {tuple(bad[0])}: gpu {a[tuple(bad[0])]} oracle {b[tuple(bad[0])]}"


def _check(g, orc, V, port_off, port_peer, region, req, prio, max_hops, weight=None, n_ports=None):
    args = (V, port_off, port_peer, region, req["src"], req["target"], req["allowed"], req["via"], req["forbid"],
            req["key"], req["out_port"], prio, max_hops)
    hg, pg, rg, eg = g.synthesize(*args, weight=weight, n_ports=n_ports)
    ho, po, ro, eo = orc.synthesize(*args, weight=weight, n_ports=n_ports)
    _same(hg, ho, "hops")
    _same(pg, po, "path")
    _same(rg.view(np.uint8).reshape(rg.shape[0], rg.shape[1] * 40),
          ro.view(np.uint8).reshape(ro.shape[0], ro.shape[1] * 40), "rules")
    assert eg == eo, (eg, eo)
    return ho, po, ro


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("kind,Kv,Kf", [("random", 0, 0), ("random", 2, 3), ("fat_tree", 1, 2), ("fat_tree", 3, 5)])
def test_synthesis_parity(g, orc, kind, Kv, Kf, weighted):
    rng = np.random.default_rng(11)
    topo = synth.random_graph(rng, 300, 700, 2, 6) if kind == "random" else synth.fat_tree(12, 6)
    weight = synth.port_weights(4, topo["port_peer"].shape[0], 9) if weighted else None
    req = synth.synthesis_requests(5, topo, 700, Kv=max(Kv, 1), Kf=max(Kf, 1))
    if Kv == 0:
        req["via"] = np.full((700, 1), -1, np.int32)
    if Kf == 0:
        req["forbid"] = np.full((700, 1), -1, np.int32)
    ho, _, _ = _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req, 4321, 40, weight)
    assert (ho >= 0).sum() > 100 and (ho == -1).sum() > 0


@pytest.mark.parametrize("kind", ["random", "fat_tree"])
def test_synthesis_huge_weights(g, orc, kind):
    """Link weights up to 2^32 - 1, so that legs cross the 2^31 - 1 distance
    bound (beyond it a switch is unreachable) and 64-bit sums would differ from
    32-bit ones."""
    rng = np.random.default_rng(21)
    topo = synth.random_graph(rng, 300, 700, 2, 6) if kind == "random" else synth.fat_tree(8, 4)
    n = topo["port_peer"].shape[0]
    choices = np.array([1, 2, 7, 1 << 28, 1 << 29, (1 << 30) - 1, 1 << 30, (1 << 31) - 3, (1 << 31) - 2,
                        (1 << 31) - 1, 1 << 31, (1 << 32) - 1], np.uint64)
    weight = choices[rng.integers(0, choices.shape[0], n)].astype(np.uint32)
    req = synth.synthesis_requests(7, topo, 600, Kv=1, Kf=1)
    ho, _, _ = _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req, 99, 40, weight)
    assert (ho >= 0).sum() > 10 and (ho == -1).sum() > 10


def test_synthesis_max_hops_and_tiny_budgets(g, orc):
    topo = synth.fat_tree(8, 4)
    req = synth.synthesis_requests(6, topo, 400, Kv=2, Kf=1)
    for max_hops in (0, 1, 2, 4, 7, 255):
        _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req, 7, max_hops)


def test_synthesis_largest_graph(g, orc):
    """A random graph at the size limit (12,288 switches): the LDS state of
    one request at its largest."""
    rng = np.random.default_rng(2)
    topo = synth.random_graph(rng, 12288, 30000, 1, 3)
    req = synth.synthesis_requests(9, topo, 64, Kv=1, Kf=2)
    ho, _, _ = _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req, 1, 255,
                      synth.port_weights(1, topo["port_peer"].shape[0]))
    assert (ho > 0).any()


def test_synthesis_malformed(g, orc):
    topo = synth.fat_tree(6, 3)
    req = synth.synthesis_requests(0, topo, 60, Kv=1, Kf=1)
    pp = topo["port_peer"].copy()
    pp[3] = 999
    pp[10] = -7
    region = topo["jur"].copy()
    region[5] = 40
    w = np.ones(pp.shape[0], np.uint32)
    w[7] = 0
    req["via"][0, 0] = -5
    req["src"][1] = 1 << 20
    req["target"][2] = -3
    req["out_port"][3] = 77
    req["forbid"][4, 0] = 4000
    po = topo["port_off"].copy()
    po[9] = po[10] + 1  # a bad offset pair for switch 9 (and 8)
    _check(g, orc, topo["S"], po, pp, region, req, 1, 20, weight=w)


def test_synthesis_empty(g, orc):
    topo = synth.fat_tree(4, 2)
    req = synth.synthesis_requests(0, topo, 3, Kv=1, Kf=1)
    empty = {k: v[:0] for k, v in req.items()}
    _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], empty, 1, 10)
    # no switches: every request fails (its endpoints are out of range)
    _check(g, orc, 0, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.uint8), req, 1, 10)


@pytest.mark.parametrize("weighted", [False, True])
def test_synthesized_rules_deliver_on_the_gpu(g, orc, weighted):
    """The compiled rules of every walk that repeats no switch, installed as
    the switches' flow tables and traced on the GPU: EGRESS at the target's
    host port after exactly the walk's links, inside the allowed
    jurisdictions."""
    topo = synth.fat_tree(16, 8)
    weight = synth.port_weights(8, topo["port_peer"].shape[0]) if weighted else None
    Q = 3000
    req = synth.synthesis_requests(12, topo, Q, Kv=1, Kf=2)
    hops, path, rules, err = g.synthesize(topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req["src"],
                                          req["target"], req["allowed"], req["via"], req["forbid"], req["key"],
                                          req["out_port"], 900, 32, weight=weight)
    assert err == 0
    simple = np.array([h >= 0 and len(set(p[:h + 1])) == h + 1 for h, p in zip(hops, path)])
    ok = np.flatnonzero(simple)
    assert ok.size > 1000
    S = topo["S"]
    sw = path[ok].ravel()
    rl = rules[ok].ravel()
    live = sw >= 0
    sw, rl = sw[live], rl[live]
    order = np.argsort(sw, kind="stable")
    sw, rl = sw[order], rl[order]
    rule_off = np.zeros(S + 1, np.int32)
    rule_off[1:] = np.cumsum(np.bincount(sw, minlength=S))
    tr = g.trace(S, topo["port_off"], topo["port_peer"], topo["jur"], rule_off, rl, req["key"][ok],
                 req["src"][ok], 255)
    assert (tr["state"] == 0).all()
    assert np.array_equal(tr["last_switch"], req["target"][ok])
    assert np.array_equal(tr["last_port"].astype(np.int32), req["out_port"][ok])
    assert np.array_equal(tr["hops"].astype(np.int32), hops[ok])
    assert ((tr["jmask"] & ~req["allowed"][ok]) == 0).all()


def _line(V, rng):
    """A line of V switches with one host port each (a search runs through hundreds of switches)."""
    peer, off = [], [0]
    for s in range(V):
        p = [x for x in (s - 1, s + 1) if 0 <= x < V] + [-1]
        peer += p
        off.append(len(peer))
    host = np.arange(V)
    return dict(S=V, J=4, H=V, port_off=np.array(off, np.int32), port_peer=np.array(peer, np.int32),
                jur=(host // 7 % 4).astype(np.uint8), host_switch=host.astype(np.int32),
                host_port=(np.diff(off) - 1).astype(np.int32))


# enough legs for the bounds to pay: the directed search with its fallbacks (a full table: sparse1500, line; rows
# missing: line900; one weight)
@pytest.mark.parametrize("kind,Kv,Kf,hops,wmax", [
    ("random", 2, 3, 40, 9), ("random", 0, 0, 255, 3), ("fat_tree", 1, 32, 16, 10), ("fat_tree", 3, 1, 1, 1),
    ("fat_tree", 1, 2, 40, 2), ("random", 1, 2, 40, 2**32 - 1), ("fat_tree", 1, 2, 40, 1 << 20),
    ("sparse1500", 1, 2, 64, 10), ("line900", 1, 1, 255, 5), ("malformed", 2, 2, 40, 9)])
def test_directed_search(g, orc, kind, Kv, Kf, hops, wmax):
    rng = np.random.default_rng(21)
    if kind == "fat_tree":
        topo = synth.fat_tree(12, 6)
    elif kind == "line900":
        topo = _line(900, rng)
    else:
        V = 1500 if kind == "sparse1500" else 300
        topo = synth.random_graph(rng, V, 2 * V + V // 3, 2, 6)
    n_ports = topo["port_peer"].shape[0]
    Q = (topo["S"] + 25_000_000 // n_ports) // (Kv + 1) + 40
    weight = np.random.default_rng(5).integers(1, wmax + 1, size=n_ports).astype(np.uint32)
    req = synth.synthesis_requests(5, topo, Q, Kv=max(Kv, 1), Kf=max(Kf, 1), p_other_jur=0.8)
    if Kv == 0:
        req["via"] = np.full((Q, 1), -1, np.int32)
    off, peer, jur = topo["port_off"].copy(), topo["port_peer"].copy(), topo["jur"].copy()
    if kind == "malformed":
        off[17] = off[18] + 1
        peer[rng.integers(0, n_ports, 40)] = 1 << 20
        weight[rng.integers(0, n_ports, 40)] = 0
        jur[rng.integers(0, 300, 9)] = 77
        req["src"][::50], req["target"][7::50], req["out_port"][9::50] = -3, 300, 99
        req["via"][11::50, 0], req["forbid"][13::50, 0] = 4000, -9
    ho, _, _ = _check(g, orc, topo["S"], off, peer, jur, req, 4321, hops, weight)
    assert (ho == -1).sum() > 0 and (hops < 2 or (ho >= 0).sum() > 50)


@pytest.mark.parametrize("weighted,Q", [(False, 60), (True, 60), (True, 24_000)])
def test_overlapping_port_ranges(g, orc, weighted, Q):
    """Every other switch owns all ports (the offset pairs between are bad), so there are many times more links
    than ports: no in-link list can hold them."""
    topo = synth.random_graph(np.random.default_rng(3), 40, 520, 2, 4)
    n = topo["port_peer"].shape[0]
    off = np.where(np.arange(41) % 2 == 0, 0, n).astype(np.int32)
    req = synth.synthesis_requests(2, topo, Q, Kv=1, Kf=1)
    req["target"] = (req["target"] // 2 * 2).astype(np.int32)
    w = synth.port_weights(4, n, 9) if weighted else None
    ho, _, _ = _check(g, orc, 40, off, topo["port_peer"], topo["jur"], req, 5, 20, w)
    assert (ho > 0).any()


def _spread(kind, n, rng):
    """Link weights that no single scale of 16 bits suits, or that one outlier must not spoil."""
    if kind == "log32":
        return np.minimum(np.exp2(rng.random(n) * 32), 2**32 - 1).astype(np.uint32)
    w = rng.integers(1, 11, n).astype(np.uint32)
    at = rng.permutation(n)
    if kind == "outlier":
        w[at[:1]] = 65535
    elif kind == "drained":      # a link in a hundred
        w[at[:n // 100]] = 65535
    elif kind == "two_scales":   # a third of them
        w[at[:n // 3]] *= 100_000
    return w


@pytest.mark.parametrize("weights", ["log32", "drained", "two_scales"])
@pytest.mark.parametrize("kind", ["random300", "random1500", "fat_tree12", "fat_tree24", "line700"])
def test_bound_forms(g, orc, kind, weights):
    """Bounds of 16 and of 32 bits, clamped links and sums that saturate, with every split of the bounds kernel."""
    rng = np.random.default_rng(31)
    size = int("".join(c for c in kind if c.isdigit()))
    topo = synth.fat_tree(size, 6) if kind.startswith("fat") else _line(size, rng) if kind.startswith("line") else \
        synth.random_graph(rng, size, 2 * size + size // 3, 2, 6)
    n = topo["port_peer"].shape[0]
    Q = (topo["S"] + 25_000_000 // n) // 2 + 40
    req = synth.synthesis_requests(5, topo, Q, Kv=1, Kf=2, p_other_jur=0.8)
    ho, _, _ = _check(g, orc, topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req, 7, 64,
                      _spread(weights, n, rng))
    assert (ho >= 0).sum() > 50


@pytest.mark.parametrize("weights", ["log32", "outlier", "drained", "two_scales"])
def test_spread_weights_are_directed(g, orc, weights):
    """Whatever the weights' range, the directed search settles nearly every request: the workgroup search is left a
    small share of what it takes for the same requests in batches too small for the directed one, with the same
    results."""
    import paper_2602_16100_amd as pc
    topo = synth.fat_tree(32, 8)
    w = _spread(weights, topo["port_peer"].shape[0], np.random.default_rng(3))
    Q, batch = 8000, 900
    req = synth.synthesis_requests(5, topo, Q, Kv=1, Kf=2)
    ctx = pc.context()

    def run(q0, q1):
        r = {k: v[q0:q1] for k, v in req.items()}
        return g.synthesize(topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], r["src"], r["target"],
                            r["allowed"], r["via"], r["forbid"], r["key"], r["out_port"], 7, 32, weight=w)[:3]

    run(0, batch)
    ctx.profile(True)
    parts = [run(q, min(q + batch, Q)) for q in range(0, Q, batch)]
    alone = ctx.profile_read()
    assert "k_ps_goal" not in alone
    run(0, Q)
    ctx.profile(True)
    whole = run(0, Q)
    left = ctx.profile_read()
    ctx.profile(False)
    for x, y in zip(whole, zip(*parts)):
        assert np.array_equal(x, np.concatenate(y))
    assert left["k_ps_search"][1] < alone["k_ps_search"][1] / 5, (left, alone)


@pytest.mark.parametrize("share,other,directed", [(0, 11, False), (1e-9, 11, False), (1e-9, 65535, False), (0.002, 11, False),
                                                  (0.1, 11, True), (0.1, 65535, True), (0.02, 1, True)])
def test_nearly_equal_weights(g, orc, share, other, directed):
    """Weight 10 on all links but a share of them (at least one): a few heavier ones leave the ties of equal weights,
    and the requests with the workgroup search."""
    import paper_2602_16100_amd as pc
    topo = synth.fat_tree(32, 8)
    n = topo["port_peer"].shape[0]
    links = np.random.default_rng(4).permutation(np.flatnonzero(topo["port_peer"] >= 0))
    w = np.full(n, 10, np.uint32)
    w[links[:int(np.ceil(share * links.size))]] = other
    req = synth.synthesis_requests(5, topo, 8000, Kv=1, Kf=2)
    args = (topo["S"], topo["port_off"], topo["port_peer"], topo["jur"], req["src"], req["target"], req["allowed"],
            req["via"], req["forbid"], req["key"], req["out_port"], 7, 32)
    ctx = pc.context()
    g.synthesize(*args, weight=w)
    ctx.profile(True)
    hg, pg, rg, _ = g.synthesize(*args, weight=w)
    t = ctx.profile_read()
    ctx.profile(False)
    goal, search = t["k_ps_goal"][1], t["k_ps_search"][1]
    assert search < goal if directed else goal < search / 5, t
    part = [a[:200] if isinstance(a, np.ndarray) and a.shape[0] == 8000 else a for a in args]
    ho, po, ro, _ = orc.synthesize(*part, weight=w)
    assert np.array_equal(hg[:200], ho) and np.array_equal(pg[:200], po) and np.array_equal(rg[:200], ro)


@pytest.mark.parametrize("weighted", [False, True])
def test_more_links_than_32_bits_count(g, orc, weighted):
    """6,144 switches own all 699,051 ports: 2^32 + 2,048 links, a count whose low 32 bits would pass for a list that
    fits.  Two switches are usable, so that the searches and the walk back stay short."""
    V, n = 12288, 699_051
    rng = np.random.default_rng(1)
    off = np.where(np.arange(V + 1) % 2 == 0, 0, n).astype(np.int32)
    region = np.full(V, 40, np.uint8)
    region[[0, 2]] = 0
    peer = rng.integers(0, V, n).astype(np.int32)
    req = dict(src=np.array([0, 2, 0, 0, 2], np.int32), target=np.array([2, 0, 0, 2, 4], np.int32),
               allowed=np.ones(5, np.uint32), via=np.full((5, 1), -1, np.int32),
               forbid=np.array([[-1], [-1], [-1], [2], [-1]], np.int32), key=synth.random_keys(rng, 5),
               out_port=np.array([0, n - 1, 9, 0, 0], np.int32))
    w = synth.port_weights(4, n, 9) if weighted else None
    ho, _, _ = _check(g, orc, V, off, peer, region, req, 5, 8, w)
    assert ho.tolist() == [1, 1, 0, -1, -1]
