"""Parity of the map search of pc_masked_reach / pc_masked_reach_via (graphs past the 6,016 vertices of the bitset
search, and few queries on smaller sparse ones) with the CPU oracle: narrow and wide frontiers and the hand-over between them, more levels than are
deferred while the row is filled, vertices of more neighbours than a record holds, dense graphs without
records, rows of every alignment, invalid entries, and the largest size of its range and the first beyond it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_run
    return gpu_run


def _csr(V, pairs):
    pairs = np.unique(np.concatenate([pairs, pairs[:, ::-1]]), axis=0)
    off = np.zeros(V + 1, np.int32)
    off[1:] = np.cumsum(np.bincount(pairs[:, 0], minlength=V))
    return off, pairs[:, 1].astype(np.int32)


def _graph(kind, V, rng):
    v = np.arange(V)
    if kind == "line":      # a vertex a level: thousands of narrow levels
        return _csr(V, np.stack([v[:-1], v[1:]], 1))
    if kind == "blocks":    # short lines of ten
        return _csr(V, np.stack([v[:-1], v[1:]], 1)[(v[1:] % 10) != 0])
    if kind == "hubs":      # a line with hubs of 17-400 entries
        hubs = rng.integers(0, V, 40)
        spokes = np.concatenate([np.stack([np.full(n, h), rng.integers(0, V, n)], 1)
                                 for h, n in zip(hubs, rng.integers(17, 400, 40))])
        return _csr(V, np.concatenate([np.stack([v[:-1], v[1:]], 1), spokes[spokes[:, 0] != spokes[:, 1]]]))
    if kind == "star":      # hubs of V entries: on narrow levels, then, past 64 of 300 entries, on wide ones
        a, b = np.arange(100), rng.integers(100, V, (100, 300))
        return _csr(V, np.concatenate([np.stack([np.full(V - 1, 0), v[1:]], 1), np.stack([np.full(V - 2, 1), v[2:]], 1),
                                       np.stack([np.repeat(a, 300), b.ravel()], 1)]))
    deg = {"sparse": 3, "mixed": 8, "mean20": 20, "dense": 60}[kind]  # random: wide levels
    return _csr(V, np.stack([rng.integers(0, V, V * deg // 2), rng.integers(0, V, V * deg // 2)], 1))


@pytest.mark.parametrize("kind,V,Q", [
    ("line", 6017, 5), ("line", 7003, 3), ("hubs", 9001, 9), ("sparse", 20001, 300), ("mixed", 12007, 40),
    ("mean20", 8191, 20), ("dense", 6100, 12), ("sparse", 512, 1000), ("sparse", 4001, 1024), ("sparse", 4001, 1025), ("sparse", 4001, 1000), ("sparse", 4001, 1001),
    ("sparse", 4001, 333), ("sparse", 4001, 334), ("sparse", 512, 256), ("sparse", 600, 257), ("blocks", 1_259_000, 4), ("blocks", 1_300_001, 4),
    ("star", 40_001, 30), ("star", 12_000, 600)])
def test_map_rows_and_targets(g, orc, kind, V, Q):
    rng = np.random.default_rng(V)
    off, adj = _graph(kind, V, rng)
    region = (np.arange(V) // 64 % 5 if kind in ("line", "hubs") else rng.integers(0, 5, V)).astype(np.uint8)
    region[rng.integers(0, V, 5)] = 40
    bad = rng.integers(0, adj.shape[0], 7)
    adj[bad] = [-1, V, V + 9, -7, 1 << 30, -(1 << 31), V]
    src = rng.integers(0, V, Q).astype(np.int32)
    src[1] = V
    allowed = rng.integers(1, 32, Q).astype(np.uint32)
    allowed[::2] = 31
    target = rng.integers(0, V, Q).astype(np.int32)
    target[0] = src[0]
    target[Q // 2] = -1
    near = np.flatnonzero(np.arange(Q) % 3 == 2)
    target[near] = np.minimum(np.clip(src[near], 0, V - 1) + rng.integers(0, 900, near.shape[0]), V - 1)
    rows = slice(0, min(Q, 24))
    _, flags = orc.reach(V, off, adj, region, src, allowed, target)
    for t, part in ((None, rows), (target, slice(0, Q))):
        tt = None if t is None else t[part]
        dg = g.reach(V, off, adj, region, src[part], allowed[part], tt)
        do, _ = orc.reach(V, off, adj, region, src[part], allowed[part], tt)
        assert np.array_equal(dg, do), (kind, t is None, np.argwhere(dg != do)[:3])
    via = rng.integers(-1, V, (Q, 2)).astype(np.int32)
    forbid = rng.integers(-1, V, (Q, 3)).astype(np.int32)
    dg = g.reach_via(V, off, adj, region, src, allowed, target, via, forbid)
    do, _ = orc.reach_via(V, off, adj, region, src, allowed, target, via, forbid)
    assert np.array_equal(dg, do), kind


@pytest.mark.parametrize("call", ["rows", "targets", "via", "queue_rows"])
def test_map_scratch_refused(g, orc, monkeypatch, call):
    """Where the map search's scratch is refused, the searches that need less of it answer: on a new context the
    bitset search (which needs none), past its sizes the queue search in an arena that holds its lists."""
    import torch
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(7)
    V, Q = (8000, 400) if call == "queue_rows" else (1500, 50)
    off, adj = _graph("mean20" if call == "queue_rows" else "sparse", V, rng)
    region = rng.integers(0, 4, V).astype(np.uint8)
    src, target = (rng.integers(0, V, Q).astype(np.int32) for _ in range(2))
    allowed = rng.integers(1, 16, Q).astype(np.uint32)
    via, forbid = rng.integers(-1, V, (Q, 1)).astype(np.int32), rng.integers(-1, V, (Q, 2)).astype(np.int32)
    d = g.dev
    ctx = pc.Context(0)

    def run(n):
        a = (V, d(off), d(adj), d(region), d(src[:n]), d(allowed[:n]))
        if call == "via":
            return pc.pc_masked_reach_via(*a, d(target[:n]), d(via[:n]), d(forbid[:n]), ctx=ctx)
        return pc.pc_masked_reach(*a, d(target[:n]) if call == "targets" else None, ctx=ctx)

    if call == "queue_rows":
        run(256)  # as many lists as the queue search has
    monkeypatch.setenv("PC_FAIL_ALLOC", "1")
    ctx.profile(True)
    got = run(Q)
    torch.cuda.synchronize()
    used = ctx.profile_read()
    ctx.profile(False)
    assert ("k_rc_queue" if call == "queue_rows" else "k_rc_bitset") in used and "k_rc_map" not in used
    if call == "via":
        want, _ = orc.reach_via(V, off, adj, region, src, allowed, target, via, forbid)
    else:
        want, _ = orc.reach(V, off, adj, region, src, allowed, target if call == "targets" else None)
    assert np.array_equal(got.cpu().numpy(), want)


def test_map_hubs_at_once(g, orc):
    """5,000 vertices joined to four hubs: a hub's 5,000 entries are the whole workgroup's (64 queries 107 us by one
    wavefront, which took them 64 at a time)."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(2)
    V, Q = 5000, 64
    v = np.arange(4, V)
    off, adj = _csr(V, np.concatenate([np.stack([np.full(V - 4, h), v], 1) for h in range(4)]))
    region = np.zeros(V, np.uint8)
    src, target = (rng.integers(0, V, Q).astype(np.int32) for _ in range(2))
    allowed = np.ones(Q, np.uint32)
    ctx = pc.context()
    for _ in range(2):
        ctx.profile(True)
        dg = g.reach(V, off, adj, region, src, allowed, target)
        used = ctx.profile_read()
        ctx.profile(False)
    do, _ = orc.reach(V, off, adj, region, src, allowed, target)
    assert np.array_equal(dg, do)
    assert used["k_rc_map"][1] < 0.06, used


@pytest.mark.parametrize("V,Q,rows,targets", [(1000, 256, True, True), (1000, 257, False, False), (3600, 300, True, True),
                                              (3600, 301, True, False), (3600, 900, True, False), (3600, 901, False, False)])
def test_few_queries_of_sparse_graphs(g, orc, V, Q, rows, targets):
    """The map search takes rows up to a quarter of the vertices, targets and legs up to a twelfth, and 256 either way."""
    rng = np.random.default_rng(V + Q)
    off, adj = _graph("mixed", V, rng)
    region = rng.integers(0, 4, V).astype(np.uint8)
    src, target = (rng.integers(0, V, Q).astype(np.int32) for _ in range(2))
    allowed = rng.integers(1, 16, Q).astype(np.uint32)
    none = np.zeros((Q, 0), np.int32)
    for t, by_map in ((None, rows), (target, targets)):
        dg, used = g.kernels(lambda: g.reach(V, off, adj, region, src, allowed, t))
        assert ("k_rc_map" in used) == by_map and ("k_rc_bitset" in used) != by_map
        do, _ = orc.reach(V, off, adj, region, src, allowed, t)
        assert np.array_equal(dg, do)
    via = rng.integers(-1, V, (Q // 2, 1)).astype(np.int32)
    args = (V, off, adj, region, *(x[:Q // 2] for x in (src, allowed, target)), via, none[:Q // 2])
    dg, used = g.kernels(lambda: g.reach_via(*args))
    assert ("k_rc_map" in used) == (Q // 2 * 2 <= max(256, V // 12))
    do, _ = orc.reach_via(*args)
    assert np.array_equal(dg, do)
