"""Parity of pc_trace_flows_delta (through the C ABI) with the CPU oracle:
after the rules of some switches change, re-tracing only the traces whose
visited-switch summary meets a changed switch gives exactly the oracle's
full trace on the new tables (records and summaries, bit-exact), starting
from the oracle's old results or from the GPU's own, over chains of
changes, with resized tables, repeated and out-of-range ids, no change,
every switch changed and no traces; and at the combined workload's size."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
F_SWITCH = 8


@pytest.fixture(scope="module")
def g():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_run
    return gpu_run


def _run(wl, rule_off, rules, out, vsum, changed, walk=None, use_walk=True, ctx=None):
    """One delta call; out / vsum / walk as numpy (records, u64, int32
    [T, 8]) or None for a first call.  Returns (records, vsum, walk,
    n_retraced, flags); walk is None with use_walk=False.  Without ctx a
    fresh context (no prepared tables kept) serves the call; a chain of calls
    on the same tables passes its own context."""
    import torch
    import paper_2602_16100_amd as pc
    ctx = ctx or pc.Context(0)
    ctx.data_errors(clear=True)
    T = wl["ingress"].shape[0]
    d = lambda a: pc.to_device(a, "cuda")
    o = torch.zeros((T, 12), dtype=torch.uint8, device="cuda") if out is None else \
        torch.from_numpy(np.ascontiguousarray(out).view(np.uint8).reshape(T, 12).copy()).cuda()
    v = torch.zeros(T, dtype=torch.int64, device="cuda") if vsum is None else \
        torch.from_numpy(np.ascontiguousarray(vsum, np.uint64).view(np.int64).copy()).cuda()
    ch = None if changed is None else torch.from_numpy(np.ascontiguousarray(changed, np.int32)).cuda()
    w = None
    if use_walk:
        w = torch.full((T, 8), -5, dtype=torch.int32, device="cuda") if walk is None else \
            torch.from_numpy(np.ascontiguousarray(walk, np.int32).copy()).cuda()
    n = pc.pc_trace_flows_delta(wl["S"], d(wl["port_off"]), d(wl["port_peer"]), d(wl["jur"]), d(rule_off), d(rules),
                                d(np.ascontiguousarray(wl["hdr"], np.uint32)), d(wl["ingress"]), wl["ttl"], o, v,
                                changed=ch, walk=w, ctx=ctx)
    torch.cuda.synchronize()
    flags = ctx.data_errors(clear=True)
    return (pc.records(o, pc.TRACE_OUT_DT), v.cpu().numpy().view(np.uint64),
            None if w is None else w.cpu().numpy(), int(n.cpu().numpy()[0]), flags)


def _oracle(orc, wl, rule_off, rules, idx=None):
    return orc.trace(wl["S"], wl["port_off"], wl["port_peer"], wl["jur"], rule_off, rules, wl["hdr"], wl["ingress"],
                     wl["ttl"], idx=idx, summary=True)


def _same_records(a, b):
    for f in ("jmask", "last_switch", "last_port", "hops", "state"):
        bad = np.flatnonzero(a[f] != b[f])
        assert bad.size == 0, f"{f}: first mismatch at trace {bad[0]}: gpu {a[bad[0]]} oracle {b[bad[0]]}"


def _mask(changed):
    m = 0
    for s in changed:
        m |= 1 << (int(s) & 63)
    return np.uint64(m)


def _expected_count(ro, vo, wo, changed, use_walk=True):
    """Traces to trace again: exact for walks that fit their record, by
    summary bits otherwise (or always, without records)."""
    by_sum = (vo & _mask(changed)) != 0
    if not use_walk:
        return int(by_sum.sum())
    ch = np.asarray([c for c in changed if c >= 0], np.int64)
    short = ro["hops"].astype(np.int64) + 1 <= 8
    hit = np.isin(wo, ch).any(axis=1)
    return int(np.where(short, hit, by_sum).sum())


def _workloads():
    return {"cfg1-dense": lambda: synth.cfg1(0, "dense"),
            "fat-tree-80-dense": lambda: synth.trace_workload(5, 8, 4, 24, 3000, 12, 200, variant="dense"),
            "fat-tree-320-rpath": lambda: synth.trace_workload(6, 16, 8, 300, 20000, 32, 4000)}


@pytest.mark.parametrize("name", list(_workloads()))
def test_first_call_matches_oracle(g, orc, name):
    wl = _workloads()[name]()
    rec, vs, wk, n, flags = _run(wl, wl["rule_off"], wl["rules"], None, None, None)
    ro, vo, wo, err = _oracle(orc, wl, wl["rule_off"], wl["rules"])
    _same_records(rec, ro)
    assert np.array_equal(vs, vo) and np.array_equal(wk, wo) and n == wl["ingress"].shape[0] and flags == err


@pytest.mark.parametrize("use_walk", [True, False])
@pytest.mark.parametrize("resize", [False, True])
@pytest.mark.parametrize("name", list(_workloads()))
def test_delta_from_oracle_state(g, orc, name, resize, use_walk):
    wl = _workloads()[name]()
    S = wl["S"]
    ro, vo, wo, _ = _oracle(orc, wl, wl["rule_off"], wl["rules"])
    changed = np.random.default_rng(3).choice(S, size=min(4, S), replace=False)
    r_off2, rules2 = synth.mutate_tables(3, wl["port_off"], wl["rule_off"], wl["rules"], changed, resize=resize)
    rec, vs, wk, n, flags = _run(wl, r_off2, rules2, ro, vo, changed, walk=wo, use_walk=use_walk)
    ro2, vo2, wo2, err2 = _oracle(orc, wl, r_off2, rules2)
    _same_records(rec, ro2)
    assert np.array_equal(vs, vo2) and flags == err2
    if use_walk:
        assert np.array_equal(wk, wo2)
    assert n == _expected_count(ro, vo, wo, changed, use_walk) and 0 < n < wl["ingress"].shape[0]


@pytest.mark.parametrize("name", ["fat-tree-80-dense", "fat-tree-320-rpath"])
def test_chained_deltas_on_gpu(g, orc, name):
    wl = _workloads()[name]()
    S = wl["S"]
    rule_off, rules = wl["rule_off"], wl["rules"]
    import paper_2602_16100_amd as pc
    ctx = pc.Context(0)  # one context: later calls re-prepare only the changed switches
    ctx.keep_tables(True)
    rec, vs, wk, _, _ = _run(wl, rule_off, rules, None, None, None, ctx=ctx)
    rng = np.random.default_rng(9)
    for step in range(4):
        changed = rng.choice(S, size=int(rng.integers(1, 6)), replace=True)  # repeats allowed
        rule_off, rules = synth.mutate_tables(20 + step, wl["port_off"], rule_off, rules, changed, resize=step % 2 == 1)
        rec, vs, wk, n, flags = _run(wl, rule_off, rules, rec, vs, changed, walk=wk, ctx=ctx)
        ro, vo, wo, err = _oracle(orc, wl, rule_off, rules)
        _same_records(rec, ro)
        assert np.array_equal(vs, vo) and np.array_equal(wk, wo) and flags == err


def test_chain_across_group_boundaries(g, orc):
    """Tables of exactly 32 rules per switch: resizing a switch to 31 or 33
    rules changes its number of 32-rule groups, so the kept tables cannot
    serve and every switch is prepared again; the next delta (sizes kept)
    re-prepares only its changed switch.  Every step equals the oracle."""
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(7, 8, 4, 32, 4000, 12, 300, variant="dense")
    ctx = pc.Context(0)
    ctx.keep_tables(True)
    rule_off, rules = wl["rule_off"], wl["rules"]
    rec, vs, wk, _, _ = _run(wl, rule_off, rules, None, None, None, ctx=ctx)
    for step, (sw, resize) in enumerate([([4, 9], True), ([30], False), ([4, 11, 70], True), ([5], False)]):
        rule_off, rules = synth.mutate_tables(40 + step, wl["port_off"], rule_off, rules, sw, resize=resize)
        rec, vs, wk, n, flags = _run(wl, rule_off, rules, rec, vs, np.array(sw, np.int32), walk=wk, ctx=ctx)
        ro, vo, wo, err = _oracle(orc, wl, rule_off, rules)
        _same_records(rec, ro)
        assert np.array_equal(vs, vo) and np.array_equal(wk, wo) and flags == err


def test_edge_cases(g, orc):
    wl = synth.trace_workload(5, 8, 4, 24, 3000, 12, 200, variant="dense")
    S, T = wl["S"], wl["ingress"].shape[0]
    ingress = wl["ingress"].copy()
    ingress[:4] = [-1, S, -7, 10 ** 6]  # invalid ingresses: MISS records, empty summaries and walks, SWITCH flag
    wl.arrays["ingress"] = ingress
    ro, vo, wo, err = _oracle(orc, wl, wl["rule_off"], wl["rules"])
    assert err == F_SWITCH and (vo[:4] == 0).all() and (wo[:4] == -1).all()
    rec, vs, wk, n, flags = _run(wl, wl["rule_off"], wl["rules"], None, None, None)
    _same_records(rec, ro)
    assert np.array_equal(vs, vo) and np.array_equal(wk, wo) and flags == F_SWITCH
    # no change: nothing traced again, nothing moves
    rec2, vs2, wk2, n, flags = _run(wl, wl["rule_off"], wl["rules"], ro, vo, np.zeros(0, np.int32), walk=wo)
    _same_records(rec2, ro)
    assert np.array_equal(vs2, vo) and np.array_equal(wk2, wo) and n == 0 and flags == F_SWITCH
    # out-of-range ids are ignored and flagged; a valid one still counts
    r_off2, rules2 = synth.mutate_tables(4, wl["port_off"], wl["rule_off"], wl["rules"], [17])
    ids = np.array([-1, 17, S, 17], np.int32)
    rec3, vs3, wk3, n, flags = _run(wl, r_off2, rules2, ro, vo, ids, walk=wo)
    ro3, vo3, wo3, err3 = _oracle(orc, wl, r_off2, rules2)
    _same_records(rec3, ro3)
    assert np.array_equal(vs3, vo3) and np.array_equal(wk3, wo3) and flags == err3 | F_SWITCH
    assert n == _expected_count(ro, vo, wo, [17])
    # every switch changed: every trace with a valid ingress is traced again
    r_off4, rules4 = synth.mutate_tables(5, wl["port_off"], wl["rule_off"], wl["rules"], np.arange(S), resize=True)
    rec4, vs4, wk4, n, flags = _run(wl, r_off4, rules4, ro, vo, np.arange(S, dtype=np.int32), walk=wo)
    ro4, vo4, wo4, _ = _oracle(orc, wl, r_off4, rules4)
    _same_records(rec4, ro4)
    assert np.array_equal(vs4, vo4) and np.array_equal(wk4, wo4) and n == T - 4
    # no traces
    wl0 = synth.trace_workload(5, 8, 4, 24, 3000, 12, 200, variant="dense")
    wl0.arrays["hdr"] = wl0["hdr"][:0]
    wl0.arrays["ingress"] = wl0["ingress"][:0]
    rec5, vs5, wk5, n, flags = _run(wl0, wl0["rule_off"], wl0["rules"], np.zeros(0, ro.dtype), np.zeros(0, np.uint64),
                                    np.array([3], np.int32), walk=np.zeros((0, 8), np.int32))
    assert n == 0 and rec5.shape[0] == 0


def test_delta_combined_workload_size(g, orc):
    """The combined workload's 699,050 traces over 2,880 switches of 16,384
    rules: a full first call, then the tables of one core, two aggregation
    and three edge switches rewritten.  Every record, summary and walk
    record equals a full GPU trace on the new tables; the traces traced
    again are exactly those whose walk visited a changed switch, except walks
    longer than their record (selected by summary bits); 4,000 sampled traces
    (half of them re-traced) equal the oracle."""
    import paper_2602_16100_amd as pc
    wl = synth.cfg5()
    ctx = pc.Context(0)
    ctx.keep_tables(True)
    rec, vs, wk, n, _ = _run(wl, wl["rule_off"], wl["rules"], None, None, None, ctx=ctx)
    k, h = 48, 24  # pod p: edge switches p*k + [0, h), aggregation p*k + [h, k); core from k*k
    changed = np.array([k * k + 5, 3 * k + h + 6, 10 * k + h + 16, 0, 5 * k + 2, 20 * k + 7], np.int32)
    assert changed.max() < wl["S"]
    r_off2, rules2 = synth.mutate_tables(8, wl["port_off"], wl["rule_off"], wl["rules"], changed)
    rec2, vs2, wk2, n2, flags = _run(wl, r_off2, rules2, rec, vs, changed, walk=wk, ctx=ctx)
    full, vfull, wfull, _, _ = _run(wl, r_off2, rules2, None, None, None)
    _same_records(rec2, full)
    assert np.array_equal(vs2, vfull) and np.array_equal(wk2, wfull) and flags == 0
    short = rec["hops"].astype(np.int64) + 1 <= 8
    assert short.mean() > 0.95  # nearly every walk fits its record
    assert n2 == _expected_count(rec, vs, wk, changed) and 0 < n2 < wl["ingress"].shape[0] // 10
    hit = np.flatnonzero(np.isin(wk, changed).any(axis=1) & short)
    rng = np.random.default_rng(4)
    idx = np.sort(np.concatenate([rng.choice(hit, min(2000, hit.shape[0]), replace=False),
                                  rng.choice(wl["ingress"].shape[0], 2000, replace=False)]))
    ro, vo, wo, err = _oracle(orc, wl, r_off2, rules2, idx=idx)
    _same_records(rec2[idx], ro)
    assert np.array_equal(vs2[idx], vo) and np.array_equal(wk2[idx], wo) and err == 0


@pytest.mark.parametrize("keep", [False, True])
def test_two_workloads_of_equal_size_on_one_context(g, orc, keep):
    """A delta chain on one workload, then a first call and a delta on a
    second workload with the same switch count, all on one context.  Without
    the keep-tables promise every call prepares anew; with it, the second
    workload's first call (C < 0) replaces the kept tables.  Either way the
    second workload's delta equals the oracle's full trace."""
    import paper_2602_16100_amd as pc
    wa = synth.trace_workload(11, 8, 4, 40, 3000, 12, 250, variant="dense")
    wb = synth.trace_workload(12, 8, 4, 40, 3000, 12, 250, variant="dense")
    assert wa["S"] == wb["S"]
    ctx = pc.Context(0)
    ctx.keep_tables(keep)
    rec, vs, wk, _, _ = _run(wa, wa["rule_off"], wa["rules"], None, None, None, ctx=ctx)
    ra, rules_a = synth.mutate_tables(3, wa["port_off"], wa["rule_off"], wa["rules"], [5, 9])
    _run(wa, ra, rules_a, rec, vs, np.array([5, 9], np.int32), walk=wk, ctx=ctx)
    # workload B: its results from the oracle, then a delta on the same context
    ro, vo, wo, _ = _oracle(orc, wb, wb["rule_off"], wb["rules"])
    if keep:  # the promise covers calls on the same tables: B starts with a full call
        rec_b, vs_b, wk_b, _, _ = _run(wb, wb["rule_off"], wb["rules"], None, None, None, ctx=ctx)
        _same_records(rec_b, ro)
    rb, rules_b = synth.mutate_tables(4, wb["port_off"], wb["rule_off"], wb["rules"], [7])
    rec2, vs2, wk2, n, flags = _run(wb, rb, rules_b, ro, vo, np.array([7], np.int32), walk=wo, ctx=ctx)
    ro2, vo2, wo2, err = _oracle(orc, wb, rb, rules_b)
    _same_records(rec2, ro2)
    assert np.array_equal(vs2, vo2) and np.array_equal(wk2, wo2) and flags == err


def test_default_context_prepares_every_call(g, orc):
    """Without the promise, a delta call on tables that differ from the
    context's previous call in unlisted switches as well still equals the
    oracle: every call prepares every switch.  (The previous results passed
    in are those of the tables' last version, as the delta contract asks.)"""
    import paper_2602_16100_amd as pc
    wl = synth.trace_workload(13, 8, 4, 40, 3000, 12, 250, variant="dense")
    ctx = pc.Context(0)
    _run(wl, wl["rule_off"], wl["rules"], None, None, None, ctx=ctx)          # the context's last tables: A
    r2, rules2 = synth.mutate_tables(6, wl["port_off"], wl["rule_off"], wl["rules"], [3, 17, 40])   # B
    rb, vb, wb_, _ = _oracle(orc, wl, r2, rules2)
    r3, rules3 = synth.mutate_tables(7, wl["port_off"], r2, rules2, [20, 21])                     # C
    rec3, vs3, wk3, n, flags = _run(wl, r3, rules3, rb, vb, np.array([20, 21], np.int32), walk=wb_, ctx=ctx)
    ro3, vo3, wo3, err3 = _oracle(orc, wl, r3, rules3)
    _same_records(rec3, ro3)
    assert np.array_equal(vs3, vo3) and np.array_equal(wk3, wo3) and flags == err3
    # the selected walks meet the switches that changed between A and B as well
    both = np.isin(wb_, [20, 21]).any(axis=1) & np.isin(wb_, [3, 17, 40]).any(axis=1)
    assert both.sum() > 0


@pytest.mark.parametrize("walk_max", [None, "0", "50"])
@pytest.mark.parametrize("ring", [False, True])
def test_delta_forms(g, orc, monkeypatch, walk_max, ring):
    """The traces to trace again walked in place, or gathered for a pass by levels; kept tables that serve, that do not
    (a table resized past a group boundary) and none; a ring of more switches than one workgroup plans; repeated and
    invalid ids in the list, actions that become invalid and valid again."""
    import paper_2602_16100_amd as pc
    if walk_max is not None:
        monkeypatch.setenv("PC_TRACE_WALK_MAX", walk_max)
    rng = np.random.default_rng(12)
    if ring:
        S = 16390
        off = np.arange(S + 1, dtype=np.int32)
        peer = np.roll(np.arange(S, dtype=np.int32), -1)
        peer[100::1000] = -1
        wl = dict(S=S, port_off=off, port_peer=peer, jur=(np.arange(S) % 31).astype(np.uint8), rule_off=off,
                  rules=np.zeros(S, synth.RULE_DT), hdr=synth.random_keys(rng, 3000),
                  ingress=rng.integers(0, S, 3000).astype(np.int32), ttl=40)
    else:
        wl = synth.trace_workload(7, 8, 4, 4200, 2500, 12, 300, variant="dense")
        S = wl["S"]
    for keep in (True, False):
        ctx = pc.Context(0)
        ctx.keep_tables(keep)
        rule_off, rules = wl["rule_off"], wl["rules"]
        rec, vs, wk, _, _ = _run(wl, rule_off, rules, None, None, None, ctx=ctx)
        for step in range(4):
            sw = rng.choice(S, size=200 if ring else 5, replace=False).astype(np.int32)
            resize = step == 2 and not ring
            rule_off, rules = synth.mutate_tables(60 + step, wl["port_off"], rule_off, rules, sw, resize=resize)
            if step == 1:  # an action beyond the switch's ports, put right by the next step
                bad = sw[0]
                rules = rules.copy()
                rules["action"][rule_off[bad]:rule_off[bad + 1]] = 5000
            if step == 2:
                sw = np.append(sw, bad).astype(np.int32)
                rules["action"][rule_off[bad]:rule_off[bad + 1]] = 0
            listed = np.concatenate([sw, sw[:3], [-1, S]]).astype(np.int32)
            rec, vs, wk, n, flags = _run(wl, rule_off, rules, rec, vs, listed, walk=wk, ctx=ctx)
            ro, vo, wo, err = _oracle(orc, wl, rule_off, rules)
            _same_records(rec, ro)
            assert np.array_equal(vs, vo) and np.array_equal(wk, wo) and flags == err | F_SWITCH
            assert n > 0


@pytest.mark.parametrize("S,T,walks", [(320, 60_000, True), (320, 65_536, False), (16_390, 60_000, True), (16_390, 65_536, False)])
def test_walk_limit_with_one_large_table(g, orc, monkeypatch, S, T, walks):
    """550,000 rules on the switch where every trace enters (17,188 groups of 32): 60,000 traces are walked, 65,536
    (past 2^30 groups for all) go by levels; also when the switch's rules change, with the tables kept and anew."""
    import torch
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(S + T)
    n = 550_000
    if S == 320:
        wl = synth.trace_workload(3, 16, 4, 16, T, 12, 50)
        port_off, peer, jur, off, rules = (wl[k] for k in ("port_off", "port_peer", "jur", "rule_off", "rules"))
    else:
        off = port_off = np.arange(S + 1, dtype=np.int32)
        peer = np.roll(np.arange(S, dtype=np.int32), -1)
        jur = (np.arange(S) % 31).astype(np.uint8)
        rules = np.zeros(S, synth.RULE_DT)
    own = off[1]
    hub = np.zeros(n, synth.RULE_DT)
    hub["value"], hub["mask"] = synth.random_keys(rng, n), np.array([0xFFFFFFFF] * 3 + [0xFF], np.uint32)
    hub["priority"] = rng.integers(0, 65536, n)
    hub["action"] = rng.integers(0, port_off[1], n)
    hub[:own] = rules[:own]
    off = off.copy()
    off[1:] += n - own
    rules = np.concatenate([hub, rules[own:]])
    hdr = synth.random_keys(rng, T)
    hdr[::2] = hub["value"][rng.integers(own, n, hdr[::2].shape[0])]
    w = synth.Workload("hub", 0)
    w.arrays.update(port_off=port_off, port_peer=peer, jur=jur, hdr=hdr, ingress=np.zeros(T, np.int32))
    w.sizes.update(S=S, ttl=12)
    ctx = pc.Context(0)
    ctx.keep_tables(True)
    some = np.sort(rng.choice(T, 40, replace=False))
    new = rules.copy()
    new["action"][:n] = (new["action"][:n] + 1) % port_off[1]

    def call(r, *state, c=ctx):
        c.profile(True)
        out = _run(w, off, r, *state[:2], state[2] if len(state) > 2 else None, walk=state[3] if len(state) > 3 else None, ctx=c)
        used = c.profile_read()
        c.profile(False)
        return out[:3], out[3], used

    first, _, used = call(rules, None, None)
    assert ("k_tr_plan" in used) != walks
    whole = pc.records(pc.pc_trace_flows(S, *(g.dev(x) for x in (port_off, peer, jur, off, rules, hdr, w["ingress"])), 12), pc.TRACE_OUT_DT)
    _same_records(whole, first[0])
    monkeypatch.setenv("PC_TRACE_WALK_MAX", "0" if walks else str(10**9))
    other, _, used = call(rules, None, None, c=pc.Context(0))
    assert ("k_tr_plan" in used) == walks
    for x, y in zip(first, other):
        assert np.array_equal(x, y)
    monkeypatch.delenv("PC_TRACE_WALK_MAX")
    for c in (ctx, pc.Context(0)):
        again, count, used = call(new, first[0], first[1], [0], first[2], c=c)
        assert count == T and ("k_delta_gather" in used) != walks
        ro, vo, wo, _ = _oracle(orc, w, off, new, idx=some)
        _same_records(again[0][some], ro)
        assert np.array_equal(again[1][some], vo) and np.array_equal(again[2][some], wo)
    ro, vo, wo, _ = _oracle(orc, w, off, rules, idx=some)
    _same_records(first[0][some], ro)
    assert np.array_equal(first[1][some], vo) and np.array_equal(first[2][some], wo)


@pytest.mark.parametrize("form,kernel", [("one", "listed"), ("few", "marked"), ("all", "marked"), ("repeated", "marked"), ("others", "listed")])
def test_delta_one_large_table_changed(g, orc, form, kernel):
    """300,000 rules on one of 320 switches: a delta on kept tables prepares them with a workgroup for each of their
    blocks (by those of the mean table 310 us), by the list or, past all tables' blocks, by the marked switches."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(4)
    wl = synth.trace_workload(3, 16, 4, 16, 1000, 12, 50)
    S, n = wl["S"], 300_000
    extra = np.zeros(n, synth.RULE_DT)
    extra["value"], extra["mask"] = synth.random_keys(rng, n), np.array([0xFFFFFFFF] * 3 + [0xFF], np.uint32)
    extra["priority"] = rng.integers(0, 65536, n)
    extra["action"] = rng.integers(0, wl["port_off"][1], n)
    own = wl["rule_off"][1]
    rules = np.concatenate([wl["rules"][:own], extra, wl["rules"][own:]])
    off = wl["rule_off"].copy()
    off[1:] += n
    hdr = wl["hdr"].copy()
    hdr[::2] = extra["value"][rng.integers(0, n, 500)]
    w = synth.Workload("hub", 0)
    w.arrays.update(port_off=wl["port_off"], port_peer=wl["port_peer"], jur=wl["jur"], hdr=hdr,
                    ingress=np.where(rng.random(1000) < 0.5, 0, wl["ingress"]).astype(np.int32))
    w.sizes.update(S=S, ttl=12)
    changed = dict(one=[0], few=[5, 0, S + 1, 7, -1, *range(10, 20)], all=np.arange(S), repeated=[0] * 500,
                   others=[3, 4])[form]
    inside = np.unique([c for c in changed if 0 <= c < S])
    new = rules.copy()
    for s in inside:
        t = new[off[s]:off[s + 1]]
        t["action"] = (t["action"] + 1) % (wl["port_off"][s + 1] - wl["port_off"][s])
    new["action"][off[inside[0]] + 3] = 5000
    ctx = pc.Context(0)
    ctx.keep_tables(True)
    first = _run(w, off, rules, None, None, None, ctx=ctx)
    for _ in range(2):
        ctx.profile(True)
        again = _run(w, off, new, *first[:2], changed, walk=first[2], ctx=ctx)
        used = ctx.profile_read()
        ctx.profile(False)
        ro, vo, wo, err = _oracle(orc, w, off, new)
        _same_records(again[0], ro)
        assert np.array_equal(again[1], vo) and np.array_equal(again[2], wo)
        assert again[4] == err | (F_SWITCH if form == "few" else 0)
        assert "k_tr_prep" not in used
    assert used["k_tr_prep_" + kernel][1] < 0.15, used


@pytest.mark.parametrize("T", [2048, 2049])
def test_walks_through_one_large_table(g, orc, T):
    """1.1 million rules on the switch where every trace enters: up to 2,048 traces walk with a whole workgroup each
    (1,000 traces 47 us, with a wavefront 122)."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(T)
    wl = synth.trace_workload(3, 16, 4, 16, T, 12, 50)
    n, own = 1_100_000, wl["rule_off"][1]
    hub = np.zeros(n, synth.RULE_DT)
    hub["value"], hub["mask"] = synth.random_keys(rng, n), np.array([0xFFFFFFFF] * 3 + [0xFF], np.uint32)
    hub["priority"] = rng.integers(0, 65536, n)
    hub["action"] = rng.integers(0, wl["port_off"][1], n)
    off = wl["rule_off"].copy()
    off[1:] += n
    rules = np.concatenate([wl["rules"][:own], hub, wl["rules"][own:]])
    hdr = wl["hdr"].copy()
    hdr[::2] = hub["value"][rng.integers(0, n, hdr[::2].shape[0])]
    w = synth.Workload("hub", 0)
    w.arrays.update(port_off=wl["port_off"], port_peer=wl["port_peer"], jur=wl["jur"], hdr=hdr, ingress=np.zeros(T, np.int32))
    w.sizes.update(S=wl["S"], ttl=12)
    some = np.sort(rng.choice(T, 60, replace=False))
    ro, vo, wo, _ = _oracle(orc, w, off, rules, idx=some)
    d = [g.dev(x) for x in (w["port_off"], w["port_peer"], w["jur"], off, rules, hdr)]
    ctx = pc.Context(0)
    for k in (1000, T):
        for _ in range(2):
            ctx.profile(True)
            got = pc.records(pc.pc_trace_flows(w["S"], *d[:5], d[5][:k], g.dev(w["ingress"][:k]), 12, ctx=ctx), pc.TRACE_OUT_DT)
            used = ctx.profile_read()
            ctx.profile(False)
        _same_records(got[some[some < k]], ro[some < k])
        if k == 1000:
            assert used["k_tr_walk"][1] < 0.09, used
    first = _run(w, off, rules, None, None, None)
    again = _run(w, off, rules, *first[:2], [0], walk=first[2])
    for r in (first, again):
        _same_records(r[0][some], ro)
        assert np.array_equal(r[1][some], vo) and np.array_equal(r[2][some], wo)


def test_delta_priorities_refused(g, orc, monkeypatch):
    """Where the kept tables' buffer holds the chunk sets but not the rules' priorities, levels of many lookups are matched
    in registers, also by the deltas that follow."""
    import paper_2602_16100_amd as pc
    T, S = 100_000, 720
    small, wl = (synth.trace_workload(3, 24, 4, R, T, 12, 2000) for R in (2016, 2400))
    some = np.arange(0, T, 5000)
    changed = np.arange(0, S, 3)
    off2, new = synth.mutate_tables(4, wl["port_off"], wl["rule_off"], wl["rules"], changed)
    ctx, other = pc.Context(0), pc.Context(0)
    for c in (ctx, other):
        c.keep_tables(True)

    def call(c, off, rules, *state):
        c.profile(True)
        r = _run(wl, off, rules, *(state[:2] or (None, None)), changed if state else None, walk=state[2] if state else None, ctx=c)
        used = c.profile_read()
        c.profile(False)
        return r, used

    _run(small, small["rule_off"], small["rules"], None, None, None, ctx=ctx)  # all buffers; 504 bytes a group for the sets'
    _run(small, small["rule_off"], small["rules"], np.zeros(T, pc.TRACE_OUT_DT), np.zeros(T, np.uint64), [], walk=np.full((T, 8), -1), ctx=ctx)
    monkeypatch.setenv("PC_FAIL_ALLOC", "1")
    first, used = call(ctx, wl["rule_off"], wl["rules"])
    assert "k_tr_match_wide" in used and "k_tr_match" not in used
    again, used = call(ctx, off2, new, *first[:3])
    monkeypatch.delenv("PC_FAIL_ALLOC")
    first2, used = call(other, wl["rule_off"], wl["rules"])
    assert "k_tr_match" in used
    again2, used = call(other, off2, new, *first2[:3])
    for a, b, off, rules in ((first, first2, wl["rule_off"], wl["rules"]), (again, again2, off2, new)):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
        ro, vo, wo, _ = _oracle(orc, wl, off, rules, idx=some)
        _same_records(a[0][some], ro)
        assert np.array_equal(a[1][some], vo) and np.array_equal(a[2][some], wo)
