"""Timed workloads of the compliance checker.

Every case is work that a validator has the library do, through the public
binding: a whole validation pass over a snapshot (placement, routing,
reachability, verdict) at three scales, and the calls that are also made on
their own: selector evaluation, affinity with scoring, flow tracing,
reachability maps, path synthesis, and re-validation after relabelled nodes
or rewritten flow tables.  Inputs are made on the GPU from a seed; their
statistics are those of the repository's synthetic generators (R-path and
prefix flow tables on fat-trees, selector rows over labels of cardinality
2-64, random geometric graphs with Voronoi regions).

All results are bitsets, counts, records and distances: integers, which
every correct implementation gives exactly.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2602_16100_amd as pc

CARDS = (2, 4, 16, 64)
DROP = 0xFFFF


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one deployment of the paper's test-bed size: a few nodes, a small fabric, some dozen intents; the whole
        # pass is a few kilobytes of input, so launches and host work count
        dict(name="validate_paper", kind="validate", mode="full", N=16, L=8, k=4, J=4, R=32, I=64, per=24, ttl=16),
        # one site: a thousand nodes, a 180-switch fabric of odd table sizes, waypoints and forbidden switches
        dict(name="validate_site", kind="validate", mode="paths", N=1503, L=32, k=12, J=6, R=777, I=9001, per=1,
             ttl=32),
        # a fleet: the repository's combined benchmark workload, full bitsets
        dict(name="validate_fleet", kind="validate", mode="full", N=50_000, L=64, k=48, J=12, R=16_384,
             I=1_048_576, per=1, ttl=32),
        # selector rows against a large cluster (the repository's selector configuration)
        dict(name="place_cluster", kind="place", N=100_000, L=64, I=16_384, absent=0.0),
        # required and preferred affinity of one batch of pods; labels that some nodes lack
        dict(name="schedule_batch", kind="schedule", N=5037, L=64, I=3001, absent=0.05),
        # the same for a fleet's worth of rows
        dict(name="schedule_fleet", kind="schedule", N=50_000, L=64, I=233_017, absent=0.0),
        # millions of headers through per-flow tables (the repository's trace configuration)
        dict(name="trace_fabric", kind="trace", tables="rpath", k=32, J=8, R=4096, T=4_194_304, ttl=32),
        # headers through routing tables: destination prefixes, several matching rules per lookup, some loops
        dict(name="trace_routed", kind="trace", tables="prefix", k=24, J=8, R=2048, T=500_009, ttl=32),
        # distance maps over a metropolitan graph (the repository's reachability configuration)
        dict(name="reach_metro", kind="reach", V=1_000_000, Q=256, degree=4.0, rows=True),
        # path requests over a fleet's fabric with link costs (the repository's synthesis pass)
        dict(name="synthesize_fleet", kind="synthesize", k=48, J=12, Q=65_536, Kv=1, Kf=2, weighted=True, hops=32),
        # a few nodes taken into maintenance and back: every row's bits of these nodes
        dict(name="relabel_nodes", kind="relabel", N=20_011, L=64, I=200_003, M=9),
        # the flow tables of a few switches rewritten and restored, the affected traces traced again
        dict(name="rules_changed", kind="rules", k=32, J=8, R=4096, T=300_007, C=16, ttl=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["validate", "validate", "place", "schedule", "trace", "reach", "synthesize", "relabel",
                       "rules"])
    if kind == "validate":
        k = 2 * _log(rng, 2, 20)
        return dict(kind=kind, mode=rng.choice(["full", "paths", "counts"]), N=_log(rng, 16, 40_000),
                    L=rng.randint(8, 64), k=k, J=rng.randint(2, min(16, k)), R=_log(rng, 32, 8192),
                    I=_log(rng, 64, 500_000), per=rng.choice([1, 1, 2]), ttl=rng.choice([16, 32, 64]))
    if kind == "place":
        return dict(kind=kind, N=_log(rng, 64, 100_000), L=rng.randint(8, 64), I=_log(rng, 64, 200_000),
                    absent=rng.choice([0.0, 0.05]))
    if kind == "schedule":
        return dict(kind=kind, N=_log(rng, 64, 50_000), L=rng.randint(8, 64), I=_log(rng, 64, 233_017),
                    absent=rng.choice([0.0, 0.05]))
    if kind == "trace":
        k = 2 * _log(rng, 2, 16)
        tables = rng.choice(["rpath", "rpath", "prefix"])
        return dict(kind=kind, tables=tables, k=k, J=rng.randint(2, min(16, k)),
                    R=_log(rng, 32, 2048 if tables == "prefix" else 4096),
                    T=_log(rng, 1000, 500_009 if tables == "prefix" else 4_194_304), ttl=rng.choice([16, 32, 64]))
    if kind == "reach":
        rows = rng.random() < 0.5
        return dict(kind=kind, V=_log(rng, 1000, 1_000_000), Q=_log(rng, 16, 256), degree=4.0, rows=rows)
    if kind == "synthesize":
        k, Kv = 2 * _log(rng, 2, 24), rng.randint(0, 2)
        return dict(kind=kind, k=k, J=rng.randint(2, min(16, k)), Q=_log(rng, 16, min(65_536, 131_072 // (Kv + 1))),
                    Kv=Kv, Kf=rng.randint(0, 3), weighted=rng.random() < 0.5, hops=rng.choice([16, 32, 64]))
    if kind == "relabel":
        return dict(kind=kind, N=_log(rng, 1000, 50_000), L=rng.randint(8, 64), I=_log(rng, 1000, 200_003),
                    M=_log(rng, 1, 64))
    k = 2 * _log(rng, 2, 16)
    return dict(kind=kind, k=k, J=rng.randint(2, min(16, k)), R=_log(rng, 32, 4096), T=_log(rng, 1000, 300_007),
                C=_log(rng, 1, 16), ttl=32)


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------ generators
class _Rng:
    """Seeded draws on the GPU."""

    def __init__(self, seed, device):
        self.g = torch.Generator(device=device)
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 12345)
        self.dev = device

    def unit(self, *shape):
        return torch.rand(shape, generator=self.g, device=self.dev)

    def below(self, n, *shape):
        """Uniform integers in [0, n) (int64); n a number or a tensor that broadcasts to the shape."""
        u = torch.rand(shape, generator=self.g, device=self.dev, dtype=torch.float64)
        return (u * n).to(torch.int64)

    def words(self, *shape):
        return torch.randint(-(1 << 31), 1 << 31, shape, generator=self.g, device=self.dev).to(torch.int32)

    def care(self, *shape):
        """Words whose bits are set with probability 11/16 (the tables' care bits: about 0.7)."""
        return self.words(*shape) | (self.words(*shape) & (self.words(*shape) | self.words(*shape)))


def _offsets(n):
    off = torch.zeros(n.shape[0] + 1, dtype=torch.int64, device=n.device)
    off[1:] = torch.cumsum(n, 0)
    return off


def _cluster(r, N, L, absent):
    cards = torch.tensor(CARDS, device=r.dev)[r.below(len(CARDS), L)]
    labels = r.below(cards, N, L).to(torch.uint8)
    if absent:
        labels[r.unit(N, L) < absent] = 255
    return cards, labels


def _preds(label, op, vals0):
    """40-byte predicate records as int64 [P, 5]; values stay below 64, so one word of the set is used."""
    p = torch.zeros((label.shape[0], 5), dtype=torch.int64, device=label.device)
    p[:, 0] = label | (op << 16)
    p[:, 1] = vals0
    return p


def _value_set(r, card, most=4):
    """1..most values of each label's domain as a 64-bit set."""
    m = r.below(most, card.shape[0]) + 1
    s = torch.zeros_like(card)
    for j in range(most):
        s |= torch.where(m > j, torch.ones_like(card) << r.below(card, card.shape[0]), torch.zeros_like(card))
    return s


def _selector_rows(r, I, cards, kmax=8):
    n = r.below(kmax, I) + 1
    off = _offsets(n)
    P = int(off[-1])
    lab = r.below(cards.shape[0], P)
    op = r.below(3, P)
    vals = torch.where(op == 2, torch.zeros_like(op), _value_set(r, cards[lab]))
    return n, off, lab, op, vals


def _affinity_rows(r, I, cards, kmax):
    """Rows of 1-3 terms of 1..kmax expressions over all six operators."""
    row_off = _offsets(r.below(3, I) + 1)
    T = int(row_off[-1])
    term_off = _offsets(r.below(kmax, T) + 1)
    P = int(term_off[-1])
    lab = r.below(cards.shape[0], P)
    op = r.below(6, P)
    card = cards[lab]
    thr = r.below(card + 2, P) - 1
    vals = torch.where(op < 2, _value_set(r, card), torch.where(op > 3, thr, torch.zeros_like(thr)))
    return row_off.to(torch.int32), term_off.to(torch.int32), _preds(lab, op, vals)


def _fat_tree(k, J, dev):
    """k-ary fat-tree (Al-Fares numbering): ports, jurisdictions, hosts and the sorted adjacency lists."""
    h, n_pod = k // 2, k * k
    S = n_pod + h * h
    peer = np.full((S, k), -1, np.int64)
    pod, x = np.divmod(np.arange(n_pod), k)
    edge = x < h
    ids = np.arange(h)
    peer[np.flatnonzero(edge), h:] = (pod[edge] * k)[:, None] + h + ids
    peer[np.flatnonzero(~edge), :h] = (pod[~edge] * k)[:, None] + ids
    peer[np.flatnonzero(~edge), h:] = n_pod + (x[~edge] - h)[:, None] * h + ids
    core = np.arange(h * h)
    peer[n_pod:, :] = np.arange(k)[None, :] * k + h + (core // h)[:, None]
    jur = np.concatenate([pod * J // k, core % J]).astype(np.uint8)
    hosts = np.arange(k * h * h)
    adj = [np.sort(p[p >= 0]) for p in peer]
    t = lambda a, d=torch.int32: torch.from_numpy(np.ascontiguousarray(a)).to(device=dev, dtype=d)  # noqa: E731
    return dict(k=k, S=S, H=hosts.shape[0], port_off=t(np.arange(S + 1) * k), port_peer=t(peer.reshape(-1)),
                jur=t(jur, torch.uint8), host_switch=t(hosts // (h * h) * k + hosts // h % h, torch.int64),
                host_port=t(hosts % h, torch.int64),
                host_ip=t(10 << 24 | hosts // (h * h) << 16 | hosts // h % h << 8 | hosts % h + 2, torch.int64),
                adj_off=t(np.concatenate([[0], np.cumsum([len(a) for a in adj])])), adj=t(np.concatenate(adj)))


def _flows(r, topo, hs, hd):
    """Per flow its 5-tuple and its ECMP path: switches and out-ports [F, 5] (-1 past the end), hop count."""
    F, k = hs.shape[0], topo["k"]
    h, n_pod = k // 2, k * k
    key = torch.empty((F, 4), dtype=torch.int32, device=r.dev)
    key[:, 0] = topo["host_ip"][hs].to(torch.int32)
    key[:, 1] = topo["host_ip"][hd].to(torch.int32)
    key[:, 2] = r.words(F)
    key[:, 3] = r.words(F) & 0xFF
    es, ed, dp = topo["host_switch"][hs], topo["host_switch"][hd], topo["host_port"][hd]
    a, j = r.below(h, F), r.below(h, F)
    same, pod = es == ed, es // k == ed // k
    no = torch.full_like(es, -1)
    up, down = es // k * k + h + a, ed // k * k + h + a
    w = torch.where
    sw = torch.stack([es, w(same, no, up), w(same, no, w(pod, ed, n_pod + a * h + j)), w(pod, no, down),
                      w(pod, no, ed)], 1)
    port = torch.stack([w(same, dp, h + a), w(pod, ed % k, h + j), w(pod, dp, ed // k), ed % k, dp], 1)
    nh = w(same, 1, w(pod, 3, 5))
    return key, sw, port, nh


def _tables(r, topo, R, kind, key, sw, port):
    """R rules per switch: one per hop of every flow at random slots, the rest noise of the same statistics;
    5 % of the actions drop, 2 % go to a random port; priorities are distinct within a switch."""
    S, k = topo["S"], topo["k"]
    n = S * R

    def masks(m):
        if kind == "prefix":
            x = torch.zeros((m, 4), dtype=torch.int32, device=r.dev)
            x[:, 1] = (torch.full((m,), 0xFFFFFFFF, device=r.dev) << (32 - 16 - r.below(17, m))).to(torch.int32)
            return x
        x = r.care(m, 4)
        x[:, 3] &= 0xFF
        return x

    def actions(out):
        u = r.unit(out.shape[0])
        bad = torch.where(u < 0.05, torch.full_like(out, DROP), r.below(k, out.shape[0]))
        return torch.where(u < 0.07, bad, out)

    rules = torch.zeros((n, 10), dtype=torch.int32, device=r.dev)
    m = masks(n)
    rules[:, 0:4] = r.words(n, 4) & m
    rules[:, 4:8] = m
    del m
    i = torch.arange(R, device=r.dev)[None, :]
    prio = (i * (2 * r.below(1 << 15, S) + 1)[:, None] + r.below(1 << 16, S)[:, None]) & 0xFFFF
    act = torch.where(r.unit(n) < 0.05, torch.full((n,), DROP, device=r.dev), r.below(k, n))
    rules[:, 8] = (prio.reshape(-1) | act << 16).to(torch.int32)
    # the flows' rules: rank r of a switch takes slot (step * r + start) mod R, step coprime to R
    at = sw >= 0
    flow = torch.arange(sw.shape[0], device=r.dev)[:, None].expand_as(sw)[at]
    e_sw, order = torch.sort(sw[at], stable=True)
    flow, out = flow[order], port[at][order]
    start = torch.zeros(S + 1, dtype=torch.int64, device=r.dev)
    start[1:] = torch.cumsum(torch.bincount(e_sw, minlength=S), 0)
    rank = torch.arange(e_sw.shape[0], device=r.dev) - start[e_sw]
    keep = rank < R
    flow, out, e_sw, rank = flow[keep], out[keep], e_sw[keep], rank[keep]
    step = next(x for x in range(int(R * 0.618) | 1, 2 * R + 3) if math.gcd(x, R) == 1)
    pos = e_sw * R + (rank * step + r.below(R, S)[e_sw]) % R
    m = masks(pos.shape[0])
    rules[pos, 0:4] = key[flow] & m
    rules[pos, 4:8] = m
    rules[pos, 8] = (rules[pos, 8] & 0xFFFF) | (actions(out) << 16).to(torch.int32)
    rule_off = (torch.arange(S + 1, device=r.dev) * R).to(torch.int32)
    return rule_off, rules


def _allowed(r, jur, J, a, b):
    """Both endpoints' jurisdictions and each other one with probability 1/2."""
    m = (1 << jur[a].to(torch.int64)) | (1 << jur[b].to(torch.int64)) | r.below(1 << J, a.shape[0])
    return m.to(torch.int32)


def _other(r, H, hs):
    return (hs + 1 + r.below(H - 1, hs.shape[0])) % H


# ------------------------------------------------------------------ states
def _prep_validate(c, r):
    N, L, I, per = c["N"], c["L"], c["I"], c["per"]
    cards, labels = _cluster(r, N, L, 0.0)
    topo = _fat_tree(c["k"], c["J"], r.dev)
    H = topo["H"]
    kind = torch.tensor([1, 2, 3], device=r.dev)[torch.arange(I, device=r.dev) % 3]
    has_sel, has_net, hyb = (kind & 1) == 1, (kind & 2) == 2, kind == 3
    rows, nets = int(has_sel.sum()), int(has_net.sum())
    sel_row = torch.where(has_sel, torch.cumsum(has_sel, 0) - 1, -1)
    net_id = torch.cumsum(has_net, 0) - 1
    # hybrid intents: two nodes that their row admits, but for 1 in 16 whose second pod sits elsewhere
    a, b = r.below(N, I), r.below(N, I)
    n, off, lab, op, vals = _selector_rows(r, rows, cards)
    owner = torch.repeat_interleave(torch.nonzero(has_sel)[:, 0], n)
    va, vb = labels[a[owner], lab].to(torch.int64), labels[b[owner], lab].to(torch.int64)
    both = (torch.ones_like(va) << va) | (torch.ones_like(vb) << vb)
    h = hyb[owner]
    vals = torch.where(h & (op == 0), vals | both, torch.where(h & (op == 1), vals & ~both, vals))
    op = torch.where(h & (op == 1) & (vals == 0), torch.full_like(op, 2), op)
    b = torch.where(r.unit(I) < 1 / 16, r.below(N, I), b)
    # flows: `per` of each network or hybrid intent, between its hosts
    hs = torch.where(hyb, a % H, r.below(H, I))[has_net]
    hd = torch.where(hyb[has_net], b[has_net] % H, _other(r, H, hs))
    hs, hd = hs.repeat_interleave(per), hd.repeat_interleave(per)
    key, sw, port, nh = _flows(r, topo, hs, hd)
    rule_off, rules = _tables(r, topo, c["R"], "rpath", key, sw, port)
    e_src, e_dst = topo["host_switch"][hs], topo["host_switch"][hd]
    q_src, q_dst = e_src[::per].contiguous(), e_dst[::per].contiguous()
    allowed = _allowed(r, topo["jur"], c["J"], q_src, q_dst)
    it = torch.zeros((I, 8), dtype=torch.int32, device=r.dev)
    it[:, 0] = kind
    it[:, 1] = sel_row
    it[:, 2] = torch.where(hyb, a, -1)
    it[:, 3] = torch.where(hyb, b, -1)
    it[:, 4] = torch.where(has_net, net_id * per, 0)
    it[:, 5] = torch.where(has_net, net_id * per + per, 0)
    it[has_net, 6] = allowed
    ex = torch.full((I, 3), -1, dtype=torch.int32, device=r.dev)
    ex[has_net, 0] = q_dst.to(torch.int32)
    ex[has_net, 1] = topo["host_port"][hd][::per].to(torch.int32)
    ex[has_net, 2] = torch.arange(nets, dtype=torch.int32, device=r.dev)
    st = dict(labels=labels, pred_off=off.to(torch.int32), preds=_preds(lab, op, vals), topo=topo, rule_off=rule_off,
              rules=rules, hdr=key, ingress=e_src.to(torch.int32), src=q_src.to(torch.int32),
              target=q_dst.to(torch.int32), allowed=allowed, intents=it, expect=ex, N=N)
    if c["mode"] == "paths":
        # a waypoint (on the flow's path for half of them) and two forbidden switches per intent
        mid = sw[::per].gather(1, (nh[::per] // 2)[:, None])[:, 0]
        way = torch.where(r.unit(nets) < 0.5, mid, r.below(topo["S"], nets))
        bad = torch.where(r.unit(nets, 2) < 0.125, sw[::per, 1:2].clamp(min=0), r.below(topo["S"], nets, 2))
        bad = torch.where(bad == way[:, None], -1, bad)
        st["via"], st["forbid"] = way[:, None].to(torch.int32).contiguous(), bad.to(torch.int32).contiguous()
        st["watch"] = torch.cat([st["via"], st["forbid"]], 1).repeat_interleave(per, 0).contiguous()
        st["pexp"] = torch.zeros((I, 2), dtype=torch.int32, device=r.dev)
        st["pexp"][has_net] = torch.tensor([1, 6], dtype=torch.int32, device=r.dev)
    if c["mode"] == "counts":
        st["probe_row"] = torch.where(hyb, sel_row, 0).repeat_interleave(2).to(torch.int32)
        st["probe_node"] = torch.stack([torch.where(hyb, a, 0), torch.where(hyb, b, 0)], 1).reshape(-1).to(torch.int32)
    return st


def _run_validate(c, s):
    t = s["topo"]
    trace = (t["S"], t["port_off"], t["port_peer"], t["jur"], s["rule_off"], s["rules"], s["hdr"], s["ingress"],
             c["ttl"])
    graph = (t["S"], t["adj_off"], t["adj"], t["jur"], s["src"], s["allowed"], s["target"])
    if c["mode"] == "counts":
        cnt = pc.pc_eval_selectors_count(s["labels"], s["pred_off"], s["preds"])
        ends = pc.pc_probe_selectors(s["labels"], s["pred_off"], s["preds"], s["probe_row"], s["probe_node"])
        out = pc.pc_trace_flows(*trace)
        dist = pc.pc_masked_reach(*graph)
        return (cnt, ends, out, dist) + pc.pc_report_counts(s["intents"], cnt, s["N"], ends, out, s["expect"], dist)
    feas, cnt = pc.pc_eval_selectors(s["labels"], s["pred_off"], s["preds"])
    if c["mode"] == "paths":
        out, visit = pc.pc_trace_flows_watch(*trace, s["watch"])
        dist = pc.pc_masked_reach_via(*graph, s["via"], s["forbid"])
        return (feas, cnt, out, visit, dist) + pc.pc_report_paths(s["intents"], feas, cnt, s["N"], out, s["expect"],
                                                                  dist, visit, s["pexp"])
    out = pc.pc_trace_flows(*trace)
    dist = pc.pc_masked_reach(*graph)
    return (feas, cnt, out, dist) + pc.pc_report(s["intents"], feas, cnt, s["N"], out, s["expect"], dist)


def _prep_place(c, r):
    cards, labels = _cluster(r, c["N"], c["L"], c["absent"])
    _, off, lab, op, vals = _selector_rows(r, c["I"], cards)
    return dict(labels=labels, pred_off=off.to(torch.int32), preds=_preds(lab, op, vals))


def _run_place(c, s):
    return pc.pc_eval_selectors(s["labels"], s["pred_off"], s["preds"])


def _prep_schedule(c, r):
    cards, labels = _cluster(r, c["N"], c["L"], c["absent"])
    req = _affinity_rows(r, c["I"], cards, 4)
    pref = _affinity_rows(r, c["I"], cards, 3)
    weight = (r.below(100, pref[1].shape[0] - 1) + 1).to(torch.int32)
    return dict(labels=labels, req=req, pref=pref, weight=weight)


def _run_schedule(c, s):
    feas, cnt, unknown = pc.pc_eval_affinity(s["labels"], *s["req"])
    best = pc.pc_score_preferred(s["labels"], s["pref"][0], s["pref"][1], s["weight"], s["pref"][2], feasible=feas)
    return (feas, cnt, unknown) + best


def _prep_trace(c, r):
    topo = _fat_tree(c["k"], c["J"], r.dev)
    F = max(1, c["T"] // 8)
    hs = r.below(topo["H"], F)
    key, sw, port, _ = _flows(r, topo, hs, _other(r, topo["H"], hs))
    rule_off, rules = _tables(r, topo, c["R"], c["tables"], key, sw, port)
    pick = r.below(F, c["T"])
    return dict(topo=topo, rule_off=rule_off, rules=rules, hdr=key[pick].contiguous(),
                ingress=topo["host_switch"][hs[pick]].to(torch.int32))


def _run_trace(c, s):
    t = s["topo"]
    return pc.pc_trace_flows(t["S"], t["port_off"], t["port_peer"], t["jur"], s["rule_off"], s["rules"], s["hdr"],
                             s["ingress"], c["ttl"])


def _prep_reach(c, r):
    """Random geometric graph on the unit square (neighbours through a grid of cells of the edge length)."""
    V, Q = c["V"], c["Q"]
    p = r.unit(V, 2).to(torch.float64)
    d = math.sqrt(c["degree"] / (math.pi * V))
    G = max(1, int(1 / d))
    cell = (p * G).to(torch.int64).clamp(max=G - 1)
    cid = cell[:, 0] * G + cell[:, 1]
    order = torch.argsort(cid)
    first = torch.zeros(G * G + 1, dtype=torch.int64, device=r.dev)
    first[1:] = torch.cumsum(torch.bincount(cid, minlength=G * G), 0)
    us, vs = [], []
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            x, y = cell[:, 0] + dx, cell[:, 1] + dy
            inside = (x >= 0) & (x < G) & (y >= 0) & (y < G)
            nb = torch.where(inside, x * G + y, 0)
            cnt = torch.where(inside, first[nb + 1] - first[nb], 0)
            u = torch.repeat_interleave(torch.arange(V, device=r.dev), cnt)
            base = _offsets(cnt)[:-1]
            v = order[first[nb][u] + torch.arange(u.shape[0], device=r.dev) - base[u]]
            near = (u != v) & (((p[u] - p[v]) ** 2).sum(1) < d * d)
            us.append(u[near])
            vs.append(v[near])
    e = torch.sort(torch.cat(us) * V + torch.cat(vs))[0]
    off = torch.zeros(V + 1, dtype=torch.int64, device=r.dev)
    off[1:] = torch.cumsum(torch.bincount(e // V, minlength=V), 0)
    seeds = r.unit(16, 2).to(torch.float64)
    region = ((p[:, None, :] - seeds[None]) ** 2).sum(2).argmin(1).to(torch.uint8)
    # 1..8 of the 16 regions per query, its source in one of them
    n = r.below(8, Q) + 1
    rank = torch.argsort(torch.argsort(r.unit(Q, 16), 1), 1)
    allowed = ((rank < n[:, None]).to(torch.int64) << torch.arange(16, device=r.dev)).sum(1)
    tries = r.below(V, Q, 64)
    ok = (allowed[:, None] >> region[tries].to(torch.int64)) & 1
    src = tries.gather(1, ok.argmax(1, keepdim=True))[:, 0]
    target = None if c["rows"] else r.below(V, Q).to(torch.int32)
    return dict(adj_off=off.to(torch.int32), adj=(e % V).to(torch.int32), region=region, src=src.to(torch.int32),
                allowed=allowed.to(torch.int32), target=target)


def _run_reach(c, s):
    return pc.pc_masked_reach(c["V"], s["adj_off"], s["adj"], s["region"], s["src"], s["allowed"], s["target"])


def _prep_synthesize(c, r):
    topo = _fat_tree(c["k"], c["J"], r.dev)
    Q, S, Kv, Kf = c["Q"], topo["S"], c["Kv"], c["Kf"]
    a = r.below(topo["H"], Q)
    b = _other(r, topo["H"], a)
    src, dst = topo["host_switch"][a], topo["host_switch"][b]
    n_via = (r.unit(Q, Kv) < 0.7).sum(1) if Kv else None
    via = torch.where(torch.arange(Kv, device=r.dev)[None] < n_via[:, None], r.below(S, Q, Kv), -1) if Kv else None
    forbid = r.below(S, Q, Kf)
    for x in [src[:, None], dst[:, None]] + [via[:, j:j + 1] for j in range(Kv)]:
        forbid = torch.where(forbid == x, -1, forbid)
    key = r.words(Q, 4)
    key[:, 3] &= 0xFF
    empty = torch.empty((Q, 0), dtype=torch.int32, device=r.dev)
    weight = (r.below(10, topo["port_peer"].shape[0]) + 1).to(torch.int32) if c["weighted"] else None
    return dict(topo=topo, src=src.to(torch.int32), target=dst.to(torch.int32),
                allowed=_allowed(r, topo["jur"], c["J"], src, dst),
                via=via.to(torch.int32).contiguous() if Kv else empty,
                forbid=forbid.to(torch.int32).contiguous() if Kf else empty, key=key,
                out_port=topo["host_port"][b].to(torch.int32), weight=weight)


def _run_synthesize(c, s):
    t = s["topo"]
    return pc.pc_synthesize_paths(t["S"], t["port_off"], t["port_peer"], t["jur"], s["src"], s["target"],
                                  s["allowed"], s["via"], s["forbid"], s["key"], s["out_port"], 40_000, c["hops"],
                                  weight=s["weight"])


def _prep_relabel(c, r):
    s = _prep_place(dict(c, absent=0.0), r)
    cards = s["labels"].max(0)[0].to(torch.int64) + 1
    nodes = torch.argsort(r.unit(c["N"]))[: c["M"]]
    s["nodes"] = nodes.to(torch.int32)
    s["relabelled"] = s["labels"].clone()
    s["relabelled"][nodes] = r.below(cards, nodes.shape[0], c["L"]).to(torch.uint8)
    s["feasible"], s["popcnt"] = pc.pc_eval_selectors(s["labels"], s["pred_off"], s["preds"])
    return s


def _run_relabel(c, s):
    args = (s["pred_off"], s["preds"], s["nodes"], s["feasible"], s["popcnt"])
    pc.pc_update_nodes(s["relabelled"], *args)
    during = s["popcnt"].clone()
    pc.pc_update_nodes(s["labels"], *args)
    return s["feasible"], s["popcnt"], during


def _prep_rules(c, r):
    s = _prep_trace(dict(c, tables="rpath"), r)
    t, T, R = s["topo"], c["T"], c["R"]
    s["ctx"] = pc.Context(torch.cuda.current_device())
    s["ctx"].keep_tables(True)
    s["out"] = torch.empty((T, 12), dtype=torch.uint8, device=r.dev)
    s["vsum"] = torch.empty(T, dtype=torch.int64, device=r.dev)
    s["walk"] = torch.empty((T, 8), dtype=torch.int32, device=r.dev)
    sw = torch.argsort(r.unit(t["S"]))[: c["C"]]
    s["changed"] = sw.to(torch.int32)
    s["rows"] = (sw[:, None] * R + torch.arange(R, device=r.dev)[None]).reshape(-1)
    s["old"] = s["rules"][s["rows"]]
    s["new"] = s["old"].clone()
    n = s["new"].shape[0]
    act = torch.where(r.unit(n) < 0.1, torch.full((n,), DROP, device=r.dev), r.below(c["k"], n))
    s["new"][:, 8] = (s["new"][:, 8] & 0xFFFF) | (act << 16).to(torch.int32)
    s["args"] = (t["S"], t["port_off"], t["port_peer"], t["jur"], s["rule_off"], s["rules"], s["hdr"], s["ingress"],
                 c["ttl"], s["out"], s["vsum"])
    pc.pc_trace_flows_delta(*s["args"], walk=s["walk"], ctx=s["ctx"])
    return s


def _run_rules(c, s):
    s["rules"][s["rows"]] = s["new"]
    n1 = pc.pc_trace_flows_delta(*s["args"], changed=s["changed"], walk=s["walk"], ctx=s["ctx"])
    during = s["out"].clone()
    s["rules"][s["rows"]] = s["old"]
    n2 = pc.pc_trace_flows_delta(*s["args"], changed=s["changed"], walk=s["walk"], ctx=s["ctx"])
    return during, n1, s["out"], s["vsum"], s["walk"], n2


_KINDS = {
    "validate": (_prep_validate, _run_validate),
    "place": (_prep_place, _run_place),
    "schedule": (_prep_schedule, _run_schedule),
    "trace": (_prep_trace, _run_trace),
    "reach": (_prep_reach, _run_reach),
    "synthesize": (_prep_synthesize, _run_synthesize),
    "relabel": (_prep_relabel, _run_relabel),
    "rules": (_prep_rules, _run_rules),
}


def prepare(case, seed):
    r = _Rng(seed, torch.device("cuda", torch.cuda.current_device()))
    s = _KINDS[case["kind"]][0](case, r)
    s["case"] = case
    return s


def run(state):
    return _KINDS[state["case"]["kind"]][1](state["case"], state)


# ------------------------------------------------------------------ necessary work
def work(case):
    """Bytes of the inputs read once and the outputs written once.  The paths compare, AND and count bits: no
    arithmetic of theirs is a floating-point operation."""
    c, kind = case, case["kind"]
    fat = lambda k: (5 * k * k // 4, 5 * k * k // 4 * k)  # noqa: E731  switches, ports
    if kind == "validate":
        S, ports = fat(c["k"])
        sel, net = c["I"] * 2 // 3, c["I"] * 2 // 3
        W = (c["N"] + 63) // 64
        b = c["N"] * c["L"] + sel * (4.5 * 40 + 8) + (0 if c["mode"] == "counts" else sel * W * 8)
        b += S * c["R"] * 40 + ports * 8 + net * c["per"] * 32 + net * 16 + c["I"] * 46
        b += net * (24 + 24 * c["per"]) if c["mode"] == "paths" else 0
        b += c["I"] * 18 if c["mode"] == "counts" else 0
    elif kind == "place":
        b = c["N"] * c["L"] + c["I"] * (4.5 * 40 + 8 + (c["N"] + 63) // 64 * 8)
    elif kind == "schedule":
        W = (c["N"] + 63) // 64
        b = 2 * c["N"] * c["L"] + c["I"] * (5 * 40 + 12 + 9 + 2 * W * 8 + 4 * 40 + 20 + 12)
    elif kind == "trace":
        S, ports = fat(c["k"])
        b = S * c["R"] * 40 + ports * 4 + c["T"] * 32
    elif kind == "reach":
        b = c["V"] * (5 + 4 * c["degree"]) + c["Q"] * (c["V"] * 4 if c["rows"] else 16)
    elif kind == "synthesize":
        S, ports = fat(c["k"])
        b = ports * 8 + c["Q"] * (32 + 4 * c["Kv"] + 4 * c["Kf"] + 4 + 44 * (c["hops"] + 1))
    elif kind == "relabel":
        # the rows' predicates, and one 64-bit word per row and listed node read (changed ones also written)
        b = 2 * (c["I"] * (4.5 * 40 + 8 + 12 * c["M"]) + c["M"] * c["L"])
    else:
        S, _ = fat(c["k"])
        b = 2 * (c["C"] * c["R"] * 40 * 2 + c["T"] * (12 + 8 + 32))
    return {"bytes": float(b), "flops": 0.0}


# ------------------------------------------------------------------ plain answers
def exact(case, seed):
    """Plain torch answers of the two calls that have a short one; the others' outputs are compared bit by bit."""
    c = case
    if c["kind"] == "place" and c["N"] * c["I"] <= 1 << 31:
        s = prepare(case, seed)
        labels, preds = s["labels"].to(torch.int64), s["preds"]
        N, I, W = c["N"], c["I"], (c["N"] + 63) // 64
        off = s["pred_off"].to(torch.int64)
        row = torch.repeat_interleave(torch.arange(I, device=off.device), off[1:] - off[:-1])
        nth = torch.arange(preds.shape[0], device=off.device) - off[:-1][row]
        bit = torch.ones((), dtype=torch.int64, device=off.device) << torch.arange(64, device=off.device)
        feas = torch.empty((I, W), dtype=torch.int64, device=off.device)
        for r0 in range(0, I, 4096):
            n = min(4096, I - r0)
            ok = torch.ones((n, W * 64), dtype=torch.bool, device=off.device)
            ok[:, N:] = False
            for j in range(8):
                p = preds[(row >= r0) & (row < r0 + n) & (nth == j)]
                at = row[(row >= r0) & (row < r0 + n) & (nth == j)] - r0
                for a0 in range(0, p.shape[0], 256):
                    q, w = p[a0:a0 + 256], at[a0:a0 + 256]
                    x = labels.T[q[:, 0] & 0xFFFF]
                    there = x != 255
                    inside = there & (((q[:, 1:2] >> x.clamp(max=63)) & 1) == 1) & (x < 64)
                    op = (q[:, 0:1] >> 16) & 0xFF
                    ok[w, :N] &= torch.where(op == 0, inside, torch.where(op == 1, ~inside, there))
            feas[r0:r0 + n] = (ok.reshape(n, W, 64).to(torch.int64) * bit).sum(2)
            del ok
        cnt = torch.zeros(I, dtype=torch.int64, device=off.device)
        for b in range(64):
            cnt += ((feas >> b) & 1).sum(1)
        return feas, cnt.to(torch.int32)
    if c["kind"] == "reach" and c["V"] * c["Q"] <= 1 << 28:
        s = prepare(case, seed)
        V, Q = c["V"], c["Q"]
        off = s["adj_off"].to(torch.int64)
        u = torch.repeat_interleave(torch.arange(V, device=off.device), off[1:] - off[:-1])
        v = s["adj"].to(torch.int64)
        ok = ((s["allowed"].to(torch.int64)[:, None] >> s["region"].to(torch.int64)[None]) & 1) == 1
        dist = torch.full((Q, V), -1, dtype=torch.int32, device=off.device)
        for q in range(Q):
            at = s["src"][q:q + 1].to(torch.int64)
            at = at[ok[q][at]]
            alive = ok[q][u] & ok[q][v]
            uq, vq = u[alive], v[alive]
            first = torch.zeros(V + 1, dtype=torch.int64, device=off.device)
            first[1:] = torch.cumsum(torch.bincount(uq, minlength=V), 0)
            dist[q, at] = 0
            d = 0
            while at.numel():
                d += 1
                n = first[at + 1] - first[at]
                e = torch.repeat_interleave(first[at] - _offsets(n)[:-1], n) + torch.arange(int(n.sum()),
                                                                                            device=off.device)
                at = torch.unique(vq[e])
                at = at[dist[q, at] < 0]
                dist[q, at] = d
        return dist if c["rows"] else dist.gather(1, s["target"].to(torch.int64)[:, None])[:, 0]
    return None
