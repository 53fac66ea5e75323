"""Parity of the selector, affinity and preferred calls with the CPU oracle where their preparation kernels change
form: label arrays of every alignment and of more labels than the presence table holds, labels of few and of
many values, node counts at the edges of the plane builder's 1,024-node pieces, and rows at the edges of what a
group of lanes compiles (terms, expressions, inline program words, row counts)."""
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


@pytest.mark.parametrize("N,L,shift", [(1, 1, 0), (1023, 3, 1), (1024, 4, 4), (1025, 5, 15), (2049, 64, 3),
                                       (3000, 16, 8), (300, 1024, 2), (300, 1025, 0), (5037, 7, 0)])
def test_label_layouts(g, orc, N, L, shift):
    import torch
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(N)
    cards = rng.choice([1, 2, 8, 9, 64, 65, 255], size=L)
    labels = synth.gen_labels(rng, N, cards, 0.05)
    off, preds = synth.gen_preds(rng, 300, cards, 0, 6, mmax=4)
    flat = torch.zeros(N * L + shift, dtype=torch.uint8, device="cuda")
    flat[shift:] = torch.from_numpy(labels.reshape(-1)).cuda()
    f, p = pc.pc_eval_selectors(flat[shift:].view(N, L), g.dev(off), g.dev(preds))
    torch.cuda.synchronize()
    fo, po, _ = orc.selectors(labels, off, preds)
    assert np.array_equal(f.cpu().numpy().view(np.uint64), fo)
    assert np.array_equal(p.cpu().numpy().view(np.uint32), po)


def _rows(rng, cards, counts):
    """Affinity rows whose terms have the given expression counts (a list of lists)."""
    row_off = np.concatenate([[0], np.cumsum([len(r) for r in counts])]).astype(np.int32)
    k = np.array([x for r in counts for x in r], np.int64)
    term_off = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    P = int(term_off[-1])
    lab = rng.integers(0, len(cards), P)
    op = rng.integers(0, 6, P)
    preds = np.zeros(P, synth.PRED_DT)
    preds["label"], preds["op"] = lab, op
    vals = synth.distinct_values(rng, cards[lab], np.minimum(rng.integers(1, 5, P), cards[lab]), 4)
    bm = synth.values_to_bitmap(vals)
    bm[op > 1] = 0
    thr = rng.integers(-1, cards[lab] + 1)
    bm[op > 3, 0] = thr[op > 3].astype(np.int64).view(np.uint64)
    preds["vals"] = bm
    return row_off, term_off, preds


@pytest.mark.parametrize("kind", ["terms", "expressions", "inline", "malformed"])
def test_compiled_rows(g, orc, kind):
    rng = np.random.default_rng(len(kind))
    cards = rng.choice([2, 5, 16, 64], size=20)
    labels = synth.gen_labels(rng, 700, cards, 0.1)
    if kind == "terms":          # 0 to 18 terms, empty ones among them
        counts = [[int(x) for x in rng.integers(0, 2, n)] for n in range(19) for _ in range(8)]
    elif kind == "expressions":  # 14 to 18 expressions, and many
        counts = [[1] * 2 + [n - 2] for n in list(range(14, 19)) + [40, 200] for _ in range(12)] + [[16], [17], [0, 16, 0]]
    else:                        # programs around the inline sizes
        counts = [[int(x) for x in rng.integers(1, 5, int(rng.integers(1, 4)))] for _ in range(900)]
    row_off, term_off, preds = _rows(rng, cards, counts)
    weight = rng.integers(1, 101, term_off.shape[0] - 1).astype(np.uint32)
    if kind == "malformed":
        at = rng.integers(0, preds.shape[0], 60)
        preds["op"][at[:20]], preds["label"][at[20:40]], preds["rsv1"][at[40:]] = 9, 20, 1
        weight[rng.integers(0, weight.shape[0], 40)] = [0, 101] * 20
        term_off = term_off.copy()
        term_off[rng.integers(1, term_off.shape[0] - 1, 12)] += 7
        row_off = row_off.copy()
        row_off[rng.integers(1, row_off.shape[0] - 1, 6)] += 5
    fg, pg, ug, eg = g.affinity(labels, row_off, term_off, preds)
    fo, po, uo, eo = orc.affinity(labels, row_off, term_off, preds)
    assert np.array_equal(fg, fo) and np.array_equal(pg, po) and np.array_equal(ug, uo) and eg == eo
    bg, sg, cg, eg = g.preferred(labels, row_off, term_off, weight, preds)
    bo, so, co, eo = orc.preferred(labels, row_off, term_off, weight, preds)
    assert np.array_equal(bg, bo) and np.array_equal(sg, so) and np.array_equal(cg, co) and eg == eo


@pytest.mark.parametrize("I", [65535, 65536, 131071, 131072])
def test_row_counts_at_the_compile_rules(g, orc, I):
    rng = np.random.default_rng(I)
    cards = rng.choice([2, 4, 16], size=8)
    labels = synth.gen_labels(rng, 100, cards, 0.1)
    row_off, term_off, preds = synth.gen_affinity(rng, I, cards, 0, 3, 1, 3)
    weight = rng.integers(1, 101, term_off.shape[0] - 1).astype(np.uint32)
    fg, pg, ug, eg = g.affinity(labels, row_off, term_off, preds)
    fo, po, uo, eo = orc.affinity(labels, row_off, term_off, preds)
    assert np.array_equal(fg, fo) and np.array_equal(pg, po) and np.array_equal(ug, uo) and eg == eo
    bg, sg, cg, eg = g.preferred(labels, row_off, term_off, weight, preds)
    bo, so, co, eo = orc.preferred(labels, row_off, term_off, weight, preds)
    assert np.array_equal(bg, bo) and np.array_equal(sg, so) and np.array_equal(cg, co) and eg == eo


@pytest.mark.parametrize("I,L,t,k", [(32767, 64, 3, 6), (32768, 64, 3, 6), (33100, 65, 20, 1), (65536, 64, 3, 5), (65800, 65, 3, 5),
                                     (65999, 3, 3, 8)])
def test_many_rows(g, orc, I, L, t, k):
    """Rows compiled a thread each: label tables that fit LDS and one label more, programs around and past the words a
    thread holds, terms that are not adjacent, malformed expressions and offsets, all classes of preferred rows."""
    rng = np.random.default_rng(I + L)
    cards = rng.choice([2, 16, 64], size=L)
    labels = synth.gen_labels(rng, 100, cards, 0.1)
    row_off, term_off, preds = synth.gen_affinity(rng, I, cards, 0, t, 1, k)
    weight = rng.integers(1, 101, term_off.shape[0] - 1).astype(np.uint32)
    at = rng.integers(0, preds.shape[0], 600)
    preds["op"][at[:200]], preds["label"][at[200:400]], preds["rsv0"][at[400:]] = 9, L, 1
    weight[rng.integers(0, weight.shape[0], 100)] = [0, 101] * 50
    x = rng.integers(1, term_off.shape[0] - 1, 300)
    term_off[x] += rng.integers(-9, 10, 300).astype(np.int32)  # terms that share expressions, run backwards, are negative
    row_off[rng.integers(1, row_off.shape[0] - 1, 60)] += 5
    fg, pg, ug, eg = g.affinity(labels, row_off, term_off, preds)
    fo, po, uo, eo = orc.affinity(labels, row_off, term_off, preds)
    assert np.array_equal(fg, fo) and np.array_equal(pg, po) and np.array_equal(ug, uo) and eg == eo
    bg, sg, cg, eg = g.preferred(labels, row_off, term_off, weight, preds)
    bo, so, co, eo = orc.preferred(labels, row_off, term_off, weight, preds)
    assert np.array_equal(bg, bo) and np.array_equal(sg, so) and np.array_equal(cg, co) and eg == eo


@pytest.mark.parametrize("N,L,I,shift", [(1, 1, 1, 1), (63, 8, 15, 3), (64, 200, 17, 0), (65, 9, 300, 2), (255, 32, 1500, 0),
                                         (257, 5, 40, 1), (512, 64, 700, 0), (512, 127, 33, 0), (512, 128, 33, 0),
                                         (513, 8, 50, 0), (64, 4, 20000, 0), (64, 4, 70000, 0)])
def test_small_clusters(g, orc, N, L, I, shift):
    """Rows evaluated from the labels themselves, and the sizes past its limits (words, labels in LDS, predicates):
    sets of values on both sides of 64, rows without predicates, malformed rows, every alignment of the labels; also
    the counting and the allocation-free entry point."""
    import torch
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(N * L + I)
    cards = rng.choice([1, 2, 16, 64, 65, 200, 255], size=L)
    labels = synth.gen_labels(rng, N, cards, 0.1)
    off, preds = synth.gen_preds(rng, I, cards, 0, 7, mmax=4)
    if I > 30:
        off[11] = off[12] + 1
        preds["op"][off[20]:off[21]] = 3
        preds["label"][off[25]:off[26]] = L
    flat = torch.zeros(N * L + shift, dtype=torch.uint8, device="cuda")
    flat[shift:] = torch.from_numpy(labels.reshape(-1)).cuda()
    lab, o, p = flat[shift:].view(N, L), g.dev(off), g.dev(preds)
    fo, po, err = orc.selectors(labels, off, preds)
    ctx = pc.context()
    for call in ("full", "noalloc", "count"):
        ctx.data_errors(clear=True)
        f = torch.full((I, (N + 63) // 64), -1, dtype=torch.int64, device="cuda")
        c = torch.full((I,), -1, dtype=torch.int32, device="cuda")
        if call == "full":
            pc.pc_eval_selectors(lab, o, p, feasible=f, popcnt=c)
        elif call == "noalloc":
            pc.pc_eval_selectors_noalloc(lab, o, p, f, c)
        else:
            c = pc.pc_eval_selectors_count(lab, o, p)
        assert ctx.data_errors(clear=True) == err
        assert np.array_equal(c.cpu().numpy().view(np.uint32), po)
        if call != "count":
            assert np.array_equal(f.cpu().numpy().view(np.uint64), fo)


@pytest.mark.parametrize("N", [16384, 16385])
def test_presence_workgroups(g, orc, N):
    """Planes numbered by the last of 256 workgroups, and by a launch of their own from 257 on; several passes."""
    rng = np.random.default_rng(N)
    cards = rng.choice([2, 64, 255], size=64)
    off, preds = synth.gen_preds(rng, 200, cards, 1, 6, mmax=4)
    for _ in range(3):
        labels = synth.gen_labels(rng, N, cards, 0.05)
        f, p = g.selectors(labels, off, preds)
        fo, po, _ = orc.selectors(labels, off, preds)
        assert np.array_equal(f, fo) and np.array_equal(p, po)


@pytest.mark.parametrize("L", [64, 65])
def test_many_selectors(g, orc, L):
    """More rows than the compile's workgroups take at once; label tables that fit LDS and one label more."""
    rng = np.random.default_rng(L)
    cards = rng.choice([2, 16, 64], size=L)
    labels = synth.gen_labels(rng, 70, cards, 0.1)
    off, preds = synth.gen_preds(rng, 8192 * 32 + 33, cards, 0, 6, mmax=4)
    preds["op"][rng.integers(0, preds.shape[0], 100)] = 9
    fo, po, _ = orc.selectors(labels, off, preds)
    fg, pg = g.selectors(labels, off, preds)[:2]
    assert np.array_equal(fg, fo) and np.array_equal(pg, po)


@pytest.mark.parametrize("N,I,small", [(500, 32_768, True), (500, 32_769, False), (250, 262_144, True),
                                       (250, 262_145, False), (64, 1_048_576, True), (60, 1_048_577, False)])
def test_small_clusters_of_many_rows(g, orc, N, I, small):
    """A wavefront per row pays up to a number of rows that falls with their words, however few predicates they have."""
    import paper_2602_16100_amd as pc
    rng = np.random.default_rng(I)
    cards = rng.choice([2, 16, 64], size=8)
    labels = synth.gen_labels(rng, N, cards, 0.1)
    some_off, preds = synth.gen_preds(rng, 5000, cards, 0, 4, mmax=3)
    off = np.zeros(I + 1, np.int32)
    at = np.sort(rng.choice(I, 5000, replace=False))
    off[at + 1] = np.diff(some_off)
    off = np.cumsum(off, dtype=np.int64).astype(np.int32)
    ctx = pc.context()
    ctx.profile(True)
    f, p = g.selectors(labels, off, preds)
    used = ctx.profile_read()
    ctx.profile(False)
    assert ("k_sel_small" in used) == small
    fo, po, _ = orc.selectors(labels, off, preds)
    assert np.array_equal(f, fo) and np.array_equal(p, po)
