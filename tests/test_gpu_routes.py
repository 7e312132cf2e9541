"""Which kernel counts: plain and weighted triangle counts on both sides of the
lines in row length, bins and points, restricted counts and 6-edge counts
likewise. Each count is repeated by the other kernel and equals it bit for bit;
a restricted count leaves the schedule of the last full count in the timings."""
import numpy as np
import pytest

import synth
from tests import test_gpu_restricted_paged as restricted

pytestmark = pytest.mark.gpu

RMAX = 10.0


@pytest.fixture(scope="module")
def ctx():
    import paper_2607_06604_amd as gsn
    gsn.load()
    with gsn.Context(0) as c:
        yield c


def catalogue(n, row, nb, seed=821):
    """n uniform points with `row` forward neighbours each."""
    box = (n * 4.18879 * RMAX ** 3 / (2.0 * row)) ** (1.0 / 3.0)
    return synth.uniform(n, box, seed), box


def same(a, b):
    return (np.array_equal(a.hist, b.hist) and a.n_triangles == b.n_triangles
            and (a.wsum is None or np.array_equal(a.wsum, b.wsum)))


def took_paged(ctx, capfd, count):
    """The count's result and whether the paged kernel was launched for it."""
    capfd.readouterr()
    r = count()
    return r, "count3p launch" in capfd.readouterr().err


# points, row, bins, weighted, anchored -> paged
FULL = [
    (20_000, 12, 10, False, False, True),
    (20_000, 12, 20, False, False, True),
    (20_000, 10, 20, True, False, False),
    (20_000, 15, 20, True, False, True),
    (20_000, 2.5, 10, False, True, False),
    (20_000, 2.5, 10, False, False, True),
    (20_000, 4, 10, True, True, True),
    (40_000, 20, 10, False, False, True),
    (40_000, 20, 10, True, False, False),
    (50_000, 20, 10, False, False, False),
    (50_000, 32, 10, False, False, False),
    (50_000, 37, 10, False, False, True),
    (50_000, 39, 10, False, True, False),
    (50_000, 37, 10, True, True, True),
    (50_000, 31, 10, True, False, True),
    (50_000, 31, 15, True, False, False),
    (30_000, 40, 18, False, False, True),
    (30_000, 48, 18, False, True, False),
    (30_000, 48, 20, True, False, False),
    (30_000, 56, 20, True, False, True),
    (30_000, 56, 18, False, True, True),
    (110_000, 60, 20, False, False, False),
    (30_000, 60, 24, False, False, False),
    (30_000, 70, 24, False, False, True),
    (30_000, 60, 24, True, True, False),
    (30_000, 60, 24, True, False, True),
]


@pytest.mark.parametrize("case", FULL, ids=lambda c: "-".join(map(str, c)))
def test_full_counts(ctx, monkeypatch, capfd, case):
    n, row, nb, weighted, anchored, paged = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    x, box = catalogue(n, row, nb)
    w = synth.uniform_values(n, 0.5, 1.0, 822) if weighted else None
    g = ctx.build_graph(x, box, 0.0, RMAX, nb, weights=w)
    count = lambda: ctx.count_3pcf(g, weighted=weighted, anchors=(n // 5, n // 2) if anchored else None)
    print("routes", case, g.info().n_edges / n, flush=True)
    got, p = took_paged(ctx, capfd, count)
    assert p == paged and (ctx.timings().table_log2 == 0) == paged
    monkeypatch.setenv("GS_PAGED", "0" if paged else "1")
    other, p = took_paged(ctx, capfd, count)
    assert p != paged and same(got, other)
    g.free()


# points, row, bins, mu bins (0: equilateral), weighted, anchored -> paged
RESTRICTED = [
    (45_000, 42, 10, 0, False, False, False),
    (45_000, 55, 12, 0, False, False, False),
    (45_000, 75, 10, 0, False, False, True),
    (45_000, 75, 10, 0, True, True, True),
    (45_000, 75, 20, 0, False, False, False),
    (45_000, 110, 20, 0, False, True, True),
    (45_000, 110, 20, 0, True, False, False),
    (45_000, 180, 20, 0, True, False, True),
    (45_000, 180, 24, 0, True, False, False),
    (120_000, 31, 10, 0, False, False, True),
    (120_000, 31, 10, 5, False, False, True),
    (45_000, 39, 10, 5, False, False, False),
    (45_000, 50, 10, 5, False, False, True),
    (45_000, 50, 16, 5, False, False, False),
    (45_000, 65, 16, 5, False, False, True),
    (45_000, 65, 16, 2, False, False, False),
    (60_000, 45, 15, 10, False, False, True),
    (45_000, 75, 20, 5, False, False, True),
]


@pytest.mark.parametrize("case", RESTRICTED, ids=lambda c: "-".join(map(str, c)))
def test_restricted_counts(ctx, monkeypatch, capfd, case):
    n, row, nb, nmu, weighted, anchored, paged = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    x, box = catalogue(n, row, nb)
    w = synth.uniform_values(n, 0.5, 1.0, 822) if weighted else None
    g = ctx.build_graph(x, box, 0.0, RMAX, nb, weights=w, keep_coords=True)
    an = (n // 5, n // 2) if anchored else None
    count = lambda: (ctx.count_3pcf_mu(g, nmu, weighted=weighted, anchors=an) if nmu else
                     ctx.count_3pcf_equilateral(g, weighted=weighted, anchors=an))
    print("routes", case, g.info().n_edges, flush=True)
    monkeypatch.setenv("GS_PAGED", "0")
    ctx.count_3pcf(g, weighted=weighted)
    kept = ctx.timings()
    monkeypatch.delenv("GS_PAGED")
    got, p = took_paged(ctx, capfd, count)
    t = ctx.timings()
    assert p == paged
    for f in ("probes", "table_log2", "block", "group", "hash_load"):
        assert getattr(t, f) == getattr(kept, f), f
    monkeypatch.setenv("GS_PAGED", "0" if paged else "1")
    other, p = took_paged(ctx, capfd, count)
    assert p != paged and same(got, other)
    g.free()


@pytest.mark.parametrize("case", restricted.CASES, ids=[c[0] for c in restricted.CASES])
def test_forced_restricted_routes(ctx, monkeypatch, capfd, case):
    """GS_PAGED=1 sends every plain restricted count of these catalogues to the
    paged kernel, except in the box of one cell (few labels of a cell are
    neighbours, and the mu bins' separations wrap); 0 sends none."""
    name, mk, L, rmax, nb, nmu, periodic = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    g = ctx.build_graph(mk(), L, 0.0, rmax, nb, keep_coords=True, periodic=periodic)
    for forced in ("1", "0"):
        monkeypatch.setenv("GS_PAGED", forced)
        print("forced", name, forced, flush=True)
        e = took_paged(ctx, capfd, lambda: ctx.count_3pcf_equilateral(g))
        m = took_paged(ctx, capfd, lambda: ctx.count_3pcf_mu(g, nmu))
        assert e[1] == m[1] == (forced == "1" and name != "wraps")
    g.free()


# points, row, bins, weighted -> adjacency bytes
SIX = [
    (6_000, 20, 7, False, True),
    (6_000, 12, 8, False, True),
    (6_000, 12, 8, True, False),
    (6_000, 16, 8, False, False),
    (6_000, 18, 10, False, True),
    (6_000, 18, 10, True, False),
]


@pytest.mark.parametrize("case", SIX, ids=lambda c: "-".join(map(str, c)))
def test_six_edge_counts(ctx, monkeypatch, capfd, case):
    n, row, nb, weighted, by_bytes = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    x, box = catalogue(n, row, nb)
    w = synth.uniform_values(n, 0.5, 1.0, 822) if weighted else None
    g = ctx.build_graph(x, box, 0.0, RMAX, nb, weights=w, keep_coords=True)
    print("six", case, g.info().max_deg, flush=True)
    out = []
    for mode in (None, "0" if by_bytes else "1"):
        if mode:
            monkeypatch.setenv("GS_MATRIX4", mode)
        capfd.readouterr()
        out.append(ctx.count_4pcf_full(g, weighted=weighted))
        assert ("count4m" in capfd.readouterr().err) == (by_bytes if mode is None else not by_bytes)
    a, b = out
    assert np.array_equal(a.hist, b.hist) and a.n_cliques == b.n_cliques
    assert not weighted or np.array_equal(a.wsum, b.wsum)
    g.free()


# crowd, points in all, kind, bins, weighted -> adjacency bytes take part
CLASSES = [
    (470, 3_470, "parity", 8, False, False),
    (470, 4_500, "parity", 8, False, True),
    (470, 4_500, "parity", 8, True, False),
    (300, 900, "parity", 8, False, False),
    (300, 900, "pixel", 8, False, True),
    (300, 1_500, "parity", 1, True, False),
    (300, 1_500, "parity", 5, True, True),
    (300, 3_000, "parity", 1, True, True),
    (600, 1_200, "six", 4, False, False),
    (470, 6_000, "pixel", 8, False, False),
    (600, 2_400, "six", 4, True, False),
    (600, 2_800, "six", 4, False, True),
]


@pytest.mark.parametrize("case", CLASSES, ids=lambda c: "-".join(map(str, c)))
def test_degree_classes(ctx, monkeypatch, capfd, case):
    """Few hubs take one kernel, more are split by degree; both equal each
    kernel on its own (GS_MATRIX4=0) and the forced split (1)."""
    crowd, n, kind, nb, weighted, split = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    box = 100.0
    x = np.concatenate([np.mod(50.0 + 4.0 * (synth.uniform(crowd, 1.0, 823) - 0.5), box), synth.uniform(n - crowd, box, 824)])
    w = synth.uniform_values(n, 0.5, 1.0, 825) if weighted else None
    g = ctx.build_graph(x, box, 0.0, RMAX, nb, weights=w, keep_coords=True)
    assert g.info().max_deg >= crowd - 1
    print("classes", case, g.info().max_deg, flush=True)
    out = []
    for mode in (None, "0", "1"):
        if mode:
            monkeypatch.setenv("GS_MATRIX4", mode)
        capfd.readouterr()
        if kind == "six":
            r = ctx.count_4pcf_full(g, weighted=weighted)
            vals = [r.hist, r.n_cliques]
        else:
            r = ctx.count_4pcf_pixel(g) if kind == "pixel" else ctx.count_4pcf_parity(g, weighted=weighted)
            vals = [r.even, r.pos, r.neg, r.n_cliques]
        out.append(vals + ([r.wsum] if weighted else []))
        assert ("count4m" in capfd.readouterr().err) == (split if mode is None else mode == "1")
    assert all(np.array_equal(a, b) for o in out[1:] for a, b in zip(out[0], o))
    g.free()


# catalogues, points each, row, bins -> paged
BATCHES = [(2, 8_000, 8, 20, True), (8, 8_000, 8, 20, False), (8, 8_000, 8, 18, True), (2, 30_000, 8, 18, True),
           (2, 30_000, 50, 20, False), (2, 30_000, 70, 20, True)]


@pytest.mark.parametrize("case", BATCHES, ids=lambda c: "-".join(map(str, c)))
def test_batches(ctx, monkeypatch, capfd, case):
    count, n, row, nb, paged = case
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    gs = []
    for k in range(count):
        x, box = catalogue(n, row, nb, 830 + k)
        gs.append(ctx.build_graph(x, box, 0.0, RMAX, nb))
    print("batch", case, flush=True)
    got, p = took_paged(ctx, capfd, lambda: ctx.count_3pcf_batch(gs))
    assert p == paged
    monkeypatch.setenv("GS_PAGED", "0" if paged else "1")
    other, p = took_paged(ctx, capfd, lambda: ctx.count_3pcf_batch(gs))
    assert p != paged and all(np.array_equal(a.hist, b.hist) and a.n_triangles == b.n_triangles for a, b in zip(got, other))
    for g in gs:
        g.free()


# points, row, weighted -> threads per work group (the LDS plan ties)
BLOCKS = [(15_000, 230, True, 512), (15_000, 180, True, 256), (36_000, 230, True, 256), (15_000, 600, False, 512)]


@pytest.mark.parametrize("case", BLOCKS, ids=lambda c: "-".join(map(str, c)))
def test_group_size_of_few_long_hubs(ctx, monkeypatch, case):
    n, row, weighted, block = case
    x, box = catalogue(n, row, 10)
    w = synth.uniform_values(n, 0.5, 1.0, 826) if weighted else None
    g = ctx.build_graph(x, box, 0.0, RMAX, 10, weights=w)
    print("block", case, flush=True)
    got = ctx.count_3pcf(g, weighted=weighted)
    t = ctx.timings()
    assert t.table_log2 == 0 and t.block == block
    monkeypatch.setenv("GS_PBLOCK", "256" if block == 512 else "512")
    other = ctx.count_3pcf(g, weighted=weighted)
    assert ctx.timings().block != block and same(got, other)
    g.free()
