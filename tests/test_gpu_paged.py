"""Triangle counts through the paged label table (csrc/count3p.hip) against the
CPU oracle, bit for bit, at the sizes where it can go wrong: tables of a few
pages (rows in rounds of labels, groups split), every step length and the
whole-wavefront rows, 32-bit and 64-bit row offsets, boxes of one cell to many
(rows that wrap), long rows, signed and wide weights, anchors, tiles, batches,
forced flushes."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2607_06604_amd as gsn
    gsn.load()
    with gsn.Context(0) as c:
        yield c


PLANS = [
    {},
    {"GS_PTAB": "1024"},                                     # rounds of labels, groups of one
    {"GS_PTAB": "3072", "GS_PBLOCK": "512", "GS_PGLOG": "5"},
    {"GS_PGLOG": "6"},                                       # whole-wavefront rows, packed hub rows
    {"GS_PGLOG": "6", "GS_PTAB": "1024", "GS_PBLOCK": "256"},
    {"GS_PGLOG": "6", "GS_PBLOCK": "768", "GS_PORDER": "0"},
    {"GS_PMODE": "1", "GS_GROUP": "3"},
    {"GS_WIDE": "1"},
    {"GS_FLUSH_LIMIT": "4096"},                              # (raised to two chunks of spokes)
]

# (catalogue, box, rmax, bins)
SHAPES = [
    (lambda: synth.neyman_scott(9_000, 40, 1.5, 60.0, 601), 60.0, 3.5, 9),      # many cells, short rows
    (lambda: synth.uniform(4_000, 12.0, 602), 12.0, 3.9, 5),                    # three cells an axis: all wrap
    (lambda: synth.uniform(1_500, 9.0, 603), 9.0, 4.4, 17),                     # one cell; table counters
    (lambda: synth.neyman_scott(6_000, 500, 1.0, 40.0, 604), 40.0, 4.0, 24),    # crowded: rows of hundreds
]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("plan", PLANS, ids=lambda p: "-".join(f"{k[3:].lower()}{v}" for k, v in p.items()) or "built-in")
def test_paged_counts_match_oracle(ctx, monkeypatch, plan, shape):
    mk, L, rmax, nb = SHAPES[shape]
    x = mk()
    print("paged", plan, shape, flush=True)
    monkeypatch.setenv("GS_PAGED", "1")   # also where short rows would go to the hash table
    for k, v in plan.items():
        monkeypatch.setenv(k, v)
    w = synth.uniform_values(len(x), 0.5, 1.0, 610 + shape)
    g = ctx.build_graph(x, L, 0.0, rmax, nb, weights=w)
    got = ctx.count_3pcf(g, weighted=True)
    assert ctx.timings().table_log2 == 0, "the hash table counted"
    part = ctx.count_3pcf(g, weighted=True, anchors=(len(x) // 7, len(x) // 2))
    g.free()
    ref = oracle.count_3pcf(x, L, 0.0, rmax, nb, weights=w)
    assert got.n_triangles == ref.n_triangles and np.array_equal(got.hist, ref.hist)
    assert got.wsum_int() == ref.wsum_int() and np.array_equal(got.whist, ref.whist())
    refp = oracle.count_3pcf(x, L, 0.0, rmax, nb, weights=w, anchors=(len(x) // 7, len(x) // 2))
    assert part.n_triangles == refp.n_triangles and part.wsum_int() == refp.wsum_int()
    # unweighted, alone and in a batch
    g = ctx.build_graph(x, L, 0.0, rmax, nb)
    plain = ctx.count_3pcf(g)
    anch = ctx.count_3pcf(g, anchors=(len(x) // 7, len(x) // 2))
    bat = ctx.count_3pcf_batch([g, g])
    g.free()
    assert np.array_equal(plain.hist, ref.hist) and np.array_equal(anch.hist, refp.hist)
    assert np.array_equal(bat[0].hist, ref.hist) and np.array_equal(bat[1].hist, ref.hist)


@pytest.mark.parametrize("glog", ["4", "6"])
def test_paged_general_weights_and_tiles(ctx, monkeypatch, glog):
    """Signed weights, magnitudes far enough apart for terms beyond 2^63, in
    survey geometry, resident and host-tiled."""
    monkeypatch.setenv("GS_PGLOG", glog)
    x = synth.neyman_scott(5_000, 100, 1.2, 40.0, 621)
    u = synth.uniform_values(len(x), 0.0, 1.0, 622)
    w = (0.5 + u) * np.where(u < 0.4, -1.0, 1.0) * np.where((u * 16) % 1 < 0.3, 900.0, 1.0)
    L, rmax, nb = 40.0, 3.3, 11
    ref = oracle.count_3pcf(x, L, 0.0, rmax, nb, weights=w, periodic=False)
    for windows in (0, 3):
        print("paged general weights", glog, windows, flush=True)
        if windows:
            monkeypatch.setenv("GS_WINDOWS", str(windows))
        g = ctx.build_graph(x, L, 0.0, rmax, nb, weights=w, periodic=False)
        got = ctx.count_3pcf(g, weighted=True)
        assert ctx.timings().table_log2 == 0
        g.free()
        assert np.array_equal(got.hist, ref.hist) and got.wsum_int() == ref.wsum_int()
