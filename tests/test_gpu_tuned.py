"""Tuned schedules stay with the kernel they were timed on: after tuning a
weighted catalogue of long rows, counts that cannot take all of the schedule
(anchors go with fewer threads) still run the paged label table, and the hash
walk plans as if nothing had been tuned. Counts equal those of an untuned
context bit for bit."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

L, RMAX, NB = 12.0, 4.0, 20


def clump(n, seed):
    """n points that are all neighbours (a cube of side 2 inside one cell)."""
    return 5.0 + synth.uniform(n, 2.0, seed)


def same(a, b):
    return np.array_equal(a.hist, b.hist) and np.array_equal(a.wsum, b.wsum) and a.n_triangles == b.n_triangles


# 9100: a hash table of 2^15 slots, which leaves LDS for no larger step table
# than the hash walk's own choice
@pytest.mark.parametrize("n", [2_600, 9_100])
def test_anchored_counts_after_tuning_long_rows(monkeypatch, n):
    import paper_2607_06604_amd as gsn
    x, w = clump(n, 801), synth.uniform_values(n, 0.5, 1.0, 802)
    an = (1, 4)
    want = sum(math.comb(n - 1 - i, 2) for i in range(*an))
    print("tuned", n, flush=True)
    with gsn.Context(0) as c, gsn.Context(0) as plain:
        g = c.build_graph(x, L, 0.0, RMAX, NB, weights=w)
        assert g.info().n_edges == math.comb(n, 2)
        first = plain.count_3pcf(g, weighted=True, anchors=an)
        block = plain.timings().block
        assert plain.timings().table_log2 == 0 and first.n_triangles == want
        plan = c.tune_3pcf(g, weighted=True)
        print(plan, flush=True)
        assert plan["hash_load"] == 5 and plan["trials"] >= 2
        got = c.count_3pcf(g, weighted=True, anchors=an)
        t = c.timings()
        assert t.table_log2 == 0 and t.block == block, "the tuned schedule took the paged table away"
        assert same(got, first)
        if n < 5_000:
            assert same(c.count_3pcf(g, weighted=True), plain.count_3pcf(g, weighted=True))
        monkeypatch.setenv("GS_PAGED", "0")
        assert same(c.count_3pcf(g, weighted=True, anchors=an), first)
        assert c.timings().table_log2 > 0
        g.free()


def test_long_rows_report_lone_hubs(monkeypatch):
    """Whole-wavefront rows take hubs one at a time: the timings say so."""
    import paper_2607_06604_amd as gsn
    x, w = clump(1_500, 803), synth.uniform_values(1_500, 0.5, 1.0, 804)
    monkeypatch.setenv("GS_PGLOG", "6")
    with gsn.Context(0) as c:
        for weights in (w, None):
            g = c.build_graph(x, L, 0.0, RMAX, NB, weights=weights)
            for an in (None, (10, 900)):
                print("lone hubs", weights is not None, an, flush=True)
                c.count_3pcf(g, weighted=weights is not None, anchors=an)
                t = c.timings()
                assert t.table_log2 == 0 and t.group == 1
            g.free()
