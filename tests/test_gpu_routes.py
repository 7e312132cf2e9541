"""Which kernel counts: plain and weighted triangle counts on both sides of the
lines in row length, bins and points. Each count is repeated by the other
kernel and equals it bit for bit."""
import numpy as np
import pytest

import synth

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
    (20_000, 12, 20, True, False, False),
    (20_000, 2.5, 10, False, True, False),
    (20_000, 2.5, 10, False, False, True),
    (20_000, 4, 10, True, True, True),
    (30_000, 20, 10, False, False, False),
    (30_000, 33, 10, False, False, False),
    (30_000, 39, 10, False, False, True),
    (30_000, 39, 10, False, True, False),
    (30_000, 46, 10, True, True, True),
    (30_000, 60, 18, False, False, False),
    (30_000, 60, 20, True, False, False),
    (30_000, 76, 20, True, False, True),
    (30_000, 76, 18, False, True, True),
    (30_000, 90, 24, False, False, False),
    (30_000, 120, 24, False, False, True),
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
