"""4-clique counts from adjacency bytes (k_count4m) against the bitset kernel
and the CPU oracle, bit for bit: hubs of every degree class in one catalogue
(a crowd whose forward degrees run from 0 to beyond the largest class), the
1024-lane form alone, every kind, weighted and anchored, tiles, ragged rows
around the 64-candidate and 16-entry windows."""
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


def counts(ctx, g, nb, anchors=None, weighted=True):
    p = ctx.count_4pcf_parity(g, anchors=anchors, weighted=weighted)
    out = [p.even, p.pos, p.neg, p.n_cliques, ctx.count_4pcf_parity(g, anchors=anchors).even]
    x = ctx.count_4pcf_pixel(g, anchors=anchors)
    out += [x.even, x.pos, x.neg, x.n_cliques]
    s = ctx.count_4pcf_full(g, anchors=anchors, weighted=weighted)
    out += [s.hist, s.n_cliques, ctx.count_4pcf_full(g, anchors=anchors).hist]
    if weighted:
        out += [p.wsum, s.wsum]
    return out


def same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


# bins: 6-edge table and counters in LDS (4), counters in LDS (6), global (9);
# 17: no ordered-triple table in the parity kinds
@pytest.mark.parametrize("nb", [4, 6, 9, 17])
def test_every_degree_class_matches_the_bitset_kernel(ctx, monkeypatch, nb):
    L, rmax = 40.0, 4.0
    crowd = np.mod(20.0 + 0.9 * (synth.uniform(470, 1.0, 701) - 0.5) * 4.0, L)      # degrees 0..469
    x = np.concatenate([crowd, synth.neyman_scott(2_500, 130, 1.0, L, 702), synth.uniform(500, L, 703)])
    w = synth.uniform_values(len(x), 0.5, 1.0, 704) * np.where(np.arange(len(x)) % 3 == 0, -1.0, 1.0)
    g = ctx.build_graph(x, L, 0.0, rmax, nb, weights=w, keep_coords=True)
    assert g.info().max_deg > 440
    if nb > 12:   # (6-edge counts take at most 12 bins)
        run = lambda an=None: [v for k in (ctx.count_4pcf_parity(g, anchors=an, weighted=True), ctx.count_4pcf_pixel(g, anchors=an))
                               for v in (k.even, k.pos, k.neg, k.n_cliques)]
    else:
        run = lambda an=None: counts(ctx, g, nb, an)
    an = (200, 1700)
    got, part = run(), run(an)
    for mode in ("0", "2"):
        print("matrix4", nb, mode, flush=True)
        monkeypatch.setenv("GS_MATRIX4", mode)
        assert same(run(), got) and same(run(an), part)
    monkeypatch.delenv("GS_MATRIX4")
    g.free()
    # two anchors of the crowd against the oracle
    ref = oracle.count_4pcf_parity(x, L, 0.0, rmax, nb, anchors=(100, 102))
    g = ctx.build_graph(x, L, 0.0, rmax, nb, keep_coords=True)
    p = ctx.count_4pcf_parity(g, anchors=(100, 102))
    g.free()
    assert p.n_cliques == ref.n_cliques and np.array_equal(p.even, ref.even)
    assert np.array_equal(p.pos, ref.pos) and np.array_equal(p.neg, ref.neg)


def test_tiles_and_noalloc(ctx, monkeypatch):
    L, rmax, nb = 30.0, 3.0, 7
    x = synth.neyman_scott(4_000, 150, 0.8, L, 711)
    g = ctx.build_graph(x, L, 0.0, rmax, nb, keep_coords=True)
    ref = ctx.count_4pcf_parity(g)
    again = ctx.count_4pcf_parity(g, noalloc=True)
    six = ctx.count_4pcf_full(g)
    g.free()
    monkeypatch.setenv("GS_WINDOWS", "3")
    t = ctx.build_graph(x, L, 0.0, rmax, nb, keep_coords=True)
    print("matrix4 tiles", flush=True)
    tiled, six_t = ctx.count_4pcf_parity(t), ctx.count_4pcf_full(t)
    t.free()
    for a in (again, tiled):
        assert a.n_cliques == ref.n_cliques and np.array_equal(a.even, ref.even)
        assert np.array_equal(a.pos, ref.pos) and np.array_equal(a.neg, ref.neg)
    assert np.array_equal(six.hist, six_t.hist) and six.n_cliques == ref.n_cliques
