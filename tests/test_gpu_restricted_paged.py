"""Equilateral and mu-binned counts by the paged label table against the hash
kernel and the CPU oracle, bit for bit: hubs taken in rounds, flushes, mu
values at the bin edges (lattice points, planes seen edge on and face on),
separations that wrap and that do not, boxes where the float32 bins serve
and where they do not."""
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


def flat(r, weighted):
    return [r.hist, r.n_triangles] + ([r.wsum] if weighted else [])


def counts(ctx, g, nmu, weighted=False, anchors=None):
    e = ctx.count_3pcf_equilateral(g, weighted=weighted, anchors=anchors)
    m = ctx.count_3pcf_mu(g, nmu, weighted=weighted, anchors=anchors)
    return flat(e, weighted) + flat(m, weighted)


def same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def lattice():
    s = np.arange(12) * 1.0
    return np.stack(np.meshgrid(s, s, s, indexing="ij"), -1).reshape(-1, 3)


def sheet(axis):
    x = synth.uniform(1500, 20.0, 743)
    x[:, axis] = 7.25
    return x


CASES = [   # points, box, rmax, bins, mu bins, periodic
    ("uniform", lambda: synth.uniform(9000, 60.0, 741), 60.0, 5.0, 7, 5, True),
    ("crowd", lambda: np.mod(np.concatenate([20.0 + 4.0 * (synth.uniform(700, 1.0, 742) - 0.5),
                                             synth.uniform(3000, 40.0, 744)]), 40.0), 40.0, 4.2, 9, 4, True),
    ("survey", lambda: synth.neyman_scott(6000, 80, 1.0, 50.0, 745), 50.0, 3.0, 16, 3, False),
    ("lattice", lattice, 12.0, 1.8, 3, 2, True),
    ("face_on", lambda: sheet(2), 20.0, 1.7, 4, 6, True),
    ("edge_on", lambda: sheet(0), 20.0, 1.7, 4, 6, True),
    ("wraps", lambda: synth.uniform(500, 8.0, 746), 8.0, 2.9, 5, 64, True),
    ("just_no_wrap", lambda: synth.uniform(700, 8.0, 748), 8.0, 1.99, 5, 64, True),
    ("large_box", lambda: np.concatenate([900.0 + synth.uniform(2000, 12.0, 749), synth.uniform(2000, 1000.0, 750)]),
     1000.0, 3.95, 4, 7, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_paged_restricted(ctx, monkeypatch, case):
    name, mk, L, rmax, nb, nmu, periodic = case
    x = mk()
    w = synth.uniform_values(len(x), 0.5, 1.0, 747) * np.where(np.arange(len(x)) % 3 == 0, -1.0, 1.0)
    g = ctx.build_graph(x, L, 0.0, rmax, nb, weights=w, keep_coords=True, periodic=periodic)
    monkeypatch.setenv("GS_PAGED", "1")
    print("paged restricted", name, len(x), g.info().max_deg, flush=True)
    an = (len(x) // 5, len(x) // 2)
    got, part = counts(ctx, g, nmu, True), counts(ctx, g, nmu, True, an)
    plain = counts(ctx, g, nmu)
    monkeypatch.setenv("GS_FLUSH_LIMIT", "300000")
    assert same(counts(ctx, g, nmu, True), got) and same(counts(ctx, g, nmu), plain)
    monkeypatch.delenv("GS_FLUSH_LIMIT")
    monkeypatch.setenv("GS_PAGED", "0")
    assert same(counts(ctx, g, nmu, True), got) and same(counts(ctx, g, nmu, True, an), part)
    assert same(counts(ctx, g, nmu), plain)
    g.free()
    ref = oracle.count_3pcf_mu(x, L, 0.0, rmax, nb, nmu, periodic=periodic)
    assert plain[3] == ref.n_triangles and np.array_equal(plain[2], ref.hist)
