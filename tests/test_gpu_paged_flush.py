"""Paged triangle counts whose LDS counters are handed in while the count runs:
a crowd under the least flush limit, few bins (counters that fill up) and many
(the look at the fullest counter puts the flush off, or is left out), short steps and
whole-wavefront rows, positive and signed weights, against the CPU oracle bit
for bit."""
import re

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

N, L, RMAX = 6_000, 40.0, 4.0


def crowd():
    return synth.neyman_scott(N, 500, 1.0, L, 604)


def weights(signed):
    w = synth.uniform_values(N, 0.5, 1.0, 613)
    return w * np.where(np.arange(N) % 3 == 0, -1.0, 1.0) if signed else w


@pytest.fixture(scope="module")
def refs():
    """Oracle counts by (bins, signed), each worked out once."""
    kept = {}

    def get(nb, signed):
        if (nb, signed) not in kept:
            kept[nb, signed] = oracle.count_3pcf(crowd(), L, 0.0, RMAX, nb, weights=weights(signed))
        return kept[nb, signed]
    return get


@pytest.mark.parametrize("signed", [False, True], ids=["positive", "signed"])
@pytest.mark.parametrize("nb,look", [(2, "1"), (24, "1"), (24, "0")])
@pytest.mark.parametrize("glog", ["4", "6"])
def test_counts_across_flushes(monkeypatch, capfd, refs, glog, nb, look, signed):
    import paper_2607_06604_amd as gsn
    monkeypatch.setenv("GS_PGLOG", glog)
    monkeypatch.setenv("GS_FLUSH_LIMIT", "4096")   # (raised to two chunks of spokes)
    monkeypatch.setenv("GS_FLUSH_LOOK", look)
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    print("flushes", glog, nb, look, signed, flush=True)
    with gsn.Context(0) as ctx:
        g = ctx.build_graph(crowd(), L, 0.0, RMAX, nb, weights=weights(signed))
        capfd.readouterr()
        got = ctx.count_3pcf(g, weighted=True)
        err = capfd.readouterr().err
        g.free()
        g = ctx.build_graph(crowd(), L, 0.0, RMAX, nb)
        capfd.readouterr()
        plain = ctx.count_3pcf(g)
        err_plain = capfd.readouterr().err
        g.free()
    ref = refs(nb, signed)
    assert got.n_triangles == ref.n_triangles and np.array_equal(got.hist, ref.hist)
    assert got.wsum_int() == ref.wsum_int() and np.array_equal(plain.hist, ref.hist)
    events = [tuple(map(int, re.search(r"count3p: (\d+) flushes in mid-count, (\d+) put off", e).groups()))
              for e in (err, err_plain)]
    # weighted: two bins fill four counters, 24 bins spread over 2600
    assert events[0][1 if nb == 24 and look == "1" else 0] > 0
    assert events[1][0] > 0
