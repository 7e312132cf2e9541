"""Weighted and anchored counts of long rows keep packed hub rows in device
memory: they fit the context's budget beside the graph (host-tiled: beside its
windows, which leave room for them), or the count takes steps that need none.
Counts are the same bit for bit."""
import math
import re

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def step_log(capfd):
    """log2 of the entries per step of the last planned count."""
    return int(re.findall(r"count3p plan: .* glog (\d+)", capfd.readouterr().err)[-1])


def same(a, b):
    return np.array_equal(a.hist, b.hist) and np.array_equal(a.wsum, b.wsum) and a.n_triangles == b.n_triangles


def test_resident_rows_fit_the_budget(monkeypatch, capfd):
    import paper_2607_06604_amd as gsn
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    n = 3_000
    x, w = 5.0 + synth.uniform(n, 2.0, 841), synth.uniform_values(n, 0.5, 1.0, 842)   # all neighbours
    out = []
    for spare in (None, 64 * MIB, 4 * MIB):
        with gsn.Context(0, budget_bytes=held + spare if spare else 0) as c:
            g = c.build_graph(x, 12.0, 0.0, 4.0, 12, weights=w)
            info = g.info()
            held = info.device_bytes
            assert info.n_windows == 1
            print("budget", spare, held, flush=True)
            for an in (None, (10, 1200)):
                out.append(c.count_3pcf(g, weighted=True, anchors=an))
                assert step_log(capfd) == (5 if spare == 4 * MIB else 6)
            g.free()
    assert out[0].n_triangles == math.comb(n, 3)
    assert all(same(out[k], out[k + 2]) for k in range(4))


def test_windows_leave_room_for_the_rows(monkeypatch, capfd):
    import paper_2607_06604_amd as gsn
    monkeypatch.setenv("GS_PLAN_LOG", "1")
    n, L, rmax = 40_000, 68.0, 15.8     # about 1050 entries a row, 210 MB of them
    x, w = synth.uniform(n, L, 843), synth.uniform_values(n, 0.5, 1.0, 844)
    out = []
    for budget, steps in ((0, 6), (140 * MIB, 6), (60 * MIB, 5)):
        with gsn.Context(0, budget_bytes=budget) as c:
            g = c.build_graph(x, L, 0.0, rmax, 9, weights=w)
            info = g.info()
            print("windows", budget, info.n_windows, info.n_edges / n, info.max_deg, flush=True)
            assert (info.n_windows == 1) == (budget == 0) and info.n_edges >= 1000 * n
            capfd.readouterr()
            out.append(c.count_3pcf(g, weighted=True))
            assert step_log(capfd) == steps
            g.free()
    assert same(out[0], out[1]) and same(out[0], out[2])
