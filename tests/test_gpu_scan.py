"""Graph builds at the edges of the prefix sums' tiles (2048 values): points
and cells just below, at and above one tile, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


# points, cells per axis (12^3 = 1728 cells, 13^3 = 2197)
@pytest.mark.parametrize("n,nc", [(1, 3), (2, 12), (2047, 12), (2048, 13), (2049, 12), (4097, 13)])
def test_build_at_scan_tile_edges(n, nc):
    import paper_2607_06604_amd as gsn
    L, rmax = 40.0, 40.0 / (nc + 0.5)
    x = synth.uniform(n, L, 760 + n % 97)
    print("scan tiles", n, nc, flush=True)
    with gsn.Context(0) as ctx:
        g = ctx.build_graph(x, L, 0.0, rmax, 4)
        info = g.info()
        t = ctx.count_3pcf(g)
        g.free()
    ref = oracle.count_3pcf(x, L, 0.0, rmax, 4)
    d = x[:, None, :] - x[None, :, :]
    d -= L * np.round(d / L)
    pairs = (int(((d * d).sum(-1) < rmax * rmax).sum()) - n) // 2
    assert info.n_edges == pairs
    assert t.n_triangles == ref.n_triangles and np.array_equal(t.hist, ref.hist)
