"""The work this library is timed on: catalogues through the public entry points.

Each case is one call pattern of a clustering analysis -- build the r < rmax
graph of a catalogue and count on it, or hand catalogues to the estimators or
the server -- over the sizes such an analysis meets, from a 20 000 point test
box to a quarter of a million points with 150 Mpc/h reach. `listed` gives the
fixed cases, `draw` further ones of the same ranges.

A case: "kind" (the call pattern, see `run`), "n" points in a cube of side
"box", "rmax", "nbins", and the options of that kind.
"""
from __future__ import annotations

import math
import time

import numpy as np
import torch

import paper_2607_06604_amd as gsn

PER_BLOB, SIGMA = 50, 3.0       # Neyman-Scott clusters: points and width (Mpc/h)


def listed():
    return [
        # the smallest everyday call: a 20 000 point box from host memory
        # (launches, copies and host work weigh most)
        dict(name="uniform_20k", kind="tri", n=20_000, box=250.0, rmax=20.0, nbins=10, field="uniform",
             weighted=False, host=True),
        # one clustered survey-sized catalogue, resident coordinates
        dict(name="clustered_1m", kind="tri", n=1_000_000, box=1000.0, rmax=30.0, nbins=15, field="clustered",
             weighted=False, host=False),
        # BAO-scale reach: thousands of neighbours per point, float64 weights
        dict(name="bao_weighted", kind="tri", n=250_000, box=1000.0, rmax=150.0, nbins=20, field="lognormal",
             weighted=True, host=False),
        # parity-decomposed 4-point counts of a clustered catalogue
        dict(name="parity4", kind="parity", n=200_000, box=400.0, rmax=20.0, nbins=8, weighted=False),
        # full 6-edge 4-point configurations (276 of them)
        dict(name="full6", kind="six", n=200_000, box=400.0, rmax=20.0, nbins=4, weighted=False),
        # parity by direction pixels
        dict(name="pixel4", kind="pixel", n=100_000, box=317.48, rmax=20.0, nbins=8, weighted=False),
        # restricted and anisotropic triangles of one graph
        dict(name="equilateral_mu", kind="restricted", n=500_000, box=793.7, rmax=30.0, nbins=15, nmu=5),
        # survey geometry, signed data-minus-random weights, one shard of the
        # points (anchor range) and the pair sums beside it; odd sizes
        dict(name="survey_shard", kind="survey", n=150_001, box=531.0, rmax=33.0, nbins=13),
        # several resident catalogues of uneven size in one launch
        dict(name="batch_6", kind="batch", n=100_000, box=600.0, rmax=40.0, nbins=10, count=6),
        # a burst of requests to the server
        dict(name="serve_12", kind="serve", n=100_000, box=600.0, rmax=40.0, nbins=10, count=12),
        # the estimators: data and randoms from host memory
        dict(name="zeta3_small", kind="zeta3", n=3_000, box=125.0, rmax=20.0, nbins=8),
        dict(name="zeta4", kind="zeta4", n=40_000, box=294.7, rmax=20.0, nbins=4),
    ]


def draw(rng):
    def logu(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    kind = rng.choice(["tri", "tri", "tri", "bao", "parity", "six", "pixel", "restricted", "survey", "batch",
                       "serve", "zeta3", "zeta4"])
    if kind == "tri":
        n = int(logu(2_000, 1_000_000))
        box = round(10.0 * n ** (1.0 / 3.0) * rng.uniform(0.9, 1.4), 2)
        return dict(kind="tri", n=n, box=box, rmax=round(min(rng.uniform(10.0, 30.0), 0.45 * box), 2),
                    nbins=rng.randint(3, 20), field=rng.choice(["uniform", "clustered"]),
                    weighted=rng.random() < 0.3, host=rng.random() < 0.3)
    if kind == "bao":
        n = int(logu(20_000, 240_000))
        box = round((n / 2.5e-4) ** (1.0 / 3.0) * rng.uniform(1.0, 1.1), 1)
        return dict(kind="tri", n=n, box=box, rmax=round(min(rng.uniform(60.0, 150.0), 0.45 * box), 1),
                    nbins=rng.randint(8, 22), field="lognormal", weighted=rng.random() < 0.7, host=False)
    if kind in ("parity", "six", "pixel"):
        n = int(logu(5_000, 200_000 if kind != "pixel" else 100_000))
        box = round(400.0 * (n / 200_000.0) ** (1.0 / 3.0) * rng.uniform(1.0, 1.2), 2)
        return dict(kind=kind, n=n, box=box, rmax=round(min(rng.uniform(9.0, 20.0), 0.45 * box), 2),
                    nbins=rng.randint(3, 6) if kind == "six" else rng.randint(3, 12),
                    weighted=kind != "pixel" and rng.random() < 0.4)
    if kind == "restricted":
        n = int(logu(5_000, 500_000))
        box = round(10.0 * n ** (1.0 / 3.0) * rng.uniform(1.0, 1.4), 2)
        return dict(kind=kind, n=n, box=box, rmax=round(min(rng.uniform(10.0, 30.0), 0.45 * box), 2),
                    nbins=rng.randint(4, 15), nmu=rng.randint(2, 10))
    if kind == "survey":
        n = int(logu(5_000, 150_000))
        box = round(10.0 * n ** (1.0 / 3.0) * rng.uniform(1.0, 1.4), 2)
        return dict(kind=kind, n=n, box=box, rmax=round(rng.uniform(10.0, 35.0), 2), nbins=rng.randint(4, 18))
    if kind in ("batch", "serve"):
        return dict(kind=kind, n=int(logu(50_000, 140_000)), box=600.0, rmax=round(rng.uniform(20.0, 40.0), 1),
                    nbins=rng.randint(5, 12), count=rng.randint(2, 6 if kind == "batch" else 12))
    n = int(logu(1_000, 60_000 if kind == "zeta3" else 30_000))
    box = round((2.0 * n / 3.2e-3) ** (1.0 / 3.0) * rng.uniform(1.0, 1.2), 2)
    return dict(kind=kind, n=n, box=box, rmax=round(min(rng.uniform(9.0, 20.0), 0.45 * box), 2),
                nbins=rng.randint(3, 12) if kind == "zeta3" else rng.randint(2, 5))


# ---------------------------------------------------------------- inputs ---

def _inside(x, box):
    x = np.mod(x, box)
    x[x >= box] = 0.0
    return x


def _uniform(n, box, r):
    return _inside(r.random((n, 3)) * box, box)


def _clustered(n, box, r):
    centres = r.random(((n + PER_BLOB - 1) // PER_BLOB, 3)) * box
    x = np.repeat(centres, PER_BLOB, axis=0)[:n]
    return _inside(x + r.normal(0.0, SIGMA, (n, 3)), box)


def _lognormal(n, box, r, smooth=20.0, spread=0.5):
    m = max(8, int(round(128 * box / 2000.0)))
    k = 2.0 * np.pi * np.fft.fftfreq(m, box / m)
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    g = np.fft.ifftn(np.fft.fftn(r.normal(size=(m, m, m))) * np.exp(-0.5 * k2 * smooth ** 2)).real
    g = (g - g.mean()) * (spread / g.std())
    rho = np.exp(g).ravel()
    cell = r.choice(m ** 3, size=n, p=rho / rho.sum())
    x = np.stack(np.unravel_index(cell, (m, m, m)), axis=1) + r.random((n, 3))
    return _inside(x * (box / m), box)


FIELDS = {"uniform": _uniform, "clustered": _clustered, "lognormal": _lognormal}


def _catalogue_sizes(case):
    """Uneven sizes around n, from half to twice."""
    c = case["count"]
    return [int(case["n"] * 2.0 ** (2.0 * k / max(1, c - 1) - 1.0)) for k in range(c)]


def _catalogues(case, r):
    return [(_clustered if k % 2 == 0 else _uniform)(n, case["box"], r)
            for k, n in enumerate(_catalogue_sizes(case))]


def _inputs(case, seed):
    """Host arrays of the case's catalogue(s), from the seed alone."""
    r = np.random.default_rng(seed)
    kind, n, box = case["kind"], case["n"], case["box"]
    if kind == "tri":
        return dict(x=FIELDS[case["field"]](n, box, r), w=r.random(n) + 0.5 if case["weighted"] else None)
    if kind in ("parity", "six", "pixel"):
        return dict(x=_clustered(n, box, r), w=r.random(n) + 0.5 if case["weighted"] else None)
    if kind == "restricted":
        return dict(x=_clustered(n, box, r), w=None)
    if kind == "survey":
        half = n // 2
        x = np.concatenate([_clustered(half, box, r), _uniform(n - half, box, r)])
        w = np.concatenate([(r.random(half) + 0.5) / half, -(r.random(n - half) + 0.5) / (n - half)])
        return dict(x=x, w=w)
    if kind in ("batch", "serve"):
        return dict(cats=_catalogues(case, r))
    return dict(data=_clustered(n, box, r), wd=r.random(n) + 0.5, rand=_uniform(n, box, r), wr=r.random(n) + 0.5)


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case, ctx=gsn.Context(0))
    kind = case["kind"]
    if kind in ("parity", "six", "pixel", "restricted", "survey") or (kind == "tri" and not case["host"]):
        s["x"] = torch.from_numpy(s["x"]).to("cuda:0")
        if s["w"] is not None:
            s["w"] = torch.from_numpy(s["w"]).to("cuda:0")
        torch.cuda.synchronize()
    if kind == "batch":
        s["graphs"] = [s["ctx"].build_graph(x, case["box"], 0.0, case["rmax"], case["nbins"]) for x in s["cats"]]
    return s


# ------------------------------------------------------------------- run ---

def run(s):
    c, ctx = s["case"], s["ctx"]
    kind, box, rmax, nb = c["kind"], c["box"], c["rmax"], c["nbins"]
    if kind == "tri":
        g = ctx.build_graph(s["x"], box, 0.0, rmax, nb, weights=s["w"])
        t = ctx.count_3pcf(g, weighted=c["weighted"])
        g.free()
        out = dict(hist=t.hist, n=t.n_triangles)
        if c["weighted"]:
            out.update(wsum=t.wsum, whist=t.whist, wscale=t.wscale)
        return out
    if kind in ("parity", "six", "pixel"):
        g = ctx.build_graph(s["x"], box, 0.0, rmax, nb, weights=s["w"], keep_coords=True)
        if kind == "six":
            q = ctx.count_4pcf_full(g, weighted=c["weighted"])
            out = dict(hist=q.hist, n=q.n_cliques)
        else:
            q = (ctx.count_4pcf_pixel(g) if kind == "pixel"
                 else ctx.count_4pcf_parity(g, weighted=c["weighted"]))
            out = dict(even=q.even, pos=q.pos, neg=q.neg, n=q.n_cliques)
        g.free()
        if c["weighted"]:
            out.update(wsum=q.wsum, wscale=q.wscale)
        return out
    if kind == "restricted":
        g = ctx.build_graph(s["x"], box, 0.0, rmax, nb, keep_coords=True)
        e = ctx.count_3pcf_equilateral(g)
        m = ctx.count_3pcf_mu(g, c["nmu"])
        g.free()
        return dict(equilateral=e.hist, ne=e.n_triangles, mu=m.hist, nm=m.n_triangles)
    if kind == "survey":
        g = ctx.build_graph(s["x"], box, 0.0, rmax, nb, weights=s["w"], periodic=False)
        p = ctx.pair_sums(g, weighted=True)
        t = ctx.count_3pcf(g, anchors=(c["n"] // 4, c["n"] // 2), weighted=True)
        g.free()
        return dict(pairs=p.pairs, psum=p.wsum, hist=t.hist, wsum=t.wsum, whist=t.whist, n=t.n_triangles)
    if kind == "batch":
        return [dict(hist=t.hist, n=t.n_triangles) for t in ctx.count_3pcf_batch(s["graphs"])]
    if kind == "serve":
        tickets = [ctx.submit(x, box, 0.0, rmax, nb) for x in s["cats"]]
        done = {}
        while len(done) < len(tickets):
            for k, t in enumerate(tickets):
                if k not in done:
                    r = ctx.poll(t, nb)
                    if r is not None:
                        done[k] = r
            time.sleep(0.0002)
        return [dict(hist=done[k]["hist"], n=done[k]["n_triangles"]) for k in range(len(tickets))]
    if kind == "zeta3":
        z = gsn.compute_3pcf(s["data"], s["wd"], s["rand"], s["wr"], 0.0, rmax, nb, box, ctx=ctx)
        return dict(zeta=z.zeta, nnn=z.NNN, rrr=z.RRR)
    z = gsn.compute_4pcf(s["data"], s["wd"], s["rand"], s["wr"], 0.0, rmax, nb, box, ctx=ctx)
    return dict(even=z.zeta_even, odd=z.zeta_odd, nnnn=z.nnnn_even, rrrr=z.rrrr_even, conn=z.zeta_even_conn,
                z6=z.zeta6, z6c=z.zeta6_conn, xi=z.xi)


# ------------------------------------------------------------------ work ---

def _tuples(n, box, rmax, blob_share):
    """Expected pairs, triangles and 4-cliques: Poisson background (a third
    point closes a triangle of two neighbours with probability 15/32, a
    4-clique a little over a sixth) plus the clusters' own tuples."""
    deg = n * 4.0 / 3.0 * math.pi * rmax ** 3 / box ** 3
    f = blob_share * min(1.0, (rmax / (4.0 * SIGMA)) ** 2)
    m = PER_BLOB * f
    pairs = n * (deg + m) / 2.0
    tri = n * (deg ** 2 * 15.0 / 32.0 + m ** 2 + 3.0 * m * deg * 0.6) / 6.0
    quad = n * (deg ** 3 * 0.17 + m ** 3 + 6.0 * m * m * deg * 0.5 + 4.0 * m * deg ** 2 * 0.3) / 24.0
    return pairs, tri, quad


def work(case):
    """Catalogue in (24 bytes a point, 8 a weight), counts out; 8 operations
    a pair (its squared length), 1 a triangle (3 weighted), 20 a parity
    4-clique (its signed volume and four counters), 7 a 6-edge one."""
    kind, n, box, rmax, nb = (case[k] for k in ("kind", "n", "box", "rmax", "nbins"))
    conf = (nb + 2) * (nb + 1) * nb // 6
    if kind in ("batch", "serve"):
        flops = bts = 0.0
        for k, m in enumerate(_catalogue_sizes(case)):
            p, t, _ = _tuples(m, box, rmax, 1.0 if k % 2 == 0 else 0.0)
            bts += (24 * m if kind == "serve" else 5 * p + 8 * m) + 8 * conf
            flops += t + (8 * p if kind == "serve" else 0)
        return dict(bytes=bts, flops=flops)
    share = {"tri": 1.0 if case.get("field") == "clustered" else 0.0, "survey": 0.5}.get(kind, 1.0)
    weighted = case.get("weighted", kind in ("survey", "zeta3", "zeta4"))
    p, t, q = _tuples(n, box, rmax, share)
    bts = n * (24 + 8 * weighted) + 8 * conf * (4 if weighted else 1)
    if kind == "tri":
        return dict(bytes=bts, flops=8 * p + (3 if weighted else 1) * t)
    if kind == "restricted":
        return dict(bytes=bts * 1.0, flops=8 * p + 20 * t)
    if kind == "survey":
        return dict(bytes=bts, flops=9 * p + 3 * t / 4.0)
    if kind == "zeta3":
        p2, t2, _ = _tuples(2 * n, box, rmax, 0.5)
        pr, tr, _ = _tuples(n, box, rmax, 0.0)
        return dict(bytes=2 * bts, flops=8 * (p2 + pr) + 3 * (t2 + tr))
    if kind == "zeta4":
        p2, _, q2 = _tuples(2 * n, box, rmax, 0.5)
        pr, _, qr = _tuples(n, box, rmax, 0.0)
        return dict(bytes=2 * bts, flops=9 * (p2 + pr) + 27 * (q2 + qr))
    return dict(bytes=bts, flops=8 * p + (7 if kind == "six" else 20) * q)


# ----------------------------------------------------------------- exact ---

def _bins(x, box, rmax, nb, periodic=True):
    """Bin of every pair (-1: no edge) of float64 coordinates on the GPU."""
    q = None
    for a in range(3):
        d = x[None, :, a] - x[:, None, a]
        if periodic:
            d = torch.where(d > box / 2, d - box, torch.where(d < -box / 2, d + box, d))
        q = d * d if q is None else q + d * d
    step = rmax / nb
    edges = torch.tensor([0.0] + [(k * step) ** 2 for k in range(1, nb)] + [rmax * rmax], dtype=torch.float64,
                         device=x.device)
    b = torch.bucketize(q, edges, right=True) - 1
    b[(q >= edges[-1])] = -1
    b.fill_diagonal_(-1)
    return b


def _triangle_sums(x, w, box, rmax, nb):
    """Weighted triangle sums per sorted-side configuration, float64."""
    x, w = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    b = _bins(x, box, rmax, nb)
    masks = [(b == k).to(torch.float64) for k in range(nb)]
    ww = w[:, None] * w[None, :]
    out = []
    for b1 in range(nb):
        for b2 in range(b1, nb):
            m = (masks[b1] * w[None, :]) @ masks[b2]      # sum over the shared vertex
            for b3 in range(b2, nb):
                same = 6.0 if b1 == b2 == b3 else (2.0 if b1 == b2 or b2 == b3 else 1.0)
                out.append(float((m * masks[b3] * ww).sum()) / same)
    return np.array(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "tri" and case["weighted"] and case["n"] <= 8_000:
        i = _inputs(case, seed)
        return dict(hist=None, n=None, wsum=None, wscale=None,
                    whist=_triangle_sums(i["x"], i["w"], case["box"], case["rmax"], case["nbins"]))
    if kind == "zeta3" and case["n"] <= 4_000:
        i = _inputs(case, seed)
        wd, wr = i["wd"] / i["wd"].sum(), i["wr"] / i["wr"].sum()
        geo = (case["box"], case["rmax"], case["nbins"])
        nnn = _triangle_sums(np.concatenate([i["data"], i["rand"]]), np.concatenate([wd, -wr]), *geo)
        rrr = _triangle_sums(i["rand"], wr, *geo)
        return dict(zeta=None, nnn=nnn, rrr=rrr)
    return None
