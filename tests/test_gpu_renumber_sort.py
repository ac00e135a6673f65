"""The order that GP_RENUMBER puts vertices and triangles in: a stable sort of
their Morton codes, against numpy's, element by element.  The inputs sit where
the sort by sampling can go wrong: fewer elements than samples, many equal
codes (within a bucket's list and beyond it), codes that agree in the bits a
bucket's words hold, and lengths either side of its limit."""
import numpy as np
import pytest

import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gp.Context(0)
    yield c
    c.close()


def spread(v):
    x = v.astype(np.uint64) & np.uint64(0x7FFFFFFF)
    for s, m in ((16, 0x0000FFFF0000FFFF), (8, 0x00FF00FF00FF00FF), (4, 0x0F0F0F0F0F0F0F0F),
                 (2, 0x3333333333333333), (1, 0x5555555555555555)):
        x = (x | (x << np.uint64(s))) & np.uint64(m)
    return x


def order(x, y):
    return np.argsort(spread(x) | (spread(y) << np.uint64(1)), kind="stable")


def with_vertices(m, extra, seed):
    """m and further vertices in no triangle, the whole numbered at random"""
    xy = np.concatenate([m.xy, np.asarray(extra, np.int32).reshape(-1, 2)])
    p = np.random.default_rng(seed).permutation(len(xy))
    out = np.empty_like(xy)
    out[p] = xy
    return out, np.ascontiguousarray(p[m.tri].astype(np.int32))


def case(name):
    rng = np.random.default_rng(7)
    if name == "one":
        return np.array([[0, 0], [4, 0], [0, 4]], np.int32), np.array([[0, 1, 2]], np.int32)
    if name == "grid":
        m = W.scrambled(W.jittered_grid(40, seed=3), 1)
        return m.xy, m.tri
    if name == "delaunay":
        m = W.scrambled(W.random_delaunay(70000, 4, order="morton"), 2)
        return m.xy, m.tri
    m = W.random_delaunay(3000, 5)
    if name == "equal":          # 300 equal codes
        return with_vertices(m, np.full((300, 2), 12345), 6)
    if name == "many_equal":     # more than any bucket holds
        return with_vertices(m, np.full((9000, 2), 12345), 6)
    if name == "cluster":        # a bucket from a dense cluster to the far corner
        return with_vertices(m, np.concatenate([(1 << 30) - 3000 + rng.integers(0, 40, (2500, 2)), [[0, 0]],
                                                rng.integers(0, 40, (2500, 2)), [[1 << 30, 1 << 30]]]), 8)
    # four times the mean fits the smaller lists, then the larger ones, then none
    n = {"small_lists": 1 << 20, "large_lists": (1 << 20) + 1, "large_equal": 1500000, "at_limit": 1 << 21,
         "over_limit": (1 << 21) + 1}[name]
    extra = rng.integers(0, 1 << 30, (n - m.nv, 2))
    if name == "large_equal":
        extra[:5000] = 12345
    return with_vertices(m, extra, 9)


@pytest.mark.parametrize("name", ["one", "grid", "delaunay", "equal", "many_equal", "cluster",
                                  "small_lists", "large_lists", "large_equal", "at_limit", "over_limit"])
def test_order(ctx, name):
    xy, tri = case(name)
    print(f"[gpu] renumber order {name}: nv={len(xy)} nt={len(tri)}", flush=True)
    h = ctx.build_halfedges(xy, tri, gp.GP_RENUMBER)
    tp, vp = h.permutation()
    h.free()
    assert np.array_equal(vp, order(xy[:, 0], xy[:, 1]))
    c = xy.astype(np.int64)[tri].sum(axis=1) // 3
    assert np.array_equal(tp, order(c[:, 0], c[:, 1]))


def test_capped_pool():
    """a pool with room for the build but not for the sampling sort's lists"""
    m = W.scrambled(W.random_delaunay(200000, 10, order="morton"), 3)
    print(f"[gpu] renumber capped: nt={m.nt}", flush=True)
    with gp.Context(0, pool_bytes=64 << 20) as c:
        for flags in (0, gp.GP_COMPACT):
            h = c.build_halfedges(m.xy, m.tri, gp.GP_RENUMBER | flags)
            tp, vp = h.permutation()
            h.free()
            assert np.array_equal(vp, order(m.xy[:, 0], m.xy[:, 1]))
            s = m.xy.astype(np.int64)[m.tri].sum(axis=1) // 3
            assert np.array_equal(tp, order(s[:, 0], s[:, 1]))
