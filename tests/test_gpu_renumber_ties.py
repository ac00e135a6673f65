"""GP_RENUMBER where many codes are equal, or agree in the leading bits that a
bucket's words hold: the order is numpy's stable sort's, and a build takes about
as long as without them (it took up to 26 times as long where they were
ordered by swapping neighbours, 1.5 times where they overflowed a bucket and the
input was sorted and built again)."""
import time

import numpy as np
import pytest

import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests import polycheck as pc
from tests.test_gpu_renumber_sort import order, with_vertices

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gp.Context(0)
    yield c
    c.close()


def extra(name):
    rng = np.random.default_rng(17)
    if name == "none":
        return np.zeros((0, 2), np.int32)
    if name.startswith("equal"):     # one code
        return np.full((int(name[5:]), 2), 12345)
    if name == "few_codes":          # runs of equal codes among neighbours
        return rng.integers(0, 3, (60_000, 2)) + (1 << 29)
    if name == "cluster":            # 5,000 codes within 2^12 of each other, in a bucket that spans far more
        return np.concatenate([rng.integers(0, 60, (5000, 2)), [[1 << 30, 1 << 30]]])
    # lists of the largest size: a million other vertices, and
    n = (1 << 20) + 5000
    e = rng.integers(0, 1 << 30, (n, 2))
    if name == "large_equal":
        e[:30_000] = 12345
    elif name == "large_cluster":
        e[:7000] = rng.integers(0, 90, (7000, 2))
    return e


@pytest.fixture(scope="module")
def mesh():
    return W.scrambled(W.random_delaunay(40_000, 16, order="morton"), 4)


NAMES = ["equal257", "equal1000", "equal4097", "equal100000", "few_codes", "cluster", "large", "large_equal", "large_cluster"]


@pytest.mark.parametrize("name", NAMES)
def test_order(ctx, mesh, name):
    xy, tri = with_vertices(mesh, extra(name), 6)
    print(f"[gpu] renumber ties {name}: nv={len(xy)} nt={len(tri)}", flush=True)
    h = ctx.build_halfedges(xy, tri, gp.GP_RENUMBER)
    tp, vp = h.permutation()
    h.free()
    assert np.array_equal(vp, order(xy[:, 0], xy[:, 1]))
    c = xy.astype(np.int64)[tri].sum(axis=1) // 3
    assert np.array_equal(tp, order(c[:, 0], c[:, 1]))


def unsampled(n=60_000, samples=2048):
    """n vertices of which those that the sort samples (sample_place in
    renumber.hip) lie far apart, a mesh's among them, and all others in one
    place's neighbourhood: a bucket that no list holds"""
    m = W.random_delaunay(1500, 27)
    i = np.arange(samples, dtype=np.uint64)
    h = (i * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)
    at = ((i * np.uint64(n) + (h * np.uint64(n) >> np.uint64(32))) // np.uint64(samples)).astype(np.int64)
    rng = np.random.default_rng(28)
    q = rng.permutation(300 * 300)[:n]
    xy = np.stack([q % 300, q // 300], -1).astype(np.int32) + (1 << 29)
    xy[at] = rng.integers(0, 1 << 30, (samples, 2))
    xy[at[:m.nv]] = m.xy
    return xy, at[m.tri].astype(np.int32)


def test_overflow():
    """the library's sort in its place, in pools with room for the lists and
    without: where there is none at all the error, else the same order"""
    xy, tri = unsampled()
    c = xy.astype(np.int64)[tri].sum(axis=1) // 3
    want, fits = (order(xy[:, 0], xy[:, 1]), order(c[:, 0], c[:, 1])), 0
    for pool in [0] + [k << 18 for k in range(4, 60, 3)]:
        with gp.Context(0, pool_bytes=pool) as ctx:
            print(f"[gpu] renumber overflow: pool {pool}", flush=True)
            try:
                h = ctx.build_halfedges(xy, tri, gp.GP_RENUMBER)
            except gp.GPolyllaError as e:
                assert e.code == gp.GP_ENOMEM and pool
                continue
            tp, vp = h.permutation()
            h.free()
            fits += 1
            assert np.array_equal(vp, want[0]) and np.array_equal(tp, want[1])
    assert fits > 3


def test_triangle_ties(ctx):
    """a unit grid, where neighbours' centroids round to one code, and 5,000
    triangles of their own vertices in one place"""
    xy, tri = pc.paper_grid(3600)
    k = 5000
    place = np.tile(np.array([[40, 900], [47, 900], [40, 911]], np.int32), (k, 1))
    xy, tri = np.concatenate([xy, place]), np.concatenate([tri, len(xy) + np.arange(3 * k, dtype=np.int32).reshape(-1, 3)])
    m = W.scrambled(W.Mesh(xy, tri, "ties"), 8)
    print(f"[gpu] renumber triangle ties: nt={m.nt}", flush=True)
    h = ctx.build_halfedges(m.xy, m.tri, gp.GP_RENUMBER)
    tp, vp = h.permutation()
    h.free()
    assert np.array_equal(vp, order(m.xy[:, 0], m.xy[:, 1]))
    s = m.xy.astype(np.int64)[m.tri].sum(axis=1) // 3
    assert np.array_equal(tp, order(s[:, 0], s[:, 1]))


@pytest.mark.parametrize("name", ["equal1000", "equal3500", "equal9000", "equal100000", "cluster"])
def test_time(ctx, mesh, name):
    import torch

    def build_us(which):
        xy, tri = with_vertices(mesh, extra(which), 6)
        dxy, dtri = torch.from_numpy(xy).cuda(), torch.from_numpy(tri).cuda()
        torch.cuda.synchronize()
        v = []
        for _ in range(12):
            t = time.perf_counter()
            ctx.build_halfedges(dxy, dtri, gp.GP_RENUMBER).free()
            v.append(time.perf_counter() - t)
        return 1e6 * sorted(v[2:])[4]

    plain, ties = build_us("none"), build_us(name)
    print(f"[gpu] renumber ties {name}: {plain:.0f} us without, {ties:.0f} us with", flush=True)
    assert ties < 3 * plain
