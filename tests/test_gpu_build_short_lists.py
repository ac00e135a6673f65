"""Builds in a pool with a cap of meshes numbered at random in a few of the groups
that the vertices are cut into: the lists are short, every group with a triangle
outgrows them, and the triangles are listed again.  Corners and twins against the
oracle, with groups that share a wave and groups that fill one, and the time against
that of the same mesh without the other vertices."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests.test_gpu_build_unused import with_unused

pytestmark = pytest.mark.gpu


def wheel(n):
    """n vertices on a square's sides around one in its middle: one group that a wave
    shares, and the others"""
    k, q = np.arange(n) % (n // 4), np.arange(n) // (n // 4)
    far, s = 4 * (n // 4), 4 * k
    x = np.select([q == 0, q == 1, q == 2], [s, np.full(n, far), far - s], 0)
    y = np.select([q == 0, q == 1, q == 2], [np.zeros(n, int), s, np.full(n, far)], far - s)
    xy = np.concatenate([np.stack([x, y], 1), [[far // 2, far // 2]]]).astype(np.int32)
    i = np.arange(n)
    return W.Mesh(xy, np.stack([np.full(n, n), i, (i + 1) % n], 1).astype(np.int32), f"wheel{n}")


@pytest.mark.parametrize("name,times", [("random", 10), ("random", 40), ("ordered", 40), ("wheel", 10), ("wheel", 1)])
def test_corners_and_twins(name, times):
    m = W.random_delaunay(20_000, 28, order="morton") if name != "wheel" else wheel(6000)
    m = W.scrambled(m, 8) if name == "random" else m
    xy, tri = with_unused(m, times, False)
    print(f"[gpu] short lists: {name}, {times} times", flush=True)
    o = oracle.polylla(xy, tri)
    with gp.Context(0, pool_bytes=64 << 20) as ctx:
        h = ctx.build_halfedges(xy, tri)
        org, twin, _ = h.copy()
        h.free()
    assert np.array_equal(org, o.org) and np.array_equal(twin, o.twin)


def test_time():
    m = W.scrambled(W.random_delaunay(150_000, 27, order="morton"), 7)

    def build_us(ctx, xy, tri):
        d = torch.from_numpy(np.ascontiguousarray(xy)).cuda(), torch.from_numpy(np.ascontiguousarray(tri)).cuda()
        torch.cuda.synchronize()
        v = []
        for _ in range(12):
            t = time.perf_counter()
            ctx.build_halfedges(*d).free()
            v.append(time.perf_counter() - t)
        return 1e6 * sorted(v[2:])[4]

    with gp.Context(0, pool_bytes=1 << 30) as ctx:
        alone, among = build_us(ctx, m.xy, m.tri), build_us(ctx, *with_unused(m, 10, False))
    print(f"[gpu] short lists: {alone:.0f} us without, {among:.0f} us with", flush=True)
    assert among < 3 * alone
