"""Builds of triangulations most of whose vertices are in no triangle: corners
and twins against the oracle, in pools with and without a cap, and the time of
one numbered at random against that of the same mesh without the others."""
import time

import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W

pytestmark = pytest.mark.gpu


def with_unused(m, times, spread):
    """m's vertices last among, or spread over, times as many"""
    n = times * m.nv
    at = np.arange(m.nv) * times if spread else np.arange(n - m.nv, n)
    xy = np.zeros((n, 2), np.int32)
    xy[at] = m.xy
    return xy, at[m.tri].astype(np.int32)


@pytest.fixture(scope="module")
def mesh():
    return W.scrambled(W.random_delaunay(40_000, 26, order="morton"), 6)


@pytest.mark.parametrize("pool", [0, 64 << 20])
@pytest.mark.parametrize("times,spread", [(3, False), (10, False), (10, True), (40, False)])
def test_corners_and_twins(mesh, times, spread, pool):
    xy, tri = with_unused(mesh, times, spread)
    print(f"[gpu] unused vertices: {times} times, spread {spread}, pool {pool}", flush=True)
    o = oracle.polylla(xy, tri)
    with gp.Context(0, pool_bytes=pool) as ctx:
        h = ctx.build_halfedges(xy, tri)
        org, twin, _ = h.copy()
        h.free()
    assert np.array_equal(org, o.org) and np.array_equal(twin, o.twin)


def test_time(mesh):
    import torch

    def build_us(ctx, xy, tri):
        d = torch.from_numpy(np.ascontiguousarray(xy)).cuda(), torch.from_numpy(np.ascontiguousarray(tri)).cuda()
        torch.cuda.synchronize()
        v = []
        for _ in range(12):
            t = time.perf_counter()
            ctx.build_halfedges(*d).free()
            v.append(time.perf_counter() - t)
        return 1e6 * sorted(v[2:])[4]

    with gp.Context(0) as ctx:
        alone, among = build_us(ctx, mesh.xy, mesh.tri), build_us(ctx, *with_unused(mesh, 10, False))
    print(f"[gpu] unused vertices: {alone:.0f} us without, {among:.0f} us with", flush=True)
    assert among < 2.5 * alone
