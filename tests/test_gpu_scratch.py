"""Batches of small meshes through the tiled chain in pools that just hold them:
the lists of a run take room by triangles, not by tiles."""
import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W

pytestmark = pytest.mark.gpu

# (meshes of 50 triangles, one of 7,200 beside them, launch shapes, pool).  The
# pools: what the runs took when the tip list had an entry per possible tip
# (half the triangles) and no stripes, 19.27, 7.49 and 7.18 MB.
CASES = [(1000, False, "small=0", 19_350_000), (300, True, "", 7_530_000),
         (300, True, "relink=1024x1,compact=64x1,label=64x1", 7_220_000)]


@pytest.mark.parametrize("count,large,launch,pool", CASES, ids=["1000", "300", "300_tiles"])
def test_batch_in_a_capped_pool(count, large, launch, pool):
    ms = [W.jittered_grid(5, seed=40 + k % 7) for k in range(count)] + ([W.jittered_grid(60, seed=47)] if large else [])
    os_ = {}
    print(f"[gpu] scratch: batch of {len(ms)} in {pool} bytes, {launch}", flush=True)
    with gp.Context(0, pool_bytes=pool) as ctx:
        if launch:
            ctx.set_launch(launch)
        hs = [ctx.build_halfedges(m.xy, m.tri) for m in ms]
        for m, r in zip(ms, ctx.mesh_batch(hs)):
            g = r.copy()
            r.free()
            if m.name not in os_:
                os_[m.name] = oracle.polylla(m.xy, m.tri)
            for key in ("next", "prev", "seeds", "loop_off", "loop_he"):
                assert np.array_equal(g[key], getattr(os_[m.name], key)), key
        for h in hs:
            h.free()


def test_build_in_a_capped_pool():
    """a build of a mesh most of whose vertices are in no triangle: its scratch
    is 12 bytes a vertex and 24 a triangle"""
    import torch
    m = W.scrambled(W.random_delaunay(20_000, 3, order="morton"), 4)
    xy = np.concatenate([np.zeros((10 * m.nv, 2), np.int32), m.xy])
    tri = (m.tri + 10 * m.nv).astype(np.int32)
    up = lambda n: (n + 255) // 256 * 256
    pool = up(8 * len(xy)) + 2 * up(12 * m.nt) + up(12 * len(xy) + 24 * m.nt)
    print(f"[gpu] scratch: build in {pool} bytes", flush=True)
    d = torch.from_numpy(xy).cuda(), torch.from_numpy(tri).cuda()
    torch.cuda.synchronize()
    o = oracle.polylla(xy, tri)
    with gp.Context(0, pool_bytes=pool) as ctx:
        h = ctx.build_halfedges(*d)
        org, twin, _ = h.copy()
        h.free()
    assert np.array_equal(org, o.org) and np.array_equal(twin, o.twin)


def test_debug_run_in_a_capped_pool():
    """a debug run over 20,000 triangles takes 4.62 MB with its mesh: a tip
    snapshot of an entry per possible tip"""
    m = W.jittered_grid(100, seed=100)
    print("[gpu] scratch: debug run", flush=True)
    with gp.Context(0, pool_bytes=4_640_000) as ctx:
        ctx.set_debug(True)
        h = ctx.build_halfedges(m.xy, m.tri)
        r = ctx.mesh(h)
        o, g, d = oracle.polylla(m.xy, m.tri), r.copy(), r.debug()
        assert np.array_equal(g["next"], o.next) and len(d["tips"]) == o.stats["ntips"]
        r.free()
        h.free()


def test_tips_of_many_small_meshes():
    """tips of meshes of every size about a tile, whose stripes end unevenly"""
    ms = [W.random_delaunay(n, 50 + k) for k, n in enumerate([20, 255, 258, 300, 40, 517, 600, 1100, 30, 25, 260] * 4)]
    print(f"[gpu] scratch: tips of {len(ms)} meshes", flush=True)
    with gp.Context(0) as ctx:
        for launch in ("small=0", "relink=64x1", "relink=512x2"):
            ctx.set_launch(launch)
            hs = [ctx.build_halfedges(m.xy, m.tri) for m in ms]
            for m, r in zip(ms, ctx.mesh_batch(hs)):
                g, o = r.copy(), oracle.polylla(m.xy, m.tri)
                r.free()
                assert g["info"]["ntips"] == o.stats["ntips"]
                for key in ("next", "prev", "seeds", "loop_off", "loop_he"):
                    assert np.array_equal(g[key], getattr(o, key)), key
            for h in hs:
                h.free()
