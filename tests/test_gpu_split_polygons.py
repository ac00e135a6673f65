"""Polygons that the repair splits, through the tiled chain, one mesh at a time
and as a batch: every loop once, whatever the tiles and list stripes, against
the oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests import polycheck as pc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gp.Context(0)
    yield c
    c.close()


def fixture_mesh(name):
    fx = pc.load_fixture(name)
    return fx["xy"], fx["tri"]


def meshes():
    out = [fixture_mesh("p3_fan_degree8.txt"), fixture_mesh("p4_fan_degree7.txt")]
    for n, seed, order in ((400, 31, "qhull"), (5000, 32, "morton"), (9000, 33, "morton"), (20000, 34, "qhull"), (60000, 37, "morton")):
        m = W.random_delaunay(n, seed, order=order)
        out.append((m.xy, m.tri))
    m = W.scrambled(W.random_delaunay(7000, 35, order="morton"), 5)
    out.append((m.xy, m.tri))
    # stretched: fewer tips, longer polygons
    m = W.random_delaunay(12000, 36, order="morton")
    out.append((np.ascontiguousarray(m.xy * np.array([1, 2], np.int32)), m.tri))
    return out


@pytest.fixture(scope="module")
def cases():
    return [(xy, tri, oracle.polylla(xy, tri)) for xy, tri in meshes()]


def check(r, o, name):
    g = r.copy()
    for key, a, b in (("next", g["next"], o.next), ("prev", g["prev"], o.prev), ("seeds", g["seeds"], o.seeds),
                      ("loop_off", g["loop_off"], o.loop_off), ("loop_he", g["loop_he"], o.loop_he)):
        assert np.array_equal(a, b), f"{name}: {key}"
    for k in ("npoly", "nloop_he", "ntips", "nmiddle", "nterminal"):
        assert g["info"][k] == o.stats[k], f"{name}: {k}"


@pytest.mark.parametrize("launch", ["", "relink=64x1,compact=64x1", "relink=1024x1", "relink=64x8,compact=256x8",
                                    "persist=64x1"])
def test_chain(ctx, cases, launch):
    ctx.set_launch("label=128x4,relink=256x2,compact=128x4,persist=256x2048,small=0")
    ctx.set_launch(launch)
    for k, (xy, tri, o) in enumerate(cases):
        print(f"[gpu] {launch} mesh {k}: nt={len(tri)} tips={o.stats['ntips']}", flush=True)
        h = ctx.build_halfedges(xy, tri)
        r = ctx.mesh(h)
        check(r, o, f"mesh {k}")
        r.free()
        h.free()
    hs = [ctx.build_halfedges(xy, tri) for xy, tri, _ in cases]
    for flags in (0, gp.GP_GRAPH, gp.GP_GRAPH):
        rs = ctx.mesh_batch(hs, flags)
        for k, (r, (_, _, o)) in enumerate(zip(rs, cases)):
            check(r, o, f"batch {k}")
            r.free()
    for h in hs:
        h.free()
