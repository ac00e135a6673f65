"""Loops longer than k_walk's LDS buffer through the tiled chain: lengths from
below the buffer to above what a loop's code and its longest record hold, with room for them in the
walk pool and without, their minima anywhere (numbered at random), one mesh and
a batch; against the oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests import polycheck as pc

pytestmark = pytest.mark.gpu
KEYS = ("next", "prev", "seeds", "loop_off", "loop_he")


@pytest.fixture(scope="module")
def ctx():
    c = gp.Context(0)
    c.set_launch("small=0")
    yield c
    c.close()


def case(name):
    every = [(n, top) for n in range(6, 36) for top in (False, True)]   # loops of 13 to 72 half-edges
    strips = {"every": every * 3, "short": [(8, False), (9, True)] * 400, "long": [(30, False), (30, True)] * 60,
              "longest": [(3, False)] * 900 + [(n, top) for n in (31, 32, 33, 50, 92, 93, 94, 95, 200) for top in (False, True)]
              }[name]
    xy, tri, _, lens = pc.rising_strips(strips)
    m = W.scrambled(W.Mesh(xy, tri, name), 5)
    return np.ascontiguousarray(m.xy), np.ascontiguousarray(m.tri)


CASES = ("every", "short", "long", "longest")


@pytest.fixture(scope="module")
def oracles():
    return {n: (case(n), oracle.polylla(*case(n))) for n in CASES}


@pytest.mark.parametrize("launch", ["", "persist=64x1", "compact=64x1"])
@pytest.mark.parametrize("name", CASES + ("batch",))
def test_long_loops(ctx, oracles, name, launch):
    ctx.set_launch("label=128x4,relink=256x2,compact=128x4,persist=256x2048,small=0")
    if launch:
        ctx.set_launch(launch)
    names = CASES if name == "batch" else (name,)
    print(f"[gpu] long loops {name} {launch}: nt={[len(oracles[n][0][1]) for n in names]}", flush=True)
    hs = [ctx.build_halfedges(*oracles[n][0]) for n in names]
    for flags in (0, gp.GP_GRAPH):
        for n, r in zip(names, ctx.mesh_batch(hs, flags)):
            g = r.copy()
            r.free()
            for k in KEYS:
                assert np.array_equal(g[k], getattr(oracles[n][1], k)), (n, k)
    for h in hs:
        h.free()
