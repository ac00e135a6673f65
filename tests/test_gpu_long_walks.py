"""Loops too long to be kept, or past the pool's room, through the tiled chain:
outputs against the oracle, and the run against one over short loops with as
many half-edges on the longest chain of loads."""
import time

import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from tests import polycheck as pc

pytestmark = pytest.mark.gpu


def strips(n, k):
    """k strips of one loop of 2n + 1 half-edges, of their own vertices"""
    xy, tri = pc.rising_strip(n, False)
    return np.tile(xy, (k, 1)), (tri[None] + (np.arange(k) * len(xy))[:, None, None]).reshape(-1, 3).astype(np.int32)


@pytest.fixture(scope="module")
def ctx():
    c = gp.Context(0, profile=True)
    c.set_launch("small=0")
    yield c
    c.close()


# lengths about the buffer (16), the places in the pool (68, 188), and far
# beyond; more loops than a wave, and than the pool has room for
@pytest.mark.parametrize("n,k", [(7, 70), (8, 3000), (9, 1), (33, 500), (34, 500), (93, 70), (94, 70), (95, 1), (3000, 3)])
def test_loops(ctx, n, k):
    xy, tri = strips(n, k)
    print(f"[gpu] long walks: {k} loops of {2 * n + 1}", flush=True)
    o = oracle.polylla(xy, tri)
    h = ctx.build_halfedges(xy, tri)
    r = ctx.mesh(h)
    g = r.copy()
    r.free()
    h.free()
    for key in ("next", "prev", "seeds", "loop_off", "loop_he"):
        assert np.array_equal(g[key], getattr(o, key)), key


def walk_us(ctx, n, k):
    xy, tri = strips(n, k)
    h = ctx.build_halfedges(xy, tri)
    for _ in range(4):
        ctx.mesh(h).free()
    ctx.sync()
    ctx.kernel_reset()
    for _ in range(12):
        ctx.mesh(h).free()
    ctx.sync()
    v = ctx.kernel_ms()
    h.free()
    us = {name: 1e3 * (x[0] if isinstance(x, (tuple, list)) else x) for name, x in v.items()}
    print(f"[gpu] {k} loops of {2 * n + 1}: k_walk {us['k_walk']:.1f} us, k_emit {us['k_emit']:.1f}", flush=True)
    return us


def test_time_of_long_chains(ctx):
    """k_walk and k_emit take the same steps over a loop that is not kept"""
    us = walk_us(ctx, 2000, 1)
    assert us["k_walk"] < 1.3 * us["k_emit"]


def test_time_of_many_places(ctx):
    """60,000 loops of 17 half-edges against as many of 15: the places in the
    pool cost no atomic per loop"""
    assert walk_us(ctx, 8, 60000)["k_walk"] < 1.6 * walk_us(ctx, 7, 60000)["k_walk"]


def test_room_for_every_loop(ctx):
    """12,000 loops of 81 half-edges are kept and copied (those that find no room
    are walked again: five times k_emit's time where it has nothing to write)"""
    none, many = walk_us(ctx, 7, 12000), walk_us(ctx, 40, 12000)
    assert many["k_emit"] < 2.5 * none["k_emit"]
