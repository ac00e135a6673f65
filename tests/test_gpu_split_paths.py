"""Barrier tips far from their polygon's seed, through the tiled chain: the
longest-edge path from a tip up to the terminal edge may run through more
triangles than any vertex has neighbours (2^20), and many tips may share one.
Against the oracle element by element."""
import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests import polycheck as pc

pytestmark = pytest.mark.gpu


def tipped_strip(n, tips, scale=400):
    """polycheck.rising_strip(n, False), with six triangles below each bottom
    side in `tips`, around a vertex whose spokes grow with their angle: every
    spoke but the first is the longest edge of the triangle before it, so the
    vertex is a barrier tip, and the path from it leaves through the side and
    runs along the strip to its last rung.  One polygon before the repair."""
    xy, tri = pc.rising_strip(n, False)
    xy = xy.astype(np.int64) * scale + 16 * scale
    tips = np.asarray(tips, np.int64)
    k = np.arange(6)
    u = (1 + 0.02 * k) * np.exp(1j * np.deg2rad(50.0 * k))
    z = (np.concatenate([[0], u[1:5]]) - u[0]) * 4 * scale / (u[5] - u[0])   # the vertex, then its ring's inner corners
    at = xy[tips][:, None, :] + np.stack([np.round(z.real), np.round(z.imag)], -1).astype(np.int64)[None]
    base = len(xy) + 5 * np.arange(len(tips))
    ring = np.stack([tips, base + 1, base + 2, base + 3, base + 4, tips + 1], -1)
    new = np.stack([np.stack([base, ring[:, j], ring[:, (j + 1) % 6]], -1) for j in range(6)], 1).reshape(-1, 3)
    return np.concatenate([xy, at.reshape(-1, 2)]).astype(np.int32), np.concatenate([tri, new]).astype(np.int32)


def scrambled(xy, tri, seed):
    m = W.scrambled(W.Mesh(xy, tri, "strip"), seed)
    return np.ascontiguousarray(m.xy), np.ascontiguousarray(m.tri)


# the long one's path: 1,200,000 triangles.  The short ones' lie about the
# length at which a climb is given up (64 steps).
CASES = [("long", lambda: tipped_strip(600_000, [0])),
         ("shared", lambda: tipped_strip(4000, range(0, 4000, 3))),
         ("shared_scrambled", lambda: scrambled(*tipped_strip(3000, range(0, 3000, 2)), 3))]
CASES += [(f"short_{n}", lambda n=n: tipped_strip(n, sorted({0, n // 2}))) for n in (1, 15, 28, 29, 30, 31, 32, 33, 34, 65)]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_paths(name, make):
    xy, tri = make()
    o = oracle.polylla(xy, tri)
    assert o.stats["ntips"] > 0 and o.stats["nterminal"] == 1
    print(f"[gpu] tipped strip {name}: nt={len(tri)} tips={o.stats['ntips']}", flush=True)
    with gp.Context(0) as ctx:
        ctx.set_launch("small=0")
        for flags in (0, gp.GP_COMPACT):
            h = ctx.build_halfedges(xy, tri, flags)
            r = ctx.mesh(h)
            g = r.copy()
            r.free()
            h.free()
            for key in ("next", "prev", "seeds", "loop_off", "loop_he"):
                assert np.array_equal(g[key], getattr(o, key)), key
            for key in ("npoly", "nloop_he", "ntips", "nmiddle", "nterminal"):
                assert g["info"][key] == o.stats[key], key
