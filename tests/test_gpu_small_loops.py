"""Long loops in meshes that run as one workgroup: one loop, several, and long
ones among short ones and beside barrier tips, about the length from which loops
are ranked instead of walked, in all three sizes of the kernel; alone, in a
batch and as packed jobs.  Against the oracle element by element; and a strip
takes little longer than a grid of as many triangles."""
import time

import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests import polycheck as pc
from tests.test_gpu_jobs import _check, _job
from tests.test_gpu_split_paths import scrambled, tipped_strip

pytestmark = pytest.mark.gpu


def strips(*ns):
    xy, tri, _, _ = pc.rising_strips([(n, n % 2 == 0) for n in ns])
    return xy, tri


def beside_grid(n, xy, tri):
    m = W.jittered_grid(n, seed=31)
    return np.concatenate([m.xy, xy]), np.concatenate([m.tri, tri + m.nv]).astype(np.int32)


# loops of 2n + 1 or 2n + 2: the three kernels walk up to 32, 64 and 128
CASES = [(f"strip_{n}", lambda n=n: strips(n)) for n in (14, 15, 16, 300, 511, 1000, 2047)]
CASES += [("strips_15", lambda: strips(*[15] * 30, 16)), ("strips_1500", lambda: strips(31, 30, 32, 33, 500, 3, 200)),
          ("strips_4000", lambda: strips(62, 63, 64, 65, 1200, 2, 400)),
          ("scrambled", lambda: scrambled(*strips(62, 63, 64, 65, 1200, 2, 400), 7)),
          ("grid_and_strip", lambda: beside_grid(30, *strips(600))),
          ("tipped", lambda: tipped_strip(500, range(0, 500, 7))),
          ("tipped_scrambled", lambda: scrambled(*beside_grid(20, *tipped_strip(300, range(0, 300, 2))), 9))]


@pytest.fixture(scope="module")
def cases():
    out = []
    for name, make in CASES:
        xy, tri = make()
        assert len(tri) <= 4096
        out.append((name, W.Mesh(np.ascontiguousarray(xy, np.int32), np.ascontiguousarray(tri, np.int32), name),
                    oracle.polylla(xy, tri)))
    return out


def check(g, o, name):
    for key in ("next", "prev", "seeds", "loop_off", "loop_he"):
        assert np.array_equal(g[key], getattr(o, key)), (name, key)
    for key in ("npoly", "nloop_he", "ntips", "nmiddle", "nterminal"):
        assert g["info"][key] == o.stats[key], (name, key)


def test_small_loops(cases):
    with gp.Context(0) as ctx:
        hs = []
        for name, m, o in cases:
            print(f"[gpu] small loops {name}: nt={m.nt} longest {np.diff(o.loop_off).max()}", flush=True)
            hs.append(ctx.build_halfedges(m.xy, m.tri))
            for flags in (0, gp.GP_COMPACT):
                h = ctx.build_halfedges(m.xy, m.tri, flags)
                r = ctx.mesh(h)
                check(r.copy(), o, name)
                r.free()
                h.free()
        for (name, _, o), r in zip(cases, ctx.mesh_batch(hs)):
            check(r.copy(), o, name)
            r.free()
        for h in hs:
            h.free()
        built = [_job(m) for _, m, _ in cases]
        arr = (gp.gp_job * len(built))(*[b[0] for b in built])
        assert gp.gpolylla_mesh_jobs(ctx.handle, arr) == gp.GP_OK
        for k, (name, m, _) in enumerate(cases):
            _check(arr[k], built[k][1], m, name)


@pytest.mark.parametrize("n", [300, 1000, 2040])
def test_time(n):
    def mesh_us(ctx, xy, tri):
        h = ctx.build_halfedges(xy, tri)
        v = []
        for _ in range(15):
            t = time.perf_counter()
            ctx.mesh(h).free()
            v.append(time.perf_counter() - t)
        h.free()
        return 1e6 * sorted(v[3:])[6]

    with gp.Context(0) as ctx:
        g = W.jittered_grid(int((n + 0.5) ** 0.5), seed=1)
        grid, strip = mesh_us(ctx, g.xy, g.tri), mesh_us(ctx, *strips(n))
    print(f"[gpu] small loops: {2 * n} triangles, grid {grid:.0f} us, strip {strip:.0f} us", flush=True)
    assert strip < 3 * grid
