"""The build and a run over more than 2^28 triangles, where 32-bit byte offsets
end and list entries are triangle ids alone: twins and loops checked on the
device against their definitions (an oracle run of this size takes minutes)."""
import ctypes

import numpy as np
import pytest

import paper_2403_14723_amd as gp

pytestmark = pytest.mark.gpu


class Ints:
    """int32 device memory of the library, for torch.as_tensor"""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 2}


def grid(n):
    """n x n cells, two triangles each, corners moved by up to a quarter of a cell"""
    import torch
    g = torch.Generator(device="cuda").manual_seed(1)
    c = (1 << 30) // (n + 1)
    ids = torch.arange(n + 1, device="cuda", dtype=torch.int32) * c
    xy = torch.stack([ids.repeat(n + 1), ids.repeat_interleave(n + 1)], 1)
    xy += torch.randint(0, c // 4, xy.shape, generator=g, device="cuda", dtype=torch.int32)
    tri = torch.empty((n, n, 2, 3), dtype=torch.int32, device="cuda")
    row = torch.arange(n, device="cuda", dtype=torch.int32)
    v = row[:, None] * (n + 1) + row[None, :]
    for k, (a, b, d) in enumerate(((0, 1, n + 2), (0, n + 2, n + 1))):
        for i, q in enumerate((a, b, d)):
            tri[:, :, k, i] = v + q
    return xy, tri.reshape(-1, 3)


def test_wide():
    import torch
    if torch.cuda.get_device_properties(0).total_memory < 100 << 30:
        pytest.skip("needs 60 GB of device memory")
    n = 11_586   # 2 n^2 = 2^28 + 35,336
    xy, tri = grid(n)
    nt, nh = len(tri), 3 * len(tri)
    assert nt > 1 << 28
    torch.cuda.synchronize()
    print(f"[gpu] wide build: {nt} triangles", flush=True)
    with gp.Context(0) as ctx:
        h = ctx.build_halfedges(xy, tri)
        del xy, tri
        org, twin, _ = h.copy()
        org, twin = torch.from_numpy(org).cuda(), torch.from_numpy(twin).cuda()
        edge = 0
        for a in range(0, nh, 90_000_000):
            e = torch.arange(a, min(nh, a + 90_000_000), device="cuda")
            g = twin[e].long()
            edge += int((g < 0).sum())
            e, g = e[g >= 0], g[g >= 0]
            after = lambda q: torch.where(q % 3 == 2, q - 2, q + 1)
            assert bool(((org[g] == org[after(e)]) & (org[after(g)] == org[e]) & (twin[g] == e)).all())
        assert edge == 4 * n
        del org, twin, e, g
        print("[gpu] wide run", flush=True)
        r = ctx.mesh(h)
        info, dev = r.info(), gp.gp_result_dev()
        gp.library().gpolylla_result_device(r.handle, ctypes.byref(dev))
        of = lambda p, m: torch.as_tensor(Ints(p, m), device="cuda")
        F, P = info["nloop_he"], info["npoly"]
        nxt, prv, he = of(dev.next, nh), of(dev.prev, nh), of(dev.loop_he, F)
        seeds, off = of(dev.seeds, P), of(dev.loop_off, P + 1)
        assert int((nxt >= 0).sum()) == F == int(off[-1]) and bool((off[1:] - off[:-1] >= 3).all())
        assert bool((seeds[1:] > seeds[:-1]).all()) and bool((he[off[:-1].long()] == seeds).all())
        last = torch.zeros(F, dtype=torch.bool, device="cuda")
        last[off[1:].long() - 1] = True
        first = torch.repeat_interleave(seeds, (off[1:] - off[:-1]).long())
        want = torch.where(last, first, torch.cat([he[1:], he[:1]]))
        assert torch.equal(nxt[he.long()], want) and torch.equal(prv[want.long()], he) and bool((he >= first).all())
        del nxt, prv, he, seeds, off, last, first, want
        r.free()
        h.free()
    torch.cuda.empty_cache()
