"""A list of many small jobs over arrays that the context has not seen, made by
parallel loops just before: no slower in groups, with helper threads, than in one
group on the caller's thread alone."""
import time

import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W

pytestmark = pytest.mark.gpu

KINDS = {"next": 3, "prev": 3, "seeds": 1, "loop_off": 1, "loop_he": 3}


def make_list(meshes, count):
    """jobs over pinned arrays, one output array per kind; what keeps them"""
    import torch
    ins = [(torch.from_numpy(m.xy.copy()).pin_memory(), torch.from_numpy(m.tri.copy()).pin_memory()) for m in meshes]
    nts = [meshes[k % len(meshes)].nt for k in range(count)]
    outs = {k: torch.zeros(f * sum(nts) + count, dtype=torch.int32).pin_memory() for k, f in KINDS.items()}
    jobs, done = (gp.gp_job * count)(), 0
    for k, j in enumerate(jobs):
        xy, tri = ins[k % len(ins)]
        j.xy, j.nv, j.tri, j.nt = xy.data_ptr(), len(xy), tri.data_ptr(), len(tri)
        for name, f in KINDS.items():
            setattr(j, name, outs[name].data_ptr() + 4 * (f * done + k))
        done += nts[k]
    return jobs, outs, ins


def test_first_lists():
    meshes = [W.jittered_grid(32, seed=60 + k) for k in range(16)]
    o = oracle.polylla(meshes[0].xy, meshes[0].tri)
    ms = {}
    with gp.Context(0) as ctx:
        for group in (0, 8 << 20):
            for _ in range(3):
                jobs, outs, ins = make_list(meshes, 512)
                for _ in range(8):
                    assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
            v = []
            for _ in range(15):
                jobs, outs, ins = make_list(meshes, 512)
                t = time.perf_counter()
                assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
                v.append(1e3 * (time.perf_counter() - t))
                assert jobs[0].npoly == len(o.seeds)
                assert np.array_equal(outs["loop_he"].numpy()[:jobs[0].nloop_he], o.loop_he)
            ms[group] = sorted(v)
            print(f"[gpu] new lists, group {group}: " + " ".join(f"{x:.2f}" for x in ms[group]) + " ms", flush=True)
    # three quarters of them within the middle of the others
    assert ms[0][10] < 1.2 * ms[8 << 20][7]
