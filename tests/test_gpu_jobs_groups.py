"""Packed lists of small jobs in many overlapping groups: outputs of each job's
own, and output arrays that the jobs share (the last job's results remain, as
when groups run one after the other); several lists on one context."""
import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests.test_gpu_jobs import _check, _job

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("count,group", [(1, 0), (90, 2000), (90, 20000), (300, 0)])
def test_groups(shared, count, group):
    base = [W.jittered_grid(n, seed=900 + n) for n in (3, 20, 11, 32, 7)] + [W.random_delaunay(400, 910)]
    big = W.jittered_grid(45, seed=911)
    ms = [base[k % len(base)] for k in range(count - 1)] + [big]
    print(f"[gpu] job groups: {count} jobs, group {group}, shared {shared}", flush=True)
    with gp.Context(0) as c:
        for _ in range(3):
            last = _job(big)
            built = [_job(m) for m in ms[:-1]] + [last]
            if shared:
                for j, _bufs in built[:-1]:
                    for k in ("next", "prev", "seeds", "loop_off", "loop_he"):
                        setattr(j, k, last[1][k].ctypes.data)
            arr = (gp.gp_job * count)(*[b[0] for b in built])
            assert gp.gpolylla_mesh_jobs(c.handle, arr, group) == gp.GP_OK
            for k, m in enumerate(ms):
                if not shared or k == count - 1:
                    _check(arr[k], built[k][1], m, f"job {k}")
                else:
                    o = oracle.polylla(m.xy, m.tri)
                    assert (arr[k].npoly, arr[k].nloop_he) == (len(o.seeds), len(o.loop_he))


def test_groups_in_a_capped_pool():
    """room for one group at a time: the others wait for it"""
    ms = [W.jittered_grid(20 + k % 5, seed=930 + k) for k in range(40)]
    print("[gpu] job groups: capped pool", flush=True)
    with gp.Context(0, pool_bytes=800 << 10) as c:
        built = [_job(m) for m in ms]
        arr = (gp.gp_job * len(ms))(*[b[0] for b in built])
        assert gp.gpolylla_mesh_jobs(c.handle, arr, 8000) == gp.GP_OK
        for k, m in enumerate(ms):
            _check(arr[k], built[k][1], m, f"job {k}")
