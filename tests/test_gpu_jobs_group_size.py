"""Packed lists with a group size of the caller's that is larger than the
library's: the groups in flight take no more device memory than two groups of
that size, and a list that fits one such group keeps its order of reads and writes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests.test_gpu_jobs import _job

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mesh():
    m = W.jittered_grid(31, seed=101)   # 1,922 triangles
    return m, oracle.polylla(m.xy, m.tri)


def test_memory_of_large_groups(mesh):
    m, o = mesh
    count, group = 1500, 480_000
    # a job's inputs and its outputs, five int arrays of 11 nt values and a few more
    per_job = 8 * m.nv + 12 * m.nt + 44 * m.nt + 256
    with gp.Context(0) as ctx:
        built = [_job(m) for _ in range(count)]
        jobs = (gp.gp_job * count)(*[b[0] for b in built])
        free = torch.cuda.mem_get_info()[0]
        print("[gpu] jobs: memory of large groups", flush=True)
        assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
        taken = free - torch.cuda.mem_get_info()[0]
        assert taken <= 2 * (group // m.nt) * per_job, taken
        for k, (_, b) in enumerate(built):
            assert jobs[k].nloop_he == len(o.loop_he)
            assert np.array_equal(b["next"][:3 * m.nt], o.next) and np.array_equal(b["prev"][:3 * m.nt], o.prev)


def test_outputs_over_inputs_of_one_large_group(mesh):
    """150 jobs of one group, each writing next' over the triangles of another, in
    either direction: every input is read first"""
    m, o = mesh
    count = 150
    with gp.Context(0) as ctx:
        for ahead in (97, -1):
            tris = [m.tri.reshape(-1).copy() for _ in range(count)]
            built = [_job(m) for _ in range(count)]
            jobs = (gp.gp_job * count)(*[b[0] for b in built])
            for k in range(count):
                jobs[k].tri = tris[k].ctypes.data
                jobs[k].next = tris[(k + ahead) % count].ctypes.data
            print(f"[gpu] jobs: one large group, ahead {ahead}", flush=True)
            assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, 1 << 20) == gp.GP_OK
            for k in range(count):
                assert jobs[k].status == gp.GP_OK and jobs[k].npoly == len(o.seeds)
                assert np.array_equal(built[k][1]["loop_he"][:jobs[k].nloop_he], o.loop_he), k
                assert np.array_equal(tris[(k + ahead) % count], o.next), k
