"""Packed lists of jobs whose arrays overlap: outputs of one kind over those of
another, and outputs over other jobs' inputs.  Groups are packed, and their
results handed out, in the order that a list had when it was two groups in flight
and one thread, so every array ends with the same bytes."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads as W
from tests.test_gpu_jobs import _job

pytestmark = pytest.mark.gpu
KINDS = ("next", "prev", "seeds", "loop_off", "loop_he")


def results(m):
    o = oracle.polylla(m.xy, m.tri)
    return {"next": o.next, "prev": o.prev, "seeds": o.seeds, "loop_off": o.loop_off, "loop_he": o.loop_he}


@pytest.fixture(scope="module")
def meshes():
    ms = [W.jittered_grid(n, seed=70 + n) for n in (20, 31, 25, 12, 28)]
    return ms, [results(m) for m in ms]


def write(buf, at, values):
    buf[at:at + len(values)] = values


@pytest.mark.parametrize("group", [0, 2000, 20000])
def test_outputs_of_different_kinds(meshes, group):
    """one block for all outputs of all jobs: a job's kinds lie apart in it, but
    at the places of other kinds of other jobs"""
    ms, outs = meshes
    count, cap = 300, 3 * max(m.nt for m in ms) + 8
    order = {"next": 0, "prev": 1, "seeds": 2, "loop_off": 3, "loop_he": 4}
    with gp.Context(0) as ctx:
        for _ in range(3):
            block, want = np.full(5 * cap, -7, np.int32), np.full(5 * cap, -7, np.int32)
            use = [k % len(ms) for k in range(count)]
            built = [_job(ms[u]) for u in use]
            jobs = (gp.gp_job * count)(*[b[0] for b in built])
            for k, u in enumerate(use):
                for name, q in order.items():
                    at = (q + k) % 5 * cap
                    setattr(jobs[k], name, block.ctypes.data + 4 * at)
                    write(want, at, outs[u][name])
            print(f"[gpu] shared arrays: kinds, group {group}", flush=True)
            assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
            assert np.array_equal(block, want)


@pytest.mark.parametrize("group,order", [(0, "all_first"), (8000, "two_groups")])
def test_outputs_over_inputs(meshes, group, order):
    """every job's next' goes over the triangles of a job further on: by itself a
    list is one group, whose inputs are all read first; in groups the inputs of the
    next one are read before a group's results are written"""
    ms, outs = meshes
    m, o = ms[1], outs[1]           # 1,922 triangles: four to a group of 8,000
    count, ahead = 300, (1 if group else 150)
    per = 4                         # jobs a group
    with gp.Context(0) as ctx:
        tris = [m.tri.reshape(-1).copy() for _ in range(count)]
        built = [_job(m) for _ in range(count)]
        jobs = (gp.gp_job * count)(*[b[0] for b in built])
        for k in range(count):
            jobs[k].tri = tris[k].ctypes.data
            # (in groups: a job over one of its own group or of the next one)
            to = k + ahead if not group else min(count - 1, (k // per + 1) * per + (k + 1) % per)
            if to < count:
                jobs[k].next = tris[to].ctypes.data
        print(f"[gpu] shared arrays: outputs over inputs, group {group}", flush=True)
        assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
        for k in range(count):
            assert jobs[k].status == gp.GP_OK and jobs[k].npoly == len(o["seeds"])
            assert np.array_equal(built[k][1]["loop_he"][:jobs[k].nloop_he], o["loop_he"]), k


def test_apart_lists_are_not_slowed(meshes):
    """arrays of every job's own, in any order of addresses: the helpers unpack"""
    ms, outs = meshes
    count = 400
    rng = np.random.default_rng(5)
    with gp.Context(0) as ctx:
        built = [_job(ms[k % len(ms)]) for k in range(count)]
        order = rng.permutation(count)
        jobs = (gp.gp_job * count)(*[built[k][0] for k in order])
        print("[gpu] shared arrays: apart", flush=True)
        for group in (0, 5000):
            assert gp.gpolylla_mesh_jobs(ctx.handle, jobs, group) == gp.GP_OK
            for k, q in enumerate(order):
                o = outs[q % len(ms)]
                assert np.array_equal(built[q][1]["loop_he"][:jobs[k].nloop_he], o["loop_he"])
                assert np.array_equal(built[q][1]["next"][:len(o["next"])], o["next"])
