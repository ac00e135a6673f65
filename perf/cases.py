"""Workloads of the library at the sizes users bring, timed through its public
entry points.

A case names a kind of call and the input it is made on:

  mesh      one meshing run on a half-edge structure that stays on the device
            (parameter studies, repeated meshing): gpolylla_mesh, the same as
            a graph replay, or gpolylla_mesh_noalloc into the caller's buffers
  batch     gpolylla_mesh_batch on meshes of uneven sizes, as a graph replay
  polygons  a triangulation in device arrays to its polygons: the half-edge
            build and one meshing run, the life of most inputs
  jobs      gpolylla_mesh_jobs on triangulations in host memory, outputs in
            host memory
  served    requests through the continuous-batching server, host to host

Inputs are jittered n x n grids with random diagonals (warped or not; the
paper's Grid meshes, two triangles per cell) and Delaunay triangulations of
random points (its Random meshes), numbered along a Z-order curve as mesh
generators number them, or at random.  The geometry belongs to the case; the
seed draws the corner that each triangle's triple begins with, which gives
every half-edge and every output another index and leaves the polygons, and so
the sizes of the outputs, the same (coordinates up to 2^30 leave no equal
edge lengths, whose ties the indices would break).  Every pass returns next',
prev', the seeds, the loop offsets and the loops of each mesh, whole.  All
values are integers, and equal inputs give equal outputs.
"""
from __future__ import annotations

import ctypes
import functools
import math

import numpy as np
import torch

import paper_2403_14723_amd as gp
from paper_2403_14723_amd import workloads

DOMAIN = 1 << 30       # side of the grids
PATCH = 16384          # points per Delaunay patch (a large mesh is made of mirrored patches)
NOALLOC_MAX = 3_900_000   # triangles whose scratch the no-allocation entry point holds


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest ordinary mesh (2,048 triangles): the latency of one call
        {"name": "mesh_grid32", "kind": "mesh", "input": "grid", "size": 32, "call": "plain"},
        # a 2.1M-triangle grid meshed into buffers that the caller keeps
        {"name": "mesh_grid1024", "kind": "mesh", "input": "grid", "size": 1024, "call": "noalloc"},
        # the benchmark's grid, 33.5M triangles, as a graph replay: throughput
        {"name": "mesh_warped4096", "kind": "mesh", "input": "warped", "size": 4096, "call": "graph"},
        # general position: a Delaunay mesh of 1M points, many barrier tips
        {"name": "mesh_delaunay1m", "kind": "mesh", "input": "delaunay", "size": 1_000_000, "call": "graph"},
        # uneven meshes that share their launches
        {"name": "batch_12", "kind": "batch", "count": 12, "smin": 64, "smax": 1024},
        # the smallest whole job on the device: build and mesh
        {"name": "polygons_grid32", "kind": "polygons", "input": "grid", "size": 32, "build": "plain"},
        # an ordinary, ragged one: 2,084,882 triangles
        {"name": "polygons_grid1021", "kind": "polygons", "input": "grid", "size": 1021, "build": "plain"},
        # the largest: 33.5M triangles from index triples to polygons
        {"name": "polygons_warped4096", "kind": "polygons", "input": "warped", "size": 4096, "build": "plain"},
        # general position, kept in the compact encoding
        {"name": "polygons_delaunay300k_compact", "kind": "polygons", "input": "delaunay", "size": 300_000,
         "build": "compact"},
        # a mesh numbered at random, renumbered along a Z-order curve by the build
        {"name": "polygons_scattered300k_renumber", "kind": "polygons", "input": "scattered", "size": 300_000,
         "build": "renumber"},
        # many small triangulations, host to host
        {"name": "jobs_512x32", "kind": "jobs", "count": 512, "smin": 32, "smax": 32, "loops_only": False},
        # requests of mixed sizes through the server
        {"name": "served_12", "kind": "served", "count": 12, "smin": 23, "smax": 708},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["mesh", "mesh", "mesh", "batch", "polygons", "polygons", "polygons", "jobs", "served"])
    if kind in ("mesh", "polygons"):
        name = rng.choice(["grid", "warped", "delaunay", "scattered"])
        size = log_int(5, 4096) if name in ("grid", "warped") else log_int(50, 1_000_000)
        case = {"kind": kind, "input": name, "size": size}
        if kind == "polygons":
            case["build"] = rng.choice(["plain", "compact", "renumber"])
            if case["build"] != "plain" and name in ("grid", "warped"):
                case["size"] = min(size, rng.randint(900, 1100))
        else:
            case["call"] = rng.choice(["plain", "graph", "noalloc"] if _triangles(case) <= NOALLOC_MAX
                                      else ["plain", "graph"])
        return case
    smin = log_int(16, 128)
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(2, 12), "smin": smin, "smax": smin * rng.randint(1, 8)}
    if kind == "jobs":
        smax = log_int(16, 128)
        return {"kind": kind, "count": min(rng.randint(16, 512), (1 << 20) // (smax * smax)), "smin": min(smin, smax),
                "smax": smax, "loops_only": rng.random() < 0.5}
    return {"kind": kind, "count": rng.randint(2, 12), "smin": smin, "smax": smin * rng.randint(1, 5)}


# ---------------------------------------------------------------------------
# inputs, made on the device
# ---------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7fffffff)


def _rotated(xy, tri, seed):
    """The mesh with the triangles' corners rotated as the seed draws."""
    turn = torch.randint(0, 3, (len(tri), 1), generator=_generator(seed), device="cuda")
    return xy, tri.gather(1, (torch.arange(3, device="cuda") + turn) % 3).contiguous()


def _grid(n, which=0, warp=False):
    """Grid number `which` of n x n cells, by workloads.jittered_grid's recipe
    on the device: (xy, tri), int32."""
    g = _generator(which)
    c = DOMAIN // n
    jit = int(0.2 * c)
    ids = torch.arange((n + 1) * (n + 1), device="cuda")
    ii, jj = ids % (n + 1), ids // (n + 1)
    pos = torch.stack([ii, jj], 1) * c
    move = torch.randint(-jit, jit + 1, pos.shape, generator=g, device="cuda")
    if warp:
        r = torch.rand((8, 4), generator=g, device="cuda", dtype=torch.float64).cpu()
        px, py = pos[:, 0].double(), pos[:, 1].double()
        bend = torch.zeros(pos.shape, device="cuda", dtype=torch.float64)
        for cx, cy, turn, width in r.tolist():
            sig = 4.0 * 16.0 ** width * c
            bump = torch.exp(((px - cx * DOMAIN) ** 2 + (py - cy * DOMAIN) ** 2) / (-2.0 * sig * sig))
            bend[:, 0] += 0.35 * c * math.cos(2 * math.pi * turn) * bump
            bend[:, 1] += 0.35 * c * math.sin(2 * math.pi * turn) * bump
        move += bend.clamp_(-0.35 * c, 0.35 * c).round_().long()
    move[(ii == 0) | (ii == n), 0] = 0
    move[(jj == 0) | (jj == n), 1] = 0
    xy = (pos + move).clamp_(0, n * c).int()
    cell = torch.arange(n * n, device="cuda")
    v00 = cell // n * (n + 1) + cell % n
    v10, v01, v11 = v00 + 1, v00 + n + 1, v00 + n + 2
    b = torch.randint(0, 2, (n * n,), generator=g, device="cuda").bool()
    tri = torch.stack([v00, v10, torch.where(b, v01, v11), torch.where(b, v10, v00), v11, v01], 1)
    return xy.contiguous(), tri.reshape(-1, 3).int().contiguous()


def _morton(x, y):
    def spread(v):
        for s, m in ((16, 0x0000ffff0000ffff), (8, 0x00ff00ff00ff00ff), (4, 0x0f0f0f0f0f0f0f0f),
                     (2, 0x3333333333333333), (1, 0x5555555555555555)):
            v = (v | (v << s)) & m
        return v
    return spread(x) | (spread(y) << 1)


@functools.lru_cache(maxsize=8)
def _patch(npts):
    return workloads.random_delaunay(npts, seed=21)


def _delaunay(npts, scattered=False):
    """A Delaunay mesh of random points.  A large one is a square of mirrored
    patches, which share the points on their common sides."""
    k = max(1, round(math.sqrt(npts / PATCH)))
    side, m = workloads.DOMAIN, _patch(max(4, npts // (k * k)))
    pts = torch.from_numpy(m.xy).cuda().long()
    one = torch.from_numpy(m.tri).cuda().long()
    xs, ts = [], []
    for q in range(k * k):
        i, j = q % k, q // k
        x = i * side + (side - pts[:, 0] if i % 2 else pts[:, 0])
        y = j * side + (side - pts[:, 1] if j % 2 else pts[:, 1])
        xs.append(x << 31 | y)
        ts.append(one + q * m.nv)
    keys, inv = torch.unique(torch.cat(xs), return_inverse=True)
    x, y, tri = keys >> 31, keys & 0x7fffffff, inv[torch.cat(ts)]
    if scattered:
        g = _generator(npts)
        vorder = torch.randperm(len(keys), generator=g, device="cuda")
        torder = torch.randperm(len(tri), generator=g, device="cuda")
    else:
        vorder = torch.argsort(_morton(x, y), stable=True)
        torder = torch.argsort(_morton(x[tri].sum(1) // 3, y[tri].sum(1) // 3), stable=True)
    rank = torch.empty_like(vorder)
    rank[vorder] = torch.arange(len(vorder), device="cuda")
    xy = torch.stack([x[vorder], y[vorder]], 1).int().contiguous()
    return xy, rank[tri[torder]].int().contiguous()


def _input(name, size, seed):
    base = _grid(size, 0, name == "warped") if name in ("grid", "warped") else _delaunay(size, name == "scattered")
    return _rotated(*base, seed)


def _sides(case):
    """The case's grid sides, spread over [smin, smax] on a log scale in an
    order that mixes large and small."""
    n, lo, hi = case["count"], math.log(case["smin"]), math.log(case["smax"])
    return [int(round(math.exp(lo + (hi - lo) * ((7 * i + 3) % n if n % 7 else i) / max(1, n - 1)))) for i in range(n)]


def _sizes(case):
    """(triangles, vertices, polygons, loop half-edges) of each mesh; the
    polygons of these inputs within a percent."""
    if "input" not in case or case["input"] in ("grid", "warped"):
        sides = [case["size"]] if "input" in case else _sides(case)
        return [(2 * s * s, (s + 1) * (s + 1), 0.478 * 2 * s * s, 1.956 * 2 * s * s) for s in sides]
    v = case["size"]
    return [(1.98 * v, v, 0.16 * 1.98 * v, 1.32 * 1.98 * v)]


def _triangles(case):
    return sum(s[0] for s in _sizes(case))


def work(case):
    """A meshing run reads the corners, twins and coordinates, a whole job the
    index triples and coordinates; both write next', prev', the seeds, the
    loop offsets and the loops.  The path is integer comparisons and index
    arithmetic: no floating-point operations."""
    resident = case["kind"] in ("mesh", "batch")
    total = 0.0
    for t, v, p, f in _sizes(case):
        out = 8 * p + 4 * f + 4 + (0 if case.get("loops_only") else 24 * t)
        total += (24 if resident else 12) * t + 8 * v + out
    return {"bytes": total, "flops": 0}


# ---------------------------------------------------------------------------
# calls
# ---------------------------------------------------------------------------

_keep = {}   # the context and the server that a program holds while it runs


def _context():
    if "ctx" not in _keep:
        _keep["ctx"] = gp.Context(0)
    return _keep["ctx"]


def _server():
    if "srv" not in _keep:
        _keep["srv"] = gp.Server(_context(), n_lanes=4, max_batch=32)
    return _keep["srv"]


class _DeviceInts:
    """int32 device memory of the library, for torch.as_tensor."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 2}


BUILD = {"plain": 0, "compact": gp.GP_COMPACT, "renumber": gp.GP_RENUMBER}


def prepare(case, seed):
    ctx = _context()
    state = {"case": dict(case), "results": [], "views": {}, "info": gp.gp_result_info(), "dev": gp.gp_result_dev()}
    kind = case["kind"]
    if kind in ("mesh", "polygons"):
        xy, tri = _input(case["input"], case["size"], seed)
        torch.cuda.synchronize()   # the library reads them on its own stream
        if kind == "polygons":
            state.update(xy=xy, tri=tri)
            return state
        state["mesh"] = ctx.build_halfedges(xy, tri)
        if case["call"] == "noalloc":
            with_counts = ctx.mesh(state["mesh"])   # the first run tells the output sizes
            info = with_counts.info()
            with_counts.free()
            nt = info["nt"]
            bufs = [torch.empty(n, dtype=torch.int32, device="cuda")
                    for n in (3 * nt + 1, 3 * nt + 1, nt + 1, nt + 2, 3 * nt + 1)]
            counts = torch.zeros(8, dtype=torch.int32, device="cuda")
            sizes = (3 * nt, 3 * nt, info["npoly"], info["npoly"] + 1, info["nloop_he"])
            torch.cuda.synchronize()
            state.update(bufs=bufs, counts=counts, out=gp.gp_result_dev(*[b.data_ptr() for b in bufs]),
                         outputs=[b[:n] for b, n in zip(bufs, sizes)] + [counts])
        return state
    sides = _sides(case)[:32] if kind == "jobs" else _sides(case)
    grids = [_rotated(*_grid(s, k), seed * 64 + k) for k, s in enumerate(sides)]
    if kind == "batch":
        torch.cuda.synchronize()
        state["meshes"] = [ctx.build_halfedges(xy, tri) for xy, tri in grids]
        return state
    if kind == "served":
        _server()
        state["requests"] = [(xy.cpu().numpy(), tri.cpu().numpy()) for xy, tri in grids]
        return state
    # jobs: inputs in pinned host memory, one pinned output array per kind
    # that the jobs share; at most 32 distinct meshes
    pinned = [(xy.cpu().pin_memory(), tri.cpu().pin_memory()) for xy, tri in grids]
    use = [pinned[k % len(pinned)] for k in range(case["count"])]
    nts = [len(tri) for _, tri in use]
    per = {"next": 3, "prev": 3, "seeds": 1, "loop_off": 1, "loop_he": 3}
    if case["loops_only"]:
        per = {k: v for k, v in per.items() if k not in ("next", "prev")}
    outs = {k: torch.zeros(f * sum(nts) + len(nts), dtype=torch.int32).pin_memory() for k, f in per.items()}
    jobs = (gp.gp_job * len(use))()
    done = 0
    for k, (job, (xy, tri)) in enumerate(zip(jobs, use)):
        job.xy, job.nv, job.tri, job.nt = xy.data_ptr(), len(xy), tri.data_ptr(), len(tri)
        for name, f in per.items():
            setattr(job, name, outs[name].data_ptr() + 4 * (f * done + k))
        done += nts[k]
    counts = np.frombuffer(jobs, np.int32).reshape(len(use), -1)
    at = gp.gp_job.npoly.offset // 4
    state.update(jobs=jobs, pinned=pinned, outputs=[outs, counts[:, at:at + 3]])
    return state


def _views(state, results):
    """The outputs of device results as tensors (wrapped once per buffer)."""
    lib, info, dev, views, out = gp.library(), state["info"], state["dev"], state["views"], []
    for r in results:
        lib.gpolylla_result_info(r.handle, ctypes.byref(info))
        lib.gpolylla_result_device(r.handle, ctypes.byref(dev))
        for ptr, n in ((dev.next, info.nh), (dev.prev, info.nh), (dev.seeds, info.npoly),
                       (dev.loop_off, info.npoly + 1), (dev.loop_he, info.nloop_he)):
            v = views.get((ptr, n))
            if v is None:
                v = views[ptr, n] = torch.as_tensor(_DeviceInts(ptr, n), device="cuda")
            out.append(v)
    return out


def run(state):
    case, ctx = state["case"], _context()
    kind = case["kind"]
    if kind == "jobs":
        rc = gp.gpolylla_mesh_jobs(ctx.handle, state["jobs"])
        if rc != gp.GP_OK:
            raise gp.GPolyllaError(rc, "gpolylla_mesh_jobs")
        return state["outputs"]
    if kind == "served":
        srv = _server()
        tickets = [srv.submit(xy, tri) for xy, tri in state["requests"]]
        out = []
        for t in tickets:
            r = srv.wait(t)
            d = r.copy()
            r.free()
            out.append([d[k] for k in ("next", "prev", "seeds", "loop_off", "loop_he")])
        return out
    if case.get("call") == "noalloc":
        rc = gp.gpolylla_mesh_noalloc(ctx.handle, state["mesh"].handle, state["out"], state["counts"].data_ptr())
        if rc != gp.GP_OK:
            raise gp.GPolyllaError(rc, "gpolylla_mesh_noalloc")
        return state["outputs"]
    for r in state["results"]:   # the last pass's, done with
        r.free()
    if kind == "batch":
        state["results"] = ctx.mesh_batch(state["meshes"], gp.GP_GRAPH)
    elif kind == "polygons":
        h = ctx.build_halfedges(state["xy"], state["tri"], BUILD[case["build"]])
        state["results"] = [ctx.mesh(h)]
        h.free()
    else:
        state["results"] = [ctx.mesh(state["mesh"], gp.GP_GRAPH if case["call"] == "graph" else 0)]
    return _views(state, state["results"])
