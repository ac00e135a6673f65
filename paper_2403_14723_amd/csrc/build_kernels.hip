// Half-edge construction on the device (the structure of Section 4.1-4.2,
// built on the GPU instead of the host).
//
//   k_orient  coordinates in [0, 2^30]; index check, exact int64 orientation
//             test, counter-clockwise corner order; triangles listed by the
//             vertex groups that their edges belong to
//   k_match   twins, one workgroup per group, in LDS
//
// Both half-edges of an edge {u, v} belong to the group of one of its ends
// (edge_owner): kBuildGroup consecutive vertices.  So each group's half-edges can
// be paired on their own, in a hash table in LDS keyed by the edge, and three
// half-edges of one edge, or two in the same direction, are seen where they
// meet: non-manifold.
//
// A group's list holds triangle ids, one per triangle with an edge in the
// group (about 1.3 per triangle in an ordered numbering), whose corners are
// read again from org.  Lists have room for up to kBuildGroupCap triangles,
// where a planar mesh has at most about 768 to a group.  A group with more, or with
// more edges than the LDS table holds (a vertex of high degree), is left out
// and counted, and the host then queues, for those groups alone:
//
//   k_part_alloc, k_scatter  their lists again, at full length
//   k_match_class            their edges in classes by hash, one workgroup
//                            per class
//
// Grouping by single vertices instead (a counting sort by origin, then a
// search of the target's bucket) took an atomic per vertex and tile in two
// passes and 8-byte records: 2.92 ms for the 33.5M-triangle grid against the
// figures at each kernel.
//
// Errors are reduced with a 64-bit atomicMax over ~(rank << 8 | code), so the
// reported code is deterministic and 0 means none: coordinate range first,
// then the lowest bad triangle, then the lowest non-manifold half-edge seen.
// A bad triangle joins no group, so the later kernels only ever see valid ones
// and the host needs one check, at the end.
#include "gp_internal.h"

namespace gp {

namespace {

constexpr int kCoordMax = 1 << 30;
// k_orient works in tiles of 256 threads x kTileItems triangles and counts per
// group in an LDS window of kBins groups around the tile (meshes numbered row
// by row or along a curve stay in it): one global atomic per group the tile
// touches.  Groups outside the window cost one per wave, or per triangle where
// no two of a wave share one.
constexpr int kTileItems = 4;
constexpr int kTileTri = 256 * kTileItems;
constexpr int kBins = 512;
constexpr int kCopyItems = 8;        // vertices per thread of k_orient's coordinate blocks
constexpr int kShift = 7;
static_assert(1 << kShift == kBuildGroup, "groups by shift");
constexpr int kGroupCap = kBuildGroupCap;
// slots of the LDS edge table: an ordered or random planar mesh has about 384
// edges to a group of 128 vertices
constexpr int kSlots = 1024;
constexpr int kClassSplit = 128;     // triangles per class of a large group
constexpr int kClassBlocks = 2048;

// three ints at 4-byte alignment: loads of 12-byte records; coordinates at
// 4-byte alignment (the caller's array)
typedef int v3i_a4 __attribute__((ext_vector_type(3), aligned(4)));
typedef int v2i_a4 __attribute__((ext_vector_type(2), aligned(4)));

__device__ __forceinline__ void report(unsigned long long *err, unsigned long long rank, int code) {
    atomicMax(err, ~((rank << 8) | (unsigned long long)(-code)));
}

// The end of edge {a, b} whose group pairs it.  The lower end when the two are
// near, as along the rows or the curve of an ordered numbering: then nearly all
// half-edges of a run of triangles fall into the same few groups.  Far ends
// (most edges of a random numbering) take turns by parity, since the lower end
// would give low vertices twice their share.
__device__ __forceinline__ int edge_owner(int a, int b, int near) {
    const int lo = min(a, b), hi = max(a, b);
    return (hi - lo < near || ((lo ^ hi) & 1)) ? lo : hi;
}

// The groups of a triangle's three edges, each once (-1: none, or there
// already).
__device__ __forceinline__ void triangle_groups(const BuildBuffers &b, bool ok, v3i_a4 c, int g[3]) {
    g[0] = edge_owner(c.x, c.y, b.near) >> kShift;
    g[1] = edge_owner(c.y, c.z, b.near) >> kShift;
    g[2] = edge_owner(c.z, c.x, b.near) >> kShift;
    if (g[2] == g[0] || g[2] == g[1]) g[2] = -1;
    if (g[1] == g[0]) g[1] = -1;
    if (!ok) g[0] = g[1] = g[2] = -1;
}

// Adds the lanes of `same` (this lane's group's, found by a ballot) to counter
// *c with one atomic; returns the counter's value at this lane's place.
__device__ __forceinline__ int add_together(int *c, unsigned long long same, int lane) {
    const int leader = __ffsll((long long)same) - 1;
    int b = 0;
    if (lane == leader) b = atomicAdd(c, __popcll(same));
    return __builtin_amdgcn_readlane(b, leader) + __popcll(same & ((1ull << lane) - 1ull));
}

// Adds this wave's triangles to their groups' counters: lane's group g (g < 0:
// none), counted in the LDS window s_bin of kBins groups from w0 on, or in
// count[] (global) outside it.  Lanes of one group add together (a wave of an
// ordered mesh has one to three groups; 64 atomics on one word would run one
// by one), for four groups at most, and the rest alone: a random numbering has
// hardly two lanes of one group.  Returns the counter's value at the lane's
// place.
__device__ __forceinline__ int bin_add(int *s_bin, int32_t *count, int g, int w0) {
    const int lane = __lane_id();
    const bool in = g >= 0 && (unsigned)(g - w0) < (unsigned)kBins;
    unsigned long long todo = __ballot(in);
    const unsigned long long out = __ballot(g >= 0 && !in);
    int place = 0;
#pragma unroll 1
    for (int k = 0; k < 4 && todo; k++) {
        const int gl = __builtin_amdgcn_readlane(g, __ffsll((long long)todo) - 1);
        const unsigned long long same = __ballot(g == gl);
        const int at = add_together(&s_bin[gl - w0], same, lane);
        if ((same >> lane) & 1) place = at;
        todo &= ~same;
    }
    if ((todo >> lane) & 1) place = atomicAdd(&s_bin[g - w0], 1);
    if (out) {   // (uniform)
        todo = out;
#pragma unroll 1
        for (int k = 0; k < 4 && todo; k++) {
            const int gl = __builtin_amdgcn_readlane(g, __ffsll((long long)todo) - 1);
            const unsigned long long same = __ballot(g == gl);
            if (__popcll(same) < 4) break;
            const int at = add_together(&count[gl], same, lane);
            if ((same >> lane) & 1) place = at;
            todo &= ~same;
        }
        if ((todo >> lane) & 1) place = atomicAdd(&count[g], 1);
    }
    return place;
}

// Workgroups go to the 8 XCDs round-robin; this gives each XCD one contiguous
// run of tiles, whose neighbours' coordinates then share its L2.
__device__ __forceinline__ int xcd_run(int b, int G) {
    const int q = G >> 3, r = G & 7, x = b & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

// First group of a tile's window: kBins groups around the median of the first
// corners of three of its cnt triangles (one alone may straddle a jump of the
// curve, which would leave the whole tile outside).
__device__ __forceinline__ int window_start(const BuildBuffers &b, int base, int cnt) {
    const int x = b.tri[3 * (size_t)base], y = b.tri[3 * (size_t)(base + cnt / 2)],
              z = b.tri[3 * (size_t)(base + cnt - 1)];
    return max(0, (max(min(x, y), min(max(x, y), z)) >> kShift) - kBins / 2);
}

// Blocks [0, tiles): a tile of triangles each.  The others: the coordinates,
// checked, and copied to the mesh when the caller's array is on the device.
__global__ void __launch_bounds__(256) k_orient(BuildBuffers b, int tiles) {
    __shared__ int s_bin[kBins];
    __shared__ int s_flip;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= tiles) {   // (uniform)
        const long long v0 = (long long)(blockIdx.x - tiles) * (256 * kCopyItems) + tid;
        bool bad = false;
#pragma unroll
        for (int j = 0; j < kCopyItems; j++) {
            const long long v = v0 + j * 256;
            if (v >= b.nv) continue;
            const v2i_a4 p = reinterpret_cast<const v2i_a4 *>(b.xy_in)[v];
            bad |= p.x < 0 || p.x > kCoordMax || p.y < 0 || p.y > kCoordMax;
            if (b.xy_out) b.xy_out[v] = make_int2(p.x, p.y);
        }
        if (bad) report(b.err, 0, -2);
        return;
    }
    const int base = xcd_run(blockIdx.x, tiles) * kTileTri;
    const int cnt = min(kTileTri, b.nt - base);
    const int w0 = window_start(b, base, cnt);   // (uniform; any value will do)
    for (int k = tid; k < kBins; k += 256) s_bin[k] = 0;
    if (tid == 0) s_flip = 0;
    // a wave takes 256 triangles in a row; all corners, then all coordinates
    // in flight together
    const int lt0 = (tid & ~63) * kTileItems + (tid & 63);
    v3i_a4 c[kTileItems];
    bool ok[kTileItems];
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        const int lt = lt0 + 64 * j;
        c[j] = *reinterpret_cast<const v3i_a4 *>(b.tri + 3 * (size_t)(base + (lt < cnt ? lt : 0)));
        ok[j] = (unsigned)c[j].x < (unsigned)b.nv && (unsigned)c[j].y < (unsigned)b.nv &&
                (unsigned)c[j].z < (unsigned)b.nv;
    }
    v2i_a4 p[kTileItems][3];
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        const v2i_a4 *xy = reinterpret_cast<const v2i_a4 *>(b.xy_in);
        if (b.nv > 0) {   // (uniform)
            p[j][0] = xy[ok[j] ? c[j].x : 0];
            p[j][1] = xy[ok[j] ? c[j].y : 0];
            p[j][2] = xy[ok[j] ? c[j].z : 0];
        }
    }
    int nflip = 0;
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        const int lt = lt0 + 64 * j;
        if (lt >= cnt) {
            ok[j] = false;
            continue;
        }
        const int t = base + lt;
        if (!ok[j]) {
            report(b.err, 1ull + t, -1);
        } else {
            // differences of valid coordinates fit 32 bits; others have
            // failed the build already (code -2 ranks first)
            const v2i_a4 pa = p[j][0], pb = p[j][1], pc = p[j][2];
            const long long o = (long long)(int)((unsigned)pb.x - (unsigned)pa.x) * (int)((unsigned)pc.y - (unsigned)pa.y) -
                                (long long)(int)((unsigned)pb.y - (unsigned)pa.y) * (int)((unsigned)pc.x - (unsigned)pa.x);
            if (o == 0) {
                report(b.err, 1ull + t, -3);
                ok[j] = false;
            } else if (o < 0) {
                const int s = c[j].y;
                c[j].y = c[j].z;
                c[j].z = s;
                nflip++;
            }
        }
        if (!ok[j]) c[j].x = -1;   // joins no group
        *reinterpret_cast<v3i_a4 *>(b.org + 3 * (size_t)t) = c[j];
    }
    __syncthreads();
    if (nflip) atomicAdd(&s_flip, nflip);
    int g[kTileItems][3], place[kTileItems][3];
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        triangle_groups(b, ok[j], c[j], g[j]);
#pragma unroll
        for (int i = 0; i < 3; i++) place[j][i] = bin_add(s_bin, b.count, g[j][i], w0);
    }
    __syncthreads();
    for (int k = tid; k < kBins; k += 256) {
        const int n = s_bin[k];
        if (n) s_bin[k] = atomicAdd(&b.count[w0 + k], n);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
#pragma unroll
        for (int i = 0; i < 3; i++) {
            if (g[j][i] < 0) continue;
            const int w = g[j][i] - w0, at = place[j][i] + ((unsigned)w < (unsigned)kBins ? s_bin[w] : 0);
            if (at < b.cap) b.list[(size_t)g[j][i] * b.cap + at] = base + lt0 + 64 * j;
        }
    }
    if (tid == 0 && s_flip) atomicAdd(b.nflipped, s_flip);
}

// The LDS edge table.  A slot is 0, or an edge with one or two half-edges:
//   bits 0-30   the edge's other end
//   bit 31      used
//   bits 32-38  the owner's index in its group
//   bit 39      the first half-edge leaves the owner
//   bits 40-51  the first half-edge's id in the workgroup
//   bits 52-63  the second's id + 1, 0 before it comes
// Ids are below 3 kGroupCap = 3072.
struct GroupEdge {
    uint32_t other, own, out;   // other end; owner's index in the group; 1: leaves the owner
};
constexpr uint32_t kUsed = 1u << 31;
static_assert(3 * kGroupCap < 4095, "ids of 12 bits");

// Edge i of triangle corners c, as its group sees it; false when it belongs to
// another group.
__device__ __forceinline__ bool group_edge(const BuildBuffers &b, v3i_a4 c, int i, int group, GroupEdge &e) {
    const int u = i == 0 ? c.x : (i == 1 ? c.y : c.z), v = i == 0 ? c.y : (i == 1 ? c.z : c.x);
    const int o = edge_owner(u, v, b.near);
    e.other = (uint32_t)(o == u ? v : u);
    e.own = (uint32_t)o - ((uint32_t)group << kShift);
    e.out = o == u;
    return (o >> kShift) == group;
}

__device__ __forceinline__ uint32_t edge_hash(const GroupEdge &e) {
    return e.other * 0x9E3779B1u + e.own * 0x85EBCA6Bu;
}

// Puts half-edge id into the table; returns its edge's slot, or -1 when the
// table is full.  dup: the edge has another half-edge in this direction, or
// two already.
__device__ __forceinline__ int edge_insert(unsigned long long *table, const GroupEdge &e, int id, bool &dup) {
    uint32_t q = edge_hash(e) >> (32 - 10);
    static_assert(kSlots == 1 << 10, "slots from the hash's top bits");
    const uint32_t key = e.other | kUsed;
    const unsigned long long mine = (unsigned long long)(e.own | (e.out << 7) | ((uint32_t)id << 8)) << 32 | key;
    for (int k = 0; k < kSlots; k++) {
        const unsigned long long was = atomicCAS(&table[q], 0ull, mine);
        if (was == 0ull) return (int)q;
        const uint32_t hi = (uint32_t)(was >> 32);
        if ((uint32_t)was == key && ((hi ^ e.own) & 127u) == 0) {
            const unsigned long long old = atomicOr(&table[q], (unsigned long long)(id + 1) << 52);
            dup |= (old >> 52) != 0 || ((hi >> 7) & 1u) == e.out;
            return (int)q;
        }
        q = (q + 1) & (kSlots - 1);
    }
    return -1;
}

// The id of the other half-edge in slot s, or -1 on the boundary.
__device__ __forceinline__ int edge_mate(unsigned long long s, int id) {
    const int first = (int)(s >> 40) & 0xfff, second = (int)(s >> 52) - 1;
    return id == first ? second : first;
}

__global__ void __launch_bounds__(256) k_match(BuildBuffers b) {
    __shared__ unsigned long long s_table[kSlots];
    __shared__ int s_tri[kGroupCap];
    constexpr int kIt = kGroupCap / 256;
    const int tid = threadIdx.x, g = xcd_run(blockIdx.x, b.nparts);
    const int n = b.count[g];
    if (n == 0) return;   // (uniform)
    if (n > b.cap) {
        if (tid == 0) {
            b.cursor[g] = 1;
            atomicAdd(b.nbig, 1);
        }
        return;
    }
    const int32_t *list = b.list + (size_t)g * b.cap;
    int t[kIt];
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        if (256 * j >= n) continue;   // (uniform)
        t[j] = list[256 * j + tid < n ? 256 * j + tid : 0];
    }
    for (int k = tid; k < kSlots; k += 256) s_table[k] = 0ull;
    v3i_a4 c[kIt];
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        if (256 * j >= n) continue;
        c[j] = *reinterpret_cast<const v3i_a4 *>(b.org + 3 * (size_t)t[j]);
        s_tri[256 * j + tid] = t[j];
    }
    __syncthreads();
    int slot[kIt][3];   // -1: not this group's
    bool full = false;
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        if (256 * j >= n) continue;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            slot[j][i] = -1;
            GroupEdge e;
            if (256 * j + tid >= n || !group_edge(b, c[j], i, g, e)) continue;
            bool dup = false;
            slot[j][i] = edge_insert(s_table, e, 3 * (256 * j + tid) + i, dup);
            full |= slot[j][i] < 0;
            if (dup) report(b.err, 1ull + b.nt + 3ull * t[j] + i, -4);
        }
    }
    if (__syncthreads_or(full)) {   // (uniform)
        if (tid == 0) {
            b.cursor[g] = 1;
            atomicAdd(b.nbig, 1);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        if (256 * j >= n) continue;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            if (slot[j][i] < 0) continue;
            const int m = edge_mate(s_table[slot[j][i]], 3 * (256 * j + tid) + i);
            const int q = m < 0 ? 0 : (int)((unsigned)m / 3u) & (kGroupCap - 1);   // (ids of a repeated edge run together)
            b.twin[3 * (size_t)t[j] + i] = m < 0 ? -1 : 3 * s_tri[q] + (m - 3 * q);
        }
    }
}

// ---- groups too large for k_match ------------------------------------------

// Places in the list for the groups that k_match left out (cursor != 0), in
// any order; a group's cursor is its place + 1.  Its classes, about
// kClassSplit triangles each, are listed.
__global__ void __launch_bounds__(256) k_part_alloc(BuildBuffers b) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= b.nparts || b.cursor[g] == 0) return;
    const int n = b.count[g], k = (n + kClassSplit - 1) / kClassSplit;
    b.cursor[g] = atomicAdd(b.total, n) + 1;
    const int at = atomicAdd(b.ntasks, k);
    for (int r = 0; r < k; r++) b.tasks[at + r] = {g, r, k};   // at most build_tasks() in all
}

__global__ void __launch_bounds__(256) k_scatter(BuildBuffers b) {
    const int lane = __lane_id();
    const int t = blockIdx.x * 256 + threadIdx.x;
    v3i_a4 c = {-1, -1, -1};
    if (t < b.nt) c = *reinterpret_cast<const v3i_a4 *>(b.org + 3 * (size_t)t);
    int g[3];
    triangle_groups(b, c.x >= 0, c, g);
#pragma unroll
    for (int i = 0; i < 3; i++) {
        unsigned long long todo = __ballot(g[i] >= 0 && b.cursor[g[i] < 0 ? 0 : g[i]] != 0);
        while (todo) {   // (uniform)
            const int gl = __builtin_amdgcn_readlane(g[i], __ffsll((long long)todo) - 1);
            const unsigned long long same = __ballot(g[i] == gl);
            const int at = add_together(&b.cursor[gl], same, lane) - 1;
            if ((same >> lane) & 1) b.list[at] = t;
            todo &= ~same;
        }
    }
}

// One class of a large group: the edges of the group that hash into the class.
// A class whose edges still do not fit the table (an edge repeated without
// end, so an error, or a freak of the hash) compares its half-edges one by
// one.  The scans stop once an error is known.
__device__ void match_class(const BuildBuffers &b, unsigned long long *s_table, int *s_he, int *s_n, ClassTask task) {
    const int tid = threadIdx.x, g = task.group, n = b.count[g], first = b.cursor[g] - 1 - n;
    const uint32_t classes = (uint32_t)task.classes;
    auto mine = [&](const GroupEdge &e) {
        const uint32_t x = edge_hash(e);
        return ((x ^ (x >> 15)) * 0x2C1B3C6Du >> 8) % classes == (uint32_t)task.cls;
    };
    auto failed = [&]() { return __hip_atomic_load(b.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0ull; };
    // every edge of the class, f(half-edge, edge)
    auto each = [&](int k, auto f) {
        const int t = b.list[first + k];
        const v3i_a4 c = *reinterpret_cast<const v3i_a4 *>(b.org + 3 * (size_t)t);
        for (int i = 0; i < 3; i++) {
            GroupEdge e;
            if (group_edge(b, c, i, g, e) && mine(e)) f(3 * t + i, e);
        }
    };
    __syncthreads();
    for (int k = tid; k < kSlots; k += 256) s_table[k] = 0ull;
    if (tid == 0) *s_n = 0;
    bool full = false, again = false;
    for (int k0 = 0; k0 < n; k0 += 256) {   // block-uniform
        if ((k0 & 0xffff) == 0 && __syncthreads_or(failed())) return;
        if (k0 + tid >= n) continue;
        each(k0 + tid, [&](int h, const GroupEdge &e) {
            const int id = atomicAdd(s_n, 1);
            bool dup = false;
            if (id < kSlots) {
                s_he[id] = h;
                full |= edge_insert(s_table, e, id, dup) < 0;
            }
            full |= id >= kSlots;
            if (dup) report(b.err, 1ull + b.nt + h, -4);
            again |= dup;
        });
    }
    if (__syncthreads_or(again)) return;   // (uniform)
    if (!__syncthreads_or(full)) {   // (uniform)
        for (int k = tid; k < kSlots; k += 256) {
            const unsigned long long s = s_table[k];
            if (s == 0ull) continue;
            const int x = s_he[(int)(s >> 40) & 0xfff], m = (int)(s >> 52) - 1;
            b.twin[x] = m < 0 ? -1 : s_he[m];
            if (m >= 0) b.twin[s_he[m]] = x;
        }
        return;
    }
    for (int k0 = tid; k0 < n; k0 += 256) {
        bool stop = false;
        each(k0, [&](int h, const GroupEdge &e) {
            int found = -1, others = 0;
            for (int k = 0; k < n && !stop; k++) {
                if ((k & 0xfff) == 0) stop = failed();
                each(k, [&](int h2, const GroupEdge &e2) {
                    if (h2 == h || e2.other != e.other || e2.own != e.own) return;
                    found = h2;
                    others += e2.out == e.out ? 2 : 1;
                });
            }
            if (others > 1) report(b.err, 1ull + b.nt + h, -4);
            b.twin[h] = found;
        });
        if (stop) return;
    }
}

__global__ void __launch_bounds__(256) k_match_class(BuildBuffers b) {
    __shared__ unsigned long long s_table[kSlots];
    __shared__ int s_he[kSlots];
    __shared__ int s_n;
    const int ntasks = *b.ntasks;
    for (int k = blockIdx.x; k < ntasks; k += kClassBlocks) match_class(b, s_table, s_he, &s_n, b.tasks[k]);
}

// ---------------------------------------------------------------------------
// compact half-edge encoding
// ---------------------------------------------------------------------------

// 16-bit offset of v from base, or kEsc16 when it does not fit (or is 0 and
// zero is reserved: twins, where 0 means boundary).
__device__ __forceinline__ int off16(int v, int base, bool zero_reserved) {
    const int d = v - base;
    return (d > kEsc16 && d <= 32767 && !(zero_reserved && d == 0)) ? d : kEsc16;
}

// One thread per triangle: its record and its three twin offsets; the
// escapes are counted (one atomic per wave that has any).
__global__ void __launch_bounds__(256) k_compact_encode(const int32_t *__restrict__ org,
                                                        const int32_t *__restrict__ twin, int nt, int2 *org8,
                                                        int16_t *twin16, int32_t *nesc) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    int n = 0;
    if (t < nt) {
        const int v0 = org[3 * t], v1 = org[3 * t + 1], v2 = org[3 * t + 2];
        const int d1 = off16(v1, v0, false), d2 = off16(v2, v0, false);
        n += (d1 == kEsc16) + (d2 == kEsc16);
        org8[t] = make_int2(v0, (d1 & 0xffff) | (d2 << 16));
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const int h = 3 * t + i, g = twin[h];
            const int d = g < 0 ? 0 : off16(g, h, true);
            n += d == kEsc16;
            twin16[h] = (int16_t)d;
        }
    }
    const unsigned long long any = __ballot(n != 0);
    if (any) {
        int w = n;
        for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o);
        if (__lane_id() == __ffsll((long long)any) - 1) atomicAdd(nesc, w);
    }
}

__device__ __forceinline__ void esc_insert(int32_t *esc, int32_t mask, int32_t key, int32_t val) {
    uint32_t slot = esc_hash(key) & (uint32_t)mask;
    for (int k = 0; k <= mask; k++) {
        const int32_t prev = atomicCAS(esc + 2 * slot, kEscEmpty, key);
        if (prev == kEscEmpty || prev == key) {
            esc[2 * slot + 1] = val;
            return;
        }
        slot = (slot + 1) & (uint32_t)mask;
    }
}

__global__ void k_esc_clear(int32_t *esc, int n) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
        esc[k] = (k & 1) ? 0 : kEscEmpty;
}

// Every value the encoder could not fit goes into the table.
__global__ void __launch_bounds__(256) k_compact_escapes(const int32_t *__restrict__ org,
                                                         const int32_t *__restrict__ twin, int nt, int32_t *esc,
                                                         int32_t mask) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const int v0 = org[3 * t];
#pragma unroll
    for (int i = 1; i < 3; i++) {
        const int v = org[3 * t + i];
        if (off16(v, v0, false) == kEsc16) esc_insert(esc, mask, ~(3 * t + i), v);
    }
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const int h = 3 * t + i, g = twin[h];
        if (g >= 0 && off16(g, h, true) == kEsc16) esc_insert(esc, mask, h, g);
    }
}

__device__ __forceinline__ int32_t esc_get(const int32_t *esc, int32_t mask, int32_t key) {
    uint32_t slot = esc_hash(key) & (uint32_t)mask;
    for (int k = 0; k <= mask; k++) {
        const int32_t kk = esc[2 * slot];
        if (kk == key) return esc[2 * slot + 1];
        if (kk == kEscEmpty) break;
        slot = (slot + 1) & (uint32_t)mask;
    }
    return -1;
}

__global__ void __launch_bounds__(256) k_compact_decode(const int2 *__restrict__ org8,
                                                        const int16_t *__restrict__ twin16,
                                                        const int32_t *__restrict__ esc, int32_t mask, int nt,
                                                        int32_t *org, int32_t *twin) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const int2 r = org8[t];
    const int d[3] = {0, (int)(int16_t)(r.y & 0xffff), r.y >> 16};
    org[3 * t] = r.x;
#pragma unroll
    for (int i = 1; i < 3; i++) org[3 * t + i] = d[i] == kEsc16 ? esc_get(esc, mask, ~(3 * t + i)) : r.x + d[i];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const int h = 3 * t + i, v = twin16[h];
        twin[h] = v == 0 ? -1 : (v == kEsc16 ? esc_get(esc, mask, h) : h + v);
    }
}

inline int grid_for(long long n, int block, int cap = 1 << 16) {
    long long g = (n + block - 1) / block;
    if (g < 1) g = 1;
    return (int)(g > cap ? cap : g);
}

}  // namespace

BuildSizes build_sizes(int64_t nv, int64_t nt) {
    BuildSizes z;
    z.parts = (nv + kBuildGroup - 1) / kBuildGroup;
    z.tasks = 3 * nt / kClassSplit + z.parts + 1;
    // 12 bytes a vertex and 24 a triangle are enough for full lists unless
    // most vertices are in no triangle; lists then are shorter
    const int64_t bytes = 12 * nv + 24 * nt + 65536 - 8 * z.parts - (int64_t)sizeof(ClassTask) * z.tasks;
    z.cap = z.parts > 0 ? bytes / (4 * z.parts) : kGroupCap;
    if (z.cap > kGroupCap) z.cap = kGroupCap;
    z.list = z.parts * z.cap > 3 * nt ? z.parts * z.cap : 3 * nt;   // large groups' lists: 3 nt at most
    return z;
}

hipError_t launch_build(const BuildBuffers &b, hipStream_t s) {
    const int tiles = (b.nt + kTileTri - 1) / kTileTri;
    const int copies = (int)(((int64_t)b.nv + 256 * kCopyItems - 1) / (256 * kCopyItems));
    if (tiles + copies > 0) hipLaunchKernelGGL(k_orient, dim3(tiles + copies), dim3(256), 0, s, b, tiles);
    if (tiles > 0 && b.nparts > 0) hipLaunchKernelGGL(k_match, dim3(b.nparts), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_build_large(const BuildBuffers &b, hipStream_t s) {
    hipLaunchKernelGGL(k_part_alloc, dim3((b.nparts + 255) / 256), dim3(256), 0, s, b);
    hipLaunchKernelGGL(k_scatter, dim3(b.nt / 256 + 1), dim3(256), 0, s, b);
    hipLaunchKernelGGL(k_match_class, dim3(kClassBlocks), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_compact_encode(const CompactBuffers &c, hipStream_t s) {
    if (c.nt > 0)
        hipLaunchKernelGGL(k_compact_encode, dim3((c.nt + 255) / 256), dim3(256), 0, s, c.org, c.twin, c.nt, c.org8,
                           c.twin16, c.nesc);
    return hipGetLastError();
}

hipError_t launch_compact_escapes(const CompactBuffers &c, hipStream_t s) {
    const long long n = 2ll * ((long long)c.esc_mask + 1);
    hipLaunchKernelGGL(k_esc_clear, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, c.esc, (int)n);
    if (c.nt > 0)
        hipLaunchKernelGGL(k_compact_escapes, dim3((c.nt + 255) / 256), dim3(256), 0, s, c.org, c.twin, c.nt, c.esc,
                           c.esc_mask);
    return hipGetLastError();
}

hipError_t launch_compact_decode(const CompactBuffers &c, int32_t *org, int32_t *twin, hipStream_t s) {
    if (c.nt > 0)
        hipLaunchKernelGGL(k_compact_decode, dim3((c.nt + 255) / 256), dim3(256), 0, s, c.org8, c.twin16, c.esc,
                           c.esc_mask, c.nt, org, twin);
    return hipGetLastError();
}

}  // namespace gp
