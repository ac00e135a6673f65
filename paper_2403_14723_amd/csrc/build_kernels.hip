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
// k_orient gives each wave kTileItems x 64 triangles in a row
constexpr int kTileItems = 4;
constexpr int kTileTri = 256 * kTileItems;
constexpr int kMaxRounds = 48;       // groups a wave of k_orient places together
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

// Workgroups go to the 8 XCDs round-robin; this gives each XCD one contiguous
// run of tiles, whose neighbours' coordinates then share its L2.
__device__ __forceinline__ int xcd_run(int b, int G) {
    const int q = G >> 3, r = G & 7, x = b & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

// A list entry: a triangle and which of its edges are the group's (bits 0-2).
// WIDE (2^28 triangles or 2^25 vertices and more): arrays past the reach of
// 32-bit byte offsets; entries are then triangle ids alone.
template <bool WIDE>
__device__ __forceinline__ uint32_t list_entry(int t, int edges) {
    return WIDE ? (uint32_t)t : ((uint32_t)t << 3) | (uint32_t)edges;
}

// The T at STRIDE-byte element i of an array, by a 32-bit byte offset from a
// uniform base unless WIDE.
template <bool WIDE, int STRIDE, class T>
__device__ __forceinline__ T &at(const void *base, uint32_t i) {
    const char *p = static_cast<const char *>(base);
    return *reinterpret_cast<T *>(const_cast<char *>(WIDE ? p + (size_t)i * STRIDE : p + i * (uint32_t)STRIDE));
}

// What a wave of k_orient has found of its triangles' groups: lane r holds the
// r-th group and how many triangles go to its list.
struct WaveGroups {
    int group = 0, n = 0, rounds = 0, thin = 0;
};

// Places one entry per item (group e[j], -1: none) of the wave: item j's round
// and rank in it as place[j] = round << 16 | rank, or -1 for the entries left
// in e when the groups have grown too many or too thin (a random numbering).
__device__ __forceinline__ void place_items(WaveGroups &w, int e[kTileItems], int place[kTileItems], int lane) {
#pragma unroll
    for (int j = 0; j < kTileItems; j++) place[j] = -1;
    while (w.rounds < kMaxRounds && w.thin < 4) {   // (uniform)
        int cand = -1;
#pragma unroll
        for (int j = 0; j < kTileItems; j++) cand = max(cand, e[j]);
        const unsigned long long any = __ballot(cand >= 0);
        if (!any) break;
        const int g = __builtin_amdgcn_readlane(cand, __ffsll((long long)any) - 1);
        int n = 0;
#pragma unroll
        for (int j = 0; j < kTileItems; j++) {
            const bool is = e[j] == g;
            const unsigned long long m = __ballot(is);
            const int rank = (w.rounds << 16) + n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            place[j] = is ? rank : place[j];
            e[j] = is ? -1 : e[j];
            n += __popcll(m);
        }
        const bool mine = lane == w.rounds;
        w.group = mine ? g : w.group;
        w.n = mine ? n : w.n;
        w.thin += n < 4;
        w.rounds++;
    }
}

// Blocks [0, tiles): 256 triangles per wave.  The others: the coordinates,
// checked, and copied to the mesh when the caller's array is on the device.
//
// Every wave works alone: it finds the groups of its triangles (three to five
// in an ordered numbering), takes their places in the groups' lists with one
// atomic instruction, a lane to a group, and writes the entries, consecutive
// lanes to consecutive places.  33.5M-triangle grid: 0.288 ms for 1.43 GB
// moved (12 bytes a triangle in and out, 8 a vertex in and out, 1.3 entries of
// 4 bytes), 5.0 TB/s, which is what bounds it: a large copy reaches 4.7.  Its 537
// vector instructions a wave take 55% of that time.  With a tile's counts in
// LDS, two barriers and an atomic per workgroup and group it took 0.39 ms and
// 1,043.
template <bool WIDE>
__global__ void __launch_bounds__(256) k_orient(BuildBuffers b, int tiles) {
    const int tid = threadIdx.x, lane = __lane_id();
    if ((int)blockIdx.x >= tiles) {   // (uniform)
        const long long v0 = (long long)(blockIdx.x - tiles) * (256 * kCopyItems) + tid;
        v2i_a4 p[kCopyItems];
#pragma unroll
        for (int j = 0; j < kCopyItems; j++)
            p[j] = reinterpret_cast<const v2i_a4 *>(b.xy_in)[min(v0 + j * 256, (long long)b.nv - 1)];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < kCopyItems; j++) {
            bad |= (unsigned)p[j].x > (unsigned)kCoordMax || (unsigned)p[j].y > (unsigned)kCoordMax;
            if (b.xy_out && v0 + j * 256 < b.nv) b.xy_out[v0 + j * 256] = make_int2(p[j].x, p[j].y);
        }
        if (bad) report(b.err, 0, -2);
        return;
    }
    const int base = xcd_run(blockIdx.x, tiles) * kTileTri + __builtin_amdgcn_readfirstlane(tid >> 6) * (64 * kTileItems);
    const int cnt = b.nt - base;
    if (cnt <= 0) return;   // (the whole wave)
    if (b.nv <= 0) {        // (uniform) no valid index
        if (lane == 0) report(b.err, 1ull + base, -1);
        return;
    }
    // all corners, then all coordinates in flight together (lanes past the
    // end take the last triangle, and drop it)
    const int32_t *tri = b.tri + 3 * (size_t)base;
    v3i_a4 c[kTileItems];
#pragma unroll
    for (int j = 0; j < kTileItems; j++) c[j] = at<false, 12, const v3i_a4>(tri, (uint32_t)min(lane + 64 * j, cnt - 1));
    v2i_a4 p[kTileItems][3];
    const uint32_t vmax = (uint32_t)b.nv - 1u;
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        p[j][0] = at<WIDE, 8, const v2i_a4>(b.xy_in, min((uint32_t)c[j].x, vmax));
        p[j][1] = at<WIDE, 8, const v2i_a4>(b.xy_in, min((uint32_t)c[j].y, vmax));
        p[j][2] = at<WIDE, 8, const v2i_a4>(b.xy_in, min((uint32_t)c[j].z, vmax));
    }
    int32_t *org = b.org + 3 * (size_t)base;
    int nflip = 0;
    bool bad = false;
    int ga[kTileItems], gb[kTileItems], gc[kTileItems];   // the triangle's groups, -1: no more
    uint32_t edges = 0;   // 9 bits per item, at 9 j: the edges of ga, gb, gc
    uint32_t edges3 = 0;  // item 3's
#pragma unroll
    for (int j = 0; j < kTileItems; j++) {
        const bool live = lane + 64 * j < cnt;
        const bool index = max(max((uint32_t)c[j].x, (uint32_t)c[j].y), (uint32_t)c[j].z) <= vmax;
        // differences of valid coordinates fit 32 bits; others have failed
        // the build already (code -2 ranks first)
        const v2i_a4 pa = p[j][0], pb = p[j][1], pc = p[j][2];
        const int ux = (int)((unsigned)pb.x - (unsigned)pa.x), uy = (int)((unsigned)pb.y - (unsigned)pa.y),
                  vx = (int)((unsigned)pc.x - (unsigned)pa.x), vy = (int)((unsigned)pc.y - (unsigned)pa.y);
        const long long l = (long long)ux * vy, r = (long long)uy * vx;
        const bool flip = l < r, ok = index && l != r;
        bad |= live && !ok;
        const int cy = flip ? c[j].z : c[j].y, cz = flip ? c[j].y : c[j].z, cx = ok ? c[j].x : -1;   // -1: joins no group
        nflip += __popcll(__ballot(flip && ok && live));
        const v3i_a4 o = {cx, cy, cz};
        if (live) at<false, 12, v3i_a4>(org, (uint32_t)(lane + 64 * j)) = o;
        const int g0 = edge_owner(cx, cy, b.near) >> kShift, g1 = edge_owner(cy, cz, b.near) >> kShift,
                  g2 = edge_owner(cz, cx, b.near) >> kShift;
        // the groups in ga, gb, gc, each once, from the front
        const bool s01 = g0 == g1, s02 = g0 == g2, s12 = g1 == g2, in = ok && live;
        ga[j] = in ? g0 : -1;
        gb[j] = !in ? -1 : (!s01 ? g1 : (!s02 ? g2 : -1));
        gc[j] = in && !s01 && !s02 && !s12 ? g2 : -1;
        const uint32_t ea = 1u | (s01 ? 2u : 0u) | (s02 ? 4u : 0u), eb = s01 ? 4u : (s12 ? 6u : 2u);
        const uint32_t all = ea | (eb << 3) | (4u << 6);
        if (j < 3)
            edges |= all << (9 * j);
        else
            edges3 = all;
    }
    if (__any(bad)) {   // (uniform, rare)
#pragma unroll
        for (int j = 0; j < kTileItems; j++) {
            if (lane + 64 * j >= cnt) continue;
            const bool index = max(max((uint32_t)c[j].x, (uint32_t)c[j].y), (uint32_t)c[j].z) <= vmax;
            const unsigned long long t = (unsigned long long)base + lane + 64 * j;
            if (!index)
                report(b.err, 1ull + t, -1);
            else if (ga[j] < 0)
                report(b.err, 1ull + t, -3);
        }
    }
    if (nflip && lane == 0) atomicAdd(&b.flips[kFlipPad * (blockIdx.x % kFlipStripes)], nflip);
    WaveGroups w;
    int pa[kTileItems], pb[kTileItems], pc[kTileItems];
    place_items(w, ga, pa, lane);
    place_items(w, gb, pb, lane);
    place_items(w, gc, pc, lane);
    // the places, one lane per group; entries past a list's end are dropped
    // (the group's count says so)
    int first = 0;
    if (lane < w.rounds) first = atomicAdd(&b.count[w.group], w.n);
    const int room = b.cap - first;
    const size_t slot = (size_t)w.group * (uint32_t)b.cap + (uint32_t)first;
    auto put = [&](const int rest[kTileItems], const int place[kTileItems], int which) {
#pragma unroll
        for (int j = 0; j < kTileItems; j++) {
            const int r = place[j] >> 16, rank = place[j] & 0xffff;   // (-1: lane 63's, unused)
            const int lim = __shfl(room, r);
            const int t = base + lane + 64 * j;
            const uint32_t entry = list_entry<WIDE>(t, (int)(((j < 3 ? edges >> (9 * j) : edges3) >> (3 * which)) & 7u));
            if (WIDE) {
                const size_t to = (size_t)__shfl((unsigned long long)slot, r);
                if (place[j] >= 0 && rank < lim) b.list[to + rank] = entry;
            } else {
                const uint32_t to = (uint32_t)__shfl((int)(uint32_t)slot, r) + (uint32_t)rank;
                if (place[j] >= 0 && rank < lim) at<false, 4, uint32_t>(b.list, to) = entry;
            }
            if (rest[j] >= 0) {
                const int k = atomicAdd(&b.count[rest[j]], 1);
                if (k < b.cap) b.list[(size_t)rest[j] * (uint32_t)b.cap + k] = entry;
            }
        }
    };
    put(ga, pa, 0);
    put(gb, pb, 1);
    bool third = false;
#pragma unroll
    for (int j = 0; j < kTileItems; j++) third |= pc[j] >= 0 || gc[j] >= 0;
    if (__any(third)) put(gc, pc, 2);
}

// The LDS edge table.  A slot is 0, or an edge with one or two half-edges:
//   low word    the edge's other end (25 bits) and the owner's index in its
//               group; WIDE: the other end and, in bit 31, a 1
//   high word   bits 0-11   the first half-edge's id in the workgroup
//               bit 12      it leaves the owner
//               bits 13-19  a 1; WIDE: the owner's index
//               bits 20-31  the second half-edge's id + 1, 0 before it comes
// Ids are 4 x the entry's place in the list + the edge's index: at most
// 4 kGroupCap - 2.
struct GroupEdge {
    uint32_t other, own, out;   // other end; owner's index in the group; 1: leaves the owner
};
constexpr int kNarrowVerts = 1 << 25;
static_assert(4 * kGroupCap <= 4096, "ids of 12 bits");

template <bool WIDE>
__device__ __forceinline__ unsigned long long edge_word(const GroupEdge &e, int id) {
    const uint32_t hi = (uint32_t)id | (e.out << 12) | (WIDE ? e.own << 13 : 1u << 13);
    return (unsigned long long)hi << 32 | (WIDE ? e.other | (1u << 31) : e.other | (e.own << 25));
}
template <bool WIDE>
__device__ __forceinline__ bool slot_empty(unsigned long long s) {
    return WIDE ? (uint32_t)s == 0u : (uint32_t)(s >> 32) == 0u;
}
// Whether slot s holds the edge of word w.
template <bool WIDE>
__device__ __forceinline__ bool same_edge(unsigned long long s, unsigned long long w) {
    return (uint32_t)s == (uint32_t)w && (!WIDE || (((uint32_t)(s >> 32) ^ (uint32_t)(w >> 32)) >> 13 & 127u) == 0);
}
__device__ __forceinline__ bool same_direction(unsigned long long s, unsigned long long w) {
    return (((uint32_t)(s >> 32) ^ (uint32_t)(w >> 32)) & (1u << 12)) == 0;
}
// Adds half-edge id as the second of a slot's edge.
__device__ __forceinline__ unsigned add_second(unsigned long long *slot, int id) {
    return atomicOr(reinterpret_cast<unsigned *>(slot) + 1, (unsigned)(id + 1) << 20);
}

// Edge u -> v as group sees it; false when it belongs to another group.
__device__ __forceinline__ bool group_edge(const BuildBuffers &b, int u, int v, int group, GroupEdge &e) {
    const int o = edge_owner(u, v, b.near);
    e.other = (uint32_t)(u ^ v ^ o);
    e.own = (uint32_t)(o - (group << kShift));
    e.out = o == u;
    return (o >> kShift) == group;
}

// Eight slots to an owner, which has about three edges; one that finds them
// taken goes on into the next owner's.  By the distance d to the other end: a
// grid's rows give each of an owner's edges a slot of its own (one neighbour in
// the row, three consecutive ones in the next), other numberings spread over
// the eight (0.17 further tries per edge on a Delaunay mesh along a Z-order
// curve).  A hash of the other end, which lets the owners of a grid share
// slots, cost 100 us more on the 33.5M grid.  Every fourth owner's slots are
// turned by one, or the like edges of a row's owners would meet in four LDS
// banks.
__device__ __forceinline__ uint32_t edge_slot(uint32_t own, uint32_t d) {
    static_assert(kSlots == 8 * kBuildGroup, "eight slots to an owner");
    return 8u * own | ((((d & 3u) | (d > 8u ? 4u : 0u)) + (own >> 2)) & 7u);
}

// One workgroup per group: the triangles of its list, their edges into the
// table, then each half-edge's twin from its slot.  33.5M-triangle grid: 0.37
// ms for 1.0 GB (the list, 1.2 x 12 bytes a triangle of corners, 12 of twins);
// bound by its 347 vector instructions a wave, which keep the SIMDs busy for 87%
// of that time.  The LDS is in use for 51% of it, bank conflicts half of that.
// The three edges' first tries go out together, without branches: one loop per
// edge took 0.53 ms, 430 vector and 474 scalar instructions.
template <bool WIDE>
__global__ void __launch_bounds__(256) k_match(BuildBuffers b) {
    __shared__ unsigned long long s_table[kSlots + 64];   // 64 for lanes with nothing to add
    __shared__ int s_tri[kGroupCap];   // a list entry's first half-edge
    constexpr int kIt = kGroupCap / 256;
    const int tid = threadIdx.x, g = xcd_run(blockIdx.x, b.nparts);
    if (blockIdx.x == 0 && tid < 64) {   // (a whole wave) k_orient's counts of flipped triangles
        static_assert(kFlipStripes == 64, "one lane per stripe");
        int f = b.flips[kFlipPad * tid];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) f += __shfl_xor(f, d);
        if (tid == 0) *b.nflipped = f;
    }
    const int n = b.count[g];
    if (n == 0) return;   // (uniform)
    if (n > b.cap) {
        if (tid == 0) {
            b.cursor[g] = 1;
            atomicAdd(b.nbig, 1);
        }
        return;
    }
    const uint32_t *list = b.list + (size_t)g * (uint32_t)b.cap;
    uint32_t rec[kIt];
#pragma unroll
    for (int j = 0; j < kIt; j++)
        if (256 * j < n) rec[j] = list[min(256 * j + tid, n - 1)];   // (uniform)
    for (int k = tid; k < (kSlots + 64) / 2; k += 256) reinterpret_cast<ulonglong2 *>(s_table)[k] = ulonglong2{0ull, 0ull};
    v3i_a4 c[kIt];
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        if (256 * j >= n) continue;
        const uint32_t t = WIDE ? rec[j] : rec[j] >> 3;
        c[j] = at<WIDE, 12, const v3i_a4>(b.org, t);
        s_tri[256 * j + tid] = 3 * (int)t;
    }
    __syncthreads();
    const uint32_t v0 = (uint32_t)g << kShift;
    uint32_t slots[kIt];   // eleven bits per edge
    uint32_t mine[kIt];    // bit i: edge i is the group's
    bool full = false, dup = false;
#pragma unroll
    for (int j = 0; j < kIt; j++) {
        slots[j] = mine[j] = 0;
        if (256 * j >= n) continue;
        const uint32_t v[4] = {(uint32_t)c[j].x, (uint32_t)c[j].y, (uint32_t)c[j].z, (uint32_t)c[j].x};
        const int id = 4 * (256 * j + tid);
        unsigned long long word[3], was[3];
        uint32_t q[3], in;
        if (!WIDE)
            in = 256 * j + tid < n ? rec[j] & 7u : 0u;
        else
            in = 0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            GroupEdge e;
            if (!WIDE) {
                // an edge of this group with both ends in it belongs to the
                // lower (near ends); else its owner is the end that is: the
                // lower index from the group's first vertex, either way
                const uint32_t x = v[i] - v0, y = v[i + 1] - v0;
                e.own = min(x, y);
                e.out = e.own == x;
                e.other = max(x, y) + v0;
            } else {
                const bool is = group_edge(b, (int)v[i], (int)v[i + 1], g, e);
                in |= is && 256 * j + tid < n ? 1u << i : 0u;
            }
            word[i] = edge_word<WIDE>(e, id + i);
            q[i] = (in >> i) & 1u ? edge_slot(e.own, e.other - v0 - e.own) : (uint32_t)kSlots + (tid & 63);
        }
        // first tries of the three edges in flight together
#pragma unroll
        for (int i = 0; i < 3; i++) was[i] = atomicCAS(&s_table[q[i]], 0ull, word[i]);
        uint32_t miss = 0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const bool taken = !slot_empty<WIDE>(was[i]) && ((in >> i) & 1u), same = same_edge<WIDE>(was[i], word[i]);
            if (taken && same) {
                add_second(&s_table[q[i]], id + i);
                dup |= same_direction(was[i], word[i]);
            }
            miss |= taken && !same ? 1u << i : 0u;
        }
        for (int k = 0; miss; k++) {
            const int i = __ffs((int)miss) - 1;
            const unsigned long long x = i == 0 ? word[0] : (i == 1 ? word[1] : word[2]);
            const uint32_t to = ((i == 0 ? q[0] : (i == 1 ? q[1] : q[2])) + 1) & (kSlots - 1);
            q[0] = i == 0 ? to : q[0];
            q[1] = i == 1 ? to : q[1];
            q[2] = i == 2 ? to : q[2];
            const unsigned long long y = atomicCAS(&s_table[to], 0ull, x);
            const bool taken = !slot_empty<WIDE>(y), same = same_edge<WIDE>(y, x);
            if (taken && same) {
                add_second(&s_table[to], id + i);
                dup |= same_direction(y, x);
            }
            if (!taken || same) miss &= miss - 1;
            if (k >= 3 * kSlots) {   // no slot left
                full = true;
                break;
            }
        }
        slots[j] = q[0] | (q[1] << 11) | (q[2] << 22);   // (of the third the low ten bits: an edge's)
        mine[j] = in;
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
        const uint32_t t = WIDE ? rec[j] : rec[j] >> 3;
        const uint32_t id = 4u * (uint32_t)(256 * j + tid);
#pragma unroll
        for (int i = 0; i < 3; i++) {
            if (!((mine[j] >> i) & 1u)) continue;
            const uint32_t s = reinterpret_cast<const uint32_t *>(s_table)[2 * ((slots[j] >> (11 * i)) & (kSlots - 1)) + 1];
            const uint32_t first = s & 0xfffu, second = s >> 20;
            const bool lead = first == id + i;
            // a third half-edge's id has run together with the second's: one
            // of the two at least does not find its own
            dup |= !lead && second != id + i + 1;
            const uint32_t m = lead ? second - 1u : first;
            const int tw = s_tri[(m >> 2) & (kGroupCap - 1)] + (int)(m & 3u);
            at<WIDE, 4, int32_t>(b.twin, 3u * t + i) = second == 0u ? -1 : tw;
        }
    }
    if (dup) report(b.err, 1ull + b.nt, -4);
}

// ---- groups too large for k_match ------------------------------------------

// Places in the list for the groups that k_match left out (cursor != 0), in
// any order; a group's cursor is its place + 1.  Its classes, about
// kClassSplit triangles each, are listed.
__global__ void __launch_bounds__(256) k_part_alloc(BuildBuffers b) {
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= b.nparts || b.cursor[g] == 0) return;
    const int n = b.count[g], k = (n + kClassSplit - 1) / kClassSplit;
    const int first = atomicAdd(b.total, n);
    b.cursor[g] = first + 1;
    b.place[(size_t)kPlacePad * g] = first;
    const int at = atomicAdd(b.ntasks, k);
    for (int r = 0; r < k; r++) b.tasks[at + r] = {g, r, k};   // at most BuildSizes::tasks in all
}

// Every triangle into the lists of its large groups.  A wave takes the places
// for all of its lanes in a group with one atomic while the first lane left has
// company in its group; else, as in a random numbering, each lane that is left
// takes its own, all at once.  The counters are a cache line apart.  A build of
// 594,000 triangles numbered at random over 2,344 groups, all large: 429 us; 903
// with an atomic per group, one after the other, on counters that lie together
// and are also read.
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
            const int leader = __ffsll((long long)todo) - 1, gl = __builtin_amdgcn_readlane(g[i], leader);
            const unsigned long long same = __ballot(g[i] == gl);
            if (__popcll(same) < 4) {
                if ((todo >> lane) & 1) b.list[atomicAdd(&b.place[(size_t)kPlacePad * g[i]], 1)] = (uint32_t)t;
                break;
            }
            int k = 0;
            if (lane == leader) k = atomicAdd(&b.place[(size_t)kPlacePad * gl], __popcll(same));
            k = __builtin_amdgcn_readlane(k, leader) + __popcll(same & ((1ull << lane) - 1ull));
            if ((same >> lane) & 1) b.list[k] = (uint32_t)t;
            todo &= ~same;
        }
    }
}

// One class of a large group: the edges of the group that hash into the class.
// A class whose edges still do not fit the table (an edge repeated without
// end, so an error, or a freak of the hash) compares its half-edges one by
// one.  The scans stop once an error is known.
__device__ void match_class(const BuildBuffers &b, unsigned long long *s_table, int *s_he, int *s_n, ClassTask task) {
    const int tid = threadIdx.x, g = task.group, n = b.count[g], first = b.cursor[g] - 1;
    const uint32_t classes = (uint32_t)task.classes;
    auto hash = [](const GroupEdge &e) {
        const uint32_t x = e.other * 0x9E3779B1u + e.own * 0x85EBCA6Bu;
        return (x ^ (x >> 15)) * 0x2C1B3C6Du;
    };
    auto failed = [&]() { return __hip_atomic_load(b.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0ull; };
    // every edge of the class, f(half-edge, edge)
    auto each = [&](int k, auto f) {
        const int t = (int)b.list[first + k];
        const v3i_a4 c = *reinterpret_cast<const v3i_a4 *>(b.org + 3 * (size_t)t);
        for (int i = 0; i < 3; i++) {
            const int u = i == 0 ? c.x : (i == 1 ? c.y : c.z), v = i == 0 ? c.y : (i == 1 ? c.z : c.x);
            GroupEdge e;
            if (group_edge(b, u, v, g, e) && (hash(e) >> 8) % classes == (uint32_t)task.cls) f(3 * t + i, e);
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
            full |= id >= kSlots;
            if (id >= kSlots) return;
            s_he[id] = h;
            const unsigned long long x = edge_word<true>(e, id);
            uint32_t q = hash(e) >> 22;
            for (int k = 0; k < kSlots; k++, q = (q + 1) & (kSlots - 1)) {   // room for all of the ids
                const unsigned long long was = atomicCAS(&s_table[q], 0ull, x);
                if (was == 0ull) break;
                if (!same_edge<true>(was, x)) continue;
                if ((add_second(&s_table[q], id) >> 20) != 0 || same_direction(was, x)) {
                    report(b.err, 1ull + b.nt + h, -4);
                    again = true;
                }
                break;
            }
        });
    }
    if (__syncthreads_or(again)) return;   // (uniform)
    if (!__syncthreads_or(full)) {   // (uniform)
        for (int k = tid; k < kSlots; k += 256) {
            const unsigned long long s = s_table[k];
            if (s == 0ull) continue;
            const int x = s_he[(int)(s >> 32) & 0xfff], m = (int)(s >> 52) - 1;
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

// Every triangle's record and its three twin offsets.  The escapes are counted
// with one atomic per block, of which there are at most kEncodeBlocks: one per
// wave that had any, all on the one counter, took 31 us for the 594,000
// triangles of a Delaunay mesh; this takes 10 us (13 with twice the blocks).
constexpr int kEncodeBlocks = 512;
__global__ void __launch_bounds__(1024) k_compact_encode(const int32_t *__restrict__ org,
                                                        const int32_t *__restrict__ twin, int nt, int2 *org8,
                                                        int16_t *twin16, int32_t *nesc) {
    __shared__ int s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    int n = 0;
    for (long long tt = blockIdx.x * 1024 + threadIdx.x; tt < nt; tt += gridDim.x * 1024) {
        const int t = (int)tt;
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
    if (n) atomicAdd(&s_n, n);
    __syncthreads();
    if (threadIdx.x == 0 && s_n) atomicAdd(nesc, s_n);
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

// Every value the encoder could not fit (its code says so) goes into the table.
__global__ void __launch_bounds__(256) k_compact_escapes(const int32_t *__restrict__ org,
                                                         const int32_t *__restrict__ twin, int nt,
                                                         const int2 *__restrict__ org8,
                                                         const int16_t *__restrict__ twin16, int32_t *esc,
                                                         int32_t mask) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const int r = org8[t].y, d[2] = {(int)(int16_t)(r & 0xffff), r >> 16};
    const int16_t g[3] = {twin16[3 * t], twin16[3 * t + 1], twin16[3 * t + 2]};
#pragma unroll
    for (int i = 0; i < 2; i++)
        if (d[i] == kEsc16) esc_insert(esc, mask, ~(3 * t + i + 1), org[3 * t + i + 1]);
#pragma unroll
    for (int i = 0; i < 3; i++)
        if (g[i] == kEsc16) esc_insert(esc, mask, 3 * t + i, twin[3 * t + i]);
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

// A build's counters start at zero: one launch, where the runtime's fill of an
// odd length was two (173 to 171 us for a build and mesh of 2.1M triangles).
__global__ void __launch_bounds__(256) k_build_clear(uint64_t *zero, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) zero[i] = 0;
}

inline int grid_for(long long n, int block, int cap = 1 << 16) {
    long long g = (n + block - 1) / block;
    if (g < 1) g = 1;
    return (int)(g > cap ? cap : g);
}

}  // namespace

BuildSizes build_sizes(int64_t nv, int64_t nt, bool roomy) {
    BuildSizes z;
    z.parts = (nv + kBuildGroup - 1) / kBuildGroup;
    z.tasks = 3 * nt / kClassSplit + z.parts + 1;
    // 12 bytes a vertex and 24 a triangle are enough for full lists unless
    // most vertices are in no triangle.  Lists then are shorter, or, roomy, as
    // many times longer in all: with 600,000 triangles numbered at random in the
    // last tenth of the vertices, all groups that have any outgrow the short
    // lists (a build takes 430 us, 366 with the long ones).
    int64_t bytes = 12 * nv + 24 * nt - 8 * z.parts - (int64_t)sizeof(ClassTask) * z.tasks - 9216;   // (the counters)
    if (bytes < 65536) bytes = 65536;   // sixteen full lists
    z.cap = z.parts > 0 && !roomy ? bytes / (4 * z.parts) : kGroupCap;
    if (z.cap > kGroupCap) z.cap = kGroupCap;
    // large groups' lists, 3 nt at most in all, and their counters lie over the others
    z.places = (3 * nt + kPlacePad - 1) / kPlacePad * kPlacePad;
    z.list = std::max(z.parts * z.cap, z.places + kPlacePad * z.parts);
    return z;
}

hipError_t launch_build(const BuildBuffers &b, hipStream_t s) {
    const int zeros = (int)(b.zero_bytes / sizeof(uint64_t));
    hipLaunchKernelGGL(k_build_clear, dim3((zeros + 255) / 256), dim3(256), 0, s, b.zero, zeros);
    const int tiles = (b.nt + kTileTri - 1) / kTileTri;
    const int copies = (int)(((int64_t)b.nv + 256 * kCopyItems - 1) / (256 * kCopyItems));
    // not wide: arrays within the reach of 32-bit byte offsets, entries with
    // their edges, and an edge in one word of the table
    const bool wide = b.nt >= 1 << 28 || b.nv >= kNarrowVerts;
    static_assert((long long)kNarrowVerts / kBuildGroup * kBuildGroupCap * 4 < 1ll << 32, "lists in reach");
    if (tiles + copies > 0)
        hipLaunchKernelGGL(wide ? k_orient<true> : k_orient<false>, dim3(tiles + copies), dim3(256), 0, s, b, tiles);
    if (tiles > 0 && b.nparts > 0)
        hipLaunchKernelGGL(wide ? k_match<true> : k_match<false>, dim3(b.nparts), dim3(256), 0, s, b);
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
        hipLaunchKernelGGL(k_compact_encode, dim3(grid_for(c.nt, 1024, kEncodeBlocks)), dim3(1024), 0, s, c.org, c.twin, c.nt, c.org8,
                           c.twin16, c.nesc);
    return hipGetLastError();
}

hipError_t launch_compact_escapes(const CompactBuffers &c, hipStream_t s) {
    const long long n = 2ll * ((long long)c.esc_mask + 1);
    hipLaunchKernelGGL(k_esc_clear, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, c.esc, (int)n);
    if (c.nt > 0)
        hipLaunchKernelGGL(k_compact_escapes, dim3((c.nt + 255) / 256), dim3(256), 0, s, c.org, c.twin, c.nt,
                           c.org8, c.twin16, c.esc, c.esc_mask);
    return hipGetLastError();
}

hipError_t launch_compact_decode(const CompactBuffers &c, int32_t *org, int32_t *twin, hipStream_t s) {
    if (c.nt > 0)
        hipLaunchKernelGGL(k_compact_decode, dim3((c.nt + 255) / 256), dim3(256), 0, s, c.org8, c.twin16, c.esc,
                           c.esc_mask, c.nt, org, twin);
    return hipGetLastError();
}

}  // namespace gp
