// Polylla pipeline kernels for gfx950 (wave64).
//
// One run processes a batch of meshes through a per-mesh descriptor table
// (a plain call is a batch of one).  Streaming kernels tile each mesh
// separately, so a workgroup never straddles two meshes and every index it
// handles is local to one mesh; data-dependent work (barrier tips, repair
// seeds, fix-ups) goes through small device lists read by persistent grids.
//
// Kernel chain (the eight kernels of the paper's Section 6 / Algorithm 7,
// regrouped so that every step reads its inputs contiguously):
//   k_label     longest edge of every triangle (Section 6.1, Algorithm 8);
//               also clears the run's counters and per-tile totals
//   k_relink    frontier bits of every half-edge (Section 6.2, Algorithm 9),
//               the seed bit of terminal edges (Section 6.3, Algorithm 10),
//               then next/prev of every frontier half-edge by turning around
//               its target / origin (Section 6.5, Algorithm 12); barrier tips
//   k_repair    middle edge at every barrier tip (Section 6.4, Algorithm 11)
//   k_fixup     next/prev again around both ends of every new frontier edge;
//               marks the seeds of the polygons that the repair split
//   k_walk      for every seed k_relink left open and every seed made by the
//               repair: move to a frontier half-edge of its polygon
//               (Section 6.5.1, Algorithm 13), walk the loop, and record its
//               minimum and length at the minimum's triangle (Section 6.6,
//               Algorithm 14).  Polygons of one or two triangles are settled
//               by k_relink itself.
//   k_tile_scan exclusive scan of the per-tile loop totals that k_relink and
//               k_walk accumulate (Section 6.7)
//   k_compact   writes seeds, loop offsets and the loops of up to sixteen
//               half-edges of every tile from its prefix (Section 6.7)
//   k_emit      copies the longer loops that k_walk kept to the offsets that
//               k_compact reserved, and walks those it did not keep
//
// Label byte per triangle (tflag):
//   bits 0-1  local index of the longest edge
//   bits 2-4  frontier bit of local edges 0..2 (the repair sets more of them)
//   bit  5    the longest edge is a terminal edge and this triangle holds its
//             seed half-edge
//   bit  6    the repair split the polygon whose seed this triangle holds
//   bit  7    from k_label to k_relink: the longest edge is tied; in k_walk: a
//             loop of a split polygon whose minimum lies here has been counted
#include <type_traits>

#include "gp_internal.h"

namespace gp {

const char *const kKernelNames[K_COUNT] = {"k_label",     "k_relink",  "k_repair", "k_fixup",
                                           "k_walk", "k_tile_scan", "k_compact", "k_emit", "k_small"};

constexpr uint32_t kSeedBit = 1u << 5;

// The mesh arrays reached through the descriptor table live in global
// memory; saying so lets the compiler use global (not flat) loads and stores
// with a scalar base and a 32-bit offset.
#define GLOBAL __attribute__((address_space(1)))
typedef GLOBAL const int32_t *gcint;
typedef GLOBAL int32_t *gint;
typedef GLOBAL const uint8_t *gcu8;
typedef GLOBAL uint8_t *gu8;
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v3i __attribute__((ext_vector_type(3)));
// three ints at 4-byte alignment (a v3i claims 16): loads of 12-byte records
typedef int v3i_a4 __attribute__((ext_vector_type(3), aligned(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

// Value of escaped field key of a compact mesh (the table holds every key an
// escaped field can ask for; -1 for an absent key: a corrupt table).
__device__ __forceinline__ int esc_lookup(const int32_t *__restrict__ esc, int32_t mask, int32_t key) {
    uint32_t slot = esc_hash(key) & (uint32_t)mask;
    for (int k = 0; k <= mask; k++) {
        const v2i e = ((GLOBAL const v2i *)esc)[slot];   // key and value in one load
        if (e.x == key) return e.y;
        if (e.x == kEscEmpty) break;
        slot = (slot + 1) & (uint32_t)mask;
    }
    return -1;
}

// Twins of a mesh, in either encoding: twin[h] (-1 on the boundary).  The
// encoding is the same for every lane of a launch over one mesh, so the
// branch on it is uniform.
struct TwinView {
    GLOBAL const int32_t *t32;
    GLOBAL const int16_t *t16;   // compact: twin - h (0: boundary, kEsc16: escaped)
    const int32_t *esc;
    int32_t mask;
    __device__ __forceinline__ int operator[](int h) const { return value(h, raw(h)); }
    // what is stored for h, to be loaded before it is known to be needed, and
    // the twin that it stands for
    __device__ __forceinline__ int raw(int h) const { return t16 ? t16[h] : t32[h]; }
    __device__ __forceinline__ int value(int h, int v) const {
        if (!t16) return v;
        if (v == 0) return -1;
        return v != kEsc16 ? h + v : esc_lookup(esc, mask, h);
    }
};

__device__ __forceinline__ TwinView twin_view(const MeshDesc &d) {
    return TwinView{(GLOBAL const int32_t *)d.twin, (GLOBAL const int16_t *)d.twin16, d.esc, d.esc_mask};
}
typedef GLOBAL const v2i *gcv2i;

// ---------------------------------------------------------------------------
// half-edge queries (implicit triangle layout, Section 4.2)
// ---------------------------------------------------------------------------

// (h >= 0 everywhere these are used; unsigned division by 3 is a multiply)
__device__ __forceinline__ int tri_of(int h) { return (int)((unsigned)h / 3u); }
__device__ __forceinline__ int he_next(int h) {
    const int t = tri_of(h);
    return (h - 3 * t == 2) ? h - 2 : h + 1;
}
__device__ __forceinline__ int he_prev(int h) {
    const int t = tri_of(h);
    return (h - 3 * t == 0) ? h + 2 : h - 1;
}

// Coordinates lie in [0, 2^30] (the build checks them), so a difference fits
// 32 bits and each square is one signed 32 x 32 -> 64-bit multiply.
__device__ __forceinline__ long long sq_len(int2 a, int2 b) {
    const int dx = b.x - a.x, dy = b.y - a.y;
    return (long long)dx * dx + (long long)dy * dy;
}

__device__ __forceinline__ bool fbit(uint32_t f, int i) { return (f >> (2 + i)) & 1u; }

__device__ __forceinline__ bool is_frontier(const uint8_t *__restrict__ tflag, int h) {
    const int t = h / 3;
    return fbit(tflag[t], h - 3 * t);
}

// ---------------------------------------------------------------------------
// wave / block helpers
// ---------------------------------------------------------------------------

// v read from the lane that DPP control CTRL names, in the rows ROW_MASK
// selects; 0 where there is no such lane or the row is not selected
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive scans over the 64 lanes of a wave; every lane must be active.
// Lanes form four rows of 16: shifts right by 1, 2, 4 and 8 lanes within each
// row scan the rows, then lane 15's total is added to row 1 and row 3, and
// lane 31's (rows 0-1) to rows 2 and 3.  One DPP add per step, no LDS.
__device__ __forceinline__ void wave_incl_scan2(int &a, int &b) {
    a += dpp_or_zero<0x111, 0xf>(a);   // row_shr:1
    b += dpp_or_zero<0x111, 0xf>(b);
    a += dpp_or_zero<0x112, 0xf>(a);   // row_shr:2
    b += dpp_or_zero<0x112, 0xf>(b);
    a += dpp_or_zero<0x114, 0xf>(a);   // row_shr:4
    b += dpp_or_zero<0x114, 0xf>(b);
    a += dpp_or_zero<0x118, 0xf>(a);   // row_shr:8
    b += dpp_or_zero<0x118, 0xf>(b);
    a += dpp_or_zero<0x142, 0xa>(a);   // row_bcast:15 into rows 1, 3
    b += dpp_or_zero<0x142, 0xa>(b);
    a += dpp_or_zero<0x143, 0xc>(a);   // row_bcast:31 into rows 2, 3
    b += dpp_or_zero<0x143, 0xc>(b);
}

__device__ __forceinline__ int wave_incl_scan(int a) {
    a += dpp_or_zero<0x111, 0xf>(a);
    a += dpp_or_zero<0x112, 0xf>(a);
    a += dpp_or_zero<0x114, 0xf>(a);
    a += dpp_or_zero<0x118, 0xf>(a);
    a += dpp_or_zero<0x142, 0xa>(a);
    a += dpp_or_zero<0x143, 0xc>(a);
    return a;
}

// Exclusive block scan of a pair; lds must hold 66 ints.
__device__ __forceinline__ void block_excl_scan2(int a, int b, int &ea, int &eb, int &ta, int &tb,
                                                 int *lds) {
    int ia = a, ib = b;
    wave_incl_scan2(ia, ib);
    const int lane = __lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    if (lane == kWave - 1) {
        lds[w] = ia;
        lds[16 + w] = ib;
    }
    __syncthreads();
    if (w == 0) {
        int xa = lane < nw ? lds[lane] : 0, xb = lane < nw ? lds[16 + lane] : 0;
        int sa = xa, sb = xb;
        wave_incl_scan2(sa, sb);
        if (lane < nw) {
            lds[32 + lane] = sa - xa;
            lds[48 + lane] = sb - xb;
        }
        if (lane == nw - 1) {
            lds[64] = sa;
            lds[65] = sb;
        }
    }
    __syncthreads();
    ea = lds[32 + w] + ia - a;
    eb = lds[48 + w] + ib - b;
    ta = lds[64];
    tb = lds[65];
    __syncthreads();
}

// Mesh of a tile: the last descriptor whose first tile is <= tile.
template <int FIELD>
__device__ __forceinline__ int find_mesh(const MeshDesc *__restrict__ d, int n, int tile) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        int t0 = FIELD == 0 ? d[mid].tri_tile0 : (FIELD == 1 ? d[mid].he_tile0 : d[mid].cmp_tile0);
        if (t0 <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Workgroups are dispatched to the 8 XCDs round-robin (block b on XCD b % 8)
// and each XCD has its own L2.  This gives every XCD one contiguous run of
// tiles, so the neighbour rows a tile gathers from were mostly touched by the
// same XCD.  A bijection of [0, G).
__device__ __forceinline__ int xcd_tile(int b, int G) {
    const int q = G >> 3, r = G & 7;
    const int x = b & 7, k = b >> 3;
    return x * q + (x < r ? x : r) + k;
}

// Prefix sums of the stripe sizes in LDS (s_pref[0..kStripes]); returns the
// total.  Called by every thread of the block.
__device__ __forceinline__ int striped_prefix(const int32_t *counts, int cap, int *s_pref) {
    static_assert(kStripes == kWave, "one lane per stripe");
    if (threadIdx.x < kWave) {
        int c = counts[threadIdx.x * kStripePad];
        c = c < 0 ? 0 : (c > cap ? cap : c);
        s_pref[threadIdx.x + 1] = wave_incl_scan(c);
        if (threadIdx.x == 0) s_pref[0] = 0;
    }
    __syncthreads();
    return s_pref[kStripes];
}

// Entry index of the g-th element of a striped list.
__device__ __forceinline__ int striped_index(const int *s_pref, int cap, int g) {
    int lo = 0, hi = kStripes - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_pref[mid] <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo * cap + (g - s_pref[lo]);
}

// The tip list's stripes: how many tips come before each (uniform loads).
struct TipStripes {
    int first[kTipStripes + 1];
    __device__ __forceinline__ TipStripes(const int32_t *counts, const TipSpan &span) {
        first[0] = 0;
#pragma unroll
        for (int s = 0; s < kTipStripes; s++)
            first[s + 1] = first[s] + max(0, min(counts[s * kStripePad], span.at[s + 1] - span.at[s]));
    }
    __device__ __forceinline__ int total() const { return first[kTipStripes]; }
    // place in the list of the g-th tip
    __device__ __forceinline__ int index(int g, const TipSpan &span) const {
        int at = g;
#pragma unroll
        for (int s = 1; s < kTipStripes; s++) at = g >= first[s] ? span.at[s] + g - first[s] : at;
        return at;
    }
};

// Copies n ints from global src to LDS dst; src and dst 16-byte aligned.
// PER: 16-byte loads per thread that cover n (n <= 4 * PER * blockDim.x); all
// of a thread's loads are issued before the first is used.
template <int PER>
__device__ __forceinline__ void load_to_lds(int *dst, gcint src, int n) {
    const int B = blockDim.x, tid = threadIdx.x, n4 = n / 4;
    GLOBAL const v4i *s4 = reinterpret_cast<GLOBAL const v4i *>(src);
    v4i *d4 = reinterpret_cast<v4i *>(dst);
    v4i v[PER];
#pragma unroll
    for (int p = 0; p < PER; p++) {
        const int k = tid + p * B;
        v[p] = s4[k < n4 ? k : 0];
    }
#pragma unroll
    for (int p = 0; p < PER; p++) {
        const int k = tid + p * B;
        if (k < n4) d4[k] = v[p];
    }
    for (int k = (n & ~3) + tid; k < n; k += B) dst[k] = src[k];
}

// ---------------------------------------------------------------------------
// k_label: longest edge of each triangle
// ---------------------------------------------------------------------------

// What a run clears before its kernels count into it.
struct ClearArgs {
    MeshCounters *ctrs;
    uint64_t *status;   // per compaction tile
    int nstatus;
    int32_t *tip_counts, *walk_counts, *emit_counts, *wbuf_counts;
};

// Label byte bit 7: the maximum edge length of the triangle is tied (k_label
// sets it, k_relink counts it and writes the byte back without it).
constexpr uint32_t kTieBit = 1u << 7;

//
// VALUE: one mesh, its descriptor passed by value; the first thread writes it
// where the kernels that follow read it.  (Staged by a launch of its own it cost
// a call 4 us.)
struct NoDesc {};
template <int ITEMS, bool VALUE>
__global__ void __launch_bounds__(1024) k_label(const MeshDesc *__restrict__ descs, int nmesh, ClearArgs ca,
                                                MeshDesc *desc_out,
                                                const std::conditional_t<VALUE, MeshDesc, NoDesc> one) {
    // the run's counters, list sizes and per-tile totals start at zero for
    // the kernels that follow (nothing in this kernel counts into them)
    {
        const int gid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
        for (int k = gid; k < ca.nstatus; k += stride) ca.status[k] = 0ull;
        for (int k = gid; k < nmesh; k += stride) ca.ctrs[k] = MeshCounters{};
        if (gid < kTipStripes) ca.tip_counts[gid * kStripePad] = 0;
        if (gid == 0) ca.tip_counts[kUnmarked] = 0;
        if (gid < kStripes) {
            ca.walk_counts[gid * kStripePad] = 0;
            ca.emit_counts[gid * kStripePad] = 0;
            ca.wbuf_counts[gid * kStripePad] = 0;
        }
        if constexpr (VALUE)
            if (gid == 0) *desc_out = one;
    }
    extern __shared__ int4 lds_raw[];
    int *s_org = reinterpret_cast<int *>(lds_raw);
    const int B = blockDim.x, tid = threadIdx.x;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const MeshDesc &d = [&]() -> const MeshDesc & {
        if constexpr (VALUE)
            return one;
        else
            return descs[find_mesh<0>(descs, nmesh, tile)];
    }();
    const int nt = d.nt;
    const int base = (tile - d.tri_tile0) * B * ITEMS;
    const gcv2i xy = (gcv2i)(d.xy);
    // the tile's corners in one contiguous load; item j of this thread is
    // triangle base + j*B + tid
    const int cnt_all = min(B * ITEMS, nt - base);
    if (cnt_all <= 0) return;   // an empty mesh's tile (the whole block)
    if (!d.org8) {   // (uniform)
        load_to_lds<(3 * ITEMS + 3) / 4>(s_org, (gcint)(d.org) + 3 * (size_t)base, 3 * cnt_all);
    } else {   // a compact mesh: v0 and two 16-bit offsets per triangle
        GLOBAL const v2i *o8 = (GLOBAL const v2i *)d.org8 + base;
        for (int k = tid; k < cnt_all; k += B) {
            const v2i r = o8[k];
            const int d1 = (int)(int16_t)(r.y & 0xffff), d2 = r.y >> 16;
            const int h = 3 * (base + k);
            s_org[3 * k] = r.x;
            s_org[3 * k + 1] = d1 != kEsc16 ? r.x + d1 : esc_lookup(d.esc, d.esc_mask, ~(h + 1));
            s_org[3 * k + 2] = d2 != kEsc16 ? r.x + d2 : esc_lookup(d.esc, d.esc_mask, ~(h + 2));
        }
    }
    __syncthreads();
    // every corner of every item first, so all the gathers are in flight
    // together (items past the tile read corner 0 and are dropped)
    v2i q[ITEMS][3];
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int lt = j * B + tid;
        const int l0 = lt < cnt_all ? 3 * lt : 0;
#pragma unroll
        for (int i = 0; i < 3; i++) q[j][i] = xy[s_org[l0 + i]];
    }
    gu8 tflag = (gu8)d.tflag;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int lt = j * B + tid;
        if (lt >= cnt_all) continue;
        const int t = base + lt;
        const int2 p0 = make_int2(q[j][0].x, q[j][0].y), p1 = make_int2(q[j][1].x, q[j][1].y),
                   p2 = make_int2(q[j][2].x, q[j][2].y);
        const long long l0 = sq_len(p0, p1), l1 = sq_len(p1, p2), l2 = sq_len(p2, p0);
        long long m = l0 > l1 ? l0 : l1;
        m = m > l2 ? m : l2;
        const int cnt = (l0 == m) + (l1 == m) + (l2 == m);
        int best = l0 == m ? 0 : (l1 == m ? 1 : 2);
        if (cnt > 1) {
            // tie at the maximum: the lower edge id min(h, twin h) wins
            best = -1;
            int bid = 0x7fffffff;
            const long long ls[3] = {l0, l1, l2};
            for (int i = 0; i < 3; i++) {
                if (ls[i] != m) continue;
                const int h = 3 * t + i, g = twin_view(d)[h];
                const int id = (g >= 0 && g < h) ? g : h;
                if (id < bid) {
                    bid = id;
                    best = i;
                }
            }
            best |= (int)kTieBit;   // counted by k_relink
        }
        tflag[t] = (uint8_t)best;
    }
}

// ---------------------------------------------------------------------------
// k_relink: frontier and seed bits, next/prev of every frontier half-edge,
// barrier tips
//
// One thread per triangle.  Phase 1 derives each triangle's frontier bits
// and seed bit from its own longest-edge label and its neighbours' (Section
// 6.2-6.3) and keeps them in LDS.  Phase 2 turns around the ends of every
// frontier half-edge (Section 6.5): a candidate in the tile reads its
// frontier bit from LDS; one outside derives it from the longest-edge labels,
// which no kernel changes during this pass (the tile's label bytes are
// written back with their longest-edge bits unchanged).  Each thread loads
// its triangles' twins and stores their next'/prev' itself (12 contiguous
// bytes per triangle).
//
// Vector instructions bound this kernel, so half-edges are slots 4t + i in it
// (the triangle and the local index are a shift and a mask), choices among a
// triangle's edges come from tables of its three frontier bits, and counts
// from ballots: 536 vector instructions per wave of 128 triangles, where half-
// edge ids (a division by 3 for each), masks and a block scan took 772.  33.5M
// grid: 0.415 -> 0.350 ms for 1.32 GB; 2.1M grid 32 -> 25 us.
// ---------------------------------------------------------------------------

// Loop byte of the minimum's triangle: (min(len, kPlMax) << 2) | local
// index of the minimum.  Length code 1 (no loop is that short) marks a loop
// of four whose second triangle is t + 1; its low bits then hold the local
// index of that triangle's terminal edge, and the minimum is the lower of
// the two frontier half-edges of t.
__device__ __forceinline__ uint8_t loop_code(int mn, int len) {
    return (uint8_t)(((len < kPlMax ? len : kPlMax) << 2) | (mn % 3));
}
constexpr int kPlQuadNext = 1;

// Label bits 6 and 7 (k_relink writes the label bytes with both clear).  The
// repair splits a polygon along middle edges, both sides of which then seed a
// walk, so every part has such a seed, some several, and the polygon's own seed
// is not needed: its triangle is marked and its walk left out.  Of the walks
// that a part still has several of, the first to set bit 7 at the minimum's
// triangle counts the loop; no other loop is walked twice.
constexpr uint32_t kSplitBit = 1u << 6;
constexpr uint32_t kCountedBit = 1u << 7;

// Sets a bit of triangle t's label byte; returns whether it was set before.
__device__ __forceinline__ bool set_label_bit(const MeshDesc &d, int t, uint32_t bit) {
    const uint32_t b = bit << (8 * (t & 3));
    return atomicOr(reinterpret_cast<uint32_t *>(d.tflag) + (t >> 2), b) & b;
}

// Slots: half-edge 3t + i as 4t + i; a boundary twin (-1) is kNoSlot, the only
// slot of local index 3.
constexpr uint32_t kNoSlot = ~0u;
__device__ __forceinline__ uint32_t he_slot(int h) {   // h >= -1
    return ((uint32_t)h + (uint32_t)h / 3u) | (uint32_t)(h >> 31);
}
__device__ __forceinline__ int he_of_slot(uint32_t s) { return (int)(s - (s >> 2)); }
__device__ __forceinline__ uint32_t next_slot(uint32_t s) { return (s & 2u) ? s - 2u : s + 1u; }
__device__ __forceinline__ uint32_t prev_slot(uint32_t s) { return (s & 3u) ? s - 1u : s + 2u; }

// What a turn in k_relink reads.
struct TileLabels {
    TwinView twin;
    gcu8 tflag;               // longest-edge bits (0-1) only are read
    const uint32_t *s_slot;   // the tile's half-edges by slot: their twins' slots
    const uint32_t *s_lab;    // its triangles' label bytes
    uint32_t base, cnt;       // the tile's triangles [base, base + cnt)
};

// One step of a turn around a vertex at candidate slot c (Lc: the longest-edge
// label of c's triangle, or -1 when not loaded).  Returns 1 when c is a
// frontier half-edge (the turn ends there), 0 after moving c to the next
// candidate (next: c <- next(twin(c)), else c <- prev(twin(c))), -1 when the
// mesh is inconsistent.
__device__ __forceinline__ int turn_step(const TileLabels &T, uint32_t &c, int &Lc, bool next) {
    const uint32_t tc = c >> 2, lc = c & 3u, kk = tc - T.base;
    uint32_t g;
    int Lg = -1;
    if (kk < T.cnt) {
        if (fbit(T.s_lab[kk], (int)lc)) return 1;
        g = T.s_slot[4 * kk + lc];
        if (g == kNoSlot) return -1;   // a non-frontier edge is interior
    } else {
        g = he_slot(T.twin[he_of_slot(c)]);
        const uint32_t fc = Lc < 0 ? T.tflag[tc] : 0u;   // in flight with the twin
        if (g == kNoSlot) return 1;   // boundary
        if (Lc < 0) Lc = (int)(fc & 3u);
        if (Lc != (int)lc) {   // c is not its triangle's longest edge
            // twin(c)'s triangle is often back in the tile, whose label
            // bytes (longest-edge bits unchanged) are in LDS
            const uint32_t tg = g >> 2, kg = tg - T.base;
            Lg = (int)((kg < T.cnt ? T.s_lab[kg] : (uint32_t)T.tflag[tg]) & 3u);
            if (Lg != (int)(g & 3u)) return 1;   // nor is twin(c)
        }
    }
    c = next ? next_slot(g) : prev_slot(g);
    Lc = Lg;
    return 0;
}

// The whole turn from candidate c: the frontier slot it ends at, or kNoSlot.
__device__ __forceinline__ uint32_t run_turn(const TileLabels &T, uint32_t c, bool next) {
    int Lc = -1;
    for (int k = 0; k < kRotGuard; k++) {
        const int r = turn_step(T, c, Lc, next);
        if (r != 0) return r > 0 ? c : kNoSlot;
    }
    return kNoSlot;
}

// Frontier bit of slot c of a triangle outside the tile whose longest-edge
// label is Lc.
__device__ __forceinline__ bool outside_fbit(const TileLabels &T, uint32_t c, uint32_t Lc) {
    if (Lc == (c & 3u)) return false;
    const uint32_t g = he_slot(T.twin[he_of_slot(c)]);
    return g == kNoSlot || (T.tflag[g >> 2] & 3u) != (g & 3u);
}

// Tables of a triangle's frontier bits F (edge i: bit i), two bits each.  A
// triangle has at most one frontier edge followed by an edge that is not, and
// at most one preceded by one.
//   kCrossNext  that following edge: next' of the frontier edge before it turns
//               across it (3: there is none)
//   kCrossPrev  that preceding edge: prev' of the frontier edge after it turns
//               across it
constexpr uint32_t cross_table(bool next) {
    uint32_t t = 0;
    for (uint32_t F = 0; F < 8; F++) {
        uint32_t e = 3;
        for (uint32_t i = 0; i < 3; i++) {
            const uint32_t x = next ? (i + 1) % 3 : (i + 2) % 3;
            if (((F >> i) & 1u) && !((F >> x) & 1u)) e = x;
        }
        t |= e << (2 * F);
    }
    return t;
}
constexpr uint32_t kCrossNext = cross_table(true), kCrossPrev = cross_table(false);

__device__ __forceinline__ uint32_t pick3(uint32_t i, uint32_t a, uint32_t b, uint32_t c) {
    return i == 0 ? a : (i == 1 ? b : c);
}

__host__ __device__ inline size_t relink_lds_bytes(int tile) {
    return sizeof(int) * (4 * (size_t)tile + 4 * (size_t)tile + (size_t)tile + 4);
}

// CM: some mesh of the run is compact (else the int32 twins are read
// without a test of the encoding).  NT: next'/prev' go out as streaming
// (nontemporal) stores.
template <int ITEMS, bool CM, bool NT>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) k_relink(const MeshDesc *__restrict__ descs, int nmesh,
                                                  ListEntry *tips, int32_t *tip_counts, const TipSpan tip_span,
                                                  ListEntry *walk, int32_t *walk_counts, int walk_cap,
                                                  uint64_t *agg, int cmp_tb) {
    extern __shared__ int4 lds_raw[];
    const int B = blockDim.x, tid = threadIdx.x, TB = B * ITEMS, lane = __lane_id();
    uint32_t *s_slot = reinterpret_cast<uint32_t *>(lds_raw);   // by slot in the tile: the twin's slot
    uint2 *s_q = reinterpret_cast<uint2 *>(s_slot + 4 * TB);    // queued turns (at most two per triangle)
    uint32_t *s_lab = reinterpret_cast<uint32_t *>(s_q + 2 * TB);   // label bytes; after them one without frontier edges
    // queued turns; open seeds; settled loops << 16 | their half-edges; barrier
    // tips; the open seeds' and the tips' places in their lists
    __shared__ int s_nq, s_nopen, s_tot, s_ntip, s_wbase, s_tbase;
    // loops settled here, per compaction tile, when the tile's triangles
    // span several of them (a relink tile of <= 1024 triangles, compaction
    // tiles of >= 64: at most 17)
    constexpr int kSpan = 1024 / 64 + 1;
    __shared__ int s_aggc[kSpan], s_aggl[kSpan];
    if (tid == 0) {
        s_nq = s_nopen = s_tot = s_ntip = 0;
        s_lab[TB] = 0;
    }
    if (tid < kSpan) {
        s_aggc[tid] = 0;
        s_aggl[tid] = 0;
    }
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int mi = find_mesh<1>(descs, nmesh, tile);
    const MeshDesc &d = descs[mi];
    const int nt = d.nt;
    TwinView twin = twin_view(d);
    if (!CM) twin.t16 = nullptr;
    const gu8 tflag = (gu8)(d.tflag);
    const gint nxo = (gint)(d.next_o), pvo = (gint)(d.prev_o);
    const int base = (tile - d.he_tile0) * TB;
    const int cnt = min(TB, nt - base);
    if (cnt <= 0) return;   // an empty mesh's tile (the whole block)
    // phase 1: labels of the triangle and its neighbours -> frontier, seed.
    // Each thread loads its triangles' twins itself (12 contiguous bytes per
    // triangle, so a wave's loads are contiguous) and issues the label
    // gathers as soon as they arrive; the twins go to LDS for the turns of
    // phase 2.  Every load is issued unconditionally (indices clamped,
    // results masked after) so that all of them are in flight together.
    uint32_t s[ITEMS][3], own[ITEMS], fn[ITEMS][3];
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int lt = j * B + tid;
        const int t = base + (lt < cnt ? lt : 0);
        v3i_a4 g;
        if (!twin.t16) {   // (uniform) one 12-byte load
            g = *(GLOBAL const v3i_a4 *)(twin.t32 + 3 * t);
        } else {
            g.x = twin[3 * t];
            g.y = twin[3 * t + 1];
            g.z = twin[3 * t + 2];
        }
        s[j][0] = he_slot(g.x);
        s[j][1] = he_slot(g.y);
        s[j][2] = he_slot(g.z);
        own[j] = tflag[t];
#pragma unroll
        for (int i = 0; i < 3; i++) fn[j][i] = tflag[min(s[j][i] >> 2, (uint32_t)nt - 1u)];
    }
    uint32_t F[ITEMS], lab[ITEMS];   // frontier bits; the label byte
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int lt = j * B + tid;
        const bool in = lt < cnt;
        const uint32_t L = own[j] & 3u, lbit = 1u << L, sL = pick3(L, s[j][0], s[j][1], s[j][2]);
        // bit i: the twin of edge i is not its triangle's longest edge
        // (a boundary twin's local index, 3, equals no label)
        const uint32_t E = min((fn[j][0] ^ s[j][0]) & 3u, 1u) | (min((fn[j][1] ^ s[j][1]) & 3u, 1u) << 1) |
                           (min((fn[j][2] ^ s[j][2]) & 3u, 1u) << 2);
        // frontier: the longest edge of neither triangle
        uint32_t f = E & ~lbit;
        // terminal edge: longest on both sides (the lower half-edge holds the seed)
        bool seed = !(E & lbit) && 4u * (uint32_t)(base + lt) + L < sL;
        if (__any(max(max(s[j][0], s[j][1]), s[j][2]) == kNoSlot)) {   // (uniform)
            // boundary edges are frontier edges; the longest one is terminal
            uint32_t bnd = 0;
#pragma unroll
            for (int i = 0; i < 3; i++) bnd |= s[j][i] == kNoSlot ? 1u << i : 0u;
            f |= bnd;
            seed |= (bnd & lbit) != 0;
        }
        F[j] = in ? f : 0u;
        lab[j] = in ? L | (f << 2) | (seed ? kSeedBit : 0u) : 0u;
        if (__any(in && (own[j] & kTieBit))) {   // (uniform, rare)
            const int n = __popcll(__ballot(in && (own[j] & kTieBit)));
            if (lane == 0) atomicAdd(&d.ctr->nties, n);
        }
        reinterpret_cast<uint4 *>(s_slot)[lt] = make_uint4(s[j][0], s[j][1], s[j][2], 0u);
        s_lab[lt] = lab[j];
    }
    __syncthreads();
    // phase 2: next'/prev' of every frontier half-edge.  The next (previous)
    // edge in the triangle is taken when it is frontier itself; otherwise the
    // turn continues in the neighbour across it.  Nearly all turns end at
    // their first candidate (96% on the grids), read from LDS; the others are
    // queued.  (The first candidate is never the twin of the turn's own
    // half-edge: two triangles of a valid mesh share one edge.)
    const TileLabels T = {twin, tflag, s_slot, s_lab, (uint32_t)base, (uint32_t)cnt};
    bool err = false;
    uint32_t cn[ITEMS], cp[ITEMS];       // the turns' candidates: next', prev'
    uint32_t xy[ITEMS];                  // edges crossed: x | y << 2
    int qn[ITEMS], qp[ITEMS];            // their places in the queue, -1: ended here
    int open[ITEMS];                     // place of an open seed among the tile's, -1: none
    uint8_t codes[ITEMS];
    unsigned long long mn[ITEMS], mp[ITEMS], mo[ITEMS];   // ballots: queued next', prev'; open seeds
    int wq = 0, wo = 0, wtot = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const uint32_t t = (uint32_t)(base + j * B + tid);   // past cnt: F == 0, so nothing happens
        const uint32_t x = (kCrossNext >> (2 * F[j])) & 3u, y = (kCrossPrev >> (2 * F[j])) & 3u;
        const uint32_t sx = pick3(x, s[j][0], s[j][1], s[j][2]), sy = pick3(y, s[j][0], s[j][1], s[j][2]);
        // a neighbour outside the tile reads the entry past it: no frontier edges
        const uint32_t fx = s_lab[min((sx >> 2) - (uint32_t)base, (uint32_t)TB)],
                       fy = s_lab[min((sy >> 2) - (uint32_t)base, (uint32_t)TB)];
        cn[j] = next_slot(sx);
        cp[j] = prev_slot(sy);
        xy[j] = x | (y << 2);
        mn[j] = __ballot(x != 3u && !fbit(fx, (int)(cn[j] & 3u)));
        mp[j] = __ballot(y != 3u && !fbit(fy, (int)(cp[j] & 3u)));
        wq += __popcll(mn[j]) + __popcll(mp[j]);
        // A seed whose polygon is one triangle (boundary terminal edge, both
        // other edges frontier) or two (interior terminal edge, the four
        // other edges frontier) is settled here: its loop is those 3 or 4
        // half-edges.  Such polygons have no interior vertex, so no barrier
        // tip and no repair touches them.  The seed is the lower half-edge of
        // its terminal edge, so the loop's minimum lies in this triangle and
        // its byte is written here with the rest of the tile.
        const uint32_t L = lab[j] & 3u, lbit = 1u << L;
        const bool seed = lab[j] & kSeedBit;
        const bool cand = seed && F[j] == (7u ^ lbit);   // then x == y == L
        bool quad = cand && ((fx >> 2) & 7u) == (7u ^ (1u << (sx & 3u)));
        if (cand && (sx >> 2) - (uint32_t)base >= (uint32_t)TB) {   // partner outside the tile (rare on ordered meshes)
            const uint32_t Lp = sx & 3u;
            quad = outside_fbit(T, cn[j], Lp) && outside_fbit(T, prev_slot(sx), Lp);
        }
        const bool one = seed && F[j] == 7u;
        codes[j] = quad ? (uint8_t)((sx >> 2) == t + 1 ? (kPlQuadNext << 2) | (sx & 3u) : (4u << 2) | (L == 0 ? 1u : 0u))
                        : (one ? (uint8_t)(3u << 2) : (uint8_t)0);
        const unsigned long long mq = __ballot(quad), m1 = __ballot(one);
        mo[j] = __ballot(seed && !quad && !one);
        wo += __popcll(mo[j]);
        const int nq = __popcll(mq), n1 = __popcll(m1);
        wtot += ((nq + n1) << 16) | (4 * nq + 3 * n1);
    }
    // the block's triangles lie in one compaction tile unless that tile is
    // smaller than this one or not aligned with it
    const int ct0 = base / cmp_tb;   // first compaction tile of this tile
    const bool one_tile = ct0 == (base + cnt - 1) / cmp_tb;
    // the wave's places in the queue and among the open seeds; its settled loops
    int q0 = 0, o0 = 0;
    if (lane == 0) {
        if (wq) q0 = atomicAdd(&s_nq, wq);
        if (wo) o0 = atomicAdd(&s_nopen, wo);
        if (one_tile && wtot) atomicAdd(&s_tot, wtot);
    }
    q0 = __builtin_amdgcn_readfirstlane(q0);
    o0 = __builtin_amdgcn_readfirstlane(o0);
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const uint32_t src = 4u * (uint32_t)(j * B + tid), x = xy[j] & 3u, y = xy[j] >> 2;
        const auto before = [](unsigned long long m) {
            return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        };
        qn[j] = qp[j] = open[j] = -1;
        if ((mn[j] >> lane) & 1) {   // from the frontier edge before x
            qn[j] = q0 + before(mn[j]);
            s_q[qn[j]] = make_uint2(cn[j], (src | (x == 0 ? 2u : x - 1u)) << 1 | 1u);
        }
        q0 += __popcll(mn[j]);
        if ((mp[j] >> lane) & 1) {   // from the frontier edge after y
            qp[j] = q0 + before(mp[j]);
            s_q[qp[j]] = make_uint2(cp[j], (src | (y == 2 ? 0u : y + 1u)) << 1);
        }
        q0 += __popcll(mp[j]);
        if ((mo[j] >> lane) & 1) open[j] = o0 + before(mo[j]);
        o0 += __popcll(mo[j]);
        if (!one_tile && codes[j]) {   // totals per compaction tile in LDS, one global atomic each below
            const int k = (base + j * B + tid) / cmp_tb - ct0;
            atomicAdd(&s_aggc[k], 1);
            atomicAdd(&s_aggl[k], (codes[j] >> 2) == kPlQuadNext ? 4 : (codes[j] >> 2));
        }
    }
    __syncthreads();
    const int stripe = tile % kStripes;
    if (tid == B - kWave) {   // (in the last wave: the first ones have the turns)
        s_wbase = s_nopen > 0 ? atomicAdd(&walk_counts[stripe * kStripePad], s_nopen) : 0;
        if (one_tile && s_tot != 0)
            atomicAdd(reinterpret_cast<unsigned long long *>(agg + d.cmp_tile0 + ct0),
                      ((unsigned long long)(uint32_t)(s_tot >> 16) << 32) | (unsigned long long)(s_tot & 0xffff));
    }
    if (!one_tile && tid <= (base + cnt - 1) / cmp_tb - ct0 && s_aggc[tid] != 0)
        atomicAdd(reinterpret_cast<unsigned long long *>(agg + d.cmp_tile0 + ct0 + tid),
                  ((unsigned long long)(uint32_t)s_aggc[tid] << 32) | (unsigned long long)(uint32_t)s_aggl[tid]);
    // the queued turns, one per thread: only the first lanes of the block work
    const int nq = s_nq;
    for (int q = tid; q < nq; q += B) {
        const uint2 w = s_q[q];
        const uint32_t src = w.y >> 1;
        const bool nxt = w.y & 1u;
        const uint32_t res = run_turn(T, w.x, nxt);
        err |= res == kNoSlot;
        s_q[q].x = res;   // the owner picks it up after the barrier
        // next'(h) == twin(h): the target of h is a barrier tip (its place
        // among the tile's in the entry's other word)
        if (nxt) s_q[q].y = res != kNoSlot && res == s_slot[src] ? (uint32_t)atomicAdd(&s_ntip, 1) : kNoSlot;
    }
    __syncthreads();
    const int ntip = s_ntip;
    if (ntip > 0) {   // (uniform)
        if (tid == 0) s_tbase = atomicAdd(&tip_counts[tile % kTipStripes * kStripePad], ntip);
        __syncthreads();
    }
    const int wbase = s_wbase;
    err |= wbase + s_nopen > walk_cap;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int lt = j * B + tid, t = base + lt, h0 = 3 * t;
        if (open[j] >= 0 && wbase + open[j] < walk_cap) {
            ListEntry &e = walk[stripe * walk_cap + wbase + open[j]];
            e.mesh = mi;
            e.he = h0 + (int)(lab[j] & 3u);
        }
        if (lt >= cnt) continue;
        // next'/prev' of the triangle's edges, the queued turns' results in
        // place, as one 12-byte store each, so every line is written once
        // and whole (kNoSlot becomes -1 or thereabouts: an error was set)
        if (qn[j] >= 0) {
            const uint2 w = s_q[qn[j]];
            cn[j] = w.x;
            if (w.y != kNoSlot) {
                const int k = s_tbase + (int)w.y, x = (int)(xy[j] & 3u);
                const int first = tip_span.at[tile % kTipStripes];
                if (k < tip_span.at[tile % kTipStripes + 1] - first)
                    tips[first + k] = {mi, h0 + (x == 0 ? 2 : x - 1)};
                else
                    err = true;
            }
        }
        if (qp[j] >= 0) cp[j] = s_q[qp[j]].x;
        const int hn = he_of_slot(cn[j]), hp = he_of_slot(cp[j]);
        const uint32_t x = xy[j] & 3u, y = xy[j] >> 2;
        const int none[3] = {(F[j] & 1u) ? 0 : -1, (F[j] & 2u) ? 0 : -1, (F[j] & 4u) ? 0 : -1};
        const v3i nv = v3i{x == 1u ? hn : (h0 + 1) | none[0], x == 2u ? hn : (h0 + 2) | none[1],
                           x == 0u ? hn : h0 | none[2]};
        const v3i pv = v3i{y == 2u ? hp : (h0 + 2) | none[0], y == 0u ? hp : h0 | none[1],
                           y == 1u ? hp : (h0 + 1) | none[2]};
        if (NT) {
            __builtin_nontemporal_store(nv, reinterpret_cast<GLOBAL v3i *>(nxo + h0));
            __builtin_nontemporal_store(pv, reinterpret_cast<GLOBAL v3i *>(pvo + h0));
        } else {
            *reinterpret_cast<GLOBAL v3i *>(nxo + h0) = nv;
            *reinterpret_cast<GLOBAL v3i *>(pvo + h0) = pv;
        }
        // the label byte keeps its longest-edge bits, which other tiles may
        // be reading
        tflag[t] = (uint8_t)lab[j];
        ((gu8)d.pl)[t] = codes[j];
    }
    if (err) atomicOr(&d.ctr->err, kErrCorrupt);
}

// ---------------------------------------------------------------------------
// k_repair: middle edge of each barrier tip
// ---------------------------------------------------------------------------

// Sets the frontier bit of half-edge h; returns whether it was set before.
__device__ __forceinline__ uint32_t set_frontier_bit(uint8_t *tflag, int h) {
    int t = h / 3, i = h - 3 * t;
    uint32_t *word = reinterpret_cast<uint32_t *>(tflag) + (t >> 2);
    uint32_t bit = (1u << (2 + i)) << (8 * (t & 3));
    return atomicOr(word, bit) & bit;
}

// Appends 2 entries per lane with pred set; one atomic per wave.  Must be
// reached by every lane of the wave.
__device__ __forceinline__ int wave_reserve2(int32_t *counter, bool pred) {
    const unsigned long long mask = __ballot(pred);
    if (mask == 0ull) return -1;
    const int lane = __lane_id(), leader = __ffsll((long long)mask) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(counter, 2 * __popcll(mask));
    base = __shfl(base, leader);
    return pred ? base + 2 * __popcll(mask & ((1ull << lane) - 1ull)) : -1;
}

// Middle edge of every barrier tip.  Whole waves take consecutive tips, so the
// list appends and counters cost one atomic per wave (tips are many on
// general-position meshes, and atomics on one address serialize).  Tip k's two
// anchors for k_fixup go to entries 2k and 2k + 1 (half-edge -1: none).
template <bool ONE>
__global__ void k_repair(const MeshDesc *__restrict__ descs, const ListEntry *tips, const int32_t *tip_counts,
                         const TipSpan tip_span, int cap_tips, ListEntry *walk, int32_t *walk_counts, int walk_cap,
                         ListEntry *fixes) {
    const TipStripes stripes(tip_counts, tip_span);
    const int all = stripes.total(), ntips = min(all, cap_tips);
    const int lane = __lane_id();
    const int stride = gridDim.x * blockDim.x;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (all > cap_tips) atomicOr(&descs[0].ctr->err, kErrCorrupt);
        if (ONE) descs[0].ctr->ntips = ntips;
    }
    for (int wbase = blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); wbase < ntips; wbase += stride) {
        const int k = wbase + lane;
        bool ok = k < ntips;
        int mesh = 0, a = -1, m = -1, mt = -1;
        bool newmid = false;
        if (ok) {
            const ListEntry e = tips[stripes.index(k, tip_span)];
            mesh = ONE ? 0 : e.mesh;
            const MeshDesc &d = descs[ONE ? 0 : mesh];
            const TwinView twin = twin_view(d);
            // a: the only frontier edge at the tip v = target(e.he), leaving v.
            // The middle edge is the outgoing half-edge floor(deg / 2)
            // clockwise steps from a.  Turning clockwise (c) and counter-
            // clockwise (b) from a at once, the two meet there after about
            // deg / 2 steps: c one step short of b after k steps means deg =
            // 2k + 1 and the middle is c; c and b equal after k + 1 steps
            // means deg = 2k + 2 and the middle is that half-edge.
            a = twin[e.he];
            bool err = a < 0;
            if (!err) {
                int c = a, b = a;
                for (int k = 0;; k++) {
                    const int gc = twin[c], gb = twin[he_prev(b)];   // both loads in flight
                    if (gc < 0 || gb < 0 || k > kRotGuard) {
                        err = true;
                        break;
                    }
                    const int c1 = he_next(gc);
                    if (c1 == b && k > 0) {   // odd degree
                        m = c;
                        break;
                    }
                    if (c1 == gb) {   // even degree
                        m = c1;
                        break;
                    }
                    c = c1;
                    b = gb;
                }
                if (!err) {
                    mt = twin[m];
                    err = mt < 0;
                }
            }
            if (err) {
                atomicOr(&d.ctr->err, kErrCorrupt);
                ok = false;
            } else {
                newmid = !set_frontier_bit(d.tflag, m < mt ? m : mt);
                set_frontier_bit(d.tflag, m < mt ? mt : m);
            }
        }
        // both halves of the middle edge seed the polygons on either side
        const int stripe = (wbase / kWave) % kStripes;
        const int c = wave_reserve2(&walk_counts[stripe * kStripePad], ok);
        if (k < ntips) {
            fixes[2 * k] = {mesh, ok ? a : -1};        // leaves the tip
            fixes[2 * k + 1] = {mesh, ok ? mt : -1};   // leaves the other end of the middle edge
        }
        if (ok) {
            if (c + 1 < walk_cap) {
                walk[stripe * walk_cap + c].mesh = mesh;
                walk[stripe * walk_cap + c].he = ~m;
                walk[stripe * walk_cap + c + 1].mesh = mesh;
                walk[stripe * walk_cap + c + 1].he = ~mt;
            } else {
                atomicOr(&descs[ONE ? 0 : mesh].ctr->err, kErrCorrupt);
            }
        }
        // tips (of a batch) and new middle edges, counted per mesh: one atomic each per mesh in the wave
        unsigned long long pending = __ballot(k < ntips);
        while (pending) {
            const int leader = __ffsll((long long)pending) - 1;
            const int lm = __shfl(mesh, leader);
            const unsigned long long same = __ballot(k < ntips && mesh == lm), mid = __ballot(ok && newmid && mesh == lm);
            if (lane == leader) {
                if (!ONE) atomicAdd(&descs[ONE ? 0 : lm].ctr->ntips, __popcll(same));
                if (mid) atomicAdd(&descs[ONE ? 0 : lm].ctr->nmiddle, __popcll(mid));
            }
            pending &= ~same;
        }
    }
}

// The tip list in one piece (debug runs).
__global__ void k_gather_tips(const ListEntry *tips, const int32_t *tip_counts, const TipSpan tip_span, int cap,
                              ListEntry *out, int32_t *ntips) {
    const TipStripes stripes(tip_counts, tip_span);
    const int n = min(stripes.total(), cap), first = blockIdx.x * blockDim.x + threadIdx.x;
    for (int k = first; k < n; k += gridDim.x * blockDim.x) out[k] = tips[stripes.index(k, tip_span)];
    if (first == 0) *ntips = n;
}

hipError_t launch_gather_tips(const RunBuffers &rb, ListEntry *out, int32_t *ntips, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_tips, dim3(64), dim3(256), 0, s, rb.tips, rb.tip_counts, rb.tip_span, rb.cap_tips, out,
                       ntips);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_fixup: recompute next/prev of every frontier half-edge at a vertex
// ---------------------------------------------------------------------------

// One lane per anchor (a half-edge leaving a vertex x at either end of a new
// frontier edge, and so a frontier half-edge itself) takes next'/prev' around
// x again: of two frontier edges that follow each other clockwise around x, the
// outgoing half-edge of the second is next' of the first's incoming one.  The
// lane turns clockwise (c) and counter-clockwise (b) from the anchor at once,
// so a vertex of degree deg takes about deg / 2 dependent steps, its two loads
// of twins in flight together, and links the last frontier edges of both sides
// where they meet.  (The chains bound the kernel: 22 us for a compact Delaunay
// mesh of 300,000 points, 30 with one sweep round the vertex and with all three
// escaped twins looked up in each step of mark_split.)  A vertex on the
// boundary is open: each side goes to its end.  Anchors at one vertex write
// the same values.
__device__ __forceinline__ bool fix_around(const MeshDesc &d, int o) {
    const TwinView twin = twin_view(d);
    const gint nxo = (gint)d.next_o, pvo = (gint)d.prev_o;
    if (!is_frontier(d.tflag, o)) return false;
    int c = o, b = o;                        // the latest half-edges of either side
    int last = o, last_in = -1, cur = o;     // their latest frontier ones; last's twin
    bool cend = false, bend = false;
    for (int k = 0; k <= kRotGuard; k++) {
        const int in = he_prev(b), gc = cend ? -1 : twin[c], gb = bend ? -1 : twin[in];
        if (last == c) last_in = gc;
        const int c1 = gc < 0 ? -1 : he_next(gc);
        if (!cend && !bend && c1 == b) {   // nothing lies between them
            if (last_in < 0) return false;
            nxo[last_in] = cur;
            pvo[cur] = last_in;
            return true;
        }
        const bool meet = c1 >= 0 && c1 == gb;   // one half-edge is left
        if (c1 >= 0) {
            if (is_frontier(d.tflag, c1)) {
                nxo[last_in] = c1;
                pvo[c1] = last_in;
                last = c1;
                last_in = in;   // (its twin, if the sides meet in it)
            }
            c = c1;
        } else {
            cend = true;   // (the boundary edge is the last frontier edge of this side)
        }
        if (meet) {
            nxo[last_in] = cur;
            pvo[cur] = last_in;
            return true;
        }
        if (gb >= 0) {
            if (is_frontier(d.tflag, gb)) {
                nxo[in] = cur;
                pvo[cur] = in;
                cur = gb;
            }
            b = gb;
        } else if (!bend) {
            bend = true;
            nxo[in] = cur;   // the boundary edge into x
            pvo[cur] = in;
        }
        if (cend && bend) return true;
    }
    return false;
}

// Marks the seed of triangle t's polygon as split: up the longest edges from t
// (Lepp, Definition 1) to the terminal edge, whose lower half-edge is the seed.
// A triangle's label and its three twins are loaded together, so a step is one
// dependent load (two where a compact mesh's twin has escaped).  A path may
// run through every triangle of the mesh, and then takes longer than the walk
// that the mark saves: past kClimb steps it is given up, and k_walk told so.
// (The longest path of a Delaunay mesh of 1M points takes 31 steps.  A run over a
// strip of 200,000 triangles with a tip at its low end: 156 ms with the whole
// path climbed, 102 so; of 200 triangles, 241 us and 208.)  Returns whether
// the seed was marked.
constexpr int kClimb = 64;
__device__ __forceinline__ bool mark_split(const MeshDesc &d, int t) {
    const TwinView twin = twin_view(d);
    const gcu8 tfl = (gcu8)d.tflag;
    int L = (int)(tfl[t] & 3u), g0 = twin.raw(3 * t), g1 = twin.raw(3 * t + 1), g2 = twin.raw(3 * t + 2);
    for (int k = 0; k < kClimb; k++) {
        const int g = twin.value(3 * t + L, L == 0 ? g0 : (L == 1 ? g1 : g2));
        if (g < 0) {   // a boundary terminal edge
            set_label_bit(d, t, kSplitBit);
            return true;
        }
        const int u = tri_of(g), Lu = (int)(tfl[u] & 3u);
        g0 = twin.raw(3 * u);
        g1 = twin.raw(3 * u + 1);
        g2 = twin.raw(3 * u + 2);
        if (Lu == g - 3 * u) {
            set_label_bit(d, 3 * t + L < g ? t : u, kSplitBit);
            return true;
        }
        t = u;
        L = Lu;
    }
    return false;
}

// The anchors of every tip, and its polygon's mark: in waves of its own, beside
// those of the anchors, since both are chains of dependent loads.
template <bool ONE>
__global__ void __launch_bounds__(256) k_fixup(const MeshDesc *__restrict__ descs, const ListEntry *tips,
                                               int32_t *tip_counts, const TipSpan tip_span, int cap_tips,
                                               const ListEntry *fixes) {
    const TipStripes stripes(tip_counts, tip_span);
    const int ntips = min(stripes.total(), cap_tips), nfix = 2 * ntips, mark0 = (nfix + kWave - 1) & ~(kWave - 1);
    const int stride = gridDim.x * blockDim.x;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < mark0 + ntips; q += stride) {
        if (q >= nfix) {
            if (q < mark0) continue;
            const ListEntry tip = tips[stripes.index(q - mark0, tip_span)];
            const MeshDesc &d = descs[ONE ? 0 : tip.mesh];
            if (!mark_split(d, tri_of(tip.he))) tip_counts[kUnmarked] = 1;
            continue;
        }
        const ListEntry en = fixes[q];
        if (en.he < 0) continue;
        const MeshDesc &d = descs[ONE ? 0 : en.mesh];
        if (!fix_around(d, en.he)) atomicOr(&d.ctr->err, kErrCorrupt);
    }
}

// ---------------------------------------------------------------------------
// k_walk: seed -> frontier half-edge -> loop minimum and length
// ---------------------------------------------------------------------------

// From seed s, turn clockwise around origin(s) until a frontier half-edge.
__device__ __forceinline__ int seek_frontier(const MeshDesc &d, int s) {
    int f = s;
    for (int k = 0; k < kRotGuard; k++) {
        if (is_frontier(d.tflag, f)) return f;
        const int g = twin_view(d)[f];
        if (g < 0) return -1;
        f = he_next(g);
    }
    return -1;
}


// Every entry of the walk list (a repair seed's half-edge complemented): from
// the seed to a frontier half-edge of its polygon (a frontier half-edge of the
// seed's own triangle if it has one), around the loop, and the loop recorded:
// its code at the minimum's triangle, one more loop for that triangle's
// compaction tile.  A loop still open after kWalkBoth steps (or after the
// first, when the loops are few and so latency decides) is walked from both
// ends from then on: forward along next' and backward along prev' from the
// start, the two loads of a step in flight together, until the ends meet, so
// a long loop of len half-edges takes about len / 2 dependent steps (short
// loops, the most, read no prev').  A step loads the three links of its triangle
// and follows the loop until it leaves it, one or two half-edges on (loading one
// link a step, the kernel took 100 us on the 33.5M grid, this 91; 37 and 35 on
// 64 mirrored Delaunay patches of 16,384 points).  Each chain also writes the
// half-edges it visits to an LDS buffer (forward ones from the front, backward ones from
// the back), so a loop of at most BUF half-edges is copied to the scratch pool
// (rotation index of the minimum, then the half-edges in loop order from the
// first backward one) and k_compact places it without walking it again.  A
// chain that fills the buffer takes kLongWords of the pool and empties the buffer
// there each time it is full, forward half-edges from the front and backward ones
// from the back (and from there to a larger place), so that k_emit copies a loop
// of up to kHugeMax half-edges instead of walking it again (its chain of
// dependent steps took 22 us for the longest loops of those patches, some 65
// half-edges; the copies take 6, and this kernel 37 instead of 33).  Such
// chains go on in a loop of their own, one link of either end at a
// step: few lanes are left then, and a wave's time is the instructions of its
// steps (one loop of 200 half-edges: 71 us with the steps of the short ones, 46
// so).
//
// Whole waves iterate together, with nothing but the two loads in a step.  What
// bounds the kernel is its device-scope atomics: one per wave for the pool, one
// per wave and compaction tile for the totals (a wave's loops end in a few
// tiles), one per repair seed.  With a claim, a total and a mark per loop,
// settled in the step in which it closed, the patches (280,000 loops) took 61
// us.  With an atomic per lane for the larger places, one triangulation of 1M
// points, whose loops are longer, took 46, now 40, and 60,000 loops of 17
// half-edges 44, now 20.
constexpr int kWalkBoth = 8;
// lpos of a loop of kPlMax or more that is stored: the sign bit, its length and
// its place in the pool in units of kPoolUnit.  (With the place alone, and the
// length read from the pool, k_compact took 183 us on the 33.5M grid, not 170.)
// Places from 2^24 units on do not pack, and their loops are walked again: some
// of a run's from 57 million triangles on.
__device__ __forceinline__ bool packs_long(int len, int pos) {
    return pos >= 0 && pos < kPoolUnit << 24 && len - kPlMax < 128;
}
__device__ __forceinline__ int pack_long(int len, int pos) {
    return (int)(0x80000000u | (uint32_t)(len - kPlMax) << 24 | (uint32_t)pos / kPoolUnit);
}
__device__ __forceinline__ int packed_len(int lp) { return ((lp >> 24) & 127) + kPlMax; }
__device__ __forceinline__ int packed_pos(int lp) { return (lp & 0xffffff) * kPoolUnit; }
constexpr int kLongHead = 4, kLongMax = 68, kLongWords = kLongHead + kLongMax, kHugeMax = 188, kNotTried = -2;
static_assert(kHugeMax - kPlMax < 128, "a stored loop's length packs");
static_assert(kLongWords % kPoolUnit == 0 && (kLongHead + kHugeMax) % kPoolUnit == 0 && kPoolUnit % 4 == 0, "its place packs");
static_assert(kPlMax - 1 <= kLongMax, "every loop whose code holds its length fits");

// ONE (here and in the other list-driven kernels): a run of one mesh, whose
// descriptor is read once, uniformly, and not per entry.
template <int BUF, bool ONE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) k_walk(const MeshDesc *__restrict__ descs, const ListEntry *walk,
                                              const int32_t *walk_counts, int walk_cap, const int32_t *tip_counts,
                                              uint64_t *agg, int cmp_tb, int32_t *wbuf, int32_t *wbuf_counts,
                                              int wbuf_cap) {
    constexpr int kSlots = 256;
    constexpr int kHeld = BUF + 3;   // a step takes up to four half-edges
    __shared__ int s_pref[kStripes + 1];
    __shared__ int s_buf[kHeld * kSlots];   // element k of thread q's chain at k * kSlots + q
    const int total = striped_prefix(walk_counts, walk_cap, s_pref);
    const int nthreads = gridDim.x * blockDim.x;
    const bool claim_all = tip_counts[kUnmarked] != 0;   // (uniform)
    const int lane = __lane_id(), tid = threadIdx.x;
    const int wstripe = ((blockIdx.x * blockDim.x + tid) >> 6) % kStripes;   // this wave's pool stripe
    // few loops (a quarter of the threads or fewer): every walk is its own
    // critical path, so all go both ways from the first step; otherwise only
    // the long ones
    const int both = total <= nthreads / 4 ? 1 : kWalkBoth;
    for (int b0 = blockIdx.x * blockDim.x; b0 < total; b0 += nthreads) {   // block-uniform
        gcint nx = nullptr, pv = nullptr;
        // forward end fc (fa half-edges taken, from the start on), backward
        // end bc (bb taken before the start; the start itself while bb == 0);
        // the minimum so far and where: forward index, or ~backward index
        int mesh = 0, fc = -1, bc = -1, fa = 0, bb = 0, mn = -1, mpos = 0, lim = 0;
        // the chain's place in the pool, or -1; what it holds; the half-edges that are there already
        int far = kNotTried, room = kLongMax, f0 = 0, k0 = 0;
        bool live = false, closed = false, repair = false, more = false;
        if (b0 + tid < total) {
            const ListEntry e = walk[striped_index(s_pref, walk_cap, b0 + tid)];
            mesh = ONE ? 0 : e.mesh;
            const MeshDesc &d = descs[mesh];
            repair = e.he < 0;
            const int he = repair ? ~e.he : e.he, t = tri_of(he);
            nx = (gcint)d.next_o;
            pv = (gcint)d.prev_o;
            lim = 3 * d.nt;
            const uint32_t f = ((gcu8)d.tflag)[t];
            if (repair || !(f & kSplitBit)) {
                int st = fbit(f, he - 3 * t) ? he : -1;
#pragma unroll
                for (int i = 0; i < 3; i++)
                    if (st < 0 && fbit(f, i)) st = 3 * t + i;
                if (st < 0) st = seek_frontier(d, he);
                if (st < 0) atomicOr(&d.ctr->err, kErrCorrupt);
                live = st >= 0;
                fc = bc = mn = st;
                fa = 1;
                s_buf[tid] = st;
            }
        }
        // words of the pool for each lane that is here: one atomic for all
        const auto take = [&](int words) {
            const unsigned long long here = __ballot(true);
            const int leader = __ffsll((long long)here) - 1;
            int at = 0;
            if (lane == leader) at = atomicAdd(&wbuf_counts[wstripe * kStripePad], words * __popcll(here));
            return __builtin_amdgcn_readlane(at, leader) + words * __popcll(here & ((1ull << lane) - 1ull));
        };
        // the buffered half-edges go to the chain's place in the pool, if there is one
        const auto flush = [&]() {
            if (far == kNotTried) {
                const int at = take(kLongWords);
                far = at + kLongWords <= wbuf_cap ? wstripe * wbuf_cap + at : -1;
            }
            if (far >= 0 && fa + bb > room) {
                int at = wbuf_cap;
                if (room == kLongMax) at = take(kLongHead + kHugeMax);
                const int to = at + kLongHead + kHugeMax <= wbuf_cap ? wstripe * wbuf_cap + at : -1;
                if (to >= 0) {
                    // the whole place to both ends of the larger one, four
                    // 16-byte groups in flight
                    const GLOBAL v4i *in = (const GLOBAL v4i *)((gcint)wbuf + far + kLongHead);
                    GLOBAL v4i *out = (GLOBAL v4i *)((gint)wbuf + to + kLongHead);
                    constexpr int kGroups = kLongMax / 4, kBack = (kHugeMax - kLongMax) / 4;
                    static_assert(kLongMax % 4 == 0 && kHugeMax % 4 == 0 && kHugeMax >= 2 * kLongMax, "16-byte groups, apart");
                    for (int k = 0; k < kGroups; k += 4) {
                        v4i v[4];
#pragma unroll
                        for (int g = 0; g < 4; g++) v[g] = in[min(k + g, kGroups - 1)];
#pragma unroll
                        for (int g = 0; g < 4; g++) out[min(k + g, kGroups - 1)] = out[kBack + min(k + g, kGroups - 1)] = v[g];
                    }
                }
                far = to;
                room = kHugeMax;
            }
            if (far >= 0) {
                const gint out = (gint)wbuf + far + kLongHead;
                for (int k = f0; k < fa; k++) out[k] = s_buf[(k - f0) * kSlots + tid];
                for (int k = k0; k < bb; k++) out[room - 1 - k] = s_buf[(kHeld - 1 - (k - k0)) * kSlots + tid];
            }
            f0 = fa;
            k0 = bb;
        };
        while (__any(live)) {
            if (!live) continue;
            if (fa + bb >= BUF) {   // the buffer may be full after this step
                more = true;
                live = false;
                continue;
            }
            const bool two = fa >= both;
            const int tf = tri_of(fc), tb = tri_of(bc);
            const v3i nn = *(GLOBAL const v3i_a4 *)(nx + 3 * tf);
            const v3i pp = two ? *(GLOBAL const v3i_a4 *)(pv + 3 * tb) : v3i{0, 0, 0};
            bool done = false, bad = false;
            const auto forward = [&]() {
                const int i = fc - 3 * tf, nf = i == 0 ? nn.x : i == 1 ? nn.y : nn.z;
                done = nf == bc;   // the forward end reached the backward one
                bad = nf < 0;
                if (done || bad) return;
                fc = nf;
                s_buf[fa * kSlots + tid] = nf;
                if (nf < mn) {
                    mn = nf;
                    mpos = fa;
                }
                ++fa;
            };
            const auto backward = [&]() {
                const int i = bc - 3 * tb, nb = i == 0 ? pp.x : i == 1 ? pp.y : pp.z;
                done = nb == fc;   // the backward end reached the forward one
                bad = nb < 0;
                if (done || bad) return;
                bc = nb;
                s_buf[(kHeld - 1 - bb) * kSlots + tid] = nb;
                if (nb < mn) {
                    mn = nb;
                    mpos = ~bb;
                }
                ++bb;
            };
            forward();
            if (!done && !bad && (unsigned)(fc - 3 * tf) < 3u) forward();   // (in the same triangle still)
            if (two && !done && !bad) {
                backward();
                if (!done && !bad && (unsigned)(bc - 3 * tb) < 3u) backward();
            }
            bad |= fa + bb > lim;
            if (bad) atomicOr(&descs[ONE ? 0 : mesh].ctr->err, kErrCorrupt);
            closed = done && !bad;
            live = !done && !bad;
        }
        // the longer loops: both ways, one link of each at a step
        while (__any(more)) {
            if (!more) continue;
            const int nf = nx[fc], nb = pv[bc];
            if (fa - f0 + bb - k0 >= BUF) flush();
            bool done = nf == bc;
            const bool bad = nf < 0 || nb < 0 || fa + bb > lim;
            if (!done) {
                fc = nf;
                s_buf[(fa - f0) * kSlots + tid] = nf;
                if (nf < mn) {
                    mn = nf;
                    mpos = fa;
                }
                ++fa;
                done = nb == nf;
                if (!done) {
                    bc = nb;
                    s_buf[(kHeld - 1 - (bb - k0)) * kSlots + tid] = nb;
                    if (nb < mn) {
                        mn = nb;
                        mpos = ~bb;
                    }
                    ++bb;
                }
            }
            if (bad) atomicOr(&descs[ONE ? 0 : mesh].ctr->err, kErrCorrupt);
            closed = done && !bad;
            more = !done && !bad;
        }
        // every loop of the wave has closed: the claims of the repair seeds,
        // in flight with one atomic for the wave's pool space (a walker that
        // loses its claim leaves its space unused)
        const MeshDesc &d = descs[ONE ? 0 : mesh];
        const int len = fa + bb, tm = closed ? tri_of(mn) : 0;
        if (closed && len > BUF && far != -1) flush();
        const bool taken = closed && (repair || claim_all) && set_label_bit(d, tm, kCountedBit);
        // whole 16-byte groups, so k_compact reads a loop with vector loads
        const int need = closed && len <= BUF ? (len + 4) & ~3 : 0;
        const int incl = wave_incl_scan(need);
        const int wtot = (__builtin_amdgcn_readlane(incl, kWave - 1) + kPoolUnit - 1) / kPoolUnit * kPoolUnit;
        int wbase = 0;
        if (lane == 0 && wtot > 0) wbase = atomicAdd(&wbuf_counts[wstripe * kStripePad], wtot);
        wbase = __builtin_amdgcn_readlane(wbase, 0);
        const int pos = wbase + wtot <= wbuf_cap ? wstripe * wbuf_cap + wbase + incl - need : -1;
        const bool won = closed && !taken;
        const int key = won ? d.cmp_tile0 + tm / cmp_tb : -1;
        if (won) {
            ((gu8)d.pl)[tm] = loop_code(mn, len);
            // where the loop is stored (-1: nowhere), or its length when the
            // code does not hold it
            // (both for a stored one, packed: k_compact needs the length at once)
            ((gint)d.lpos)[tm] = len <= BUF ? pos : len < kPlMax ? far : packs_long(len, far) ? pack_long(len, far) : len;
            if (len > BUF && far >= 0)   // a record's head:
                // forward half-edges, the minimum's position from the start
                *(GLOBAL v4i *)((gint)wbuf + far) = v4i{fa, mpos >= 0 ? mpos : len - 1 - ~mpos, len, room};
            if (need && pos >= 0) {
                // position of the minimum in loop order from the first backward
                // half-edge; then the backward half-edges (from the back of the
                // buffer) and the forward ones, in 16-byte groups
                GLOBAL v4i *out = (GLOBAL v4i *)((gint)wbuf + pos);
                const int rot = mpos >= 0 ? bb + mpos : bb - 1 - ~mpos;
                const int back = (kHeld - bb) * kSlots + tid, fore = -bb * kSlots + tid;
                const auto at = [&](int k) { return s_buf[(k < bb ? back : fore) + min(k, len - 1) * kSlots]; };
                for (int k = -1; k < len; k += 4) *out++ = v4i{k < 0 ? rot : at(k), at(k + 1), at(k + 2), at(k + 3)};
            }
        }
        // the loops into their compaction tiles' totals, tile by tile for up
        // to four tiles, then one by one
        unsigned long long todo = __ballot(won);
        for (int k = 0; k < 4 && todo; k++) {
            const int leader = __ffsll((long long)todo) - 1, kt = __builtin_amdgcn_readlane(key, leader);
            const unsigned long long same = __ballot(key == kt);
            const int sum = __builtin_amdgcn_readlane(wave_incl_scan(key == kt ? len : 0), kWave - 1);
            if (lane == leader)
                atomicAdd(reinterpret_cast<unsigned long long *>(agg + kt),
                          ((unsigned long long)(uint32_t)__popcll(same) << 32) | (unsigned long long)(uint32_t)sum);
            todo &= ~same;
        }
        if ((todo >> lane) & 1)
            atomicAdd(reinterpret_cast<unsigned long long *>(agg + key), (1ull << 32) | (unsigned long long)(uint32_t)len);
    }
}

// The loops k_compact left out, each written from its minimum at its offset
// from both ends at once: position s forward along next' and position len - s
// backward along prev', so the two loads of a step are in flight together and
// a loop of len half-edges takes about len / 2 dependent steps.
template <int ITEMS, bool ONE>
__global__ void __launch_bounds__(256) k_emit(const MeshDesc *__restrict__ descs, const EmitEntry *emit,
                                              const int32_t *emit_counts, int emit_cap, const int32_t *wbuf,
                                              int wbuf_cap, int nmesh) {
    // the counts are complete but for errors found here
    if (blockIdx.x == 0)
        for (int m = threadIdx.x; m < nmesh; m += blockDim.x) {
            const MeshDesc &d = descs[m];
            if (!d.ctr_out) continue;
            const MeshCounters c = *d.ctr;
            d.ctr_out->ntips = c.ntips;
            d.ctr_out->nmiddle = c.nmiddle;
            d.ctr_out->nties = c.nties;
            d.ctr_out->npoly = c.npoly;
            d.ctr_out->nloop = c.nloop;
            if (c.err) d.ctr_out->err = c.err;
        }
    const auto corrupt = [](const MeshDesc &d) {
        atomicOr(&d.ctr->err, kErrCorrupt);
        if (d.ctr_out) d.ctr_out->err = kErrCorrupt;
    };
    __shared__ int s_pref[kStripes + 1];
    const int total = striped_prefix(emit_counts, emit_cap, s_pref);
    const int nthreads = gridDim.x * blockDim.x;
    // loops that k_walk kept: kCopyLanes lanes copy one, from its minimum on
    constexpr int kCopyLanes = 16;
    const int sub = threadIdx.x % kCopyLanes;
    for (int g = (blockIdx.x * blockDim.x + threadIdx.x) / kCopyLanes; g < total; g += nthreads / kCopyLanes) {
        const EmitEntry e = emit[striped_index(s_pref, emit_cap, g)];
        if (e.mn >= 0) continue;
        const MeshDesc &d = descs[ONE ? 0 : e.mesh];
        // its lanes, all of one wave, read these before any of them writes
        const bool in = e.off >= 0 && e.off < 3 * d.nt - 1;
        const int L = in ? ((gcint)d.loop_he)[e.off] : -1, at = in ? ((gcint)d.loop_he)[e.off + 1] : -1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int pos = L < kPlMax ? at : packed_pos(at);
        const bool ok = L > 0 && (long long)e.off + L <= 3ll * d.nt && pos >= 0 &&
                        pos <= kStripes * wbuf_cap - kLongWords;
        const gcint src = (gcint)wbuf + (ok ? pos : 0);
        const int fore = src[0], rot = src[1], room = src[3];
        if (!ok || L != src[2] || L > room || (room != kLongMax && room != kHugeMax) ||
            pos > kStripes * wbuf_cap - kLongHead - room || fore < 1 || fore > L || rot < 0 || rot >= L) {
            if (sub == 0) corrupt(d);
            continue;
        }
        const gint out = (gint)d.loop_he + e.off;
        constexpr int kCopies = 4;
        for (int k0 = sub; k0 < L; k0 += kCopies * kCopyLanes) {
            int v[kCopies];
#pragma unroll
            for (int j = 0; j < kCopies; j++) {
                const int k = k0 + j * kCopyLanes;
                v[j] = src[kLongHead + (k < fore ? k : min(k + room - L, room - 1))];
            }
#pragma unroll
            for (int j = 0; j < kCopies; j++) {
                const int k = k0 + j * kCopyLanes;
                if (k >= L) continue;
                if (k == rot && v[j] != ~e.mn) corrupt(d);
                out[k >= rot ? k - rot : k - rot + L] = v[j];
            }
        }
    }
    // the others: walked again, from both ends
    for (int g0 = blockIdx.x * blockDim.x + threadIdx.x; g0 < total; g0 += nthreads * ITEMS) {
        gcint nx[ITEMS], pv[ITEMS];
        gint out[ITEMS];
        int mesh[ITEMS], f[ITEMS], b[ITEMS], len[ITEMS];
        bool live[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            live[j] = false;
            f[j] = b[j] = len[j] = mesh[j] = 0;
            nx[j] = pv[j] = nullptr;
            out[j] = nullptr;
            const int g = g0 + j * nthreads;
            if (g >= total) continue;
            const EmitEntry e = emit[striped_index(s_pref, emit_cap, g)];
            if (e.mn < 0) continue;
            const MeshDesc &d = descs[ONE ? 0 : e.mesh];
            mesh[j] = ONE ? 0 : e.mesh;
            // k_compact left the loop's length in its first slot
            const int L = (e.off >= 0 && e.off < 3 * d.nt) ? ((gcint)d.loop_he)[e.off] : -1;
            if (L < 1 || (long long)e.off + L > 3ll * d.nt) {
                corrupt(d);
                continue;
            }
            nx[j] = (gcint)d.next_o;
            pv[j] = (gcint)d.prev_o;
            out[j] = (gint)d.loop_he + e.off;
            f[j] = b[j] = e.mn;
            len[j] = L;
            out[j][0] = e.mn;
            live[j] = L > 1;
        }
        for (int s = 1;; s++) {
            bool active = false;
#pragma unroll
            for (int j = 0; j < ITEMS; j++) {
                if (!live[j]) continue;
                const int bi = len[j] - s;   // the backward end's position; the forward end's is s
                if (s > bi) {
                    live[j] = false;
                    continue;
                }
                const int nf = nx[j][f[j]], nb = pv[j][b[j]];   // both in flight together
                if (nf < 0 || nb < 0) {
                    corrupt(descs[ONE ? 0 : mesh[j]]);
                    live[j] = false;
                    continue;
                }
                out[j][s] = nf;
                if (s < bi) out[j][bi] = nb;
                f[j] = nf;
                b[j] = nb;
                active = true;
            }
            if (!active) break;
        }
    }
}

// ---------------------------------------------------------------------------
// k_tile_scan: exclusive scan of the compaction tiles' loop totals
//
// k_relink (settled loops) and k_walk (walked loops) add every loop, once, to
// the total of the compaction tile holding its minimum: (loops << 32 |
// half-edges).  One block per mesh turns the totals into exclusive prefixes
// in place and records the mesh's polygon and loop half-edge counts, so each
// k_compact tile starts with its output offsets known.
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(1024) k_tile_scan(const MeshDesc *__restrict__ descs, uint64_t *status,
                                                     uint64_t *cpre, int cmp_tb) {
    // block (mesh, chunk): tiles [chunk * kScanChunk, ...) of that mesh,
    // kTileScanItems consecutive ones per thread, read and written contiguously
    __shared__ int s_scan[72];
    __shared__ int s_last;
    const MeshDesc &d = descs[blockIdx.x];
    const int ntiles = d.nt > 0 ? (d.nt + cmp_tb - 1) / cmp_tb : 1;
    const int nchunks = (ntiles + kScanChunk - 1) / kScanChunk;
    const int chunk = blockIdx.y;
    if (chunk >= nchunks) return;   // the whole block
    const int tid = threadIdx.x, k0 = chunk * kScanChunk + tid * kTileScanItems;
    uint64_t *st = status + d.cmp_tile0;
    uint64_t v[kTileScanItems];
    int lc = 0, lh = 0;
#pragma unroll
    for (int i = 0; i < kTileScanItems; i++) {
        v[i] = k0 + i < ntiles ? st[k0 + i] : 0ull;
        lc += (int)(v[i] >> 32);
        lh += (int)(uint32_t)v[i];
    }
    int ec, eh, tc, th;
    block_excl_scan2(lc, lh, ec, eh, tc, th, s_scan);
#pragma unroll
    for (int i = 0; i < kTileScanItems; i++) {
        if (k0 + i < ntiles) st[k0 + i] = ((uint64_t)(uint32_t)ec << 32) | (uint32_t)eh;
        ec += (int)(v[i] >> 32);
        eh += (int)(uint32_t)v[i];
    }
    if (nchunks == 1) {   // (uniform) the whole mesh in one block: its totals at once
        if (tid == 0) {
            cpre[d.cmp_tile0] = 0ull;
            const bool ok = tc >= 0 && th >= 0 && tc <= d.nt && th <= 3 * d.nt;
            d.ctr->npoly = ok ? tc : 0;
            d.ctr->nloop = ok ? th : 0;
            if (ok)
                d.loop_off[tc] = th;
            else
                atomicOr(&d.ctr->err, kErrCorrupt);
        }
        return;
    }
    // chunk total at the chunk's first tile; the last block of the mesh turns
    // the totals into prefixes
    if (tid == 0) {
        cpre[d.cmp_tile0 + chunk * kScanChunk] = ((uint64_t)(uint32_t)tc << 32) | (uint32_t)th;
        __threadfence();
        s_last = atomicAdd(&d.ctr->chunks_done, 1) == nchunks - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    int c = 0, h = 0;
    for (int base = 0; base < nchunks; base += blockDim.x) {   // chunks beyond 1024: further rounds
        const int q = base + tid;
        uint64_t *slot = cpre + d.cmp_tile0 + (size_t)q * kScanChunk;
        const uint64_t w = q < nchunks ? __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
        int ec2, eh2, tc2, th2;
        block_excl_scan2((int)(w >> 32), (int)(uint32_t)w, ec2, eh2, tc2, th2, s_scan);
        if (q < nchunks) *slot = ((uint64_t)(uint32_t)(c + ec2) << 32) | (uint32_t)(h + eh2);
        c += tc2;
        h += th2;
    }
    if (tid == 0) {
        const bool ok = c >= 0 && h >= 0 && c <= d.nt && h <= 3 * d.nt;
        d.ctr->npoly = ok ? c : 0;
        d.ctr->nloop = ok ? h : 0;
        if (ok)
            d.loop_off[c] = h;
        else
            atomicOr(&d.ctr->err, kErrCorrupt);
    }
}

// ---------------------------------------------------------------------------
// k_compact: seeds, loop offsets and loops of every tile, from the tile's
// prefix; each tile assembles its part in LDS and writes it contiguously
// ---------------------------------------------------------------------------


template <int ITEMS>
__global__ void __launch_bounds__(1024) k_compact(const MeshDesc *__restrict__ descs, int nmesh,
                                                  const uint64_t *status, const uint64_t *cpre, EmitEntry *emit,
                                                  int32_t *emit_counts, int emit_cap, const int32_t *wbuf) {
    // LDS: loop half-edges (compact_he_cap of them), seeds and local offsets
    // (one per triangle)
    extern __shared__ int4 lds_raw[];
    const int B = blockDim.x, tid = threadIdx.x;
    const int TB = B * ITEMS;
    const int he_cap = compact_he_cap(TB);
    int *s_he = reinterpret_cast<int *>(lds_raw);
    int *s_seed = s_he + he_cap;
    int *s_off = s_seed + TB;
    __shared__ int s_scan[72];
    __shared__ int s_ebase;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int mi = find_mesh<2>(descs, nmesh, tile);
    const MeshDesc &d = descs[mi];
    const int nt = d.nt, nh = 3 * nt;
    const int ltile = tile - d.cmp_tile0;
    const int mesh_tiles = nt > 0 ? (nt + TB - 1) / TB : 1;
    const int t0 = ltile * TB + tid * ITEMS;
    const gcint nx = (gcint)d.next_o;
    const gcu8 plb = (gcu8)d.pl, tfl = (gcu8)d.tflag;
    // prefix within the chunk plus the chunk's prefix (no field carries)
    const uint64_t pre = status[tile] + cpre[d.cmp_tile0 + ltile / kScanChunk * kScanChunk];
    const int pc = (int)(pre >> 32), ps = (int)(uint32_t)pre;

    // 1. loop minima and lengths of this thread's ITEMS contiguous triangles;
    //    which loops are longer than a quad, and which of those k_walk stored
    //    (the rest k_emit writes)
    //    (the walk-pool positions come with them, read whether or not a loop
    //    was stored there, so a stored loop's pool read follows directly)
    uint8_t code[ITEMS], fl[ITEMS];
    int lp[ITEMS];
    const gcint lpos = (gcint)d.lpos;
    if (ITEMS == 4 && t0 + 4 <= nt) {
        const uint32_t w = *reinterpret_cast<GLOBAL const uint32_t *>(plb + t0);
        const uint32_t v = *reinterpret_cast<GLOBAL const uint32_t *>(tfl + t0);
        const v4i l4 = *(GLOBAL const v4i *)(lpos + t0);
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            code[j] = (uint8_t)(w >> (8 * (j & 3)));
            fl[j] = (uint8_t)(v >> (8 * (j & 3)));
        }
        lp[0] = l4.x;
        lp[1 % ITEMS] = l4.y;
        lp[2 % ITEMS] = l4.z;
        lp[3 % ITEMS] = l4.w;
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            code[j] = t0 + j < nt ? plb[t0 + j] : 0;
            fl[j] = t0 + j < nt ? tfl[t0 + j] : 0;
            lp[j] = t0 + j < nt ? lpos[t0 + j] : 0;
        }
    }
    int lens[ITEMS];
    bool defer[ITEMS], stored[ITEMS];
    int cnt = 0, sum = 0, nd = 0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        lens[j] = 0;
        defer[j] = stored[j] = false;
        if (!code[j]) continue;
        int len = code[j] >> 2;
        if (len == kPlQuadNext) len = 4;
        // longer than the code holds: k_walk left the length in lpos
        if (len >= kPlMax) {
            len = lp[j] < 0 ? packed_len(lp[j]) : lp[j];
            len = len >= kPlMax && len <= nh ? len : -1;
        }
        if (len <= 0) {
            bad = true;
            len = 0;
        }
        lens[j] = len;
        // loops of three and two-triangle loops of four are written here
        defer[j] = len > 0 && len != 3 && !(len == 4 && __popc((fl[j] >> 2) & 7u) == 2);
        cnt += 1;
        sum += len;
        stored[j] = defer[j] && len <= kWalkBuf && lp[j] >= 0;
        nd += defer[j] && !stored[j];
    }
    // 2. block scan: tile-local loop index and offset, emit-list slot
    int ecn, esum, tcn, tsum;
    block_excl_scan2(cnt | (nd << 16), sum, ecn, esum, tcn, tsum, s_scan);
    const int tcnt = tcn & 0xffff, tnd = tcn >> 16;
    const int stripe = tile % kStripes;
    if (tid == 0) {
        s_ebase = tnd > 0 ? atomicAdd(&emit_counts[stripe * kStripePad], tnd) : 0;
        // the tiles' prefixes must add up to the mesh totals
        if (ltile == mesh_tiles - 1 && (pc + tcnt != d.ctr->npoly || ps + tsum != d.ctr->nloop)) bad = true;
    }
    const bool fits = tsum <= he_cap && pc + tcnt <= nt && ps + tsum <= nh;
    // 3. seeds, local offsets and loops; into LDS, or straight to global
    //    memory for a tile whose loops do not fit
    // A loop of 3 is one triangle: (mn, next, prev).  A loop of 4 is two
    // triangles: the minimum's triangle has frontier half-edges a, b = next(a)
    // and crosses to the other triangle at b, whose two frontier half-edges
    // follow as p1 = next'(b), next(p1).  Longer loops get their offset here
    // and are written by k_emit.
    __syncthreads();
    const int elim = (stripe + 1) * emit_cap;
    bad |= s_ebase + tnd > emit_cap;
    // the body is instantiated twice: loops into LDS (the tile fits, the
    // usual case), or straight to global memory; the tile decides for all
    // its threads
    auto place_loops = [&](auto he_out) {
    int q = ecn & 0xffff, off = esum, e = (ecn >> 16) + stripe * emit_cap + s_ebase;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        if (!code[j]) continue;
        const int t = t0 + j;
        const uint32_t fb = (fl[j] >> 2) & 7u;
        const bool qn = (code[j] >> 2) == kPlQuadNext;
        const int mn = 3 * t + (qn ? __builtin_ctz(fb | 8u) : (code[j] & 3));
        const bool place = fits || (pc + q < nt && ps + off + lens[j] <= nh);
        if (!place) {
            bad = true;
        } else {
            if (fits) {
                s_seed[q] = mn;
                s_off[q] = off;
            } else {
                d.seeds[pc + q] = mn;
                d.loop_off[pc + q] = ps + off;
            }
            if (lens[j] == 3) {
                he_out[off] = mn;
                he_out[off + 1] = he_next(mn);
                he_out[off + 2] = he_prev(mn);
            } else if (!defer[j] && lens[j] == 4) {
                // non-frontier edge sx; a = next(sx), b = prev(sx); the loop
                // crosses sx's twin into the other triangle
                const int sx = (fb & 1u) == 0 ? 0 : ((fb & 2u) == 0 ? 1 : 2);
                const int aa = 3 * t + (sx == 2 ? 0 : sx + 1), bb = 3 * t + (sx == 0 ? 2 : sx - 1);
                int p1;
                if (qn) {   // the second triangle is t + 1: next'(b) leaves its terminal edge
                    const int Lp = code[j] & 3;
                    p1 = 3 * (t + 1) + (Lp == 2 ? 0 : Lp + 1);
                } else {
                    p1 = nx[bb];
                }
                if (p1 < 0 || (mn != aa && mn != bb)) {
                    bad = true;
                } else if (mn == aa) {
                    he_out[off] = aa;
                    he_out[off + 1] = bb;
                    he_out[off + 2] = p1;
                    he_out[off + 3] = he_next(p1);
                } else {
                    he_out[off] = bb;
                    he_out[off + 1] = p1;
                    he_out[off + 2] = he_next(p1);
                    he_out[off + 3] = aa;
                }
            } else if (stored[j]) {
                // stored by k_walk in walk order from some start; rotate so
                // the loop begins at its minimum (loads first, all in flight)
                static_assert(kWalkBuf % 4 == 0, "stored loops are read in 16-byte groups");
                const int len = lens[j];
                const GLOBAL v4i *src = (GLOBAL const v4i *)((gcint)wbuf + lp[j]);
                v4i g[kWalkBuf / 4 + 1];   // rotation index, then the half-edges
#pragma unroll
                for (int c = 0; c <= kWalkBuf / 4; c++) g[c] = src[c];
                int v[kWalkBuf + 4];
#pragma unroll
                for (int c = 0; c <= kWalkBuf / 4; c++) {
                    v[4 * c] = g[c].x;
                    v[4 * c + 1] = g[c].y;
                    v[4 * c + 2] = g[c].z;
                    v[4 * c + 3] = g[c].w;
                }
                const int rot = v[0];
                if (rot < 0 || rot >= len || len > kWalkBuf || v[1 + rot] != mn) bad = true;
                else
#pragma unroll
                    for (int k = 0; k < kWalkBuf; k++)
                        if (k < len) he_out[off + (k >= rot ? k - rot : k - rot + len)] = v[1 + k];
            } else if (defer[j]) {
                if (e < elim) {
                    emit[e].mesh = mi;
                    emit[e].mn = lens[j] > kWalkBuf && (lens[j] < kPlMax) == (lp[j] >= 0) ? ~mn : mn;
                    emit[e].off = ps + off;
                }
                // the loop's length and place in the walk pool in its own
                // first slots, which k_emit reads and then overwrites
                he_out[off] = lens[j];
                if (lens[j] > 1) he_out[off + 1] = lp[j];
                ++e;
            }
        }
        ++q;
        off += lens[j];
    }
    };
    if (fits)
        place_loops(s_he);
    else
        place_loops((gint)d.loop_he + ps);
    if (fits) {
        __syncthreads();
        // contiguous stores of the tile's part of seeds, loop_off, loop_he;
        // all of a thread's LDS reads are issued before its first store
        constexpr int kSeedIt = ITEMS;                  // tcnt <= TB
        constexpr int kHeIt = (kCompactHe4 * ITEMS + 3) / 4;   // tsum <= he_cap
        const gint seeds = (gint)d.seeds, loff = (gint)d.loop_off, lhe = (gint)d.loop_he;
        int vs[kSeedIt], vo[kSeedIt], vh[kHeIt];
#pragma unroll
        for (int it = 0; it < kSeedIt; it++) {
            const int k = tid + it * B;
            vs[it] = s_seed[k < tcnt ? k : 0];
            vo[it] = s_off[k < tcnt ? k : 0];
        }
#pragma unroll
        for (int it = 0; it < kHeIt; it++) {
            const int k = tid + it * B;
            vh[it] = s_he[k < tsum ? k : 0];
        }
#pragma unroll
        for (int it = 0; it < kSeedIt; it++) {
            const int k = tid + it * B;
            if (k < tcnt) {
                seeds[pc + k] = vs[it];
                loff[pc + k] = ps + vo[it];
            }
        }
#pragma unroll
        for (int it = 0; it < kHeIt; it++) {
            const int k = tid + it * B;
            if (k < tsum) lhe[ps + k] = vh[it];
        }
    }
    if (bad) atomicOr(&d.ctr->err, kErrCorrupt);
}

// ---------------------------------------------------------------------------
// k_small: the whole chain for one small mesh in one workgroup
//
// Below a few thousand triangles the chain's time is its eight launches and
// the memory round trips that open each of them, not its bytes.  A mesh of at
// most kSmallMaxTri triangles keeps every intermediate array in LDS, and one
// workgroup runs the steps with block barriers between them:
//   1. longest edge of every triangle (Section 6.1, Algorithm 8);
//   2. frontier bits and the seeds of terminal edges (Sections 6.2-6.3);
//   3. next' of every frontier half-edge, as in k_relink: the turn across the
//      edge that its triangle's frontier bits name (Section 6.5, Algorithm
//      12).  The same turns find the barrier tips (Section 6.4, Algorithm 11):
//      one that comes all the way round to the twin of its half-edge met no
//      other frontier edge, so that target is a tip whose degree is the turn's
//      length; its middle edge lies half the degree further round.  The turns
//      around both ends of every middle edge are then taken again with the
//      repaired frontier;
//   4. prev' as the inverse of next'; every seed's loop walked once for its
//      minimum and length (Section 6.6, Algorithm 14; the first walker of a
//      loop that several seeds reach records it), or, when some loop is long,
//      all loops ranked by pointer doubling;
//   5. seeds and loop offsets from a block scan over the triangles that hold a
//      minimum (Section 6.7);
//   6. every loop walked again from its minimum into its place, or by its ranks.
// In LDS a half-edge 3t + i is slot 4t + i, so next and the triangle of a
// slot are bit operations (the order of slots is the order of half-edges),
// and slot 4t + 3 holds what belongs to the triangle.  The vector instructions
// of a single CU bound the kernel: a thread handles whole triangles, most with
// one turn that ends at its first candidate, and a thread per loop walks it:
// 12.5 us for a 2,048-triangle grid, where one item per half-edge, and loop
// minima by pointer doubling over all of them, took 22 us.  The outputs equal the tiled chain's
// element by element.  One workgroup per mesh: a batch whose meshes are all
// small is one launch.
// ---------------------------------------------------------------------------

constexpr uint32_t kNo16 = 0xffff;   // no slot (boundary), in 16 bits
// The word of slot 4t + 3: bits 0-1 the longest edge, bits 2-4 the label
// phase's frontier bits, bits 5-7 the edges the repair adds, bit 8 the loop
// whose minimum lies in t has been recorded.
constexpr uint32_t kRecorded = 1u << 8;
__device__ __forceinline__ uint32_t repaired_bits(uint32_t lab) { return ((lab >> 2) | (lab >> 5)) & 7u; }

// The corners and twin slots of a thread's triangles t = tid + j * kSmallBlock.
template <int TI>
struct SmallTris {
    int v[TI][3];
    uint32_t s[TI][3];
};

template <int TI>
__device__ __forceinline__ void small_load(const MeshDesc &d, SmallTris<TI> &tr) {
    const TwinView twin = twin_view(d);
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = threadIdx.x + j * kSmallBlock, tt = t < d.nt ? t : 0;
        if (!d.org8) {
            const gcint org = (gcint)(d.org);
#pragma unroll
            for (int i = 0; i < 3; i++) tr.v[j][i] = org[3 * tt + i];
        } else {
            const v2i r = ((GLOBAL const v2i *)d.org8)[tt];
            const int d1 = (int)(int16_t)(r.y & 0xffff), d2 = r.y >> 16;
            tr.v[j][0] = r.x;
            tr.v[j][1] = d1 != kEsc16 ? r.x + d1 : esc_lookup(d.esc, d.esc_mask, ~(3 * tt + 1));
            tr.v[j][2] = d2 != kEsc16 ? r.x + d2 : esc_lookup(d.esc, d.esc_mask, ~(3 * tt + 2));
        }
#pragma unroll
        for (int i = 0; i < 3; i++) tr.s[j][i] = he_slot(max(twin[3 * tt + i], -1));
    }
}

// The counts of a run go to the mesh's device counters and to the host's
// coherent copy, where there are such.
__device__ __forceinline__ void small_counts(const MeshDesc &d, const MeshCounters &c) {
    if (d.ctr) *d.ctr = c;
    if (d.ctr_out) *d.ctr_out = c;
}

// Loops longer than this are not walked by one thread.
template <int TI>
constexpr int kSmallWalk = 16 * (TI + 1);

// The minimum of every loop, its length, and every half-edge's place in its
// loop, by pointer doubling along prev': for meshes with a long loop, which one
// thread would walk twice, 55 ns a step (a strip of 4,079 triangles, one loop:
// 474 us for a run with the walks, 64 so; 599 triangles, 89 and 29).  First each
// half-edge's minimum over ever longer stretches (most: half-edges on the long
// loops together), then its distance from that minimum.  Value and link of a half-edge are one word, so
// a round needs no barrier between its reads and its writes: a word that has
// moved on already only makes the stretch longer.  A round follows two links.
// Leaves by slot: minimum | place << 16; and 4t + 3: the length of the loop with its
// minimum in t, or 0.
template <int TI>
__device__ __forceinline__ void small_rank(uint32_t *s_pk, const uint16_t *s_pv, const uint32_t (&F)[TI], int nt,
                                           int most) {
    uint32_t p[TI][3], m[TI][3], n[TI][3];
    bool on[TI][3];
    // every frontier half-edge of the thread: f(its slot, j, i)
    const auto each = [&](auto f) {
#pragma unroll
        for (int j = 0; j < TI; j++)
#pragma unroll
            for (int i = 0; i < 3; i++)
                if (on[j][i]) f(4u * (threadIdx.x + j * kSmallBlock) + i, j, i);
    };
#pragma unroll
    for (int j = 0; j < TI; j++)
#pragma unroll
        for (int i = 0; i < 3; i++) on[j][i] = (int)threadIdx.x + j * kSmallBlock < nt && ((F[j] >> i) & 1u);
    each([&](uint32_t q, int j, int i) { p[j][i] = s_pv[q]; });
    __syncthreads();   // (s_pk lies over s_pv)
    each([&](uint32_t q, int j, int i) {
        m[j][i] = q;
        n[j][i] = p[j][i];
        s_pk[q] = q | p[j][i] << 16;
    });
#pragma unroll
    for (int j = 0; j < TI; j++)
        if ((int)threadIdx.x + j * kSmallBlock < nt) s_pk[4 * (threadIdx.x + j * kSmallBlock) + 3] = 0;
    __syncthreads();
    for (int w = 1; w < most; w *= 3) {   // stretches of w at least
        each([&](uint32_t, int j, int i) {
            const uint32_t a = s_pk[n[j][i]], b = s_pk[a >> 16];
            m[j][i] = min(m[j][i], min(a & 0xffffu, b & 0xffffu));
            n[j][i] = b >> 16;
        });
        each([&](uint32_t q, int j, int i) { s_pk[q] = m[j][i] | n[j][i] << 16; });
        __syncthreads();
    }
    uint32_t d[TI][3];
    each([&](uint32_t q, int j, int i) {
        d[j][i] = m[j][i] != q;
        n[j][i] = m[j][i] != q ? p[j][i] : q;
        s_pk[q] = d[j][i] | n[j][i] << 16;
    });
    __syncthreads();
    for (int w = 1; w < 4 * nt; w *= 3) {   // (a valid mesh's loops end it sooner)
        bool open = false;
        each([&](uint32_t, int j, int i) {
            const uint32_t a = s_pk[n[j][i]], b = s_pk[a >> 16];
            d[j][i] += (a & 0xffffu) + (b & 0xffffu);
            n[j][i] = b >> 16;
            open |= n[j][i] != m[j][i];
        });
        each([&](uint32_t q, int j, int i) { s_pk[q] = (d[j][i] & 0xffffu) | n[j][i] << 16; });
        if (!__syncthreads_or(open)) break;   // (uniform)
    }
    each([&](uint32_t q, int j, int i) {
        if (m[j][i] == q) s_pk[q | 3u] = (s_pk[p[j][i]] & 0xffffu) + 1u;
    });
    __syncthreads();
    each([&](uint32_t q, int j, int i) { s_pk[q] = m[j][i] | d[j][i] << 16; });
}

// TI: triangles per thread (1, 2 or 4).
template <int TI>
__device__ __forceinline__ void small_body(const MeshDesc &d, const SmallTris<TI> &tr) {
    extern __shared__ int4 lds_raw[];
    __shared__ int s_scan[72];
    __shared__ int s_cnt[6];   // tied maxima, tips, new middle edges, frontier half-edges, seeds, half-edges of walked loops
    const int nt = d.nt, nh = 3 * nt, tid = threadIdx.x, lane = __lane_id();
    const uint32_t ns = 4u * (uint32_t)nt;
    uint16_t *s_sl = reinterpret_cast<uint16_t *>(lds_raw);   // by slot: the twin's slot; 4t + 3: the triangle's word
    uint16_t *s_nx = s_sl + ns;     // by slot: next'; 4t + 3: length, then place, of the loop with its minimum in t
    uint16_t *s_pv = s_nx + ns;     // by slot: prev'; then the loops' half-edges in output order
    uint16_t *s_list = s_pv + ns;   // seeds (label phase, then both sides of every middle edge), then minima
    uint32_t *w32 = reinterpret_cast<uint32_t *>(s_sl);
    int bad = 0;
    __shared__ int s_longer;   // some loop was not walked to its end
    if (tid < 6) s_cnt[tid] = 0;
    if (tid == 0) s_longer = 0;

    // 1. longest edges; edge i of t runs from corner i to corner i + 1, and a
    //    tie at the maximum goes to the lower edge id min(h, twin h)
    uint32_t L[TI];
    {
        const gcv2i xy = (gcv2i)(d.xy);
        int2 p[TI][3];
#pragma unroll
        for (int j = 0; j < TI; j++) {
            const bool in = tid + j * kSmallBlock < nt;
#pragma unroll
            for (int i = 0; i < 3; i++) {
                const bool ok = tr.v[j][i] >= 0 && tr.v[j][i] < d.nv;
                bad |= in && !ok;
                const v2i q = xy[ok ? tr.v[j][i] : 0];
                p[j][i] = make_int2(q.x, q.y);
            }
        }
        __syncthreads();   // (s_cnt; and, after a build, its table)
        int ties = 0;
#pragma unroll
        for (int j = 0; j < TI; j++) {
            const int t = tid + j * kSmallBlock;
            L[j] = 0;
            if (t >= nt) continue;
            const long long l[3] = {sq_len(p[j][0], p[j][1]), sq_len(p[j][1], p[j][2]), sq_len(p[j][2], p[j][0])};
            long long bl = l[0];
            uint32_t bid = min(tr.s[j][0], 4u * t);
#pragma unroll
            for (int i = 1; i < 3; i++) {
                const uint32_t id = min(tr.s[j][i], 4u * t + i);
                if (l[i] > bl || (l[i] == bl && id < bid)) {
                    L[j] = i;
                    bl = l[i];
                    bid = id;
                }
            }
            ties += (l[0] == bl) + (l[1] == bl) + (l[2] == bl) > 1;
#pragma unroll
            for (int i = 0; i < 3; i++) bad |= tr.s[j][i] != kNoSlot && tr.s[j][i] >= ns;
            reinterpret_cast<ushort4 *>(s_sl)[t] = make_ushort4((uint16_t)tr.s[j][0], (uint16_t)tr.s[j][1], (uint16_t)tr.s[j][2], (uint16_t)L[j]);
        }
        if (ties) atomicAdd(&s_cnt[0], ties);
    }
    if (__syncthreads_or(bad)) {   // (uniform) a slot or corner out of range
        if (tid == 0) {
            MeshCounters c{};
            c.err = kErrCorrupt;
            small_counts(d, c);
        }
        return;
    }

    // 2. frontier edges: on the boundary, or the longest edge of neither
    //    triangle; seeds: the lower half-edge of a terminal edge
    uint32_t F[TI];
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
        F[j] = 0;
        bool seed = false;
        if (t < nt) {
            const uint32_t lbit = 1u << L[j], sL = pick3(L[j], tr.s[j][0], tr.s[j][1], tr.s[j][2]);
            uint32_t E = 0, bnd = 0;   // bit i: the twin of edge i is not its triangle's longest edge; is missing
#pragma unroll
            for (int i = 0; i < 3; i++) {
                const uint32_t q = tr.s[j][i], lab = s_sl[4 * min(q >> 2, (uint32_t)nt - 1u) + 3];
                E |= min((lab ^ q) & 3u, 1u) << i;
                bnd |= q == kNoSlot ? 1u << i : 0u;
            }
            F[j] = (E & ~lbit) | bnd;
            seed = (bnd & lbit) || (!(E & lbit) && 4u * t + L[j] < sL);
            s_sl[4 * t + 3] = (uint16_t)(L[j] | (F[j] << 2));   // (its longest edge as it was, for others' reads)
        }
        const unsigned long long m = __ballot(seed);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(&s_cnt[4], __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
        if (seed) s_list[at] = (uint16_t)(4 * t + L[j]);
    }
    __syncthreads();

    // 3. next': the next edge of the triangle, or the turn across it
    uint32_t mid[TI];   // the middle slot of a tip found here, or kNoSlot
    {
        uint32_t x[TI], c[TI], deg[TI];
        bool act[TI];
        bool any = false;
#pragma unroll
        for (int j = 0; j < TI; j++) {
            x[j] = (kCrossNext >> (2 * F[j])) & 3u;
            const uint32_t sx = pick3(x[j], tr.s[j][0], tr.s[j][1], tr.s[j][2]);
            act[j] = x[j] != 3u;   // (then the edge is no frontier edge: sx is a slot)
            c[j] = act[j] ? next_slot(sx) : 0u;
            deg[j] = 2;   // half-edges at the target seen so far
            mid[j] = kNoSlot;
            any |= act[j];
        }
        for (int it = 0; any && it <= 4 * nt; it++) {
            any = false;
            uint32_t f[TI], g[TI];
#pragma unroll
            for (int j = 0; j < TI; j++) {
                f[j] = act[j] ? s_sl[c[j] | 3u] : 0u;
                g[j] = act[j] ? s_sl[c[j]] : 0u;
            }
#pragma unroll
            for (int j = 0; j < TI; j++) {
                if (!act[j]) continue;
                if (fbit(f[j], (int)(c[j] & 3u))) {
                    act[j] = false;
                } else if (g[j] == kNo16) {   // a non-frontier edge on the boundary: not a valid mesh
                    act[j] = false;
                    bad = 1;
                } else {
                    c[j] = next_slot(g[j]);
                    deg[j]++;
                    any = true;
                }
            }
        }
        bad |= any;
#pragma unroll
        for (int j = 0; j < TI; j++) {
            const int t = tid + j * kSmallBlock;
            if (t >= nt) continue;
            const uint32_t q = 4u * (uint32_t)t;
            reinterpret_cast<ushort4 *>(s_nx)[t] = make_ushort4((uint16_t)(x[j] == 1u ? c[j] : q + 1), (uint16_t)(x[j] == 2u ? c[j] : q + 2),
                                                                (uint16_t)(x[j] == 0u ? c[j] : q), 0);
            const uint32_t tw = x[j] == 3u ? kNoSlot : pick3(x[j], tr.s[j][2], tr.s[j][0], tr.s[j][1]);
            if (tw == kNoSlot || c[j] != tw) continue;
            // a tip: its frontier half-edge is tw; the middle edge deg / 2
            // clockwise steps further
            uint32_t m = tw;
            for (uint32_t k = 0; k < deg[j] / 2 && m != kNo16; k++) {
                const uint32_t g = s_sl[m];
                m = g == kNo16 ? g : next_slot(g);
            }
            const uint32_t mt = m == kNo16 ? m : s_sl[m];
            if (mt == kNo16) {
                bad = 1;
                continue;
            }
            mid[j] = m;
            const uint32_t lo = min(m, mt), hi = max(m, mt);
            const uint32_t blo = 1u << (16 + 5 + (lo & 3u)), bhi = 1u << (16 + 5 + (hi & 3u));
            const uint32_t old = atomicOr(&w32[2 * (lo >> 2) + 1], blo);
            atomicOr(&w32[2 * (hi >> 2) + 1], bhi);
            atomicAdd(&s_cnt[1], 1);
            if (!(old & blo)) atomicAdd(&s_cnt[2], 1);   // the edge's first tip counts it
            const int at = atomicAdd(&s_cnt[4], 2);      // both sides seed a loop
            if (at + 1 >= 2 * nt + 8) {                  // more than a valid mesh can have
                bad = 1;
                continue;
            }
            s_list[at] = (uint16_t)m;
            s_list[at + 1] = (uint16_t)mt;
        }
    }
    __syncthreads();

    // 3b. the turns around both ends of every middle edge again, over the
    //     repaired frontier: every slot entering such a vertex.  (Two tips may
    //     share a vertex; they write the same values.)
    auto frontier2 = [&](uint32_t q) { return (repaired_bits(s_sl[q | 3u]) >> (q & 3u)) & 1u; };
    if (s_cnt[1] > 0) {   // (uniform)
        auto turn2 = [&](uint32_t c) {
            for (int k = 0; k <= 4 * nt; k++) {
                if (frontier2(c)) return c;
                const uint32_t g = s_sl[c];
                if (g == kNo16) break;
                c = next_slot(g);
            }
            return kNoSlot;
        };
        auto fix_vertex = [&](uint32_t o0) {   // o0 leaves the vertex
            bool open = false;
            uint32_t o = o0;
            for (int k = 0; k <= 4 * nt; k++) {   // clockwise
                const uint32_t pin = prev_slot(o);
                if (frontier2(pin)) {
                    const uint32_t c = turn2(next_slot(pin));
                    bad |= c == kNoSlot;
                    s_nx[pin] = (uint16_t)(c == kNoSlot ? 0u : c);
                }
                const uint32_t g = s_sl[o];
                if (g == kNo16) {
                    open = true;
                    break;
                }
                o = next_slot(g);
                if (o == o0) break;
            }
            if (!open) return;
            o = o0;
            for (int k = 0; k <= 4 * nt; k++) {   // counter-clockwise, to the other boundary edge
                const uint32_t g = s_sl[prev_slot(o)];
                if (g == kNo16) break;
                o = g;
                const uint32_t pin = prev_slot(o);
                if (frontier2(pin)) {
                    const uint32_t c = turn2(next_slot(pin));
                    bad |= c == kNoSlot;
                    s_nx[pin] = (uint16_t)(c == kNoSlot ? 0u : c);
                }
            }
        };
#pragma unroll
        for (int j = 0; j < TI; j++) {
            if (mid[j] == kNoSlot) continue;
            fix_vertex(mid[j]);         // leaves the tip
            fix_vertex(s_sl[mid[j]]);   // leaves the middle edge's other end
        }
        __syncthreads();
    }

    // 4. prev' inverts next'; then both go out, and every seed's loop is walked
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
        if (t >= nt) continue;
        F[j] = repaired_bits(s_sl[4 * t + 3]);
        const ushort4 n = reinterpret_cast<const ushort4 *>(s_nx)[t];
        if (F[j] & 1u) s_pv[n.x] = (uint16_t)(4 * t);
        if (F[j] & 2u) s_pv[n.y] = (uint16_t)(4 * t + 1);
        if (F[j] & 4u) s_pv[n.z] = (uint16_t)(4 * t + 2);
    }
    if (__syncthreads_or(bad)) {   // (uniform) no loop structure to follow
        if (tid == 0) {
            MeshCounters c{};
            c.err = kErrCorrupt;
            small_counts(d, c);
        }
        return;
    }
    int nfront = 0;
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
        const bool in = t < nt;
#pragma unroll
        for (int i = 0; i < 3; i++) nfront += __popcll(__ballot(in && ((F[j] >> i) & 1u)));
        if (!in) continue;
        const ushort4 n = reinterpret_cast<const ushort4 *>(s_nx)[t], p = reinterpret_cast<const ushort4 *>(s_pv)[t];
        const int none[3] = {(F[j] & 1u) ? 0 : -1, (F[j] & 2u) ? 0 : -1, (F[j] & 4u) ? 0 : -1};
        *(GLOBAL v3i_a4 *)((gint)d.next_o + 3 * t) =
            v3i_a4{he_of_slot(n.x) | none[0], he_of_slot(n.y) | none[1], he_of_slot(n.z) | none[2]};
        *(GLOBAL v3i_a4 *)((gint)d.prev_o + 3 * t) =
            v3i_a4{he_of_slot(p.x) | none[0], he_of_slot(p.y) | none[1], he_of_slot(p.z) | none[2]};
    }
    if (lane == 0 && nfront) atomicAdd(&s_cnt[3], nfront);
    const int nlist = s_cnt[4];   // (within s_list: checked as it grew)
    bool longer = false;
    int walked = 0;
    for (int k = tid; k < nlist; k += kSmallBlock) {
        const uint32_t s0 = s_list[k], f = repaired_bits(s_sl[s0 | 3u]);
        uint32_t st = ((f >> (s0 & 3u)) & 1u) ? s0 : (s0 & ~3u) + (uint32_t)__builtin_ctz(f | 8u);
        if (!f) {   // clockwise around the seed's origin to a frontier half-edge
            st = s0;
            for (int r = 0; !frontier2(st); r++) {
                const uint32_t g = s_sl[st];
                if (g == kNo16 || r > 4 * nt) {
                    bad = 1;
                    break;
                }
                st = next_slot(g);
            }
        }
        uint32_t cur = s_nx[st], mn = st;
        int len = 1;
        for (; cur != st && len < kSmallWalk<TI>; len++) {
            mn = min(mn, cur);
            cur = s_nx[cur];
        }
        if (cur != st) {
            longer = true;
            continue;
        }
        const uint32_t old = atomicOr(&w32[2 * (mn >> 2) + 1], kRecorded << 16);
        const bool won = !(old & (kRecorded << 16));
        if (won) s_nx[mn | 3u] = (uint16_t)len;
        walked += won ? len : 0;
        s_list[k] = (uint16_t)(won ? mn : kNo16);
    }
    if (longer) s_longer = 1;
    bad = __syncthreads_or(bad);
    const bool ranked = __builtin_expect(s_longer, 0);
    uint32_t *s_pk = reinterpret_cast<uint32_t *>(s_nx);   // (over s_nx and s_pv)
    if (ranked) {   // (uniform)
        if (walked) atomicAdd(&s_cnt[5], walked);
        __syncthreads();
        small_rank<TI>(s_pk, s_pv, F, nt, s_cnt[3] - s_cnt[5]);
        __syncthreads();
    }

    // 5. loops in the order of their minima: each thread scans a few
    //    consecutive triangles (a loop's minimum is the first frontier
    //    half-edge of its triangle, and no triangle has two loops)
    int cnt = 0, sum = 0, len[TI];
#pragma unroll
    for (int r = 0; r < TI; r++) {
        const int t = tid * TI + r;
        len[r] = t >= nt ? 0 : ranked ? (int)s_pk[4 * t + 3] : s_nx[4 * t + 3];
        cnt += len[r] != 0;
        sum += len[r];
    }
    int ec, es, tc, ts;
    block_excl_scan2(cnt, sum, ec, es, tc, ts, s_scan);
    // every frontier half-edge lies on exactly one loop
    const bool fits = !bad && tc <= nt && ts <= nh && ts == s_cnt[3];
    if (fits) {
        const gint seeds = (gint)d.seeds, loff = (gint)d.loop_off;
#pragma unroll
        for (int r = 0; r < TI; r++) {
            if (!len[r]) continue;
            const uint32_t q = 4u * (uint32_t)(tid * TI + r);
            seeds[ec] = he_of_slot(q + (uint32_t)__builtin_ctz(repaired_bits(s_sl[q + 3]) | 8u));
            loff[ec] = es;
            // the loop's first place
            if (ranked)
                s_pk[q + 3] = es;
            else
                s_nx[q + 3] = (uint16_t)es;
            ec++;
            es += len[r];
        }
        if (tid == 0) loff[tc] = ts;
    }
    __syncthreads();

    // 6. every loop from its minimum into its place (prev' is out; by the ranks:
    //    the labels are done with), then out
    if (fits) {
        uint16_t *s_out = ranked ? s_sl : s_pv;
        if (ranked) {   // (uniform)
#pragma unroll
            for (int j = 0; j < TI; j++)
#pragma unroll
                for (int i = 0; i < 3; i++) {
                    const uint32_t t = tid + j * kSmallBlock, q = 4u * t + i;
                    if ((int)t >= nt || !((F[j] >> i) & 1u)) continue;
                    const uint32_t w = s_pk[q], at = s_pk[(w & 0xffffu) | 3u] + (w >> 16);
                    if (at < (uint32_t)nh) s_out[at] = (uint16_t)q;   // (always, in a valid mesh)
                }
        } else {
            for (int k = tid; k < nlist; k += kSmallBlock) {
                const uint32_t mn = s_list[k];
                if (mn == kNo16) continue;
                uint32_t at = s_nx[mn | 3u], cur = mn;
                do {
                    s_out[at++] = (uint16_t)cur;
                    cur = s_nx[cur];
                } while (cur != mn);
            }
        }
        __syncthreads();
        const gint lhe = (gint)d.loop_he;
        for (int k = tid; k < ts; k += kSmallBlock) lhe[k] = he_of_slot(s_out[k]);
    }
    if (tid == 0) {
        MeshCounters c{};
        c.err = fits ? 0 : kErrCorrupt;
        c.nties = s_cnt[0];
        c.ntips = s_cnt[1];
        c.nmiddle = s_cnt[2];
        c.npoly = tc;
        c.nloop = ts;
        small_counts(d, c);
    }
}

template <int TI>
__device__ __forceinline__ void small_mesh(const MeshDesc &d) {
    if (d.nt <= 0 || d.nt > TI * kSmallBlock) {   // (uniform) an empty mesh; larger ones are never launched here
        if (threadIdx.x == 0) {
            MeshCounters c{};
            c.err = d.nt != 0 ? kErrCorrupt : 0;
            small_counts(d, c);
            if (d.nt == 0) d.loop_off[0] = 0;
        }
        return;
    }
    SmallTris<TI> tr;
    small_load(d, tr);
    small_body(d, tr);
}

// a batch of small meshes: one workgroup per descriptor
template <int TI>
__global__ void __launch_bounds__(kSmallBlock) k_small(const MeshDesc *__restrict__ descs) {
    small_mesh<TI>(descs[blockIdx.x]);
}

// one small mesh, its descriptor passed by value and its counts written to
// host memory: a call that needs nothing staged before it or copied after it
template <int TI>
__global__ void __launch_bounds__(kSmallBlock) k_small_one(const MeshDesc d) {
    small_mesh<TI>(d);
}

// ---------------------------------------------------------------------------
// k_small_jobs: build and mesh one small job per workgroup
//
// The half-edge build of Section 4.1-4.2 for a job small enough for LDS, with
// the error reports of the staged build kernels: every coordinate in [0,
// 2^30]; every corner index in [0, nv) and no zero-area triangle (exact int64
// orientation test), clockwise triangles reordered counter-clockwise; then
// twins by a hash table of the edges in LDS, where a third half-edge of one
// edge, or a second in the same direction, is non-manifold.  Errors keep the
// lowest (rank << 8 | code): coordinates first, then the lowest bad triangle,
// then non-manifold; the twins are matched only when the first checks pass.
// A thread keeps its triangles in registers from their loads to the labels of
// the meshing that follows (as k_small does it), so a job's structure goes to
// memory only for a build on its own.  A build of 2,048 triangles takes 9.7
// us, most of it the two dependent loads before its checks and the table's
// LDS atomics; listing the half-edges by origin vertex and searching the lists
// took 16 us.
// ---------------------------------------------------------------------------

__device__ __forceinline__ unsigned long long job_key(unsigned long long rank, int code) {
    return (rank << 8) | (unsigned long long)(-code);
}

// Slots of the build's edge table: more than the 3 nt edges a job can have.
template <int TI>
struct JobTable {
    static constexpr int kBits = TI == 1 ? 12 : (TI == 2 ? 13 : 14), kSlots = 1 << kBits;
    static_assert(kSlots > 3 * TI * kSmallBlock, "every edge finds a slot");
};

size_t small_job_lds_bytes(int max_nt) {
    const int slots = max_nt <= kSmallBlock       ? JobTable<1>::kSlots
                      : max_nt <= 2 * kSmallBlock ? JobTable<2>::kSlots
                                                  : JobTable<4>::kSlots;
    const size_t build = 8 * (size_t)slots, mesh = small_lds_bytes(max_nt);
    return build > mesh ? build : mesh;
}

template <int TI>
__device__ __forceinline__ void small_job(const SmallJob &jd) {
    extern __shared__ int4 lds_raw[];
    __shared__ unsigned long long s_key;
    __shared__ int s_flip;
    constexpr int kBits = JobTable<TI>::kBits, kSlots = JobTable<TI>::kSlots;
    const int nv = jd.nv, nt = jd.nt, tid = threadIdx.x;
    if (nv < 0 || nt < 0 || nv > kJobSmallV || nt > TI * kSmallBlock) {   // (uniform) never launched so
        if (tid == 0) {
            jd.counts[8] = (int)(uint32_t)job_key(0, -1);
            jd.counts[9] = 0;
        }
        return;
    }
    if (tid == 0) {
        s_key = ~0ull;
        s_flip = 0;
    }
    // an edge's slot: bits 0-11 and 12-23 its ends (the lower first), bit 24 a
    // 1; bits 32-45 the first half-edge's slot, bit 46 it runs from the lower
    // end, bits 48-62 the second's slot + 1 (0 before it comes)
    unsigned long long *s_table = reinterpret_cast<unsigned long long *>(lds_raw);
    for (int k = tid; k < kSlots / 2; k += kSmallBlock) reinterpret_cast<ulonglong2 *>(lds_raw)[k] = ulonglong2{0ull, 0ull};
    // corners: indices, orientation, counter-clockwise order
    SmallTris<TI> tr;
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock, tt = t < nt ? t : 0;
#pragma unroll
        for (int i = 0; i < 3; i++) tr.v[j][i] = nt > 0 ? jd.tri[3 * tt + i] : 0;
    }
    __syncthreads();
    // coordinates (and the mesh's own copy of them)
    for (int v = tid; v < nv; v += kSmallBlock) {
        const int2 p = jd.xy[v];
        if (jd.xy_out) jd.xy_out[v] = p;
        if (p.x < 0 || p.x > (1 << 30) || p.y < 0 || p.y > (1 << 30)) atomicMin(&s_key, job_key(0, -2));
    }
    int flips = 0;
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
        if (t >= nt) continue;
        const int a = tr.v[j][0], b = tr.v[j][1], c = tr.v[j][2];
        if ((unsigned)a >= (unsigned)nv || (unsigned)b >= (unsigned)nv || (unsigned)c >= (unsigned)nv) {
            atomicMin(&s_key, job_key(1ull + t, -1));
            continue;
        }
        const int2 pa = jd.xy[a], pb = jd.xy[b], pc = jd.xy[c];
        const long long o = ((long long)pb.x - pa.x) * ((long long)pc.y - pa.y) -
                            ((long long)pb.y - pa.y) * ((long long)pc.x - pa.x);
        if (o == 0) {
            atomicMin(&s_key, job_key(1ull + t, -3));
        } else if (o < 0) {
            tr.v[j][1] = c;
            tr.v[j][2] = b;
            flips++;
        }
    }
    if (flips) atomicAdd(&s_flip, flips);
    __syncthreads();
    if (s_key != ~0ull) {   // (uniform) the inputs failed their checks: no twins
        if (tid == 0) {
            jd.counts[8] = (int)(uint32_t)s_key;
            jd.counts[9] = (int)(uint32_t)(s_key >> 32);
        }
        return;
    }
    // every half-edge into its edge's slot, then its twin from there
    uint32_t q[TI][3];
    bool dup = false;
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            q[j][i] = 0;
            if (t >= nt) continue;
            const uint32_t u = (uint32_t)tr.v[j][i], v = (uint32_t)tr.v[j][i == 2 ? 0 : i + 1], slot = 4u * t + i;
            const uint32_t key = min(u, v) | (max(u, v) << 12) | (1u << 24);
            const unsigned long long word = (unsigned long long)(slot | (u < v ? 1u << 14 : 0u)) << 32 | key;
            uint32_t at = (key * 0x9E3779B1u) >> (32 - kBits);
            while (true) {
                const unsigned long long was = atomicCAS(&s_table[at], 0ull, word);
                if (was == 0ull) break;
                if ((uint32_t)was == key) {
                    atomicOr(reinterpret_cast<unsigned *>(&s_table[at]) + 1, (slot + 1u) << 16);
                    dup |= ((uint32_t)((was ^ word) >> 32) & (1u << 14)) == 0;
                    break;
                }
                at = (at + 1) & (kSlots - 1);
            }
            q[j][i] = at;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TI; j++) {
        const int t = tid + j * kSmallBlock;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            tr.s[j][i] = kNoSlot;
            if (t >= nt) continue;
            const uint32_t w = (uint32_t)(s_table[q[j][i]] >> 32), slot = 4u * t + i, first = w & 0x3fffu, second = w >> 16;
            const bool lead = first == slot;
            dup |= !lead && second != slot + 1u;   // (a third half-edge's slot has run together with the second's)
            tr.s[j][i] = !lead ? first : (second ? second - 1u : kNoSlot);
        }
    }
    if (dup) atomicMin(&s_key, job_key(1ull + nt, -4));
    __syncthreads();
    if (tid == 0) {
        jd.counts[8] = (int)(uint32_t)s_key;
        jd.counts[9] = (int)(uint32_t)(s_key >> 32);
        jd.counts[10] = s_flip;
    }
    if (s_key != ~0ull) return;   // (uniform)
    if (jd.build_only) {          // (uniform)
#pragma unroll
        for (int j = 0; j < TI; j++) {
            const int t = tid + j * kSmallBlock;
            if (t >= nt) continue;
            *(GLOBAL v3i_a4 *)((gint)jd.org + 3 * t) = v3i_a4{tr.v[j][0], tr.v[j][1], tr.v[j][2]};
            const auto he = [](uint32_t s) { return s == kNoSlot ? -1 : he_of_slot(s); };
            *(GLOBAL v3i_a4 *)((gint)jd.twin + 3 * t) = v3i_a4{he(tr.s[j][0]), he(tr.s[j][1]), he(tr.s[j][2])};
        }
        return;
    }
    MeshDesc d{};
    d.xy = jd.xy;
    d.next_o = jd.next_o;
    d.prev_o = jd.prev_o;
    d.seeds = jd.seeds;
    d.loop_off = jd.loop_off;
    d.loop_he = jd.loop_he;
    d.ctr = reinterpret_cast<MeshCounters *>(jd.counts);
    d.nt = nt;
    d.nv = nv;
    if (nt == 0) {   // (uniform)
        if (tid == 0) {
            *d.ctr = MeshCounters{};
            d.loop_off[0] = 0;
        }
        return;
    }
    small_body(d, tr);
}

template <int TI>
__global__ void __launch_bounds__(kSmallBlock) k_small_jobs(const SmallJob *__restrict__ jobs) {
    small_job<TI>(jobs[blockIdx.x]);
}

// one job, its description passed by value
template <int TI>
__global__ void __launch_bounds__(kSmallBlock) k_small_job_one(const SmallJob job) {
    small_job<TI>(job);
}

hipError_t launch_small_job_one(const SmallJob &job, hipStream_t s) {
    const dim3 grid(1), block(kSmallBlock);
    const size_t lds = small_job_lds_bytes(job.nt);
    if (job.nt <= kSmallBlock)
        hipLaunchKernelGGL(k_small_job_one<1>, grid, block, lds, s, job);
    else if (job.nt <= 2 * kSmallBlock)
        hipLaunchKernelGGL(k_small_job_one<2>, grid, block, lds, s, job);
    else
        hipLaunchKernelGGL(k_small_job_one<4>, grid, block, lds, s, job);
    return hipGetLastError();
}

hipError_t launch_small_jobs(const SmallJob *jobs, int n, int max_nt, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(n), block(kSmallBlock);
    const size_t lds = small_job_lds_bytes(max_nt);
    if (max_nt <= kSmallBlock)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_jobs<1>), grid, block, lds, s, jobs);
    else if (max_nt <= 2 * kSmallBlock)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_jobs<2>), grid, block, lds, s, jobs);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_jobs<4>), grid, block, lds, s, jobs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// small copies between device memory and coherent pinned host memory (the
// descriptor table before a run, the per-mesh counters after it): a kernel
// in stream order instead of the runtime's copy path
// ---------------------------------------------------------------------------

__global__ void k_copy_words(uint32_t *dst, const uint32_t *src, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = src[i];
}

hipError_t launch_copy_words(void *dst, const void *src, size_t bytes, hipStream_t s) {
    if (bytes % 4 || bytes / 4 > 0x7fffffff) return hipErrorInvalidValue;
    const int n = (int)(bytes / 4);
    if (n == 0) return hipSuccess;
    const int grid = (n + 255) / 256 < 64 ? (n + 255) / 256 : 64;
    hipLaunchKernelGGL(k_copy_words, dim3(grid), dim3(256), 0, s, static_cast<uint32_t *>(dst),
                       static_cast<const uint32_t *>(src), n);
    return hipGetLastError();
}

__global__ void k_export_counts(const MeshCounters *c, int32_t *out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const MeshCounters k = *c;
        out[0] = k.err ? -10 : 0;   // GP_ECORRUPT
        out[1] = k.npoly;
        out[2] = k.nloop;
        out[3] = k.ntips;
        out[4] = k.nmiddle;
        out[5] = k.nties;
        out[6] = 0;
        out[7] = 0;
    }
}

hipError_t launch_export_counts(const MeshCounters *c, int32_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_export_counts, dim3(1), dim3(64), 0, s, c, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// host launch of the whole chain
// ---------------------------------------------------------------------------

#define GP_LAUNCH_ITEMS(KER, ITEMS_RT, GRID, BLOCK, LDS, STREAM, ...)                          \
    do {                                                                                       \
        switch (ITEMS_RT) {                                                                    \
            case 1: hipLaunchKernelGGL(KER(1), GRID, BLOCK, LDS, STREAM, __VA_ARGS__); break;  \
            case 2: hipLaunchKernelGGL(KER(2), GRID, BLOCK, LDS, STREAM, __VA_ARGS__); break;  \
            case 4: hipLaunchKernelGGL(KER(4), GRID, BLOCK, LDS, STREAM, __VA_ARGS__); break;  \
            case 8: hipLaunchKernelGGL(KER(8), GRID, BLOCK, LDS, STREAM, __VA_ARGS__); break;  \
            default: return hipErrorInvalidValue;                                              \
        }                                                                                      \
    } while (0)
#define GP_LABEL(I) HIP_KERNEL_NAME(k_label<I, false>)
#define GP_LABEL_ONE(I) HIP_KERNEL_NAME(k_label<I, true>)
#define GP_COMPACT(I) HIP_KERNEL_NAME(k_compact<I>)

template <bool CM, bool NT>
hipError_t launch_relink_nt(const LaunchCfg &cfg, const RunBuffers &rb, hipStream_t s, size_t lds, int cmp_tb) {
    const dim3 grid(rb.he_tiles), block(cfg.block_relink);
#define GP_RELINK_ARGS rb.descs, rb.nmesh, rb.tips, rb.tip_counts, rb.tip_span, rb.walk, rb.walk_counts, rb.walk_cap, \
                       rb.status, cmp_tb
    switch (cfg.items_relink) {
        case 1: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_relink<1, CM, NT>), grid, block, lds, s, GP_RELINK_ARGS); break;
        case 2: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_relink<2, CM, NT>), grid, block, lds, s, GP_RELINK_ARGS); break;
        case 4: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_relink<4, CM, NT>), grid, block, lds, s, GP_RELINK_ARGS); break;
        case 8: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_relink<8, CM, NT>), grid, block, lds, s, GP_RELINK_ARGS); break;
        default: return hipErrorInvalidValue;
    }
#undef GP_RELINK_ARGS
    return hipGetLastError();
}

// next'/prev' of a run larger than the last-level cache go out as streaming
// stores: they would not stay cached for the kernels that read them, and the
// cache keeps what those kernels reuse (the run's size from its label tiles,
// at most a tile per mesh over).  Smaller runs keep them cached.
template <bool CM>
hipError_t launch_relink(const LaunchCfg &cfg, const RunBuffers &rb, hipStream_t s, size_t lds, int cmp_tb) {
    const bool stream_out = 24ll * rb.tri_tiles * cfg.block_label * cfg.items_label > kStreamOutBytes;
    return stream_out ? launch_relink_nt<CM, true>(cfg, rb, s, lds, cmp_tb)
                      : launch_relink_nt<CM, false>(cfg, rb, s, lds, cmp_tb);
}

bool small_fits(const LaunchCfg &cfg, int max_nt) {
    return max_nt >= 0 && max_nt <= cfg.small_max && max_nt <= kSmallMaxTri &&
           small_lds_bytes(max_nt) <= (size_t)cfg.lds_max;
}

bool runs_small(const LaunchCfg &cfg, const RunBuffers &rb) { return !rb.chain_only && small_fits(cfg, rb.max_nt); }

hipError_t launch_small_one(const MeshDesc &d, hipStream_t s) {
    const dim3 grid(1), block(kSmallBlock);
    const size_t lds = small_lds_bytes(d.nt);
    if (d.nt <= kSmallBlock)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_one<1>), grid, block, lds, s, d);
    else if (d.nt <= 2 * kSmallBlock)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_one<2>), grid, block, lds, s, d);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small_one<4>), grid, block, lds, s, d);
    return hipGetLastError();
}

int prepare_small(int lds_block) {
    const void *const fns[12] = {reinterpret_cast<const void *>(&k_small_job_one<1>),
                                reinterpret_cast<const void *>(&k_small_job_one<2>),
                                reinterpret_cast<const void *>(&k_small_job_one<4>),
                                reinterpret_cast<const void *>(&k_small<1>),
                                reinterpret_cast<const void *>(&k_small<2>),
                                reinterpret_cast<const void *>(&k_small<4>),
                                reinterpret_cast<const void *>(&k_small_one<1>),
                                reinterpret_cast<const void *>(&k_small_one<2>),
                                reinterpret_cast<const void *>(&k_small_one<4>),
                                reinterpret_cast<const void *>(&k_small_jobs<1>),
                                reinterpret_cast<const void *>(&k_small_jobs<2>),
                                reinterpret_cast<const void *>(&k_small_jobs<4>)};
    int fixed = 0;
    for (const void *f : fns) {
        hipFuncAttributes a{};
        if (hipFuncGetAttributes(&a, f) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        fixed = (int)a.sharedSizeBytes > fixed ? (int)a.sharedSizeBytes : fixed;
    }
    const int dyn = lds_block - fixed;
    if (dyn <= 0) return 0;
    if (dyn > 65536 - fixed)
        for (const void *f : fns)
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn) != hipSuccess) {
                (void)hipGetLastError();
                return 65536 - fixed;
            }
    return dyn;
}

hipError_t launch_pipeline(const LaunchCfg &cfg, const RunBuffers &rb, hipStream_t s, launch_hook hook,
                           void *user, const MeshDesc *one_desc) {
    auto H = [&](int k, int after) {
        if (hook) hook(user, k, after);
    };
    if (rb.nmesh <= 0) return hipSuccess;
    if (runs_small(cfg, rb)) {   // every mesh fits one workgroup: one launch
        const dim3 grid(rb.nmesh), block(kSmallBlock);
        const size_t lds = small_lds_bytes(rb.max_nt);
        H(K_SMALL, 0);
        if (one_desc) {
            const hipError_t e = launch_small_one(*one_desc, s);
            if (e != hipSuccess) return e;
        } else if (rb.max_nt <= kSmallBlock)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small<1>), grid, block, lds, s, rb.descs);
        else if (rb.max_nt <= 2 * kSmallBlock)
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small<2>), grid, block, lds, s, rb.descs);
        else
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_small<4>), grid, block, lds, s, rb.descs);
        H(K_SMALL, 1);
        return hipGetLastError();
    }
    // tips are at most half the triangles and rarely many: a quarter of the
    // blocks for them, for the time that idle ones take to start and end
    const int pb = cfg.persistent_blocks, pt = cfg.block_persistent, pq = (pb + 3) / 4;
    const int cmp_tb = cfg.block_compact * cfg.items_compact;   // triangles per compaction tile
    const bool one = rb.nmesh == 1;

    H(K_LABEL, 0);
    {
        const ClearArgs ca = {rb.ctrs, rb.status, rb.cmp_tiles, rb.tip_counts, rb.walk_counts, rb.emit_counts,
                              rb.wbuf_counts};
        const dim3 grid(rb.tri_tiles), block(cfg.block_label);
        const size_t lds = sizeof(int) * 3 * (size_t)cfg.block_label * cfg.items_label;
        MeshDesc *const out = const_cast<MeshDesc *>(rb.descs);
        if (one_desc)
            GP_LAUNCH_ITEMS(GP_LABEL_ONE, cfg.items_label, grid, block, lds, s, rb.descs, rb.nmesh, ca, out, *one_desc);
        else
            GP_LAUNCH_ITEMS(GP_LABEL, cfg.items_label, grid, block, lds, s, rb.descs, rb.nmesh, ca, out, NoDesc{});
    }
    H(K_LABEL, 1);

    H(K_RELINK, 0);
    {
        const size_t lds = relink_lds_bytes(cfg.block_relink * cfg.items_relink);
        const hipError_t e = rb.compact ? launch_relink<true>(cfg, rb, s, lds, cmp_tb)
                                        : launch_relink<false>(cfg, rb, s, lds, cmp_tb);
        if (e != hipSuccess) return e;
    }
    H(K_RELINK, 1);

    H(K_REPAIR, 0);
    hipLaunchKernelGGL(one ? k_repair<true> : k_repair<false>, dim3(pq), dim3(pt), 0, s, rb.descs, rb.tips, rb.tip_counts, rb.tip_span, rb.cap_tips,
                       rb.walk, rb.walk_counts, rb.walk_cap, rb.fixes);
    H(K_REPAIR, 1);

    H(K_FIXUP, 0);
    hipLaunchKernelGGL(one ? k_fixup<true> : k_fixup<false>, dim3(pq), dim3(256), 0, s, rb.descs, rb.tips, rb.tip_counts,
                       rb.tip_span, rb.cap_tips, rb.fixes);
    H(K_FIXUP, 1);

    H(K_WALK, 0);
    hipLaunchKernelGGL((one ? k_walk<kWalkBuf, true> : k_walk<kWalkBuf, false>), dim3(pb), dim3(256), 0, s, rb.descs, rb.walk,
                       rb.walk_counts, rb.walk_cap, rb.tip_counts, rb.status, cmp_tb, rb.wbuf, rb.wbuf_counts, rb.wbuf_cap);
    H(K_WALK, 1);

    H(K_TSCAN, 0);
    hipLaunchKernelGGL(k_tile_scan, dim3(rb.nmesh, rb.max_chunks), dim3(1024), 0, s, rb.descs, rb.status,
                       rb.cpre, cmp_tb);
    H(K_TSCAN, 1);

    H(K_COMPACT, 0);
    GP_LAUNCH_ITEMS(GP_COMPACT, cfg.items_compact, dim3(rb.cmp_tiles), dim3(cfg.block_compact),
                    compact_lds_bytes(cmp_tb), s, rb.descs, rb.nmesh,
                    rb.status, rb.cpre, rb.emit, rb.emit_counts, rb.emit_cap, rb.wbuf);
    H(K_COMPACT, 1);

    H(K_EMIT, 0);
    hipLaunchKernelGGL((one ? k_emit<4, true> : k_emit<4, false>), dim3(pb), dim3(256), 0, s, rb.descs, rb.emit,
                       rb.emit_counts, rb.emit_cap, rb.wbuf, rb.wbuf_cap, rb.nmesh);
    H(K_EMIT, 1);
    return hipGetLastError();
}

}  // namespace gp
