// Optional renumbering of a triangulation along a Z-order (Morton) curve, run
// on the device before the half-edge build (GP_RENUMBER).
//
// The meshing kernels read neighbours' labels, twins and next' by index, so
// they run fastest when neighbouring triangles have nearby indices.  Meshes
// numbered without locality (a Delaunay triangulator's output order, a
// shuffled file) are renumbered here: vertices in the Morton order of their
// coordinates, triangles in the Morton order of their centroids (corner order
// within a triangle kept).  Equal codes keep their old order.  The new-to-old
// maps are kept with the mesh.
//
// Arrays of up to kSortMax elements are sorted here by sampling: a sorted
// sample of the keys cuts their range into buckets, one pass over the input
// puts every key and index into its bucket's list, and one workgroup per
// bucket sorts its list in LDS and writes the permuted arrays.  Those are five
// launches for the vertices and triangles together, and the data moves twice:
// 300,000 vertices and 594,000 triangles take 79 us, where the library's sort
// (block sorts, then merges of pairs of ever longer runs: 38 launches of 4 to
// 8 us each at these sizes) with separate key and gather passes took 370 us.
// Larger arrays go to the library, which above a million elements sorts by
// digits in a fixed number of passes.  kSortMax is where 1,024 buckets, the most
// that k_sort_place keeps, hold a quarter at the mean of the 8,192 elements that a
// workgroup sorts, and not where the library would be as fast.
// Whole builds with this sort and with the library's: 140 and 399 us with
// 594,000 triangles, 331 and 801 us with 1,980,000 (the lists then take 250 MB
// of scratch; when that cannot be had, the library sorts).
#include <hipcub/hipcub.hpp>

#include <type_traits>

#include "gp_internal.h"

namespace gp {

namespace {

// The 31 low bits of v spread to the even bits of a 64-bit word.
__device__ __forceinline__ uint64_t spread31(uint32_t v) {
    uint64_t x = v & 0x7fffffffu;
    x = (x | (x << 16)) & 0x0000ffff0000ffffull;
    x = (x | (x << 8)) & 0x00ff00ff00ff00ffull;
    x = (x | (x << 4)) & 0x0f0f0f0f0f0f0f0full;
    x = (x | (x << 2)) & 0x3333333333333333ull;
    x = (x | (x << 1)) & 0x5555555555555555ull;
    return x;
}

// Morton code of (x, y), coordinates clamped to [0, 2^31) (valid inputs are
// in [0, 2^30]; others are reported by the build later).
__device__ __forceinline__ uint64_t morton(long long x, long long y) {
    const uint32_t cx = (uint32_t)(x < 0 ? 0 : (x > 0x7fffffff ? 0x7fffffff : x));
    const uint32_t cy = (uint32_t)(y < 0 ? 0 : (y > 0x7fffffff ? 0x7fffffff : y));
    return spread31(cx) | (spread31(cy) << 1);
}

// The Morton code of a triangle's centroid.  A triangle with an index outside
// [0, nv) gets the largest key (the build reports it later, wherever it lands).
__device__ __forceinline__ uint64_t triangle_key(const int2 *__restrict__ xy, int nv, const int32_t (&v)[3]) {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 3; i++) ok &= v[i] >= 0 && v[i] < nv;
    if (!ok) return ~0ull;
    long long sx = 0, sy = 0;
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const int2 p = xy[v[i]];
        sx += p.x;
        sy += p.y;
    }
    return morton(sx / 3, sy / 3);
}

__global__ void k_vertex_keys(const int2 *__restrict__ xy, int nv, uint64_t *keys, int32_t *vals) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const int2 p = xy[v];
    keys[v] = morton(p.x, p.y);
    vals[v] = v;
}

// vinv: old -> new vertex index; xy_out in the new order.
__global__ void k_vertex_gather(const int2 *__restrict__ xy, const int32_t *__restrict__ vperm, int nv,
                                int32_t *vinv, int2 *xy_out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nv) return;
    const int v = vperm[k];
    vinv[v] = k;
    xy_out[k] = xy[v];
}

__global__ void k_triangle_keys(const int2 *__restrict__ xy, const int32_t *__restrict__ tri, int nv, int nt,
                                uint64_t *keys, int32_t *vals) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const int32_t v[3] = {tri[3 * (size_t)t], tri[3 * (size_t)t + 1], tri[3 * (size_t)t + 2]};
    keys[t] = triangle_key(xy, nv, v);
    vals[t] = t;
}

// Triangles in the new order with new vertex indices (invalid ones kept).
__global__ void k_triangle_gather(const int32_t *__restrict__ tri, const int32_t *__restrict__ tperm,
                                  const int32_t *__restrict__ vinv, int nv, int nt, int32_t *tri_out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nt) return;
    const int t = tperm[k];
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const int v = tri[3 * t + i];
        tri_out[3 * k + i] = (v >= 0 && v < nv) ? vinv[v] : v;
    }
}

inline int blocks_for(int n) { return n > 0 ? (n + 255) / 256 : 1; }

// ---- sorting by sampling ---------------------------------------------------

constexpr int kSortBits = 21, kSortMax = 1 << kSortBits;
// A bucket's list has room for seven times the mean (and a bucket spans at
// least four samples), or for at least four times the mean beyond kBucketMean
// elements to each of the largest number of buckets (eight samples): fewer than
// one random input in a thousand has a bucket that does not fit.
constexpr int kBucketMean = 600, kMaxBuckets = 1024, kMaxSamples = 8192;
constexpr int kBucketCap = 4096, kBigCap = 2 * kBucketCap;   // (the latter: k_sort_bucket<true>)
static_assert(kSortMax / kMaxBuckets * 4 == kBigCap, "buckets fit");

__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int m) { return (uint32_t)__shfl_xor((int)v, m); }
__device__ __forceinline__ uint64_t lane_xor(uint64_t v, int m) {
    return (uint64_t)__shfl_xor((unsigned long long)v, m);
}

// Sorts TPB * E words, E per thread: in increasing order of tid * E + r when it
// returns.  A bitonic network: partners within a thread are registers, within
// a wave lanes, and only the others meet in LDS (s, TPB * E words).
template <int TPB, int E>
__device__ __forceinline__ void block_sort(uint32_t (&x)[E], uint32_t *s) {
    const int tid = threadIdx.x;
    auto in_thread = [&](int j, int k) {   // (j, E: constants once unrolled)
#pragma unroll
        for (int r = 0; r < E; r++) {
            if (r & j) continue;
            const bool up = ((tid * E + r) & k) == 0;
            const uint32_t a = min(x[r], x[r | j]), b = max(x[r], x[r | j]);
            x[r] = up ? a : b;
            x[r | j] = up ? b : a;
        }
    };
#pragma unroll
    for (int k = 2; k <= E; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) in_thread(j, k);
    for (int k = 2 * E; k <= TPB * E; k <<= 1) {
        const bool up = ((tid * E) & k) == 0;
        for (int m = k / (2 * E); m > 0; m >>= 1) {   // partner thread: tid ^ m
            const bool low = ((tid & m) == 0) == up;
            uint32_t y[E];
            if (m >= 64) {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < E; r++) s[r * TPB + tid] = x[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < E; r++) y[r] = s[r * TPB + (tid ^ m)];
            } else {
#pragma unroll
                for (int r = 0; r < E; r++) y[r] = lane_xor(x[r], m);
            }
#pragma unroll
            for (int r = 0; r < E; r++) x[r] = low ? min(x[r], y[r]) : max(x[r], y[r]);
        }
#pragma unroll
        for (int j = E >> 1; j > 0; j >>= 1) in_thread(j, k);
    }
}

// One array's sort (vertices, or triangles): n elements in `buckets` buckets,
// whose lists hold cap entries each.  A bucket begins at a sample's key and
// place in the input, so that equal keys, however many, spread over buckets too.
struct SortPart {
    int n, samples, buckets, cap;
    uint64_t *sample;    // samples: their keys
    uint64_t *split;     // buckets: the lowest key of each (the first: none)
    int32_t *split_at;   // buckets: of that key, the first place in the input
    int32_t *cursor;     // buckets: elements of each
    void *list;         // buckets * cap entries
};

// What a list holds of an element: all that the sort and the permuted arrays
// need, so that both are one run of reads per bucket: 25 us for the buckets of
// 594,000 triangles, where keys and indices alone, the corners gathered
// afterwards, took 37 (the placing takes as long with either).
struct VertexEntry {
    int32_t x, y, old;
    __device__ uint64_t key() const { return morton(x, y); }
};
struct TriangleEntry {
    uint32_t key0, key1;
    int32_t old, v[3];
    __device__ uint64_t key() const { return (uint64_t)key1 << 32 | key0; }
};
template <bool TRI>
using ListEntryOf = std::conditional_t<TRI, TriangleEntry, VertexEntry>;

// Element k as its list holds it; returns its key.
__device__ __forceinline__ uint64_t load_entry(const RenumberBuffers &b, int k, VertexEntry &e) {
    const int2 p = b.xy_in[k];
    e = VertexEntry{p.x, p.y, k};
    return e.key();
}
__device__ __forceinline__ uint64_t load_entry(const RenumberBuffers &b, int k, TriangleEntry &e) {
    const int32_t *v = b.tri_in + 3 * (size_t)k;
    e.old = k;
    e.v[0] = v[0];
    e.v[1] = v[1];
    e.v[2] = v[2];
    const uint64_t key = triangle_key(b.xy_in, b.nv, e.v);
    e.key0 = (uint32_t)key;
    e.key1 = (uint32_t)(key >> 32);
    return key;
}

// Sample i's place in the input: in the i-th of `samples` equal stretches, where
// a hash picks.
__device__ __forceinline__ int sample_place(const SortPart &p, uint32_t i) {
    const uint64_t at = (uint64_t)i * (uint32_t)p.n + ((uint64_t)(i * 0x9E3779B1u) * (uint32_t)p.n >> 32);
    return (int)(at / (uint32_t)p.samples);
}

// Samples the keys, and clears the lists.  grid: kMaxSamples / 256 blocks for
// the vertices, as many for the triangles.
__global__ void __launch_bounds__(256) k_sort_sample(const RenumberBuffers b, const SortPart pv, const SortPart pt) {
    const bool tri = blockIdx.x >= kMaxSamples / 256;
    const SortPart &p = tri ? pt : pv;
    const uint32_t i = (blockIdx.x % (kMaxSamples / 256)) * 256 + threadIdx.x;
    if (!tri && i == 0) *b.overflow = 0;
    if (i >= (uint32_t)p.samples) return;
    const int k = sample_place(p, i);
    VertexEntry ev;
    TriangleEntry et;
    p.sample[i] = tri ? load_entry(b, k, et) : load_entry(b, k, ev);
    if (i < (uint32_t)p.buckets) p.cursor[i] = 0;
}

// Ranks the samples: a lane per sample counts the lower ones (of equal keys,
// the earlier), each of the block's waves over its share of the sample.
// Counting is more work than sorting, but it spreads over the chip: 8,192
// samples of both arrays take 18 us, sorted by a workgroup per array 80 us.  The
// scalar loads of the other keys bound it, so 32 of them are in flight (8: 24
// us).
constexpr int kRankWaves = 16;
__global__ void __launch_bounds__(64 * kRankWaves) k_sort_rank(const SortPart pv, const SortPart pt) {
    __shared__ int s_rank[64];
    const bool tri = blockIdx.x >= kMaxSamples / 64;
    const SortPart &p = tri ? pt : pv;
    const int group = blockIdx.x % (kMaxSamples / 64), lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (64 * group >= p.samples) return;   // (uniform)
    if (threadIdx.x < 64) s_rank[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t *sample = p.sample;
    const uint64_t x = sample[64 * group + lane];
    int rank = 0;
    const int groups = p.samples / 64, per = (groups + kRankWaves - 1) / kRankWaves;
    for (int g = wave * per; g < min(groups, (wave + 1) * per); g++) {
        const uint64_t *y = sample + 64 * g;   // (uniform: scalar loads)
        if (g < group) {
#pragma unroll 32
            for (int k = 0; k < 64; k++) rank += y[k] <= x;
        } else if (g > group) {
#pragma unroll 32
            for (int k = 0; k < 64; k++) rank += y[k] < x;
        } else {
#pragma unroll 32
            for (int k = 0; k < 64; k++) rank += y[k] < x || (y[k] == x && k < lane);
        }
    }
    atomicAdd(&s_rank[lane], rank);
    __syncthreads();
    const int span = p.samples / p.buckets;
    if (threadIdx.x < 64 && s_rank[lane] % span == 0) {
        p.split[s_rank[lane] / span] = x;
        p.split_at[s_rank[lane] / span] = sample_place(p, 64 * group + lane);
    }
}

// Puts 2 elements per thread into their buckets' lists.  The block counts its
// elements of each bucket in LDS first, so a list is claimed once per block:
// the claims (device atomics) and the scattered writes bound this pass.
constexpr int kPlaceItems = 2, kPlaceBlock = 1024;
template <bool TRI>
__device__ __forceinline__ void place(const RenumberBuffers &b, const SortPart &p, int block, uint64_t *s_split,
                                      int *s_at, int *s_count) {
    const int tid = threadIdx.x;
    if (tid < p.buckets) {
        s_split[tid] = p.split[tid];
        s_at[tid] = p.split_at[tid];
        s_count[tid] = 0;
    }
    ListEntryOf<TRI> e[kPlaceItems];
    uint64_t key[kPlaceItems];
    int k[kPlaceItems], at[kPlaceItems], rank[kPlaceItems];
#pragma unroll
    for (int j = 0; j < kPlaceItems; j++) {
        k[j] = (block * kPlaceItems + j) * kPlaceBlock + tid;
        key[j] = load_entry(b, min(k[j], p.n - 1), e[j]);
        at[j] = 0;
    }
    __syncthreads();
    for (int step = p.buckets / 2; step > 0; step /= 2)
#pragma unroll
        for (int j = 0; j < kPlaceItems; j++) {
            // (without branches: hipcc 7.2 drops the step of equal keys from
            // the form with && and ||)
            const uint64_t first = s_split[at[j] + step];
            const bool up = (key[j] > first) | ((key[j] == first) & (k[j] >= s_at[at[j] + step]));
            at[j] += up ? step : 0;
        }
#pragma unroll
    for (int j = 0; j < kPlaceItems; j++)
        if (k[j] < p.n) rank[j] = atomicAdd(&s_count[at[j]], 1);
    __syncthreads();
    if (tid < p.buckets) {
        const int c = s_count[tid];
        const int first = c ? atomicAdd(&p.cursor[tid], c) : 0;
        if (first + c > p.cap) *b.overflow = 1;
        s_count[tid] = first;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPlaceItems; j++) {
        if (k[j] >= p.n) continue;
        const int i = s_count[at[j]] + rank[j];
        if (i >= p.cap) continue;   // (reported above)
        static_cast<ListEntryOf<TRI> *>(p.list)[(size_t)at[j] * p.cap + i] = e[j];
    }
}

// grid: `vblocks` of vertices, then the triangles'
__global__ void __launch_bounds__(kPlaceBlock) k_sort_place(const RenumberBuffers b, const SortPart pv,
                                                           const SortPart pt, int vblocks) {
    __shared__ uint64_t s_split[kMaxBuckets];
    __shared__ int s_at[kMaxBuckets], s_count[kMaxBuckets];
    if ((int)blockIdx.x < vblocks)
        place<false>(b, pv, blockIdx.x, s_split, s_at, s_count);
    else
        place<true>(b, pt, blockIdx.x - vblocks, s_split, s_at, s_count);
}

// Sorts a bucket's m <= 256 * E elements by (key, index), E elements per
// thread: their places in the list, in order, are the low bits of s[0, m).
// The words that move are the key's distance from the bucket's lowest, in as
// many leading bits as the bucket's range and the word leave room for, over
// the place in the list; elements that agree in these bits are neighbours
// afterwards, and swap by whole keys until they are in order.  Returns whether
// they are, within a few rounds.
constexpr int kBucketBlock = 256;
template <int E>
struct BucketWord {
    static constexpr int kLocal = 8 + __builtin_ctz(E), kBits = 32 - kLocal;
    static constexpr uint32_t kPlace = (1u << kLocal) - 1;
};

template <int E, class Entry>
__device__ __forceinline__ bool sort_words(const uint64_t (&key)[E], uint64_t lo, int bits,
                                           const Entry *__restrict__ list, int m, uint32_t *s) {
    constexpr int kLocal = BucketWord<E>::kLocal, kRounds = 4;
    constexpr uint32_t kPlace = BucketWord<E>::kPlace;
    const int tid = threadIdx.x;
    const int shift = max(0, bits - BucketWord<E>::kBits);
    uint32_t x[E];
#pragma unroll
    for (int r = 0; r < E; r++) {
        const int i = r * kBucketBlock + tid;
        x[r] = i < m ? (uint32_t)((key[r] - lo) >> shift) << kLocal | (uint32_t)i : ~0u;
    }
    block_sort<kBucketBlock, E>(x, s);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; r++) s[tid * E + r] = x[r];
    __syncthreads();
    bool tie = false;
#pragma unroll
    for (int r = 0; r < E; r++) {
        const int i = r * kBucketBlock + tid;
        tie |= i > 0 && i < m && (s[i] ^ s[i - 1]) >> kLocal == 0;
    }
    if (!__syncthreads_or(tie)) return true;
    for (int round = 0; round < kRounds; round++) {
        bool swapped = false;
        for (int par = 0; par < 2; par++) {
            for (int i = 2 * tid + par; i + 1 < m; i += 2 * kBucketBlock) {
                const uint32_t u = s[i], v = s[i + 1];
                if ((u ^ v) >> kLocal) continue;
                const Entry eu = list[u & kPlace], ev = list[v & kPlace];
                const uint64_t ku = eu.key(), kv = ev.key();
                if (ku < kv || (ku == kv && eu.old < ev.old)) continue;
                s[i] = v;
                s[i + 1] = u;
                swapped = true;
            }
            __syncthreads();
        }
        if (!__syncthreads_or(swapped)) return true;
    }
    return false;
}

// The same order whatever the keys: by the digits of the index in the input,
// then those of the key's distance from the bucket's lowest, the least digit
// first, each by a sort of words that hold the digit over the place in the
// order so far.  For buckets where many keys agree in the bits above: equal
// ones, or a cluster far smaller than the bucket's range (swapping neighbours
// until they were in order, a build of 594,000 triangles with 3,500 vertices in
// one place took 13.8 ms; now 0.14).
template <int E, class Entry>
__device__ __forceinline__ void sort_digits(uint64_t lo, int bits, const Entry *__restrict__ list, int m, uint32_t *s) {
    constexpr int kLocal = BucketWord<E>::kLocal, kBits = BucketWord<E>::kBits;
    constexpr int kOldDigits = (kSortBits + kBits - 1) / kBits;
    const int tid = threadIdx.x, digits = kOldDigits + (bits + kBits - 1) / kBits;
    uint32_t at[E];   // the element in place r * 256 + tid of the order so far
#pragma unroll
    for (int r = 0; r < E; r++) at[r] = r * kBucketBlock + tid;
    for (int d = 0; d < digits; d++) {
        uint32_t x[E];
#pragma unroll
        for (int r = 0; r < E; r++) {
            const int i = r * kBucketBlock + tid;
            x[r] = ~0u;
            if (i >= m) continue;
            const Entry e = list[at[r]];
            const uint64_t from = d < kOldDigits ? (uint64_t)e.old >> (d * kBits) : (e.key() - lo) >> ((d - kOldDigits) * kBits);
            x[r] = (uint32_t)from << kLocal | (uint32_t)i;
        }
        block_sort<kBucketBlock, E>(x, s);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; r++) s[tid * E + r] = x[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; r++) x[r] = s[r * kBucketBlock + tid] & BucketWord<E>::kPlace;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; r++) s[r * kBucketBlock + tid] = at[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; r++) at[r] = s[x[r]];
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < E; r++) s[r * kBucketBlock + tid] = at[r];
    __syncthreads();
}

// Sorts the bucket and writes its part of the permuted arrays, from `first`
// on.
template <bool TRI, int E>
__device__ __forceinline__ void sort_bucket(const RenumberBuffers &b, const SortPart &p, int bucket, int m,
                                            int first, uint32_t *s, uint64_t *s_range) {
    const int tid = threadIdx.x;
    const ListEntryOf<TRI> *list = static_cast<const ListEntryOf<TRI> *>(p.list) + (size_t)bucket * p.cap;
    uint64_t x[E], lo = ~0ull, hi = 0;
#pragma unroll
    for (int r = 0; r < E; r++) {
        const int i = r * kBucketBlock + tid;
        x[r] = i < m ? list[i].key() : 0;
        lo = i < m ? min(lo, x[r]) : lo;
        hi = max(hi, x[r]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, lane_xor(lo, o));
        hi = max(hi, lane_xor(hi, o));
    }
    if ((tid & 63) == 0) {
        s_range[2 * (tid >> 6)] = lo;
        s_range[2 * (tid >> 6) + 1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kBucketBlock / 64; w++) {
        lo = min(lo, s_range[2 * w]);
        hi = max(hi, s_range[2 * w + 1]);
    }
    const int bits = hi > lo ? 64 - __clzll((long long)(hi - lo)) : 0;
    if (!sort_words<E>(x, lo, bits, list, m, s)) sort_digits<E>(lo, bits, list, m, s);   // (uniform)
#pragma unroll
    for (int r = 0; r < E; r++) {
        const int i = r * kBucketBlock + tid, k = first + i;
        if (i >= m) continue;
        const ListEntryOf<TRI> e = list[s[i] & BucketWord<E>::kPlace];
        if constexpr (TRI) {
            b.tperm[k] = e.old;
#pragma unroll
            for (int c = 0; c < 3; c++) b.tri_out[3 * (size_t)k + c] = e.v[c];   // (renamed by k_rename_corners)
        } else {
            b.vperm[k] = e.old;
            b.vinv[e.old] = k;
            b.xy_out[k] = make_int2(e.x, e.y);
        }
    }
}

// A workgroup's bucket starts where the buckets before it end.
template <bool TRI, bool BIG>
__device__ __forceinline__ void place_bucket(const RenumberBuffers &b, const SortPart &p, int bucket, uint32_t *s,
                                             uint64_t *s_range, int *s_first) {
    const int tid = threadIdx.x;
    if (tid == 0) *s_first = 0;
    __syncthreads();
    int sum = 0;
    for (int k = tid; k < bucket; k += kBucketBlock) sum += p.cursor[k];
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((tid & 63) == 0 && sum) atomicAdd(s_first, sum);
    const int m = min(p.cursor[bucket], p.cap);
    __syncthreads();
    const int first = *s_first;
    if (m <= kBucketBlock)
        sort_bucket<TRI, 1>(b, p, bucket, m, first, s, s_range);
    else if (m <= 2 * kBucketBlock)
        sort_bucket<TRI, 2>(b, p, bucket, m, first, s, s_range);
    else if (m <= 4 * kBucketBlock)
        sort_bucket<TRI, 4>(b, p, bucket, m, first, s, s_range);
    else if (m <= 8 * kBucketBlock)
        sort_bucket<TRI, 8>(b, p, bucket, m, first, s, s_range);
    else if (!BIG || m <= 16 * kBucketBlock)
        sort_bucket<TRI, 16>(b, p, bucket, m, first, s, s_range);
    else if constexpr (BIG)
        sort_bucket<TRI, 32>(b, p, bucket, m, first, s, s_range);
}

// One workgroup per bucket, the triangles' first (they are more), the vertices'
// beside them: the new corner names, which need both, are a pass of their own
// (7 us for 594,000 triangles; the buckets of both then take 30, where the
// vertices' took 20 before the triangles' 25).  BIG: lists of more than kBucketCap (which need more
// registers).
template <bool BIG>
__global__ void __launch_bounds__(kBucketBlock) k_sort_bucket(const RenumberBuffers b, const SortPart pv,
                                                             const SortPart pt) {
    __shared__ uint32_t s[BIG ? kBigCap : kBucketCap];
    __shared__ uint64_t s_range[2 * (kBucketBlock / 64)];
    __shared__ int s_first;
    if (*b.overflow) {   // (uniform) a list overflowed: the caller sorts in another way
        if (blockIdx.x == 0 && threadIdx.x == 0) *b.overflow_out = 1;
        return;
    }
    if ((int)blockIdx.x < pt.buckets)
        place_bucket<true, BIG>(b, pt, blockIdx.x, s, s_range, &s_first);
    else
        place_bucket<false, BIG>(b, pv, blockIdx.x - pt.buckets, s, s_range, &s_first);
}

// The sorted triangles' corners by their new names (an index outside [0, nv)
// stays).
__global__ void __launch_bounds__(256) k_rename_corners(const RenumberBuffers b) {
    const long long n = 3ll * b.nt;
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += gridDim.x * 256ll) {
        const int w = b.tri_out[i];
        if (w >= 0 && w < b.nv) b.tri_out[i] = b.vinv[w];
    }
}

// The buckets of n elements (0: not sorted here).
SortPart sort_part(int n) {
    SortPart p{};
    if (n <= 0) return p;
    p.n = n;
    p.buckets = 64;
    while (p.buckets < kMaxBuckets && (int64_t)p.buckets * kBucketMean < n) p.buckets *= 2;
    const int mean = (n + p.buckets - 1) / p.buckets;
    p.samples = mean > kBucketMean ? kMaxSamples : 16 * p.buckets < kMaxSamples / 2 ? 16 * p.buckets : kMaxSamples / 2;
    p.cap = 7 * mean + 64 < kBucketCap ? 7 * mean + 64 : 4 * mean <= kBucketCap ? kBucketCap : kBigCap;
    return p;
}

template <bool TRI>
size_t part_bytes(const SortPart &p) {
    const size_t lists = sizeof(ListEntryOf<TRI>) * (size_t)p.buckets * (size_t)p.cap;
    return (sizeof(uint64_t) * (size_t)(p.samples + p.buckets) + lists + 2 * sizeof(int32_t) * (size_t)p.buckets + 63) / 64 * 64;
}

template <bool TRI>
char *part_layout(SortPart &p, char *at) {
    if (p.n <= 0) return at;
    p.sample = reinterpret_cast<uint64_t *>(at);
    p.split = p.sample + p.samples;
    p.list = p.split + p.buckets;
    p.cursor = reinterpret_cast<int32_t *>(static_cast<ListEntryOf<TRI> *>(p.list) + (size_t)p.buckets * p.cap);
    p.split_at = p.cursor + p.buckets;
    return at + part_bytes<TRI>(p);
}

// Whether an array of n elements is sorted by sampling.
bool sampled(int n, bool library) { return !library && n <= kSortMax; }

}  // namespace

RenumberSizes renumber_sizes(int32_t nv, int32_t nt, bool library) {
    RenumberSizes z;
    const SortPart pv = sort_part(sampled(nv, library) ? nv : 0), pt = sort_part(sampled(nt, library) ? nt : 0);
    z.sample_bytes = part_bytes<false>(pv) + part_bytes<true>(pt);
    for (int32_t k : {nv, nt})
        if (!sampled(k, library) && k > z.pairs) z.pairs = k;
    if (z.pairs > 0 &&
        hipcub::DeviceRadixSort::SortPairs(nullptr, z.sort_bytes, (const uint64_t *)nullptr, (uint64_t *)nullptr,
                                           (const int32_t *)nullptr, (int32_t *)nullptr, z.pairs, 0, 64,
                                           (hipStream_t)0) != hipSuccess) {
        (void)hipGetLastError();
        z.ok = false;
    }
    return z;
}

hipError_t launch_renumber(const RenumberBuffers &b, hipStream_t s) {
    hipError_t e = hipSuccess;
    size_t tb = b.sort_bytes;
    const bool own_v = sampled(b.nv, b.library), own_t = sampled(b.nt, b.library);
    SortPart pv = sort_part(own_v ? b.nv : 0), pt = sort_part(own_t ? b.nt : 0);
    part_layout<true>(pt, part_layout<false>(pv, static_cast<char *>(b.sample_tmp)));
    if (pv.n + pt.n > 0) {
        constexpr int per = kPlaceItems * kPlaceBlock;
        const int vblocks = (pv.n + per - 1) / per, tblocks = (pt.n + per - 1) / per;
        hipLaunchKernelGGL(k_sort_sample, dim3(2 * kMaxSamples / 256), dim3(256), 0, s, b, pv, pt);
        hipLaunchKernelGGL(k_sort_rank, dim3(2 * kMaxSamples / 64), dim3(64 * kRankWaves), 0, s, pv, pt);
        hipLaunchKernelGGL(k_sort_place, dim3(vblocks + tblocks), dim3(kPlaceBlock), 0, s, b, pv, pt, vblocks);
        const auto kernel = pv.cap > kBucketCap || pt.cap > kBucketCap ? &k_sort_bucket<true> : &k_sort_bucket<false>;
        hipLaunchKernelGGL(kernel, dim3(pv.buckets + pt.buckets), dim3(kBucketBlock), 0, s, b, pv, pt);
    }
    if (!own_v && b.nv > 0) {
        hipLaunchKernelGGL(k_vertex_keys, dim3(blocks_for(b.nv)), dim3(256), 0, s, b.xy_in, b.nv, b.keys, b.vals);
        e = hipcub::DeviceRadixSort::SortPairs(b.sort_tmp, tb, b.keys, b.keys_alt, b.vals, b.vperm, b.nv, 0, 62, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_vertex_gather, dim3(blocks_for(b.nv)), dim3(256), 0, s, b.xy_in, b.vperm, b.nv, b.vinv,
                           b.xy_out);
    }
    if (pt.n > 0) {
        hipLaunchKernelGGL(k_rename_corners, dim3(blocks_for(3 * b.nt)), dim3(256), 0, s, b);
    } else if (b.nt > 0) {
        hipLaunchKernelGGL(k_triangle_keys, dim3(blocks_for(b.nt)), dim3(256), 0, s, b.xy_in, b.tri_in, b.nv, b.nt,
                           b.keys, b.vals);
        tb = b.sort_bytes;
        e = hipcub::DeviceRadixSort::SortPairs(b.sort_tmp, tb, b.keys, b.keys_alt, b.vals, b.tperm, b.nt, 0, 64, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_triangle_gather, dim3(blocks_for(b.nt)), dim3(256), 0, s, b.tri_in, b.tperm, b.vinv,
                           b.nv, b.nt, b.tri_out);
    }
    return hipGetLastError();
}

}  // namespace gp
