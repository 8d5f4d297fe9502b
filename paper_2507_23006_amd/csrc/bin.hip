// Tile binning -- gfx950.
//
// "Processed in depth order" (§3.1) per tile, ties by input order, is built
// depth-first: the visible slots are compacted in slot order (a scan), sorted
// once by their 32-bit depth key, expanded into (tile, slot) pairs in that
// order, and the pairs are then stably sorted by tile id only
// (ceil(log2 tiles) bits, 2-3 passes) instead of sorting P pairs on a 45-49
// bit (tile, depth) key.  Stability of both sorts keeps the depth order
// inside every tile, ties by slot index.
#include <algorithm>

#include "gs_internal.h"

namespace gs {

namespace {

// Visible slots are counted and compacted kVisTile at a time.
constexpr int kVisThreads = 256, kVisIpt = 8;
constexpr uint32_t kVisTile = kVisThreads * kVisIpt;
static_assert(kVisTile == kBinVisTile, "the workspace holds one pair of counts per tile");

// Per tile of slots: how many are visible and how many pairs they emit.
__global__ __launch_bounds__(kVisThreads) void k_count_visible(const uint32_t* __restrict__ tiles, uint32_t n,
                                                               uint32_t* __restrict__ vis,
                                                               unsigned long long* __restrict__ pairs) {
    __shared__ uint32_t s_v[4];
    __shared__ unsigned long long s_p[4];
    const uint32_t base = blockIdx.x * kVisTile + threadIdx.x;
    uint32_t t[kVisIpt];
#pragma unroll
    for (int r = 0; r < kVisIpt; ++r) t[r] = base + r * kVisThreads < n ? tiles[base + r * kVisThreads] : 0u;
    uint32_t v = 0;
    unsigned long long p = 0;
#pragma unroll
    for (int r = 0; r < kVisIpt; ++r) {
        v += (uint32_t)__popcll(__ballot(t[r] != 0u));      // the wave's count
        p += t[r];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off, 64);
    if ((threadIdx.x & 63) == 0) {
        s_v[threadIdx.x >> 6] = v;
        s_p[threadIdx.x >> 6] = p;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        vis[blockIdx.x] = s_v[0] + s_v[1] + s_v[2] + s_v[3];
        pairs[blockIdx.x] = s_p[0] + s_p[1] + s_p[2] + s_p[3];
    }
}

// The binning's sizes: the pair count goes to n_pairs_out; the effective
// counts counts[0] (visible) and counts[1] (pairs), read by the launches after
// the compaction, are 0 when the pairs exceed the capacity or 32-bit indexing,
// so those launches then produce empty lists and the caller learns of it from
// the count alone.
__device__ __forceinline__ void write_counts(uint32_t visible, unsigned long long pairs, unsigned long long capacity,
                                             int64_t* __restrict__ n_pairs_out, uint32_t* __restrict__ counts) {
    const bool ok = pairs <= capacity && pairs <= 0xFFFFFF00ull;
    counts[0] = ok ? visible : 0u;
    counts[1] = ok ? (uint32_t)pairs : 0u;
    *n_pairs_out = (int64_t)pairs;
}

// Exclusive scan of the tiles' visible counts in place, and the totals, by one
// workgroup: only from kVisScanMin tiles on, where adding up the earlier
// tiles' counts in every compaction workgroup costs more (96M slots, 47k tiles:
// 4 GB of L2 reads, the compaction 940 instead of 600 us) than this launch.
constexpr uint32_t kVisScanMin = 6144;
__global__ __launch_bounds__(1024) void k_scan_visible(uint32_t* __restrict__ vis,
                                                       const unsigned long long* __restrict__ pairs, uint32_t n_tiles,
                                                       unsigned long long capacity, int64_t* __restrict__ n_pairs_out,
                                                       uint32_t* __restrict__ counts) {
    __shared__ uint32_t s_w[16];
    __shared__ unsigned long long s_p[16];
    constexpr int kPer = 16;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t before = 0;
    unsigned long long P = 0;
    for (uint32_t c0 = 0; c0 < n_tiles; c0 += 1024 * kPer) {
        const uint32_t i0 = c0 + threadIdx.x * kPer;
        uint32_t v[kPer], sum = 0;
#pragma unroll
        for (int r = 0; r < kPer; ++r) v[r] = i0 + r < n_tiles ? vis[i0 + r] : 0u;
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const uint32_t i = c0 + r * 1024 + threadIdx.x;
            P += i < n_tiles ? pairs[i] : 0ull;
            sum += v[r];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        __syncthreads();      // the previous chunk's sums are consumed
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        uint32_t pre = before + incl - sum;
        for (int w = 0; w < 16; ++w) {
            pre += w < wave ? s_w[w] : 0u;
            before += s_w[w];
        }
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            if (i0 + r < n_tiles) vis[i0 + r] = pre;
            pre += v[r];
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) P += __shfl_xor(P, off, 64);
    if (lane == 0) s_p[wave] = P;
    __syncthreads();
    if (threadIdx.x == 0) {
        P = 0;
        for (int w = 0; w < 16; ++w) P += s_p[w];
        write_counts(before, P, capacity, n_pairs_out, counts);
    }
}

// Visible slots, in slot order, with their depth keys: the input of the
// depth sort (culled slots never enter it), whose values are the compaction
// positions.  Each visible slot also leaves a 32-byte descriptor there
// (rectangle, tile mask, tile count, slot) so that the gather after the sort
// fetches one line per depth rank instead of one per source array.  Unless
// k_scan_visible ran (kScanned), a workgroup adds up the earlier tiles' counts
// itself and the last one has the totals.  A thread's kVisIpt slots have their
// gathers in flight together.  Bound by HBM: the visible sixth of a street
// scene touches nearly every line of the four source arrays (6M slots: 200 MB
// in 39 us).
template <bool kScanned>
__global__ __launch_bounds__(kVisThreads) void k_compact_visible(
    const uint32_t* __restrict__ tiles, const uint32_t* __restrict__ vis,
    const unsigned long long* __restrict__ pairs, const uint32_t* __restrict__ dkey, const uint2* __restrict__ rect,
    const uint64_t* __restrict__ mask, uint32_t n, unsigned long long capacity, uint32_t* __restrict__ keys,
    uint4* __restrict__ desc, int64_t* __restrict__ n_pairs_out, uint32_t* __restrict__ counts) {
    __shared__ uint32_t s_cnt[kVisIpt * 4], s_off[4];
    __shared__ unsigned long long s_p[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t base = blockIdx.x * kVisTile + threadIdx.x;
    uint32_t t[kVisIpt];
#pragma unroll
    for (int r = 0; r < kVisIpt; ++r) t[r] = base + r * kVisThreads < n ? tiles[base + r * kVisThreads] : 0u;
    const bool last = !kScanned && blockIdx.x == gridDim.x - 1;
    uint32_t off = 0;
    unsigned long long P = 0;
    if (kScanned) {
        if (threadIdx.x == 0) off = vis[blockIdx.x];
    } else {
        for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kVisThreads) off += vis[b];
        if (last)
            for (uint32_t b = threadIdx.x; b < gridDim.x; b += kVisThreads) P += pairs[b];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            off += __shfl_xor(off, o, 64);
            P += __shfl_xor(P, o, 64);
        }
    }
    uint64_t seen[kVisIpt];
#pragma unroll
    for (int r = 0; r < kVisIpt; ++r) seen[r] = __ballot(t[r] != 0u);
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < kVisIpt; ++r) s_cnt[r * 4 + wave] = (uint32_t)__popcll(seen[r]);
        s_off[wave] = off;
        s_p[wave] = P;
    }
    // half of the thread's slots at a time, the gathers of the first before the
    // barrier: with all in flight at once the kernel needs 88 registers, and beside
    // a compositing kernel, whose ending waves free 72, it waits for that kernel's end
    constexpr int kHalf = kVisIpt / 2;
    uint32_t k[kHalf];
    uint2 rc[kHalf];
    uint64_t m[kHalf];
    const auto gather = [&](int first) {
#pragma unroll
        for (int r = 0; r < kHalf; ++r) {
            const uint32_t i = base + (first + r) * kVisThreads;
            const bool on = t[first + r] != 0u;
            k[r] = on ? dkey[i] : 0u;
            rc[r] = on ? rect[i] : make_uint2(0u, 0u);
            m[r] = on && mask ? mask[i] : 0ull;
        }
    };
    gather(0);
    __syncthreads();
    uint32_t pos[kVisIpt], run = s_off[0] + s_off[1] + s_off[2] + s_off[3];
#pragma unroll
    for (int j = 0; j < kVisIpt * 4; ++j) {       // (r, wave) in slot order
        if ((j & 3) == wave)
            pos[j >> 2] = run + __builtin_amdgcn_mbcnt_hi((uint32_t)(seen[j >> 2] >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)seen[j >> 2], 0));
        run += s_cnt[j];
    }
    if (last && threadIdx.x == 0) write_counts(run, s_p[0] + s_p[1] + s_p[2] + s_p[3], capacity, n_pairs_out, counts);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h) gather(kHalf);
#pragma unroll
        for (int r = 0; r < kHalf; ++r) {
            const int j = h * kHalf + r;
            if (!t[j]) continue;
            const uint32_t d = pos[j];
            keys[d] = k[r];
            desc[2 * (size_t)d] = make_uint4(rc[r].x, rc[r].y, (uint32_t)m[r], (uint32_t)(m[r] >> 32));
            desc[2 * (size_t)d + 1] = make_uint4(t[j], base + j * kVisThreads, 0u, 0u);
        }
    }
}

// per depth rank: tiles covered and the emission descriptor of its slot
// (rectangle, covered-tile mask, slot), from its compaction descriptor; per
// kScanTileElems ranks the sum of the tile counts, for the scan after it
constexpr int kGatherThreads = 256, kGatherIpt = kScanTileElems / kGatherThreads;
__global__ __launch_bounds__(kGatherThreads) void k_gather_sorted(
    const uint32_t* __restrict__ sorted_pos, const uint4* __restrict__ desc, uint32_t n_max,
    const uint32_t* __restrict__ counts, uint32_t* __restrict__ tiles_s, uint2* __restrict__ rect_s,
    uint64_t* __restrict__ mask_s, uint32_t* __restrict__ slot_s, uint32_t* __restrict__ tile_sums) {
    __shared__ uint32_t s_w[4];
    const uint32_t n = min(counts[0], n_max);
    if (blockIdx.x > 0 && blockIdx.x * (uint32_t)kScanTileElems >= n) return;
    const uint32_t base = blockIdx.x * kScanTileElems + threadIdx.x;
    uint32_t c[kGatherIpt];
#pragma unroll
    for (int r = 0; r < kGatherIpt; ++r)
        c[r] = base + r * kGatherThreads < n ? sorted_pos[base + r * kGatherThreads] : 0xFFFFFFFFu;
    uint4 a[kGatherIpt];
    uint2 b[kGatherIpt];
#pragma unroll
    for (int r = 0; r < kGatherIpt; ++r) {
        const bool in = c[r] != 0xFFFFFFFFu;
        a[r] = in ? desc[2 * (size_t)c[r]] : make_uint4(0u, 0u, 0u, 0u);
        b[r] = in ? *reinterpret_cast<const uint2*>(desc + 2 * (size_t)c[r] + 1) : make_uint2(0u, 0u);
    }
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kGatherIpt; ++r) {
        if (c[r] == 0xFFFFFFFFu) continue;
        const uint32_t d = base + r * kGatherThreads;
        tiles_s[d] = b[r].x;
        rect_s[d] = make_uint2(a[r].x, a[r].y);
        mask_s[d] = (uint64_t)a[r].z | ((uint64_t)a[r].w << 32);
        slot_s[d] = b[r].y;
        sum += b[r].x;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// index of the k-th set bit (k < popcount(m)) of m, by halving
__device__ __forceinline__ uint32_t nth_set_bit(uint64_t m, uint32_t k) {
    const uint32_t lo = (uint32_t)m, c0 = (uint32_t)__popc(lo);
    const bool up = k >= c0;
    uint32_t w = up ? (uint32_t)(m >> 32) : lo, base = up ? 32u : 0u;
    k -= up ? c0 : 0u;
#pragma unroll
    for (int width = 16; width >= 1; width >>= 1) {
        const uint32_t c = (uint32_t)__popc(w & ((1u << width) - 1u));
        const bool skip = k >= c;
        k -= skip ? c : 0u;
        w >>= skip ? width : 0;
        base += skip ? width : 0;
    }
    return base;
}

constexpr int kEmitThreads = 256;
constexpr int kEmitPer = kEmitChunk / kEmitThreads;

// Pair p belongs to the last depth rank d with offsets[d] <= p.  A workgroup
// owns kEmitChunk consecutive pairs, whose ranks form one contiguous run of
// at most kEmitChunk + 1 entries (every visible rank owns >= 1 pair, culled
// ranks own none and sort last), from the rank the offsets' scan left for the
// chunk.  The run's ranks mark the places of their first pairs in LDS, and a
// running maximum over the chunk (consecutive pairs per thread, then the wave,
// then the workgroup) gives every pair its rank: about 10 instructions per pair, where a binary search of the offsets in
// LDS took 60, and the division by the rectangle's width is a multiplication
// by the reciprocal (6M Gaussians, 3.3M pairs: 24 -> 16 us).  The
// workgroups also zero the tile ranges, which the launch after the tile sort
// fills for tiles with pairs.
__global__ __launch_bounds__(kEmitThreads) void k_emit_pairs(const uint32_t* __restrict__ offsets,
                                                             const uint32_t* __restrict__ chunk_first,
                                                             const uint2* __restrict__ rect_s,
                                                             const uint64_t* __restrict__ mask_s,
                                                             const uint32_t* __restrict__ sorted_slot, uint32_t n_max,
                                                             uint32_t n_pairs_max, const uint32_t* __restrict__ counts,
                                                             uint32_t* __restrict__ pair_key,
                                                             uint32_t* __restrict__ pair_val,
                                                             uint2* __restrict__ ranges, uint32_t n_tiles) {
    for (uint32_t t = blockIdx.x * kEmitThreads + threadIdx.x; t < n_tiles; t += gridDim.x * kEmitThreads)
        ranges[t] = make_uint2(0u, 0u);
    __shared__ uint32_t s_off[kEmitChunk + 1];                 // the run's offsets
    __shared__ alignas(16) uint32_t s_rank[kEmitChunk];        // rank of the run that starts at a pair
    __shared__ uint32_t s_max[kEmitThreads / 64];
    // depth ranks and pairs: the launch's bounds, or the counts on the device
    const uint32_t n = min(counts[0], n_max);
    const uint32_t n_pairs = min(counts[1], n_pairs_max);
    const uint32_t p0 = blockIdx.x * kEmitChunk;
    if (p0 >= n_pairs) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t d0 = chunk_first[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kEmitPer; ++k) s_rank[k * kEmitThreads + threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t cnt = min((uint32_t)(kEmitChunk + 1), n - d0);
    for (uint32_t i = threadIdx.x; i < cnt; i += kEmitThreads) {
        const uint32_t o = offsets[d0 + i];
        s_off[i] = o;
        // run 0 starts at or before the chunk and is the initial 0
        if (i > 0 && o - p0 < (uint32_t)kEmitChunk) s_rank[o - p0] = i;
    }
    __syncthreads();
    // running maximum, kEmitPer consecutive pairs per thread
    uint32_t r[kEmitPer];
#pragma unroll
    for (int k = 0; k < kEmitPer; k += 4) {
        const uint4 r4 = reinterpret_cast<const uint4*>(s_rank)[(threadIdx.x * kEmitPer + k) / 4];
        r[k] = r4.x;
        r[k + 1] = r4.y;
        r[k + 2] = r4.z;
        r[k + 3] = r4.w;
    }
#pragma unroll
    for (int k = 1; k < kEmitPer; ++k) r[k] = max(r[k], r[k - 1]);
    uint32_t top = r[kEmitPer - 1];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(top, off, 64);
        if (lane >= off) top = max(top, y);
    }
    if (lane == 63) s_max[wave] = top;
    uint32_t before = __shfl_up(top, 1, 64);
    if (lane == 0) before = 0u;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before = max(before, s_max[w]);
#pragma unroll
    for (int k = 0; k < kEmitPer; ++k) r[k] = max(r[k], before);
#pragma unroll
    for (int k = 0; k < kEmitPer; k += 4)
        reinterpret_cast<uint4*>(s_rank)[(threadIdx.x * kEmitPer + k) / 4] = make_uint4(r[k], r[k + 1], r[k + 2], r[k + 3]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kEmitPer; ++k) {
        const uint32_t i = k * kEmitThreads + threadIdx.x, p = p0 + i;
        if (p >= n_pairs) break;
        const uint32_t run = s_rank[i], d = d0 + run;
        uint32_t local = p - s_off[run];
        const uint2 rs = rect_s[d];
        const uint32_t w = rs.y & 0xFFFFu, tw = rs.y >> 16;
        if (mask_s) {
            // the local-th covered tile of the rectangle (row-major bits)
            const uint64_t m = mask_s[d];
            if (m) local = nth_set_bit(m, local);
        }
        // local / w: local + 1/2 is at least 1/2 from a multiple of w, and an
        // image has at most 2^20 tiles, so the product's error (2 ulps of at
        // most 2^20 / w) stays below 1 / (2 w)
        const uint32_t row = (uint32_t)(((float)local + 0.5f) * __builtin_amdgcn_rcpf((float)w));
        const uint32_t col = local - row * w;
        pair_key[p] = rs.x + row * tw + col;
        pair_val[p] = sorted_slot[d];
    }
}

// kRangePer pairs per thread, kRangeThreads apart (coalesced), so that each
// wave keeps several loads in flight instead of one round trip per wave; a
// pair's predecessor is the neighbouring lane's
constexpr int kRangeThreads = 256, kRangePer = 8;

__global__ __launch_bounds__(kRangeThreads) void k_tile_ranges(const uint32_t* __restrict__ keys, uint32_t n_max,
                                                               const uint32_t* __restrict__ counts,
                                                               uint2* __restrict__ ranges, uint32_t n_tiles) {
    const uint32_t n = min(counts[1], n_max);
    const uint32_t base = blockIdx.x * (kRangeThreads * kRangePer) + threadIdx.x;
    if (blockIdx.x * (kRangeThreads * kRangePer) >= n) return;
    const int lane = threadIdx.x & 63;
    uint32_t k[kRangePer], prev[kRangePer];
#pragma unroll
    for (int j = 0; j < kRangePer; ++j) {
        const uint32_t p = base + j * kRangeThreads;
        k[j] = p < n ? keys[p] : 0u;
        prev[j] = lane == 0 && p > 0 && p < n ? keys[p - 1] : 0xFFFFFFFFu;      // no tile before the first pair
    }
#pragma unroll
    for (int j = 0; j < kRangePer; ++j) {
        const uint32_t p = base + j * kRangeThreads;
        const uint32_t left = __shfl_up(k[j], 1, 64);
        const uint32_t before = lane == 0 ? prev[j] : left;
        if (p >= n) break;
        // keys are tile ids by construction; the comparisons guard the writes
        if (before != k[j]) {
            if (k[j] < n_tiles) ranges[k[j]].x = p;
            if (before < n_tiles) ranges[before].y = p;
        }
        if (p == n - 1 && k[j] < n_tiles) ranges[k[j]].y = n;
    }
}

// Launch order of the tiles for compositing: longest lists first, so that
// the slowest workgroups start early instead of forming the tail of the
// launch (longest-processing-time-first list scheduling).  One workgroup:
// tiles are bucketed by 1/8-octave steps of their list length (LDS counts),
// the buckets are scanned from the longest down, and every tile takes the
// next place of its bucket.  Order inside a bucket is arbitrary; results do
// not depend on it.
constexpr int kOrderThreads = 1024;
constexpr int kOrderBuckets = 256;

__device__ __forceinline__ int order_bucket(const uint2 r) {
    const uint32_t len = r.y - r.x;
    const int b = (int)(8.0f * __log2f((float)len + 1.0f));
    return kOrderBuckets - 1 - min(b, kOrderBuckets - 1);   // longest first
}

__global__ __launch_bounds__(kOrderThreads) void k_tile_order(const uint2* __restrict__ ranges, uint32_t n_tiles,
                                                              uint32_t* __restrict__ order) {
    __shared__ uint32_t s_cnt[kOrderBuckets];
    const int tid = threadIdx.x;
    for (int b = tid; b < kOrderBuckets; b += kOrderThreads) s_cnt[b] = 0;
    __syncthreads();
    // kOrderPer tiles per thread at a time, all loads first
    constexpr int kOrderPer = 8;
    auto load = [&](uint32_t t0, uint2* r) {
#pragma unroll
        for (int u = 0; u < kOrderPer; ++u) {
            const uint32_t t = t0 + u * kOrderThreads;
            r[u] = t < n_tiles ? ranges[t] : make_uint2(0u, 0u);
        }
    };
    for (uint32_t t0 = tid; t0 < n_tiles; t0 += kOrderPer * kOrderThreads) {
        uint2 r[kOrderPer];
        load(t0, r);
#pragma unroll
        for (int u = 0; u < kOrderPer; ++u)
            if (t0 + u * kOrderThreads < n_tiles) atomicAdd(&s_cnt[order_bucket(r[u])], 1u);
    }
    __syncthreads();
    static_assert(kOrderBuckets == 256, "one wave scans the buckets, four per lane");
    if (tid < 64) wave_excl_scan256(s_cnt);
    __syncthreads();
    for (uint32_t t0 = tid; t0 < n_tiles; t0 += kOrderPer * kOrderThreads) {
        uint2 r[kOrderPer];
        load(t0, r);
#pragma unroll
        for (int u = 0; u < kOrderPer; ++u) {
            const uint32_t t = t0 + u * kOrderThreads;
            if (t < n_tiles) order[atomicAdd(&s_cnt[order_bucket(r[u])], 1u)] = t;
        }
    }
}

}  // namespace

hipError_t launch_tile_order(const uint32_t* ranges, uint32_t n_tiles, uint32_t* order, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(kOrderThreads), 0, s, reinterpret_cast<const uint2*>(ranges),
                       n_tiles, order);
    return hipGetLastError();
}

hipError_t launch_compact_visible(const Projected& proj, uint32_t n_slots, unsigned long long capacity, uint32_t* vis,
                                  unsigned long long* pairs, uint32_t* keys, uint4* desc, int64_t* n_pairs_out,
                                  uint32_t* counts, hipStream_t s) {
    const dim3 grid((unsigned)(((uint64_t)n_slots + kVisTile - 1) / kVisTile));
    hipLaunchKernelGGL(k_count_visible, grid, dim3(kVisThreads), 0, s, proj.tiles, n_slots, vis, pairs);
    if (grid.x >= kVisScanMin) {
        hipLaunchKernelGGL(k_scan_visible, dim3(1), dim3(1024), 0, s, vis, pairs, grid.x, capacity, n_pairs_out, counts);
        hipLaunchKernelGGL(k_compact_visible<true>, grid, dim3(kVisThreads), 0, s, proj.tiles, vis, pairs, proj.dkey,
                           proj.rect, proj.tile_mask, n_slots, capacity, keys, desc, n_pairs_out, counts);
    } else {
        hipLaunchKernelGGL(k_compact_visible<false>, grid, dim3(kVisThreads), 0, s, proj.tiles, vis, pairs, proj.dkey,
                           proj.rect, proj.tile_mask, n_slots, capacity, keys, desc, n_pairs_out, counts);
    }
    return hipGetLastError();
}

hipError_t launch_gather_sorted(const uint32_t* sorted_pos, const uint4* desc, uint32_t n_visible, const uint32_t* counts,
                                uint32_t* tiles_s, uint2* rect_s, uint64_t* mask_s, uint32_t* slot_s,
                                uint32_t* tile_sums, hipStream_t s) {
    if (!n_visible) return hipSuccess;
    hipLaunchKernelGGL(k_gather_sorted, dim3((unsigned)(((uint64_t)n_visible + kScanTileElems - 1) / kScanTileElems)),
                       dim3(kGatherThreads), 0, s, sorted_pos, desc, n_visible, counts, tiles_s, rect_s, mask_s, slot_s,
                       tile_sums);
    return hipGetLastError();
}

hipError_t launch_emit_pairs(const uint32_t* offsets, const uint32_t* chunk_first, const uint2* rect_s,
                             const uint64_t* mask_s,
                             const uint32_t* sorted_slot, uint32_t n_slots, uint32_t n_pairs, const uint32_t* counts,
                             uint32_t* pair_key, uint32_t* pair_val, uint32_t* ranges, uint32_t n_tiles,
                             hipStream_t s) {
    // one workgroup zeroes the ranges even with no room for a pair
    const uint32_t blocks = std::max(1u, (uint32_t)(((uint64_t)n_pairs + kEmitChunk - 1) / kEmitChunk));
    hipLaunchKernelGGL(k_emit_pairs, dim3(blocks), dim3(kEmitThreads), 0, s, offsets, chunk_first, rect_s, mask_s, sorted_slot,
                       n_slots, n_pairs, counts, pair_key, pair_val, reinterpret_cast<uint2*>(ranges), n_tiles);
    return hipGetLastError();
}

hipError_t launch_tile_ranges(const uint32_t* sorted_keys, uint32_t n_pairs, const uint32_t* counts, uint32_t* ranges,
                              uint32_t n_tiles, hipStream_t s) {
    if (!n_pairs) return hipSuccess;
    constexpr uint32_t per_block = kRangeThreads * kRangePer;
    hipLaunchKernelGGL(k_tile_ranges, dim3((n_pairs + per_block - 1) / per_block), dim3(kRangeThreads), 0, s,
                       sorted_keys, n_pairs, counts, reinterpret_cast<uint2*>(ranges), n_tiles);
    return hipGetLastError();
}

}  // namespace gs
