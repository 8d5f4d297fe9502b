// Device-wide primitives for binning: a stable LSD radix sort of
// (uint32 key, uint32 value) pairs and an exclusive scan of uint32 -- gfx950.
//
// Radix pass = two or three launches, none of which waits for another
// workgroup (so no kernel can hang on a missing predecessor):
//   1. upsweep: each workgroup counts the digits of its tile (1024 or 2048
//      keys) into a table of [digit][tile];
//   2. row scan: one workgroup per digit scans its row of the table in place
//      and leaves the row's total;
//   3. downsweep: every workgroup scans the row totals, which with its column
//      of the table gives the output offset of each of its digits; each wave64
//      ranks its keys in rounds of 64 with ballot-based digit matching (lanes
//      with equal digits find each other through one __ballot per digit bit;
//      rank = popcount of lower peers), keeping per-wave running digit counters
//      in LDS.  Keys and values are then scattered into LDS in digit order and
//      written out in runs, so global stores are contiguous per digit.
// Sorts of at most kFewTiles tiles leave out the row scan: the table is laid
// out [tile][digit] and the downsweep adds up the earlier tiles' counts itself
// (at 118 tiles 8.1 us instead of 5.9, against a launch of 3.4 and its gap: a
// render of 120k Gaussians takes 176 instead of 182 us).
// Stability: inside a wave items are ranked in (round, lane) order, waves
// and tiles are concatenated in order, so equal keys keep input order.
#include "chunks.h"
#include "gs_internal.h"

namespace gs {

namespace {

constexpr int kSortThreads = 256;
constexpr int kMaxRadixBits = 8;
// Keys per workgroup: small sorts take 4 per thread (1024 per workgroup),
// so that a sort of ~1M keys still spreads over ~1000 workgroups; larger
// ones take 8 (fewer digit-table entries to scan).
constexpr uint32_t kSmallSortMax = 1u << 21;
constexpr int kMinSortTile = kSortThreads * 4;      // digit tables are sized for this
constexpr uint32_t kFewTiles = 128;

__device__ __forceinline__ unsigned long long lanemask_lt() {
    const unsigned lane = __lane_id();
    return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Mask of the active lanes whose `digit` equals this lane's, restricted to
// lanes where `valid` holds.  `bits` ballots.
__device__ __forceinline__ unsigned long long match_digit(uint32_t digit, bool valid, int bits) {
    unsigned long long m = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool bit = (digit >> b) & 1u;
        const unsigned long long bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// n_dev (nullable): the key count on the device, at most n (the launch's bound)
__device__ __forceinline__ uint32_t count_of(uint32_t n, const uint32_t* __restrict__ n_dev) {
    return n_dev ? min(*n_dev, n) : n;
}

template <int kSortIpt, bool kFew>
__global__ __launch_bounds__(kSortThreads) void k_radix_upsweep(const uint32_t* __restrict__ keys, uint32_t n_max,
                                                                const uint32_t* __restrict__ n_dev, int shift,
                                                                int bits, uint32_t* __restrict__ hist) {
    constexpr int kSortTile = kSortThreads * kSortIpt, kWaveItems = 64 * kSortIpt;
    __shared__ uint32_t cnt[4][1 << kMaxRadixBits];
    // the digit table has one column per tile that holds keys: its row
    // stride is the tile count of the device count, and workgroups past it
    // write nothing
    const uint32_t n = count_of(n_max, n_dev);
    const uint32_t n_tab = (uint32_t)(((uint64_t)n + kSortTile - 1) / kSortTile);
    if (blockIdx.x >= n_tab) return;
    const int radix = 1 << bits;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t base = blockIdx.x * kSortTile + wave * kWaveItems;
    uint32_t key[kSortIpt];
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) key[r] = base + r * 64 + lane < n ? keys[base + r * 64 + lane] : 0u;
    // rows are (1 << kMaxRadixBits) apart: clear the whole table, not 4 * radix entries
    for (int i = threadIdx.x; i < 4 * (1 << kMaxRadixBits); i += kSortThreads) (&cnt[0][0])[i] = 0;
    __syncthreads();
    const uint32_t mask = (uint32_t)radix - 1;
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const bool valid = base + r * 64 + lane < n;
        const uint32_t d = (key[r] >> shift) & mask;
        const unsigned long long m = match_digit(d, valid, bits);
        if (valid && lane == __ffsll((unsigned long long)m) - 1) cnt[wave][d] += (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = threadIdx.x; d < radix; d += kSortThreads)
        hist[kFew ? (size_t)blockIdx.x * radix + d : (size_t)d * n_tab + blockIdx.x] =
            cnt[0][d] + cnt[1][d] + cnt[2][d] + cnt[3][d];
}

// One workgroup per digit: exclusive scan of its row of the table (one count
// per tile) in place; its total goes to row_total.  A row is walked in chunks
// of 8 per thread, one after another.  (1024 threads walk the long rows of 76M
// pairs' 37k tiles in 17 us where 256 take 19, but beside a compositing kernel
// their 16 waves wait for that many slots of one compute unit: 137 us.)
constexpr int kRowIpt = 8, kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void k_radix_rowscan(uint32_t* __restrict__ hist, uint32_t n_max,
                                                            const uint32_t* __restrict__ n_dev, uint32_t sort_tile,
                                                            uint32_t* __restrict__ row_total) {
    constexpr int kWaves = kRowThreads / 64;
    __shared__ uint32_t s_w[2][kWaves];
    const uint32_t n = count_of(n_max, n_dev);
    const uint32_t n_tab = (uint32_t)(((uint64_t)n + sort_tile - 1) / sort_tile);
    uint32_t* row = hist + (size_t)blockIdx.x * n_tab;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t before = 0;
    int buf = 0;
    uint32_t v[kRowIpt];
    auto load = [&](uint32_t c0) {
        // kRowIpt consecutive entries per thread
        const uint32_t i0 = c0 + threadIdx.x * kRowIpt;
#pragma unroll
        for (int r = 0; r < kRowIpt; ++r) v[r] = i0 + r < n_tab ? row[i0 + r] : 0u;
    };
    load(0);
    for (uint32_t c0 = 0; c0 < n_tab; c0 += kRowThreads * kRowIpt) {
        uint32_t cur[kRowIpt], sum = 0;
#pragma unroll
        for (int r = 0; r < kRowIpt; ++r) {
            cur[r] = v[r];
            sum += v[r];
        }
        load(c0 + kRowThreads * kRowIpt);      // the next chunk, beside this one's scan
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        if (lane == 63) s_w[buf][wave] = incl;
        __syncthreads();
        uint32_t pre = before + incl - sum;
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t x = s_w[buf][w];
            pre += w < wave ? x : 0u;
            before += x;
        }
        buf ^= 1;      // the other buffer is written before the next barrier
        const uint32_t i0 = c0 + threadIdx.x * kRowIpt;
#pragma unroll
        for (int r = 0; r < kRowIpt; ++r) {
            if (i0 + r < n_tab) row[i0 + r] = pre;
            pre += cur[r];
        }
    }
    if (threadIdx.x == 0) row_total[blockIdx.x] = before;
}

// vin NULL: the values are the input positions
template <int kSortIpt, bool kFew>
__global__ __launch_bounds__(kSortThreads) void k_radix_downsweep(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, uint32_t n_max, const uint32_t* __restrict__ n_dev, int shift, int bits,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ row_total) {
    constexpr int kSortTile = kSortThreads * kSortIpt, kWaveItems = 64 * kSortIpt;
    const uint32_t n = count_of(n_max, n_dev);
    if (blockIdx.x * (uint32_t)kSortTile >= n) return;     // no keys in this tile
    const uint32_t n_tab = (uint32_t)(((uint64_t)n + kSortTile - 1) / kSortTile);   // digit-table stride
    __shared__ uint32_t s_keys[kSortTile];
    __shared__ uint32_t s_vals[kSortTile];
    __shared__ uint32_t s_wcnt[4][1 << kMaxRadixBits];
    __shared__ uint32_t s_bstart[1 << kMaxRadixBits];
    __shared__ uint32_t s_goff[1 << kMaxRadixBits];
    __shared__ uint32_t s_wsum[4], s_gsum[4];

    const int radix = 1 << bits;
    const uint32_t mask = (uint32_t)radix - 1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < 4 * (1 << kMaxRadixBits); i += kSortThreads) (&s_wcnt[0][0])[i] = 0;
    __syncthreads();

    const uint32_t tile0 = blockIdx.x * kSortTile;
    const uint32_t base = tile0 + wave * kWaveItems;
    uint32_t key[kSortIpt], val[kSortIpt], rank[kSortIpt];
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const uint32_t idx = base + r * 64 + lane;
        const bool valid = idx < n;
        key[r] = valid ? kin[idx] : 0u;
        val[r] = !vin ? idx : valid ? vin[idx] : 0u;
    }
    // this thread's digit: its keys in earlier tiles, and in all
    uint32_t earlier = 0, all = 0;
    if ((int)threadIdx.x < radix) {
        if (kFew) {
#pragma unroll 16
            for (uint32_t c = 0; c < n_tab; ++c) {
                const uint32_t h = hist[(size_t)c * radix + threadIdx.x];
                all += h;
                earlier += c < blockIdx.x ? h : 0u;
            }
        } else {
            all = row_total[threadIdx.x];
            earlier = hist[(size_t)threadIdx.x * n_tab + blockIdx.x];
        }
    }
    const unsigned long long lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const uint32_t idx = base + r * 64 + lane;
        const bool valid = idx < n;
        const uint32_t d = (key[r] >> shift) & mask;
        const unsigned long long m = match_digit(d, valid, bits);
        uint32_t pre = 0;
        if (valid) pre = s_wcnt[wave][d];
        rank[r] = pre + (uint32_t)__popcll(m & lt);
        // every lane of the wave reads the counter before the group leader
        // rewrites it: one wave's LDS instructions execute in order; the
        // wave barrier keeps the compiler from moving LDS accesses across
        __builtin_amdgcn_wave_barrier();
        if (valid && lane == __ffsll((unsigned long long)m) - 1) s_wcnt[wave][d] = pre + (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // per digit: exclusive prefix over waves and block total, then exclusive
    // scans over the digits of the block totals and of the counts in all
    uint32_t total = 0;
    if ((int)threadIdx.x < radix) {
        const int d = threadIdx.x;
        const uint32_t c0 = s_wcnt[0][d], c1 = s_wcnt[1][d], c2 = s_wcnt[2][d], c3 = s_wcnt[3][d];
        s_wcnt[0][d] = 0;
        s_wcnt[1][d] = c0;
        s_wcnt[2][d] = c0 + c1;
        s_wcnt[3][d] = c0 + c1 + c2;
        total = c0 + c1 + c2 + c3;
    }
    // thread d holds digit d
    uint32_t incl = total, gincl = all;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64), g = __shfl_up(gincl, off, 64);
        if (lane >= off) {
            incl += y;
            gincl += g;
        }
    }
    if (lane == 63) {
        s_wsum[wave] = incl;
        s_gsum[wave] = gincl;
    }
    __syncthreads();
    uint32_t wpre = 0, gpre = 0;
    for (int w = 0; w < wave; ++w) {
        wpre += s_wsum[w];
        gpre += s_gsum[w];
    }
    if ((int)threadIdx.x < radix) {
        s_bstart[threadIdx.x] = wpre + incl - total;
        s_goff[threadIdx.x] = gpre + gincl - all + earlier;
    }
    __syncthreads();

#pragma unroll
    for (int r = 0; r < kSortIpt; ++r) {
        const uint32_t idx = base + r * 64 + lane;
        if (idx < n) {
            const uint32_t d = (key[r] >> shift) & mask;
            const uint32_t lp = s_bstart[d] + s_wcnt[wave][d] + rank[r];
            s_keys[lp] = key[r];
            s_vals[lp] = val[r];
        }
    }
    __syncthreads();
    const uint32_t count = min((uint32_t)kSortTile, n - tile0);
    for (uint32_t i = threadIdx.x; i < count; i += kSortThreads) {
        const uint32_t k = s_keys[i];
        const uint32_t d = (k >> shift) & mask;
        const uint32_t gp = s_goff[d] + (i - s_bstart[d]);
        if (gp < n) {     // always true for a consistent histogram; guards the write
            kout[gp] = k;
            vout[gp] = s_vals[i];
        }
    }
}

// ---------------------------------------------------------------- scan

constexpr int kScanThreads = 256;
constexpr int kScanIpt = 8;
constexpr int kScanTile = kScanThreads * kScanIpt;
static_assert(kScanTile == kScanTileElems, "tile sums are written by other kernels too");

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    return x;
}

// per-tile exclusive scan plus the tile's offset; items are blocked per
// thread (consecutive) so that the in-thread prefix is sequential.  The
// tile's offset is the sum of the earlier tiles' sums, which every
// workgroup adds up itself (64-bit, at most a few thousand values) rather
// than waiting for a separate one-workgroup launch.
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const uint32_t* __restrict__ in,
                                                            uint32_t* __restrict__ out, uint32_t n_max,
                                                            const uint32_t* __restrict__ n_dev,
                                                            const uint32_t* __restrict__ tsum,
                                                            uint32_t* __restrict__ chunk_first, uint32_t chunk) {
    __shared__ uint32_t s_buf[kScanTile];
    const uint32_t n = count_of(n_max, n_dev);
    if ((uint64_t)blockIdx.x * kScanTile >= n) return;
    __shared__ uint32_t s_w[4];
    __shared__ unsigned long long s_off[4];
    const uint32_t base = blockIdx.x * kScanTile;
#pragma unroll
    for (int r = 0; r < kScanIpt; ++r) {
        const uint32_t i = r * kScanThreads + threadIdx.x;
        s_buf[i] = base + i < n ? in[base + i] : 0u;
    }
    {
        unsigned long long acc = 0;
        for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kScanThreads) acc += tsum[t];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((threadIdx.x & 63) == 0) s_off[threadIdx.x >> 6] = acc;
    }
    __syncthreads();
    uint32_t v[kScanIpt];
    uint32_t acc = 0;
#pragma unroll
    for (int r = 0; r < kScanIpt; ++r) {
        v[r] = s_buf[threadIdx.x * kScanIpt + r];
        acc += v[r];
    }
    const uint32_t incl = wave_incl_scan(acc);
    if ((threadIdx.x & 63) == 63) s_w[threadIdx.x >> 6] = incl;
    __syncthreads();
    const unsigned long long tile_off = s_off[0] + s_off[1] + s_off[2] + s_off[3];
    uint32_t pre = (uint32_t)tile_off + incl - acc;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) pre += s_w[w];
#pragma unroll
    for (int r = 0; r < kScanIpt; ++r) {
        s_buf[threadIdx.x * kScanIpt + r] = pre;
        // the chunks of the counted items that start in this element's
        if (v[r])
            for (uint32_t c = first_chunk(pre, chunk); c <= (pre + v[r] - 1) / chunk; ++c)
                chunk_first[c] = base + threadIdx.x * kScanIpt + r;
        pre += v[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kScanIpt; ++r) {
        const uint32_t i = r * kScanThreads + threadIdx.x;
        if (base + i < n) out[base + i] = s_buf[i];
    }
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

}  // namespace

// the digit table and the row totals
size_t radix_hist_elems(uint32_t n) {
    // sized for the smallest tile, so that the size grows with n
    const size_t tiles = ((size_t)n + kMinSortTile - 1) / kMinSortTile;
    return ((tiles ? tiles : 1) + 1) * (size_t)(1 << kMaxRadixBits);
}

// tile sums
size_t scan_tmp_elems(uint32_t n) {
    const size_t t = ((size_t)n + kScanTile - 1) / kScanTile;
    return t ? t : 1;
}

hipError_t fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t s) {
    if (!n) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t exclusive_scan_sums_u32(const uint32_t* in, uint32_t* out, uint32_t n, const uint32_t* n_dev,
                                   const uint32_t* tile_sums, uint32_t* chunk_first, uint32_t chunk, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const uint32_t nt = (uint32_t)(((uint64_t)n + kScanTile - 1) / kScanTile);
    hipLaunchKernelGGL(k_scan_down, dim3(nt), dim3(kScanThreads), 0, s, in, out, n, n_dev, tile_sums,
                       chunk_first, chunk);
    return hipGetLastError();
}

int radix_passes(uint32_t n, int begin_bit, int end_bit) {
    return (n <= 1 || end_bit <= begin_bit) ? 0 : (end_bit - begin_bit + kMaxRadixBits - 1) / kMaxRadixBits;
}

// Sorts keys/vals on bits [begin_bit, end_bit) with passes of <= 8 bits of
// near-equal width.  The result lands in (keys, vals) or in the alternate
// buffers; *result_in_alt says which.  `hist` needs radix_hist_elems(n).
// With n_dev the key count is read on the device (at most n, which sizes
// the launches), so the sort needs no host knowledge of it: the digit
// table and its scan cover only the tiles that hold keys.  small_tiles: a
// device count expected well below n, 1024-key tiles up to four times the n.
// vals_are_positions: the input values are 0, 1, 2, ... and `vals` is not
// read (at least one pass has to run).
hipError_t radix_sort_pairs(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, uint32_t n,
                            int begin_bit, int end_bit, uint32_t* hist, hipStream_t s, bool* result_in_alt,
                            const uint32_t* n_dev, bool small_tiles, bool vals_are_positions) {
    *result_in_alt = false;
    if (radix_passes(n, begin_bit, end_bit) == 0) return hipSuccess;
    const int total_bits = end_bit - begin_bit;
    const int passes = (total_bits + kMaxRadixBits - 1) / kMaxRadixBits;
    const bool small = n <= (small_tiles ? 4 * kSmallSortMax : kSmallSortMax);
    const uint32_t sort_tile = (uint32_t)kSortThreads * (small ? 4u : 8u);
    const uint32_t tiles = (uint32_t)(((uint64_t)n + sort_tile - 1) / sort_tile);
    const bool few = tiles <= kFewTiles;      // then small as well
    uint32_t* row_total = hist + (size_t)tiles * (1 << kMaxRadixBits);
    uint32_t *ki = keys, *vi = vals, *ko = keys_alt, *vo = vals_alt;
    bool iota = vals_are_positions;
    auto rowscan = [&](int bits) {
        hipLaunchKernelGGL(k_radix_rowscan, dim3(1u << bits), dim3(kRowThreads), 0, s, hist, n, n_dev, sort_tile,
                           row_total);
    };
    int shift = begin_bit;
    for (int p = 0; p < passes; ++p) {
        const int remaining = end_bit - shift;
        const int bits = (remaining + (passes - p) - 1) / (passes - p);
        const dim3 grid(tiles), wg(kSortThreads);
        const uint32_t* v = iota ? nullptr : vi;
        if (few) {
            hipLaunchKernelGGL((k_radix_upsweep<4, true>), grid, wg, 0, s, ki, n, n_dev, shift, bits, hist);
            hipLaunchKernelGGL((k_radix_downsweep<4, true>), grid, wg, 0, s, ki, v, ko, vo, n, n_dev, shift, bits,
                               hist, row_total);
        } else if (small) {
            hipLaunchKernelGGL((k_radix_upsweep<4, false>), grid, wg, 0, s, ki, n, n_dev, shift, bits, hist);
            rowscan(bits);
            hipLaunchKernelGGL((k_radix_downsweep<4, false>), grid, wg, 0, s, ki, v, ko, vo, n, n_dev, shift, bits,
                               hist, row_total);
        } else {
            hipLaunchKernelGGL((k_radix_upsweep<8, false>), grid, wg, 0, s, ki, n, n_dev, shift, bits, hist);
            rowscan(bits);
            hipLaunchKernelGGL((k_radix_downsweep<8, false>), grid, wg, 0, s, ki, v, ko, vo, n, n_dev, shift, bits,
                               hist, row_total);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        iota = false;
        shift += bits;
        uint32_t* t;
        t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
        *result_in_alt = !*result_in_alt;
    }
    return hipSuccess;
}

}  // namespace gs
