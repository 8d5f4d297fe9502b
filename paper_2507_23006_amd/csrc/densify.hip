// Densification bookkeeping and the 3D smoothing filter -- gfx950.
//
// Consumers of the backward's per-view statistics between training steps:
//   accumulate  per Gaussian, the views that rasterized it add their
//               |dL/d mean2d| (or the AbsGS per-axis absolute sums' length)
//               times a per-view scale to a running sum, and count;
//   classify    mean = sum / count against the in-partition threshold of
//               Eq. 4, tau_i = tau_min (min(d_i, d_max) / d_max (eta - 1) + 1)
//               with d_i the distance to the partition box; pruning by an
//               opacity floor; a sort key of mean / tau_i for the budget cap;
//   mark        the first K candidates of the key order are cloned or split
//               (by their largest scale);
//   filter      Mip-Splatting's 3D smoothing filter: the sampling rate
//               max f_x / depth over the cameras that hold the mean, and
//               scales sqrt(s^2 + (s_f / rate)^2) with the opacity scaled by
//               prod s / s' (forward and backward).
// Streams over structure-of-arrays rows, HBM-bound but for the sampling rate.
// Decisions compare FP64 values formed from the float32 inputs (the mean is
// a float32 division, as stored).
#include "gs_internal.h"

namespace gs {

namespace {

constexpr int kDT = 256;

__global__ __launch_bounds__(kDT) void k_dens_accumulate(const uint32_t* __restrict__ tiles,
                                                         const float* __restrict__ grad_norm,
                                                         const float2* __restrict__ absgrad, int32_t n_views,
                                                         int64_t n, DensViewScale sc, float* __restrict__ accum,
                                                         int32_t* __restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * kDT + threadIdx.x;
    if (i >= n) return;
    float a = accum[i];
    int32_t c = count[i];
    for (int v = 0; v < n_views; ++v) {
        const int64_t slot = (int64_t)v * n + i;
        if (!tiles[slot]) continue;
        float val;
        if (absgrad) {
            const float2 g = absgrad[slot];
            val = sqrtf(g.x * g.x + g.y * g.y);
        } else {
            val = grad_norm[slot];
        }
        a += val * sc.s[v];
        c += 1;
    }
    accum[i] = a;
    count[i] = c;
}

__device__ __forceinline__ double box_dist(double x, double lo, double hi) {
    return fmax(fmax(lo - x, x - hi), 0.0);
}

// The budgeted selection works on blocks of kDensBlock consecutive Gaussians,
// whose candidates lie packed in index order in the block's part of (key,
// index).  The `grown` largest scores are found by three histograms over the
// key's bits instead of a sort: the counts of one narrow the key's prefix for
// the next.  6M Gaussians: 73 us, where flags and positions of every Gaussian, two
// scans over them and twelve sorting launches took 182.
constexpr int kDensBlock = 4 * kDT;
constexpr int kSelBins = 2048;               // 11 + 11 + 10 bits
constexpr int kSelGrid = 512;

// exclusive sum over the workgroup's threads; *total = all (s: one word a wave)
template <class T>
__device__ __forceinline__ T block_scan(T x, T* s, T* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    T incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    __syncthreads();
    if (lane == 63) s[wave] = incl;
    __syncthreads();
    T base = 0, all = 0;
    for (int w = 0; w < waves; ++w) {
        if (w < wave) base += s[w];
        all += s[w];
    }
    *total = all;
    return base + incl - x;
}

// action: PRUNE or KEEP; candidates with key = ~bits(mean / tau) (ascending keys
// = descending scores) packed in the block's part; their number and that of
// pruned Gaussians in count[block]
__global__ __launch_bounds__(kDT) void k_dens_classify(const float* __restrict__ accum,
                                                       const int32_t* __restrict__ count,
                                                       const float* __restrict__ means,
                                                       const float* __restrict__ opac, int64_t n, DensParams p,
                                                       uint8_t* __restrict__ action, uint2* __restrict__ cand,
                                                       uint2* __restrict__ counts) {
    __shared__ uint32_t s_cand[4][4], s_pruned[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * kDensBlock + threadIdx.x;
    float a[4], x[4], y[4], z[4], o[4];
    int32_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = i0 + k * kDT < n ? i0 + k * kDT : n - 1;      // (no branch between the loads)
        a[k] = accum[i];
        c[k] = count[i];
        x[k] = means[i];
        y[k] = means[n + i];
        z[k] = means[2 * n + i];
        o[k] = opac[i];
    }
    uint32_t key[4], below[4], pruned = 0;
    bool cd[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool in = i0 + k * kDT < n;
        const float mean = c[k] > 0 ? a[k] / (float)c[k] : 0.0f;
        const double dx = box_dist(x[k], p.box_min[0], p.box_max[0]);
        const double dy = box_dist(y[k], p.box_min[1], p.box_max[1]);
        const double dz = box_dist(z[k], p.box_min[2], p.box_max[2]);
        const double d = sqrt(dx * dx + dy * dy + dz * dz);
        const double tau = (double)p.tau_min * (fmin(d, (double)p.d_max) / (double)p.d_max * ((double)p.eta - 1.0) + 1.0);
        const bool pr = in && o[k] < p.prune_opacity;
        cd[k] = in && !pr && (double)mean > tau;
        key[k] = cd[k] ? ~__float_as_uint((float)((double)mean / tau)) : 0u;
        if (in) action[i0 + k * kDT] = pr ? (uint8_t)GS_DENSIFY_PRUNE : (uint8_t)GS_DENSIFY_KEEP;
        const uint64_t m = __ballot(cd[k]);
        below[k] = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        pruned += (uint32_t)__popcll(__ballot(pr));
        if (lane == 0) s_cand[k][wave] = (uint32_t)__popcll(m);
    }
    if (lane == 0) s_pruned[wave] = pruned;
    __syncthreads();
    uint32_t at = 0;      // candidates of the block before this wave's k-th Gaussians
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w == wave && cd[k]) cand[(int64_t)blockIdx.x * kDensBlock + at + below[k]] = make_uint2(key[k], (uint32_t)(i0 + k * kDT));
            at += s_cand[k][w];
        }
    if (threadIdx.x == 0) counts[blockIdx.x] = make_uint2(at, s_pruned[0] + s_pruned[1] + s_pruned[2] + s_pruned[3]);
}

// totals of the blocks' counts to the host's total[2], and zeroed histograms
__global__ __launch_bounds__(1024) void k_dens_totals(const uint2* __restrict__ counts, uint32_t blocks,
                                                      uint32_t* __restrict__ hist, unsigned long long* __restrict__ total) {
    __shared__ unsigned long long s[16];
    unsigned long long a = 0, b = 0, all;
    for (uint32_t i = threadIdx.x; i < blocks; i += 1024) {
        const uint2 c = counts[i];
        a += c.x;
        b += c.y;
    }
    for (uint32_t i = threadIdx.x; i < 3 * kSelBins; i += 1024) hist[i] = 0u;
    block_scan(a, s, &all);
    if (threadIdx.x == 0) total[0] = all;
    block_scan(b, s, &all);
    if (threadIdx.x == 0) total[1] = all;
}

// Selection state after the histograms 0 .. P - 1: the key's leading bits, and
// how many of the keys that share them are still to take
struct DensSel {
    uint32_t prefix, take, ties;      // ties: keys that share the whole prefix (P = 3)
};

// bin of histogram h (of `bins`) that the take-th smallest entry falls in, by the
// whole workgroup of kDT threads; *before = entries of the bins below it
__device__ __forceinline__ uint32_t find_bin(const uint32_t* __restrict__ h, uint32_t take, uint32_t* s, uint32_t* before,
                                             uint32_t* in_bin) {
    __shared__ uint32_t s_bin[3];
    constexpr int kPer = kSelBins / kDT;
    uint32_t c[kPer], sum = 0, all;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        c[k] = h[threadIdx.x * kPer + k];
        sum += c[k];
    }
    uint32_t base = block_scan(sum, s, &all);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (base < take && take <= base + c[k]) {
            s_bin[0] = threadIdx.x * kPer + k;
            s_bin[1] = base;
            s_bin[2] = c[k];
        }
        base += c[k];
    }
    __syncthreads();
    *before = s_bin[1];
    *in_bin = s_bin[2];
    return s_bin[0];
}

// the state after histogram P - 1 (every workgroup computes it from the state
// before; workgroup 0 keeps it for the next kernel)
template <int P>
__device__ __forceinline__ DensSel advance(const uint32_t* __restrict__ hist, DensSel* __restrict__ sel, uint32_t take0,
                                           uint32_t* s) {
    DensSel st{0u, take0, 0u};
    if (P > 1) st = sel[P - 2];
    if (P > 0) {
        uint32_t before, in_bin;
        const uint32_t bin = find_bin(hist + (P - 1) * kSelBins, st.take, s, &before, &in_bin);
        st.prefix = st.prefix << (P == 3 ? 10 : 11) | bin;
        st.take -= before;
        st.ties = in_bin;
        if (blockIdx.x == 0 && threadIdx.x == 0) sel[P - 1] = st;
    }
    return st;
}

// histogram P of the candidates that share the prefix found so far, a wave per block
template <int P>
__global__ __launch_bounds__(kDT) void k_dens_hist(const uint2* __restrict__ cand, const uint2* __restrict__ counts,
                                                   uint32_t blocks, uint32_t take0, uint32_t* __restrict__ hist,
                                                   DensSel* __restrict__ sel) {
    __shared__ uint32_t s_hist[kSelBins], s_scan[4];
    const DensSel st = advance<P>(hist, sel, take0, s_scan);
    for (int i = threadIdx.x; i < kSelBins; i += kDT) s_hist[i] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (uint32_t b = blockIdx.x * 4 + (threadIdx.x >> 6); b < blocks; b += gridDim.x * 4) {
        const uint32_t m = counts[b].x;
        for (uint32_t j = lane; j < m; j += 64) {
            const uint32_t key = cand[(int64_t)b * kDensBlock + j].x;
            if (P == 0) atomicAdd(&s_hist[key >> 21], 1u);
            if (P == 1 && key >> 21 == st.prefix) atomicAdd(&s_hist[(key >> 10) & 2047u], 1u);
            if (P == 2 && key >> 10 == st.prefix) atomicAdd(&s_hist[key & 1023u], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kDT)
        if (s_hist[i]) atomicAdd(&hist[P * kSelBins + i], s_hist[i]);
}

// keys equal to the last one taken, by block (nothing to do when all are taken)
__global__ __launch_bounds__(kDT) void k_dens_ties(const uint2* __restrict__ cand, const uint2* __restrict__ counts,
                                                   uint32_t blocks, const uint32_t* __restrict__ hist,
                                                   DensSel* __restrict__ sel, uint32_t* __restrict__ ties) {
    __shared__ uint32_t s_scan[4];
    const DensSel st = advance<3>(hist, sel, 0u, s_scan);
    if (st.take == st.ties) return;
    const int lane = threadIdx.x & 63;
    for (uint32_t b = blockIdx.x * 4 + (threadIdx.x >> 6); b < blocks; b += gridDim.x * 4) {
        const uint32_t m = counts[b].x;
        uint32_t c = 0;
        for (uint32_t j = 0; j < m; j += 64)
            c += (uint32_t)__popcll(__ballot(j + lane < m && cand[(int64_t)b * kDensBlock + j + lane].x == st.prefix));
        if (lane == 0) ties[b] = c;
    }
}

// ties before each block
__global__ __launch_bounds__(1024) void k_dens_tie_scan(uint32_t blocks, const DensSel* __restrict__ sel,
                                                        uint32_t* __restrict__ ties) {
    __shared__ uint32_t s[16];
    if (sel[2].take == sel[2].ties) return;
    uint32_t base = 0, all;
    for (uint32_t i0 = 0; i0 < blocks; i0 += 1024) {
        const uint32_t i = i0 + threadIdx.x, x = i < blocks ? ties[i] : 0u;
        const uint32_t at = block_scan(x, s, &all);
        if (i < blocks) ties[i] = base + at;
        base += all;
    }
}

__device__ __forceinline__ uint8_t grow_kind(const float* __restrict__ scales, int64_t n, int64_t i, float thr) {
    const float m = fmaxf(scales[i], fmaxf(scales[n + i], scales[2 * n + i]));
    return m > thr ? (uint8_t)GS_DENSIFY_SPLIT : (uint8_t)GS_DENSIFY_CLONE;
}

// the selected candidates grow: all of them (sel null), or those with smaller keys
// than the last one taken and the first of its equals in index order; a wave per
// block
__global__ __launch_bounds__(kDT) void k_dens_mark(const uint2* __restrict__ cand, const uint2* __restrict__ counts,
                                                   uint32_t blocks, const DensSel* __restrict__ sel,
                                                   const uint32_t* __restrict__ ties, const float* __restrict__ scales,
                                                   int64_t n, float thr, uint8_t* __restrict__ action) {
    const uint32_t b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= blocks) return;
    const int lane = threadIdx.x & 63;
    const uint32_t m = counts[b].x;
    DensSel st{0xFFFFFFFFu, 0u, 0u};
    uint32_t tie = 0;      // ties before this one
    if (sel) {
        st = sel[2];
        tie = st.take == st.ties ? 0u : ties[b];
    }
    const bool every = !sel || st.take == st.ties;
    for (uint32_t j = 0; j < m; j += 64) {
        const bool on = j + lane < m;
        const uint2 c = on ? cand[(int64_t)b * kDensBlock + j + lane] : make_uint2(0u, 0u);
        const uint64_t eq = __ballot(on && c.x == st.prefix);
        const uint32_t before = tie + __builtin_amdgcn_mbcnt_hi((uint32_t)(eq >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eq, 0));
        if (on && (c.x < st.prefix || (c.x == st.prefix && (every || before < st.take))))
            action[c.y] = grow_kind(scales, n, c.y, thr);
        tie += (uint32_t)__popcll(eq);
    }
}

// rate = max(rate if `accumulate`, max over the table's views holding the mean of fx / depth).
// Bound by FP64 issue, so the camera's constants arrive as doubles (converting
// them took as many instructions as the transform), a view is two distances
// |x - c z| <= h z, and the maximum is the smallest z / fx, inverted once at the
// end.  Four means a thread cover the latency of the FP64 chain.  6M means, 40
// cameras: 195 us, 411 with three launches of up to 16 views and a division each.
constexpr int kRatePer = 4;
__global__ __launch_bounds__(kDT) void k_filter_rate(const float* __restrict__ means, int64_t n, RateTable tab,
                                                     int accumulate, float* __restrict__ rate) {
    const int64_t i0 = (int64_t)blockIdx.x * (kDT * kRatePer) + threadIdx.x;
    double m[kRatePer][3], best[kRatePer];
#pragma unroll
    for (int j = 0; j < kRatePer; ++j) {
        const int64_t i = i0 + j * kDT < n ? i0 + j * kDT : n - 1;      // (no branch between the loads)
#pragma unroll
        for (int c = 0; c < 3; ++c) m[j][c] = (double)means[c * n + i];
        best[j] = __builtin_huge_val();
    }
    for (int v = 0; v < tab.n_cams; ++v) {
        const RateCam& C = tab.c[v];
#pragma unroll
        for (int j = 0; j < kRatePer; ++j) {
            const double x = fma(C.R[2], m[j][2], fma(C.R[1], m[j][1], C.R[0] * m[j][0])) + C.t[0];
            const double y = fma(C.R[5], m[j][2], fma(C.R[4], m[j][1], C.R[3] * m[j][0])) + C.t[1];
            const double z = fma(C.R[8], m[j][2], fma(C.R[7], m[j][1], C.R[6] * m[j][0])) + C.t[2];
            const double ex = fma(C.hu, z, -fabs(fma(-C.cu, z, x))), ey = fma(C.hv, z, -fabs(fma(-C.cv, z, y)));
            const double s = z * C.ifx;
            if (s < best[j] && z >= C.znear && z <= C.zfar && ex >= 0.0 && ey >= 0.0) best[j] = s;
        }
    }
#pragma unroll
    for (int j = 0; j < kRatePer; ++j) {
        const int64_t i = i0 + j * kDT;
        if (i >= n) continue;
        const float r = (float)(1.0 / best[j]);      // 0 where no camera holds the mean
        rate[i] = accumulate ? fmaxf(rate[i], r) : r;
    }
}

// filter variance (s_f / rate)^2, 0 for an unseen Gaussian
__device__ __forceinline__ double filter_var(float rate, float s_f) {
    if (!(rate > 0.0f)) return 0.0;
    const double q = (double)s_f / (double)rate;
    return q * q;
}

__global__ __launch_bounds__(kDT) void k_filter_fwd(const float* __restrict__ scales, const float* __restrict__ opac,
                                                    const float* __restrict__ rate, int64_t n, float s_f,
                                                    float* __restrict__ scales_out, float* __restrict__ opac_out) {
    const int64_t i = (int64_t)blockIdx.x * kDT + threadIdx.x;
    if (i >= n) return;
    const double var = filter_var(rate[i], s_f);
    double comp = 1.0;
    for (int k = 0; k < 3; ++k) {
        const double s = scales[k * n + i];
        const double s2 = sqrt(s * s + var);
        scales_out[k * n + i] = (float)s2;
        comp *= s / s2;
    }
    opac_out[i] = (float)((double)opac[i] * comp);
}

__global__ __launch_bounds__(kDT) void k_filter_bwd(const float* __restrict__ scales, const float* __restrict__ opac,
                                                    const float* __restrict__ rate, int64_t n, float s_f,
                                                    const float* __restrict__ d_scales_out,
                                                    const float* __restrict__ d_opac_out,
                                                    float* __restrict__ d_scales, float* __restrict__ d_opac) {
    const int64_t i = (int64_t)blockIdx.x * kDT + threadIdx.x;
    if (i >= n) return;
    const double var = filter_var(rate[i], s_f);
    double s[3], s2[3], comp = 1.0;
    for (int k = 0; k < 3; ++k) {
        s[k] = scales[k * n + i];
        s2[k] = sqrt(s[k] * s[k] + var);
        comp *= s[k] / s2[k];
    }
    const double dop = d_opac_out[i];
    const double o2 = (double)opac[i] * comp;
    for (int k = 0; k < 3; ++k) {
        // s' = sqrt(s^2 + var); d log(s / s') / ds = var / (s s'^2)
        const double g = (double)d_scales_out[k * n + i] * s[k] / s2[k] + dop * o2 * var / (s[k] * s2[k] * s2[k]);
        d_scales[k * n + i] = (float)g;
    }
    d_opac[i] = (float)(dop * comp);
}

unsigned blocks_of(int64_t n) { return (unsigned)((n + kDT - 1) / kDT); }

}  // namespace

hipError_t launch_dens_accumulate(const uint32_t* tiles, const float* grad_norm, const float* absgrad,
                                  int32_t n_views, int64_t n, const DensViewScale& sc, float* accum, int32_t* count,
                                  hipStream_t s) {
    hipLaunchKernelGGL(k_dens_accumulate, dim3(blocks_of(n)), dim3(kDT), 0, s, tiles, grad_norm,
                       reinterpret_cast<const float2*>(absgrad), n_views, n, sc, accum, count);
    return hipGetLastError();
}

uint32_t dens_blocks(int64_t n) { return (uint32_t)((n + kDensBlock - 1) / kDensBlock); }
size_t dens_cand_elems(int64_t n) { return (size_t)dens_blocks(n) * kDensBlock; }
size_t dens_hist_elems() { return 3 * kSelBins; }
size_t dens_sel_bytes() { return 3 * sizeof(DensSel); }

hipError_t launch_dens_classify(const float* accum, const int32_t* count, const float* means, const float* opac,
                                int64_t n, const DensParams& p, uint8_t* action, const DensSelect& w,
                                unsigned long long* total, hipStream_t s) {
    const uint32_t blocks = dens_blocks(n);
    hipLaunchKernelGGL(k_dens_classify, dim3(blocks), dim3(kDT), 0, s, accum, count, means, opac, n, p, action, w.cand,
                       w.counts);
    hipLaunchKernelGGL(k_dens_totals, dim3(1), dim3(1024), 0, s, w.counts, blocks, w.hist, total);
    return hipGetLastError();
}

hipError_t launch_dens_grow(const DensSelect& w, uint32_t grown, bool all, const float* scales, int64_t n,
                            float split_scale, uint8_t* action, hipStream_t s) {
    const uint32_t blocks = dens_blocks(n), per_wave = (blocks + 3) / 4;
    const dim3 grid(per_wave < (uint32_t)kSelGrid ? per_wave : (uint32_t)kSelGrid), dim(kDT);
    DensSel* sel = all ? nullptr : static_cast<DensSel*>(w.sel);
    if (!all) {
        hipLaunchKernelGGL(k_dens_hist<0>, grid, dim, 0, s, w.cand, w.counts, blocks, grown, w.hist, sel);
        hipLaunchKernelGGL(k_dens_hist<1>, grid, dim, 0, s, w.cand, w.counts, blocks, grown, w.hist, sel);
        hipLaunchKernelGGL(k_dens_hist<2>, grid, dim, 0, s, w.cand, w.counts, blocks, grown, w.hist, sel);
        hipLaunchKernelGGL(k_dens_ties, grid, dim, 0, s, w.cand, w.counts, blocks, w.hist, sel, w.ties);
        hipLaunchKernelGGL(k_dens_tie_scan, dim3(1), dim3(1024), 0, s, blocks, sel, w.ties);
    }
    hipLaunchKernelGGL(k_dens_mark, dim3(per_wave), dim, 0, s, w.cand, w.counts, blocks, sel, w.ties, scales, n,
                       split_scale, action);
    return hipGetLastError();
}

hipError_t launch_filter_rate(const float* means, int64_t n, const RateTable& tab, bool accumulate, float* rate,
                              hipStream_t s) {
    const int64_t per = kDT * kRatePer;
    hipLaunchKernelGGL(k_filter_rate, dim3((unsigned)((n + per - 1) / per)), dim3(kDT), 0, s, means, n, tab,
                       accumulate ? 1 : 0, rate);
    return hipGetLastError();
}

hipError_t launch_filter_fwd(const float* scales, const float* opac, const float* rate, int64_t n, float s_f,
                             float* scales_out, float* opac_out, hipStream_t s) {
    hipLaunchKernelGGL(k_filter_fwd, dim3(blocks_of(n)), dim3(kDT), 0, s, scales, opac, rate, n, s_f, scales_out,
                       opac_out);
    return hipGetLastError();
}

hipError_t launch_filter_bwd(const float* scales, const float* opac, const float* rate, int64_t n, float s_f,
                             const float* d_scales_out, const float* d_opac_out, float* d_scales, float* d_opac,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_filter_bwd, dim3(blocks_of(n)), dim3(kDT), 0, s, scales, opac, rate, n, s_f, d_scales_out,
                       d_opac_out, d_scales, d_opac);
    return hipGetLastError();
}

}  // namespace gs
