// D-SSIM term of the training loss (Eq. 3) and its gradient -- gfx950.
//
// SSIM per pixel and channel with an 11x11 Gaussian window (sigma 1.5,
// weights normalised to 1), zero outside the image, C1 = 0.01^2,
// C2 = 0.03^2:  s = (2 mx my + C1)(2 sxy + C2) / ((mx^2 + my^2 + C1)(sx^2 +
// sy^2 + C2)) with mx = G*x, sx^2 = G*(x^2) - mx^2, sxy = G*(xy) - mx my.
// The term is weight * (1 - mean s) over 3 W H values.
//
// An image row is 3 W floats, in which a pixel's horizontal neighbours of the
// same channel lie 3 apart and its vertical ones a row apart, so the blur needs
// no channels.  One wave owns 64 neighbouring floats of a strip of rows: it
// walks down the strip, stages each row with its halo of 15 floats in LDS,
// blurs it horizontally, and adds the result with each of the 11 weights to the
// sums of the 11 output rows it belongs to, which live in registers (the loop
// over rows is unrolled by 11, so each sum keeps its registers).  Nothing but
// the row of inputs passes through LDS and no other wave is waited for.
// Forward: blurs x, y, x^2, y^2, xy and writes s's partial derivatives with
// respect to a = G*x, b = G*(x^2), c = G*(xy) for the backward, plus the wave's
// sum of s.  Backward: the blur is self-adjoint (symmetric window, zero padding),
// so dL/dx = -weight / (3 W H) (G*Pa + 2 x G*Pb + y G*Pc), three more blurs.
// 1920x1080: 48 and 34 us, bound by FP32 issue (forward, 200 instructions a float)
// and HBM (backward, 150 MB); with 16x16 tiles, whose halos and blurred rows all
// passed through LDS, 71 and 65.
#include <type_traits>
#include <utility>

#include "gs_internal.h"
#include "rows.h"

namespace gs {

namespace {

constexpr int kR = 5;                     // window radius
constexpr int kWin = 2 * kR + 1;          // 11 taps
constexpr int kHaloF = 3 * kR;            // halo in floats
constexpr int kRowF = 64 + 2 * kHaloF;    // staged floats of a row
constexpr float kC1 = 0.01f * 0.01f, kC2 = 0.03f * 0.03f;

struct SsimWin {
    float w[kWin];
};

// normalised Gaussian taps exp(-k^2 / (2 sigma^2)), sigma = 1.5 (host side)
SsimWin ssim_window() {
    SsimWin t;
    double s = 0.0, v[kWin];
    for (int k = 0; k < kWin; ++k) {
        const double d = k - kR;
        v[k] = exp(-d * d / (2.0 * 1.5 * 1.5));
        s += v[k];
    }
    for (int k = 0; k < kWin; ++k) t.w[k] = (float)(v[k] / s);
    return t;
}

// the window's distinct weights, in vector registers (a scalar operand halves the
// rate of an FMA)
struct SsimTaps {
    float w[kR + 1];
    __device__ explicit SsimTaps(const SsimWin& win) {
#pragma unroll
        for (int k = 0; k <= kR; ++k) {
            w[k] = win.w[k];
            asm volatile("" : "+v"(w[k]));
        }
    }
    __device__ float operator[](int k) const { return w[k <= kR ? k : kWin - 1 - k]; }
};

// the floats of a row that a lane stages: j0 - kHaloF + lane and, of the first
// lanes, the one 64 further; outside the image the nearest one is read and
// replaced by 0, so that no branch parts the loads
struct RowLane {
    int64_t W3;
    int H;
    uint32_t ja, jb;
    bool a, b;
    __device__ RowLane(int W, int H_, int64_t j0, int lane) : W3(3 * (int64_t)W), H(H_) {
        const int64_t p = j0 - kHaloF + lane, q = p + 64;
        a = p >= 0 && p < W3;
        b = lane < 2 * kHaloF && q < W3;
        ja = (uint32_t)(p < 0 ? 0 : p < W3 ? p : W3 - 1);
        jb = (uint32_t)(q < W3 ? q : W3 - 1);
    }
};

// row `row` of N images, 0 outside
template <int N>
__device__ __forceinline__ void row_load(const float* const (&img)[N], const RowLane& l, int row, float (&v)[N][2]) {
    const int r = row < 0 ? 0 : row < l.H ? row : l.H - 1;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float* p = img[i] + r * l.W3;
        v[i][0] = p[l.ja];
        v[i][1] = p[l.jb];
    }
}

template <int N>
__device__ __forceinline__ void row_stage(const float (&v)[N][2], const RowLane& l, int row, int lane, float (&s)[N][kRowF]) {
    const bool in = row >= 0 && row < l.H;
    wave_sync();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        s[i][lane] = in && l.a ? v[i][0] : 0.0f;
        if (lane < 2 * kHaloF) s[i][64 + lane] = in && l.b ? v[i][1] : 0.0f;
    }
    wave_sync();
}

// adds row u's blurred values to the sums of the 11 output rows they belong to;
// the row that began 10 rows ago is complete in acc[(u + 1) % kWin]
template <int U, int Q>
__device__ __forceinline__ void column_add(const SsimTaps& w, const float (&h)[Q], float (&acc)[kWin][Q]) {
#pragma unroll
    for (int k = 0; k < kWin; ++k) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float& a = acc[(U - k + kWin) % kWin][q];
            a = k == 0 ? w[0] * h[q] : fmaf(w[k], h[q], a);
        }
    }
}

// A wave's columns and strip.  The card deals workgroups to its XCDs in turn, each
// with an L2 of its own; every XCD gets a run of neighbouring pieces, whose halos
// are then read once (dealt in turn, the halos' lines made the backward fetch 326
// MB for an image of which 125 MB are read).  Four waves a workgroup, one for each
// SIMD of a compute unit, though none waits for another.
constexpr int kXcds = 8, kWaves = 4;

__device__ __forceinline__ bool wave_piece(int columns, int strips, int& column, int& strip) {
    const int per_xcd = (int)(gridDim.x / kXcds);
    const int piece = ((int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds)) * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    strip = piece / columns;
    column = piece - strip * columns;
    return strip < strips;
}

// calls f<0> ... f<10>
template <class F, int... U>
__device__ __forceinline__ void eleven(F&& f, std::integer_sequence<int, U...>) {
    (f(std::integral_constant<int, U>{}), ...);
}

__global__ __launch_bounds__(64 * kWaves) void k_ssim_fwd(const float* __restrict__ x, const float* __restrict__ y, int W, int H,
                                                 int strip, int strips, SsimWin win, float* __restrict__ Pa, float* __restrict__ Pb,
                                                 float* __restrict__ Pc, double* __restrict__ partial) {
    __shared__ float s_all[kWaves][2][kRowF];
    const int lane = threadIdx.x & 63;
    const int64_t W3 = 3 * (int64_t)W;
    int column, row_strip;
    if (!wave_piece((int)((W3 + 63) / 64), strips, column, row_strip)) return;
    float(&s)[2][kRowF] = s_all[threadIdx.x >> 6];
    const int64_t j0 = (int64_t)column * 64, j = j0 + lane;
    const int r0 = row_strip * strip, rows = H - r0 < strip ? H - r0 : strip;
    const SsimTaps w(win);
    const float* const img[2] = {x, y};
    float acc[kWin][5] = {}, next[2][2], after[2][2];
    double sum = 0.0;
    const RowLane rl(W, H, j0, lane);
    row_load<2>(img, rl, r0 - kR, next);
    row_load<2>(img, rl, r0 - kR + 1, after);
    for (int t0 = 0; t0 < rows + 2 * kR; t0 += kWin) {
        eleven([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            const int t = t0 + u;
            if (t >= rows + 2 * kR) return;
            row_stage<2>(next, rl, r0 - kR + t, lane, s);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                next[i][0] = after[i][0];
                next[i][1] = after[i][1];
            }
            row_load<2>(img, rl, r0 - kR + t + 2, after);
            float h[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kWin; ++k) {
                const float xv = s[0][lane + 3 * k], yv = s[1][lane + 3 * k];
                h[0] = fmaf(w[k], xv, h[0]);
                h[1] = fmaf(w[k], yv, h[1]);
                h[2] = fmaf(w[k], xv * xv, h[2]);
                h[3] = fmaf(w[k], yv * yv, h[3]);
                h[4] = fmaf(w[k], xv * yv, h[4]);
            }
            column_add<u, 5>(w, h, acc);
            if (t >= 2 * kR && j < W3) {
                const float(&m)[5] = acc[(u + 1) % kWin];
                const float mx = m[0], my = m[1];
                const float vx = m[2] - mx * mx, vy = m[3] - my * my, cxy = m[4] - mx * my;
                const float A1 = 2.0f * mx * my + kC1, A2 = 2.0f * cxy + kC2;
                const float B1 = mx * mx + my * my + kC1, B2 = vx + vy + kC2;
                const float inv = 1.0f / (B1 * B2);
                const float sv = A1 * A2 * inv;
                const int64_t o = (r0 + t - 2 * kR) * W3 + j;
                Pa[o] = (2.0f * my * (A2 - A1) - sv * 2.0f * mx * (B2 - B1)) * inv;   // ds/d(G*x)
                Pb[o] = -sv / B2;                                                      // ds/d(G*x^2)
                Pc[o] = 2.0f * A1 * inv;                                               // ds/d(G*xy)
                sum += sv;
            }
        }, std::make_integer_sequence<int, kWin>{});
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == 0) partial[(size_t)row_strip * ((W3 + 63) / 64) + column] = sum;
}

__global__ __launch_bounds__(1024) void k_ssim_total(const double* __restrict__ partial, int n, double scale,
                                                     float weight, float* __restrict__ loss) {
    __shared__ double s_sum[16];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) acc += partial[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
        for (int w = 0; w < 16; ++w) b += s_sum[w];
        loss[0] = (float)((double)weight * (1.0 - b * scale));
    }
}

__global__ __launch_bounds__(64 * kWaves) void k_ssim_bwd(const float* __restrict__ x, const float* __restrict__ y, int W, int H,
                                                 int strip, int strips, SsimWin win, const float* __restrict__ Pa,
                                                 const float* __restrict__ Pb, const float* __restrict__ Pc,
                                                 float gscale, float* __restrict__ dx) {
    __shared__ float s_all[kWaves][3][kRowF];
    const int lane = threadIdx.x & 63;
    const int64_t W3 = 3 * (int64_t)W;
    int column, row_strip;
    if (!wave_piece((int)((W3 + 63) / 64), strips, column, row_strip)) return;
    float(&s)[3][kRowF] = s_all[threadIdx.x >> 6];
    const int64_t j0 = (int64_t)column * 64, j = j0 + lane;
    const int r0 = row_strip * strip, rows = H - r0 < strip ? H - r0 : strip;
    const SsimTaps w(win);
    const float* const img[3] = {Pa, Pb, Pc};
    float acc[kWin][3] = {}, next[3][2], after[3][2];
    const RowLane rl(W, H, j0, lane);
    row_load<3>(img, rl, r0 - kR, next);
    row_load<3>(img, rl, r0 - kR + 1, after);
    for (int t0 = 0; t0 < rows + 2 * kR; t0 += kWin) {
        eleven([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            const int t = t0 + u;
            if (t >= rows + 2 * kR) return;
            const int64_t o = (r0 + t - 2 * kR) * W3 + j;
            const bool out = t >= 2 * kR && j < W3;
            const int64_t oc = (r0 + (t >= 2 * kR ? t - 2 * kR : 0)) * W3 + (j < W3 ? j : W3 - 1);
            const float xv = x[oc], yv = y[oc];
            row_stage<3>(next, rl, r0 - kR + t, lane, s);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                next[i][0] = after[i][0];
                next[i][1] = after[i][1];
            }
            row_load<3>(img, rl, r0 - kR + t + 2, after);
            float h[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kWin; ++k) {
#pragma unroll
                for (int q = 0; q < 3; ++q) h[q] = fmaf(w[k], s[q][lane + 3 * k], h[q]);
            }
            column_add<u, 3>(w, h, acc);
            const float(&g)[3] = acc[(u + 1) % kWin];
            if (out) dx[o] = gscale * (g[0] + 2.0f * xv * g[1] + yv * g[2]);
        }, std::make_integer_sequence<int, kWin>{});
    }
}

}  // namespace

// Rows of a strip: as many as leave the card four waves per SIMD (4096); with 2048,
// 3072 and 5120 waves 1920x1080 takes 89, 82 and 86 us, with 4096 82.  A strip of n
// rows blurs n + 10, so not fewer than 8.
static int ssim_strip(int W, int H) {
    const int64_t columns = (3 * (int64_t)W + 63) / 64, strips = 4096 / columns;
    const int64_t rows = strips > 1 ? (H + strips - 1) / strips : H;
    return (int)(rows < 8 ? 8 : rows);
}

size_t ssim_partials(int W, int H) {
    const int strip = ssim_strip(W, H);
    return (size_t)((3 * (int64_t)W + 63) / 64) * ((H + strip - 1) / strip);
}

hipError_t launch_dssim(const float* x, const float* y, int W, int H, float weight, float* loss, float* dx, float* Pa,
                        float* Pb, float* Pc, double* partial, hipStream_t s) {
    const SsimWin win = ssim_window();
    const int strip = ssim_strip(W, H);
    const int strips = (H + strip - 1) / strip;
    const size_t per = (size_t)kWaves * kXcds;
    const dim3 grid((unsigned)((ssim_partials(W, H) + per - 1) / per * kXcds)), dim(64 * kWaves);
    hipLaunchKernelGGL(k_ssim_fwd, grid, dim, 0, s, x, y, W, H, strip, strips, win, Pa, Pb, Pc, partial);
    const double n = 3.0 * (double)W * (double)H;
    hipLaunchKernelGGL(k_ssim_total, dim3(1), dim3(1024), 0, s, partial, (int)ssim_partials(W, H), 1.0 / n, weight,
                       loss);
    hipLaunchKernelGGL(k_ssim_bwd, grid, dim, 0, s, x, y, W, H, strip, strips, win, Pa, Pb, Pc,
                       (float)(-(double)weight / n), dx);
    return hipGetLastError();
}

}  // namespace gs
