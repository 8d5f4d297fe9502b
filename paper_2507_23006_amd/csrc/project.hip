// Projection of 3D Gaussians to 2D (EWA) with SH colour -- gfx950.
//
// Two launch shapes share the per-view arithmetic: one thread per Gaussian
// walking every view of the launch (training: all views see the same
// Gaussians, whose parameters are then read from HBM once), or one thread
// per slot of a segment table (served views, each with its own selection of
// level-of-detail segments).  Geometry reads are structure-of-arrays;
// records are written as four float4s so the compositing kernels gather a
// record with 16-byte loads.  Arithmetic is FP64: the kernel is bound by HBM and
// CDNA4 executes FP64 FMAs at the non-packed FP32 rate, so the geometry that
// decides tile rectangles and depth keys carries no FP32 rounding.
//
// Paper: §3.1 (Eq. 1 for Sigma = R S S^T R^T; the projection to 2D Gaussians
// G' in the text after it), §3.5.4 (anti-aliasing dilation and opacity
// compensation), colour c of §3.1 as degree-3 SH.
#include <math.h>

#include "gs_internal.h"
#include "rows.h"

namespace gs {

namespace {

__device__ __forceinline__ void quat_rotation(double w, double x, double y, double z, double R[9]) {
    R[0] = 1.0 - 2.0 * (y * y + z * z);
    R[1] = 2.0 * (x * y - w * z);
    R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);
    R[4] = 1.0 - 2.0 * (x * x + z * z);
    R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);
    R[7] = 2.0 * (y * z + w * x);
    R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// camera-space position t = R mu + t_w of a mean in view V
__device__ __forceinline__ void view_point(const ViewK& V, double mu0, double mu1, double mu2, double& tx, double& ty,
                                           double& tz) {
    tx = (double)V.R[0] * mu0 + (double)V.R[1] * mu1 + (double)V.R[2] * mu2 + (double)V.t[0];
    ty = (double)V.R[3] * mu0 + (double)V.R[4] * mu1 + (double)V.R[5] * mu2 + (double)V.t[1];
    tz = (double)V.R[6] * mu0 + (double)V.R[7] * mu1 + (double)V.R[8] * mu2 + (double)V.t[2];
}

// M = R(q) diag(s) of Gaussian g with scales s0..s2, and its opacity op
// (times 1 - do under appearance offsets); false for a zero quaternion
__device__ __forceinline__ bool load_shape(const GaussPtrs& gp, int64_t n, int64_t g, double s0, double s1, double s2,
                                           double op, double M[9], double& opac) {
    double qw = gp.quats[g], qx = gp.quats[n + g], qy = gp.quats[2 * n + g], qz = gp.quats[3 * n + g];
    const double qn = sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    if (!(qn > 0.0)) return false;
    const double inv = 1.0 / qn;
    double Rq[9];
    quat_rotation(qw * inv, qx * inv, qy * inv, qz * inv, Rq);
    M[0] = Rq[0] * s0; M[1] = Rq[1] * s1; M[2] = Rq[2] * s2;
    M[3] = Rq[3] * s0; M[4] = Rq[4] * s1; M[5] = Rq[5] * s2;
    M[6] = Rq[6] * s0; M[7] = Rq[7] * s1; M[8] = Rq[8] * s2;
    opac = op;
    if (gp.app) opac *= 1.0 - (double)gp.app[4 * g + 3];
    return true;
}

// square root within an ulp for r in the range that projected sizes have (0
// below 1e-200): one step from the reciprocal root's estimate squares its
// 2^-26 error twice over, a third of the instructions of the general sqrt
__device__ __forceinline__ double root(double r) {
    const double s = __builtin_amdgcn_rsq(r);
    double g = r * s;
    double h = 0.5 * s;
    double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-g, g, r);
    g = fma(e, h, g);
    return !(r <= 1e-200) ? g : 0.0;
}

// Exact tile culling of a rectangle of w x h <= 64 tiles at (ix0, iy0): bit
// (ty - iy0) w + (tx - ix0) is set when the alpha ellipse
// q(d) = A dx^2 + 2 B dx dy + C dy^2 <= L, L = 2 tau (1 + 4e-6), reaches the
// tile's pixel-centre rectangle widened by 1e-3 px.  Row by row: the ellipse
// within a row's strip is convex, so it meets a tile iff its x-extent over the
// strip meets the tile's columns, a run of tiles found by division.  For fixed y
// the ellipse spans x = (-B y -+ sqrt(A L - det y^2)) / A; the upper end is
// concave in y and peaks at the rightmost point (X, -B X / C), X = sqrt(L C /
// det), the lower end is convex with its minimum at (-X, B X / C), so over a
// strip (clipped to the ellipse's y-extent +-sqrt(L A / det)) both come from
// those y clamped into it.  Two square roots a row, whose count (the tallest
// rectangle of the wave's) bounds the projection's arithmetic: with IEEE roots
// and divisions and a loop over the columns they were two thirds of it.
__device__ uint64_t covered_tiles(const ViewK& V, double mx, double my, double A, double B, double C, double tau,
                                  int ix0, int iy0, int w, int h) {
    const double L = 2.0 * tau * (1.0 + 4e-6);
    const double det = A * C - B * B;
    const double id = 1.0 / det, iA = 1.0 / A;
    const double X = root(L * C * id), Y = root(L * A * id), yr = -B / C * X;
    const double AL = A * L, BA = -B * iA;
    // in units of tiles from the rectangle's first column: the first column's
    // first pixel centre less the margin, its last pixel centre with the
    // margin, and the image's last
    const double x0 = mx - ((double)(ix0 * kTile) + 0.5 - 1e-3), x1 = mx - ((double)(ix0 * kTile + kTile - 1) + 0.5 + 1e-3);
    const double xe = (double)(V.W - 1) + 0.5 + 1e-3 - mx;
    uint64_t m = 0;
    double ylo = (double)(iy0 * kTile) + 0.5 - 1e-3 - my;
    for (int j = 0; j < h; ++j, ylo += (double)kTile) {
        int py1 = (iy0 + j) * kTile + kTile - 1;
        if (py1 > V.H - 1) py1 = V.H - 1;
        const double yhi = (double)py1 + 0.5 + 1e-3 - my;
        const double a = fmax(ylo, -Y), b = fmin(yhi, Y);
        if (a > b) continue;
        const double y1 = fmin(fmax(yr, a), b), y2 = fmin(fmax(-yr, a), b);
        const double xhi_e = fma(BA, y1, root(fma(-det * y1, y1, AL)) * iA);
        const double xlo_e = fma(BA, y2, -root(fma(-det * y2, y2, AL)) * iA);
        if (xlo_e > xe) continue;      // past the image's last pixel centre
        // column i: 16 i <= xhi_e + x0 and 16 i >= xlo_e + x1
        const double dw = (double)(w - 1);
        const int i1 = (int)fmax(fmin(floor((xhi_e + x0) * (1.0 / kTile)), dw), -1.0);
        const int i0 = (int)fmin(fmax(ceil((xlo_e + x1) * (1.0 / kTile)), 0.0), 64.0);
        if (i0 <= i1) m |= (~0ull >> (63 - (i1 - i0))) << (j * w + i0);
    }
    return m;
}

// 2D Gaussian of (t, M, opac) in view V: writes the record's geometry words
// (float4s 0, 1 and 3; the .w of float4 2 is returned in yfrac for the
// colour's write) and the rectangle of `slot`; returns the number of tiles
// covered, 0 when culled
__device__ __forceinline__ uint32_t project_view(const ViewK& V, const OptK& opt, double tx, double ty, double tz,
                                                 const double M[9], double opac, const Projected& out,
                                                 int64_t slot, float& yfrac) {
    const double W0 = V.R[0], W1 = V.R[1], W2 = V.R[2], W3 = V.R[3], W4 = V.R[4], W5 = V.R[5], W6 = V.R[6],
                 W7 = V.R[7], W8 = V.R[8];
    const double fx = V.fx, fy = V.fy;
    const double itz = 1.0 / tz;
    const double u = tx * itz, vv = ty * itz;
    const double uc = fmin(fmax(u, V.ulo), V.uhi);
    const double vc = fmin(fmax(vv, V.vlo), V.vhi);
    const double j00 = fx * itz, j02 = -j00 * uc, j11 = fy * itz, j12 = -j11 * vc;
    // Tm = J W (2x3), Vm = Tm M (2x3): Sigma_2D = Vm Vm^T
    const double T0 = j00 * W0 + j02 * W6, T1 = j00 * W1 + j02 * W7, T2 = j00 * W2 + j02 * W8;
    const double T3 = j11 * W3 + j12 * W6, T4 = j11 * W4 + j12 * W7, T5 = j11 * W5 + j12 * W8;
    const double a0 = T0 * M[0] + T1 * M[3] + T2 * M[6];
    const double a1 = T0 * M[1] + T1 * M[4] + T2 * M[7];
    const double a2 = T0 * M[2] + T1 * M[5] + T2 * M[8];
    const double b0 = T3 * M[0] + T4 * M[3] + T5 * M[6];
    const double b1 = T3 * M[1] + T4 * M[4] + T5 * M[7];
    const double b2 = T3 * M[2] + T4 * M[5] + T5 * M[8];
    const double ca = a0 * a0 + a1 * a1 + a2 * a2;
    const double cb = a0 * b0 + a1 * b1 + a2 * b2;
    const double cc = b0 * b0 + b1 * b1 + b2 * b2;
    // det(Sigma_2D) = |a x b|^2 (Lagrange identity, no cancellation)
    const double x0 = a1 * b2 - a2 * b1, x1 = a2 * b0 - a0 * b2, x2 = a0 * b1 - a1 * b0;
    const double det2 = x0 * x0 + x1 * x1 + x2 * x2;
    const double dil = (double)opt.dilation;
    const double ad = ca + dil, cd = cc + dil;
    const double detd = det2 + dil * (ca + cc) + dil * dil;
    const double mx = fx * u + (double)V.cx, my = fy * vv + (double)V.cy;
    const double lmax = 0.5 * (ad + cd) + root(0.25 * (ad - cd) * (ad - cd) + cb * cb);
    const double ext = 3.0 * root(lmax);
    if (!(detd > 0.0 && isfinite(ext) && isfinite(mx) && isfinite(my))) return 0;
    const double r = ceil(ext);
    const int TW = V.tiles_x, TH = V.tiles_y;
    double x0t = floor((floor(mx) - r) * (1.0 / kTile)), x1t = floor((floor(mx) + r) * (1.0 / kTile));
    double y0t = floor((floor(my) - r) * (1.0 / kTile)), y1t = floor((floor(my) + r) * (1.0 / kTile));
    x0t = fmax(x0t, 0.0);
    y0t = fmax(y0t, 0.0);
    x1t = fmin(x1t, (double)(TW - 1));
    y1t = fmin(y1t, (double)(TH - 1));
    // Tile-based culling: alpha = o' G' reaches 1/255 only inside the ellipse
    // x^T Sigma'^-1 x <= 2 tau, tau = ln(255 o'), whose bounding box has
    // half-widths sqrt(2 tau Sigma'_xx), sqrt(2 tau Sigma'_yy).  Widened by
    // margins for the float32 compositing arithmetic (1e-5 on tau, relative
    // 1e-6 and 1e-3 px), the box keeps the tiles whose pixel centres it
    // reaches; the rectangle drops the others, which no entry could change.
    // The box also travels in the record for the per-quadrant culling.
    const double invd = 1.0 / detd;
    const double rho = opt.aa ? root(det2 * invd) : 1.0;
    const double o2 = opac * rho;
    if (!((float)o2 >= kAlphaMin)) return 0;     // below the skip threshold everywhere
    const double tau = log(255.0 * o2) + 1e-5;
    const double hxd = root(2.0 * tau * ad) * (1.0 + 1e-6) + 1e-3;
    const double hyd = root(2.0 * tau * cd) * (1.0 + 1e-6) + 1e-3;
    x0t = fmax(x0t, floor(ceil(mx - hxd - 0.5) * (1.0 / kTile)));
    x1t = fmin(x1t, floor(floor(mx + hxd - 0.5) * (1.0 / kTile)));
    y0t = fmax(y0t, floor(ceil(my - hyd - 0.5) * (1.0 / kTile)));
    y1t = fmin(y1t, floor(floor(my + hyd - 0.5) * (1.0 / kTile)));
    if (!(x0t <= x1t && y0t <= y1t)) return 0;
    const int ix0 = (int)x0t, iy0 = (int)y0t, ix1 = (int)x1t, iy1 = (int)y1t;
    const int w = ix1 - ix0 + 1, h = iy1 - iy0 + 1;
    const double A = cd * invd, B = -cb * invd, C = ad * invd;
    uint32_t covered = (uint32_t)(w * h);
    if (out.tile_mask) {
        uint64_t m = 0;
        if (w * h <= 64) {
            m = covered_tiles(V, mx, my, A, B, C, tau, ix0, iy0, w, h);
            if (!m) return 0;     // the ellipse reaches no pixel centre of the image
            covered = (uint32_t)__popcll(m);
        }
        out.tile_mask[slot] = m;
    }
    // mean = integer part (exact in float32) + fraction, so that the
    // compositing kernels can form a tile-relative mean without the
    // rounding of a large absolute pixel coordinate
    const double fmx = floor(mx), fmy = floor(my);
    out.rec[4 * slot + 0] = make_float4((float)fmx, (float)fmy, (float)(-0.5 * kLog2e * A), (float)(-kLog2e * B));
    out.rec[4 * slot + 1] = make_float4((float)(-0.5 * kLog2e * C), (float)(opac * rho), (float)tz, (float)(mx - fmx));
    yfrac = (float)(my - fmy);
    out.rec[4 * slot + 3] = make_float4((float)hxd, (float)hyd, 0.0f, 0.0f);
    out.rect[slot] = make_uint2((uint32_t)(V.tile_off + iy0 * TW + ix0), (uint32_t)w | ((uint32_t)TW << 16));
    return covered;
}

// view-dependent colour of a mean seen by V into the record's .xyz of
// float4 2 (written whole, with yfrac as its .w); the coefficient row is
// read as 16-byte vectors; cb is the constant of the polynomial (1/2, or
// the appearance colour offset)
__device__ __forceinline__ void colour_view(const ViewK& V, const OptK& opt, double mu0, double mu1, double mu2,
                                            const F4* __restrict__ shq, float4 cb, const Projected& out,
                                            int64_t slot, float yfrac) {
    const int nb = (opt.sh_degree + 1) * (opt.sh_degree + 1);
    const int nq = (3 * nb + 3) >> 2;    // float4s that hold the used coefficients
    // direction in FP64 (mu and the camera centre are large numbers), the
    // SH polynomial in FP32
    const double e0 = mu0 - V.campos[0], e1 = mu1 - V.campos[1], e2 = mu2 - V.campos[2];
    const double inv = 1.0 / sqrt(e0 * e0 + e1 * e1 + e2 * e2);
    float Y[16];
    sh_eval_basis<float>((float)(e0 * inv), (float)(e1 * inv), (float)(e2 * inv), opt.sh_degree, Y);
    float shv[48];
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const F4 t = q < nq ? shq[q] : F4{0.0f, 0.0f, 0.0f, 0.0f};
        shv[4 * q + 0] = t.x; shv[4 * q + 1] = t.y; shv[4 * q + 2] = t.z; shv[4 * q + 3] = t.w;
    }
    float c[3] = {cb.x, cb.y, cb.z};
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k < nb) {
            c[0] = fmaf(shv[3 * k + 0], Y[k], c[0]);
            c[1] = fmaf(shv[3 * k + 1], Y[k], c[1]);
            c[2] = fmaf(shv[3 * k + 2], Y[k], c[2]);
        }
    }
    out.rec[4 * slot + 2] = make_float4(fmaxf(c[0], 0.0f), fmaxf(c[1], 0.0f), fmaxf(c[2], 0.0f), yfrac);
}

// Conservative pre-test of project_view in FP32: false only when the Gaussian
// certainly covers no tile.  With M = R(q) diag(s), R orthonormal,
// lambda_max(Sigma_2D) = |J W M|^2 <= |J|_F^2 |W|^2 s_max^2, and |J|_F <=
// sqrt(fx^2 (1 + u^2) + fy^2 (1 + v^2)) / tz for the clamped u, v, so the
// 3-sigma radius with its rounding up is at most (jn s_max) / tz + k, k =
// 3 sqrt(dilation) + 2.  Times tz > 0, "the rectangle reaches the image" is then
// linear in t for each image side, and reads no division or root.  Each sum is
// compared with the bound e on its rounding error, so that only a Gaussian
// outside by more is dropped; a NaN or an infinity drops nothing.
// 12M Gaussians in eight views: the test in FP64 took 1 of the kernel's 3 ms.
struct ViewPlane {
    float left, right, top, bottom;     // coefficients of tz
    float jn;                           // of the largest scale
    float ez, ef, tn;                   // errors of tz and of a side are <= ez (a + tn), ef (a + tn); a = |mu|_1
};

struct PlaneTable {
    ViewPlane p[GS_MAX_VIEWS];
};

__device__ __forceinline__ void view_point32(const ViewK& V, const float mu[3], float& tx, float& ty, float& tz) {
    tx = fmaf(V.R[0], mu[0], fmaf(V.R[1], mu[1], fmaf(V.R[2], mu[2], V.t[0])));
    ty = fmaf(V.R[3], mu[0], fmaf(V.R[4], mu[1], fmaf(V.R[5], mu[2], V.t[1])));
    tz = fmaf(V.R[6], mu[0], fmaf(V.R[7], mu[1], fmaf(V.R[8], mu[2], V.t[2])));
}

// between the near and the far plane, or too close to them to tell
__device__ __forceinline__ bool may_be_in_front(const ViewK& V, const ViewPlane& P, const float mu[3], float a) {
    const float tz = fmaf(V.R[6], mu[0], fmaf(V.R[7], mu[1], fmaf(V.R[8], mu[2], V.t[2])));
    const float e = P.ez * (a + P.tn);
    return !(tz + e < V.znear) && !(tz - e > V.zfar);
}

// the four image sides; smax: the largest scale's size
__device__ __forceinline__ bool may_cover(const ViewK& V, const ViewPlane& P, const float mu[3], float a, float smax) {
    float tx, ty, tz;
    view_point32(V, mu, tx, ty, tz);
    const float r = fmaf(P.jn, smax, P.ef * (a + P.tn)), x = V.fx * tx, y = V.fy * ty;
    return !(fmaf(P.left, tz, r) + x < 0.0f) && !(fmaf(P.right, tz, r) - x < 0.0f) &&
           !(fmaf(P.top, tz, r) + y < 0.0f) && !(fmaf(P.bottom, tz, r) - y < 0.0f);
}

// exact projection and colour of Gaussian g (mean mu, scales s, opacity
// op, coefficient row shq, as stored) into the views of `cand`; slot of view v
// = slot_base + v * slot_stride
__device__ __forceinline__ void project_candidate(const GaussPtrs& gp, int64_t n, const ViewTable& vt,
                                                  const OptK& opt, const Projected& out, int64_t g, uint32_t cand,
                                                  int64_t slot_base, int64_t slot_stride, const float mu[3],
                                                  const float sc[3], float op, const F4* __restrict__ shq) {
    const double mu0 = mu[0], mu1 = mu[1], mu2 = mu[2];
    double M[9], opac = 0.0;
    const bool shape_ok = load_shape(gp, n, g, sc[0], sc[1], sc[2], op, M, opac);
    const float4 cb = gp.app ? reinterpret_cast<const float4*>(gp.app)[g] : make_float4(0.5f, 0.5f, 0.5f, 0.0f);
    for (int v = 0; v < vt.n_views; ++v) {
        if (!(cand & (1u << v))) continue;
        const ViewK& V = vt.v[v];
        const int64_t slot = slot_base + v * slot_stride;
        double tx, ty, tz;
        view_point(V, mu0, mu1, mu2, tx, ty, tz);
        float yfrac = 0.0f;
        const bool front = tz >= (double)V.znear && tz <= (double)V.zfar;
        const uint32_t ntiles = shape_ok && front ? project_view(V, opt, tx, ty, tz, M, opac, out, slot, yfrac) : 0u;
        if (ntiles) colour_view(V, opt, mu0, mu1, mu2, shq, cb, out, slot, yfrac);
        out.tiles[slot] = ntiles;
        out.dkey[slot] = ntiles ? __float_as_uint((float)tz) : 0xFFFFFFFFu;
    }
}

constexpr int kPFPer = 4;                // items per lane in the scan of a chunk

// Every view of the launch sees the same n Gaussians: slot = view * n + g.  Each
// workgroup is one wave that scans chunks of 64 * per Gaussians (per <=
// kPFPer): it reads the means and, of Gaussians in front of some camera, the
// scales and opacity, runs the conservative pre-test per view, writes the
// culled slots' count and key with coalesced stores and packs the rest into an
// LDS list.  Whenever the list holds a batch of 64 (with several views after
// grouping it by the views to test), the wave runs the FP64 EWA and the colour
// on full waves of listed Gaussians (a large scene leaves most lanes culled, which
// would otherwise idle through the FP64 chain of their wave's few visible
// neighbours); their coefficient rows pass through LDS, where they stay for
// all views.  Chunk k of the wave is chunk blockIdx.x + k gridDim.x, at most
// 256 per wave.  A longer list would share views better, but its Gaussians'
// parameters are in cache no more when it comes to them: with 384 and 64
// entries 2880 and 2771 us for 12M Gaussians in eight views, timed alone.
//
// HBM-bound where most Gaussians are seen, else by the 128-byte lines of which
// one or two Gaussians are wanted.  Measured (256 threads over spans of 1024,
// FP64 pre-test, IEEE roots and divisions before): 1M Gaussians, most seen
// 108 -> 81 us, 120k 27 -> 15, 4096 29 -> 9; averages over training steps 6M with
// 16 % seen 200 -> 192, 12M in eight views 2997 -> 2974 (shortest 2970 -> 2746).
// Waves of a launch: as many as run at once, ten on a compute unit by their LDS,
// with several views eight by their registers.  (One view of 6M Gaussians takes
// 187, 186, 226 and 220 us with 2048, 2560, 2816 and 3072: a second turn of a
// few waves is a long tail.)
constexpr int64_t max_waves(bool multi) { return multi ? 2048 : 2560; }

template <bool kMulti>
__global__ __launch_bounds__(64, 3) void k_project_fwd(GaussPtrs gp, uint32_t n, ViewTable vt, PlaneTable planes,
                                                       OptK opt, Projected out, int per) {
    constexpr uint32_t kCap = 64 * (1 + kPFPer);
    __shared__ uint32_t s_list[kCap];      // index in the chunk | chunk of the wave << 8 | view mask << 16
    __shared__ uint32_t s_group[kMulti ? kCap : 1];    // the list grouped by view mask (several views)
    __shared__ uint32_t s_hist[kMulti ? 256 : 1];
    __shared__ F4 s_rows[kWaveRows];
    const int lane = threadIdx.x;
    const int n_views = kMulti ? vt.n_views : 1;
    const uint32_t span = 64u * (uint32_t)per, n_chunks = (n + span - 1) / span;
    const int nq = (3 * (opt.sh_degree + 1) * (opt.sh_degree + 1) + 3) >> 2;    // float4s of a row in use
    const RowLanes rl(lane);
    uint32_t cnt = 0, k = 0, chunk = blockIdx.x;
    for (;;) {
        while (cnt < 64 && chunk < n_chunks) {
            const uint32_t g0 = chunk * span;
            // the lane's Gaussians move through each phase together, so that
            // their independent loads are in flight at once
            float mu[kPFPer][3], a[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                const uint64_t g = (uint64_t)g0 + 64 * i + lane;
                const bool ok = i < per && g < n;
#pragma unroll
                for (int c = 0; c < 3; ++c) mu[i][c] = ok ? gp.means[(int64_t)c * n + g] : 0.0f;
            }
            uint32_t front[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                front[i] = 0;
                a[i] = fabsf(mu[i][0]) + fabsf(mu[i][1]) + fabsf(mu[i][2]);
            }
            for (int v = 0; v < n_views; ++v) {
#pragma unroll
                for (int i = 0; i < kPFPer; ++i)
                    front[i] |= may_be_in_front(vt.v[v], planes.p[v], mu[i], a[i]) ? 1u << v : 0u;
            }
            float smax[kPFPer], op[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                const uint64_t g = (uint64_t)g0 + 64 * i + lane;
                if (!(i < per && g < n)) front[i] = 0;
                float sc[3] = {0.0f, 0.0f, 0.0f};
                op[i] = 0.0f;
                if (front[i]) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) sc[c] = gp.scales[(int64_t)c * n + g];
                    op[i] = gp.opac[g];
                }
                smax[i] = fmaxf(fabsf(sc[0]), fmaxf(fabsf(sc[1]), fabsf(sc[2])));
            }
#pragma unroll
            for (int i = 0; i < kPFPer; ++i)
                if (!(op[i] >= kAlphaMin)) front[i] = 0;     // o' = o rho <= o: below the skip threshold everywhere
            uint32_t cand[kPFPer] = {};
            for (int v = 0; v < n_views; ++v) {
#pragma unroll
                for (int i = 0; i < kPFPer; ++i) {
                    const uint64_t g = (uint64_t)g0 + 64 * i + lane;
                    if ((front[i] & (1u << v)) && may_cover(vt.v[v], planes.p[v], mu[i], a[i], smax[i]))
                        cand[i] |= 1u << v;
                    else if (i < per && g < n) {
                        const int64_t slot = (int64_t)v * n + g;
                        __builtin_nontemporal_store(0u, out.tiles + slot);
                        __builtin_nontemporal_store(0xFFFFFFFFu, out.dkey + slot);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                const uint64_t m = __ballot(cand[i] != 0);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                if (cand[i]) s_list[cnt + below] = (uint32_t)(64 * i + lane) | k << 8 | cand[i] << 16;
                cnt += (uint32_t)__popcll(m);
            }
            chunk += gridDim.x;
            ++k;
        }
        wave_sync();
        const bool last = chunk >= n_chunks;
        const uint32_t* lst = s_list;
        if (kMulti) {      // Gaussians that are candidates in the same views side by side
            group_by_views(s_list, cnt, s_group, s_hist);
            lst = s_group;
        }
        // lanes past the end work on the last Gaussian and write nothing
        uint32_t b = 0;
        for (; b + 64 <= cnt || (last && b < cnt); b += 64) {
            const int m = cnt - b < 64u ? (int)(cnt - b) : 64;
            const uint32_t e = lst[b + (lane < m ? lane : m - 1)];
            const uint32_t g = (((e >> 8) & 255u) * gridDim.x + blockIdx.x) * span + (e & 255u);
            float mu[3], sc[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                mu[c] = gp.means[(int64_t)c * n + g];
                sc[c] = gp.scales[(int64_t)c * n + g];
            }
            const float op = gp.opac[g];
            load_rows(gp.sh, g, nq, rl, s_rows);
            if (lane < m)
                project_candidate(gp, n, vt, opt, out, g, e >> 16, g, n, mu, sc, op, s_rows + lane * kRowF4);
            wave_sync();
        }
        if (last) return;
        // what is left over, to the front
        const uint32_t left = cnt - b;
        const uint32_t e = lst[b + ((uint32_t)lane < left ? lane : 0)];
        wave_sync();
        if ((uint32_t)lane < left) s_list[lane] = e;
        cnt = left;
    }
}

// slot s of a segment table: the last segment with slot_start <= s
__device__ __forceinline__ int segment_of(const SlotSeg* __restrict__ segs, int32_t n_seg, uint32_t s) {
    int lo = 0, hi = n_seg;      // invariant: segs[lo].slot_start <= s, answer in [lo, hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (segs[mid].slot_start <= s) lo = mid; else hi = mid;
    }
    return lo;
}

// the same by a whole wave for one slot, 64 probes at a time
__device__ __forceinline__ int segment_of_wave(const SlotSeg* __restrict__ segs, int32_t n_seg, uint32_t s, int lane) {
    int lo = 0, hi = n_seg;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64, q = lo + lane * step;
        const bool le = lane == 0 || (q < hi && segs[q].slot_start <= s);
        const int last = 63 - __clzll(__ballot(le));       // lanes 0 .. last hold
        lo += last * step;
        hi = min(hi, lo + step);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Views with their own selections of Gaussians (served requests): slot s
// maps to Gaussian gstart + (s - slot_start) of its segment, seen by the
// segment's view.  The scan and the batches of k_project_fwd, over chunks of
// slots; a chunk's segments are held one per lane when it has fewer than 64 (else
// each slot searches them).  Batches of 8 views of 6M Gaussians, beside the
// compositing of the batch before: 405 us where 256 threads over spans of 1024
// took 967.  More waves than run at once (2304): beside another stream's kernel
// waves that end make room for it (2304, 1536, 1024 and 512 waves: 40 requests take
// 10.4, 10.7, 10.5 and 11.4 ms, 16384: 10.2).
constexpr int64_t kSlotWaves = 16384;
__global__ __launch_bounds__(64, 3) void k_project_slots(GaussPtrs gp, int64_t n, ViewTable vt, PlaneTable planes,
                                                         OptK opt, const SlotSeg* __restrict__ segs, int32_t n_seg,
                                                         uint32_t n_slots, Projected out, int per) {
    constexpr uint32_t kCap = 64 * (1 + kPFPer);
    __shared__ uint32_t s_slot[kCap], s_gid[kCap];      // listed slots and their Gaussians (n < 2^32, checked at launch)
    __shared__ uint8_t s_view[kCap];
    __shared__ F4 s_rows[kWaveRows];
    const int lane = threadIdx.x;
    const uint32_t span = 64u * (uint32_t)per;
    const uint32_t n_chunks = (uint32_t)(((uint64_t)n_slots + span - 1) / span);
    const int nq = (3 * (opt.sh_degree + 1) * (opt.sh_degree + 1) + 3) >> 2;    // float4s of a row in use
    const RowLanes rl(lane);
    constexpr uint32_t kNone = 0xFFFFFFFFu;      // view of a lane without a slot
    uint32_t cnt = 0, chunk = blockIdx.x;
    for (;;) {
        while (cnt < 64 && chunk < n_chunks) {
            const uint32_t s0 = chunk * span, s1 = n_slots - s0 < span ? n_slots : s0 + span;
            const int seg0 = segment_of_wave(segs, n_seg, s0, lane);
            SlotSeg mine = {};
            mine.slot_start = kNone;
            if (seg0 + lane < n_seg) mine = segs[seg0 + lane];
            const int n_in = __popcll(__ballot(mine.slot_start < s1));      // segments of the chunk, from lane 0 on
            uint32_t g[kPFPer], view[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                const uint32_t s = s0 + 64 * i + lane;
                const bool in = i < per && (uint64_t)s0 + 64 * i + lane < s1;
                SlotSeg sg;
                if (n_in < 64) {
                    int k = 0;
                    for (int j = 1; j < n_in; ++j)
                        if (s >= (uint32_t)__builtin_amdgcn_readlane((int)mine.slot_start, j)) k = j;
                    sg.slot_start = __shfl(mine.slot_start, k);
                    sg.view = __shfl(mine.view, k);
                    sg.gstart = __shfl(mine.gstart, k);
                } else {
                    sg = segs[seg0 + segment_of(segs + seg0, n_seg - seg0, in ? s : s0)];
                }
                g[i] = in ? (uint32_t)(sg.gstart + (int64_t)(s - sg.slot_start)) : 0u;
                view[i] = in ? (uint32_t)sg.view : kNone;
            }
            float mu[kPFPer][3], a[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
#pragma unroll
                for (int c = 0; c < 3; ++c) mu[i][c] = view[i] != kNone ? gp.means[c * n + g[i]] : 0.0f;
                a[i] = fabsf(mu[i][0]) + fabsf(mu[i][1]) + fabsf(mu[i][2]);
            }
            // views one after another, with their constants in scalar registers (a
            // chunk rarely has more than one)
            const auto of_view = [&](uint32_t v) {
                bool any = false;
#pragma unroll
                for (int i = 0; i < kPFPer; ++i) any |= view[i] == v;
                return __ballot(any) != 0;
            };
            bool cand[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) cand[i] = false;
            for (uint32_t v = 0; v < (uint32_t)vt.n_views; ++v) {
                if (!of_view(v)) continue;
#pragma unroll
                for (int i = 0; i < kPFPer; ++i)
                    if (view[i] == v) cand[i] = may_be_in_front(vt.v[v], planes.p[v], mu[i], a[i]);
            }
            float smax[kPFPer];
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                float sc[3] = {0.0f, 0.0f, 0.0f}, op = 0.0f;
                if (cand[i]) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) sc[c] = gp.scales[c * n + g[i]];
                    op = gp.opac[g[i]];
                }
                smax[i] = fmaxf(fabsf(sc[0]), fmaxf(fabsf(sc[1]), fabsf(sc[2])));
                cand[i] = op >= kAlphaMin;      // o' = o rho <= o: else below the skip threshold everywhere
            }
            for (uint32_t v = 0; v < (uint32_t)vt.n_views; ++v) {
                if (!of_view(v)) continue;
#pragma unroll
                for (int i = 0; i < kPFPer; ++i)
                    if (view[i] == v) cand[i] = cand[i] && may_cover(vt.v[v], planes.p[v], mu[i], a[i], smax[i]);
            }
#pragma unroll
            for (int i = 0; i < kPFPer; ++i) {
                const uint32_t s = s0 + 64 * i + lane;
                const uint64_t m = __ballot(cand[i]);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                if (cand[i]) {
                    s_slot[cnt + below] = s;
                    s_gid[cnt + below] = g[i];
                    s_view[cnt + below] = (uint8_t)view[i];
                } else if (view[i] != kNone) {
                    __builtin_nontemporal_store(0u, out.tiles + s);
                    __builtin_nontemporal_store(0xFFFFFFFFu, out.dkey + s);
                }
                cnt += (uint32_t)__popcll(m);
            }
            chunk += gridDim.x;
        }
        wave_sync();
        const bool last = chunk >= n_chunks;
        // lanes past the end work on the last slot and write nothing
        uint32_t b = 0;
        for (; b + 64 <= cnt || (last && b < cnt); b += 64) {
            const int m = cnt - b < 64u ? (int)(cnt - b) : 64;
            const uint32_t j = b + (lane < m ? lane : m - 1), g = s_gid[j];
            float mu[3], sc[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                mu[c] = gp.means[c * n + g];
                sc[c] = gp.scales[c * n + g];
            }
            const float op = gp.opac[g];
            load_rows(gp.sh, g, nq, rl, s_rows);
            // one view bit: the slot is s itself (stride 0)
            if (lane < m)
                project_candidate(gp, n, vt, opt, out, g, 1u << s_view[j], s_slot[j], 0, mu, sc, op, s_rows + lane * kRowF4);
            wave_sync();
        }
        if (last) return;
        // what is left over, to the front
        const uint32_t left = cnt - b, at = b + ((uint32_t)lane < left ? lane : 0);
        const uint32_t slot = s_slot[at], gid = s_gid[at];
        const uint8_t v = s_view[at];
        wave_sync();
        if ((uint32_t)lane < left) {
            s_slot[lane] = slot;
            s_gid[lane] = gid;
            s_view[lane] = v;
        }
        cnt = left;
    }
}

}  // namespace

// constants of the pre-test (see ViewPlane), rounded away from dropping
static PlaneTable build_planes(const ViewTable& vt, const OptK& opt) {
    PlaneTable pt = {};
    const double k = 3.0 * sqrt((double)opt.dilation) + 2.0, up = 1.0 + 1e-5;
    for (int v = 0; v < vt.n_views; ++v) {
        const ViewK& V = vt.v[v];
        // |W|: 1 for a rotation, else at most the Frobenius norm
        double f2 = 0.0, off = 0.0, big = 1.0;
        for (int i = 0; i < 9; ++i) {
            f2 += (double)V.R[i] * V.R[i];
            big = fmax(big, fabs((double)V.R[i]));
        }
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) {
                double d = i == j ? -1.0 : 0.0;
                for (int c = 0; c < 3; ++c) d += (double)V.R[3 * c + i] * V.R[3 * c + j];
                off = fmax(off, fabs(d));
            }
        const double w = off < 1e-3 ? 1.0 + 2e-3 : sqrt(f2);
        const double um = fmax(fabs(V.ulo), fabs(V.uhi)), vm = fmax(fabs(V.vlo), fabs(V.vhi));
        const double fx = V.fx, fy = V.fy;
        const double X = V.tiles_x * kTile, Y = V.tiles_y * kTile;
        ViewPlane& P = pt.p[v];
        P.left = (float)(V.cx + k);
        P.right = (float)(X - V.cx + k);
        P.top = (float)(V.cy + k);
        P.bottom = (float)(Y - V.cy + k);
        P.jn = (float)(up * 3.0 * w * sqrt(fx * fx * (1.0 + um * um) + fy * fy * (1.0 + vm * vm)));
        // every coordinate is a sum of four products of at most big |mu|_1 + tn,
        // rounded four times (2^-24 each), a side two such sums and three more
        // roundings: 2^-20 covers both, with the constants' own rounding
        P.tn = (float)(up * fmax(fabs((double)V.t[0]), fmax(fabs((double)V.t[1]), fabs((double)V.t[2]))));
        P.ez = (float)(up * big * 0x1p-20);
        P.ef = (float)(up * big * 0x1p-20 * (fmax(fx, fy) + fmax(fmax(fabs((double)P.left), fabs((double)P.right)),
                                                               fmax(fabs((double)P.top), fabs((double)P.bottom)))));
    }
    return pt;
}

hipError_t launch_project_fwd(const GaussPtrs& g, int64_t n, const ViewTable& vt, const OptK& opt,
                              const Projected& out, hipStream_t s) {
    if (n > 0xFFFFFFFFLL) return hipErrorInvalidValue;     // Gaussians are kept as 32-bit indices
    // chunks of 256 Gaussians when that leaves every wave several, else of 64
    const int64_t waves = max_waves(vt.n_views > 1);
    const int per = n >= waves * 64 * kPFPer ? kPFPer : 1;
    const int64_t chunks = (n + 64 * per - 1) / (64 * per);
    int64_t blocks = chunks < waves ? chunks : waves;
    if (blocks * 256 < chunks) blocks = (chunks + 255) / 256;
    const hipEvent_t timed_ = timer_begin(GS_KERNEL_PROJECT_FWD, s);
    const auto kernel = vt.n_views > 1 ? k_project_fwd<true> : k_project_fwd<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64), 0, s, g, (uint32_t)n, vt, build_planes(vt, opt), opt, out,
                       per);
    timer_end(timed_, s);
    return hipGetLastError();
}

hipError_t launch_project_slots(const GaussPtrs& g, int64_t n, const ViewTable& vt, const OptK& opt,
                                const SlotSeg* segs, int32_t n_seg, uint32_t n_slots, const Projected& out,
                                hipStream_t s) {
    if (!n_slots) return hipSuccess;
    if (n > 0xFFFFFFFFLL) return hipErrorInvalidValue;     // listed Gaussians are kept as 32-bit indices
    // chunks of 256 slots when the waves that run at once (2304) each have several, else of 64
    const int per = (int64_t)n_slots >= 2304 * 64 * kPFPer ? kPFPer : 1;
    const int64_t chunks = ((int64_t)n_slots + 64 * per - 1) / (64 * per);
    hipLaunchKernelGGL(k_project_slots, dim3((unsigned)(chunks < kSlotWaves ? chunks : kSlotWaves)), dim3(64), 0, s, g, n, vt,
                       build_planes(vt, opt), opt, segs, n_seg, n_slots, out, per);
    return hipGetLastError();
}

}  // namespace gs
