// Backward of projection and colour -- gfx950.
//
// Each workgroup is one wave that scans chunks of 256 consecutive Gaussians:
// it writes the zeros and statistics of those no view sees and packs the
// others into an LDS list.  Whenever the list holds 64 (with several views
// after grouping them by the views that see them), the wave runs the chain, one
// lane per listed Gaussian: it reads the parameters once, recomputes the
// projection in FP64 for each view that sees the Gaussian, chains that view's
// 2D gradients (mean2d, conic, opacity', colour, depth) back to the
// parameters, and writes the sums once.  Only a small fraction of a large
// scene is in view, so the list keeps the chain on full waves, and without
// barriers one wave's reads run beside another's arithmetic.  When the
// outputs were zeroed beforehand (k_zero_floats on a second stream beside the
// compositing backward), the unseen rows are left alone.  2D gradients of
// unseen slots are never read.  With
// Sigma_2D = V V^T and V = (J W) M, M = R(q) diag(s), the covariance
// gradient flows as dV = 2 G V, d(JW) = dV M^T, dM += (JW)^T dV; dM is
// accumulated over views and pushed through R(q) and s once at the end.
// HBM-bound; geometry in FP64 for the same reason as the forward.
//
// Measured (workgroups of 256 threads over spans of 1024 before, one wave
// now): 1M Gaussians, most of them seen, one view: 175 -> 119 us, 4.6 TB/s of
// the 0.55 GB that rows and parameters hold; 4096: 34 -> 7 us; 12M in eight
// views 6570 -> 2560 us (2860 with lists of 384, whose Gaussians' parameters
// are in cache no more when the chain comes to them); 6M with 16 % seen 310 -> 292 us, where 128-byte lines
// of which one or two Gaussians are wanted make 1.1 GB of the traffic.
//
// Paper: backward of Eq. 1 and of the projection of §3.1; the per-view
// |dL/d mean2d| is the image-space statistic that densification thresholds
// (§3.1, §3.3 Eq. 4), and the absolute accumulation is the AbsGS statistic
// of §3.5.4.
#include "gs_internal.h"
#include "rows.h"

namespace gs {

namespace {

// gradient of each basis polynomial of sh_eval_basis with respect to (x, y, z)
__device__ __forceinline__ void sh_basis_grad(float x, float y, float z, int k, float& gx, float& gy,
                                              float& gz) {
    const float xx = x * x, yy = y * y, zz = z * z;
    const float k1 = (float)ShK::k1, k2 = (float)ShK::k2, k6 = (float)ShK::k6, k8 = (float)ShK::k8,
                k9 = (float)ShK::k9, k10 = (float)ShK::k10, k11 = (float)ShK::k11, k12 = (float)ShK::k12,
                k14 = (float)ShK::k14;
    gx = gy = gz = 0.0f;
    switch (k) {
        case 1: gy = -k1; break;
        case 2: gz = k1; break;
        case 3: gx = -k1; break;
        case 4: gx = k2 * y; gy = k2 * x; break;
        case 5: gy = -k2 * z; gz = -k2 * y; break;
        case 6: gx = -2.0f * k6 * x; gy = -2.0f * k6 * y; gz = 4.0f * k6 * z; break;
        case 7: gx = -k2 * z; gz = -k2 * x; break;
        case 8: gx = 2.0f * k8 * x; gy = -2.0f * k8 * y; break;
        case 9: gx = -6.0f * k9 * x * y; gy = -3.0f * k9 * (xx - yy); break;
        case 10: gx = k10 * y * z; gy = k10 * x * z; gz = k10 * x * y; break;
        case 11: gx = 2.0f * k11 * x * y; gy = -k11 * (4.0f * zz - xx - 3.0f * yy); gz = -8.0f * k11 * y * z; break;
        case 12: gx = -6.0f * k12 * x * z; gy = -6.0f * k12 * y * z; gz = k12 * (6.0f * zz - 3.0f * xx - 3.0f * yy); break;
        case 13: gx = -k11 * (4.0f * zz - 3.0f * xx - yy); gy = 2.0f * k11 * x * y; gz = -8.0f * k11 * x * z; break;
        case 14: gx = 2.0f * k14 * x * z; gy = -2.0f * k14 * y * z; gz = k14 * (xx - yy); break;
        case 15: gx = -3.0f * k9 * (xx - yy); gy = 6.0f * k9 * x * y; break;
        default: break;
    }
}

constexpr int kG2 = GS_GRAD2D_FLOATS;
constexpr int kChunkPer = 4;               // Gaussians per lane in the scan of a chunk
constexpr int kMaxWaves = 2048;            // two per SIMD, what the chain's registers allow
constexpr int kRowApp = 11;

// row c of the one-float gradients (means 0-2, scales 3-5, quats 6-9,
// opacity 10, appearance offsets 11-14) of Gaussian g
__device__ __forceinline__ float* grad_row(const GradPtrs& out, int64_t n, int64_t g, int c) {
    return c < 3 ? out.means + c * n + g : c < 6 ? out.scales + (c - 3) * n + g
         : c < 10 ? out.quats + (c - 6) * n + g : c == 10 ? out.opac + g : out.app + 4 * g + (c - kRowApp);
}

// Parameters of one Gaussian as stored, but for the coefficient row; app holds
// the appearance offsets (or the polynomial's constant and 0)
struct GaussIn {
    float mu[3], s[3], q[4], o;
    float4 app;
};

__device__ __forceinline__ GaussIn load_gauss(const GaussPtrs& gp, int64_t n, int64_t g) {
    GaussIn in;
#pragma unroll
    for (int c = 0; c < 3; ++c) in.mu[c] = gp.means[c * n + g];
#pragma unroll
    for (int c = 0; c < 3; ++c) in.s[c] = gp.scales[c * n + g];
#pragma unroll
    for (int c = 0; c < 4; ++c) in.q[c] = gp.quats[c * n + g];
    in.o = gp.opac[g];
    in.app = gp.app ? reinterpret_cast<const float4*>(gp.app)[g] : make_float4(0.5f, 0.5f, 0.5f, 0.0f);
    return in;
}

// band L of the polynomial: its part of the colour and of S_c = sum_k sh_kc
// grad Y_k
template <int L>
__device__ __forceinline__ void band_colour(const float r[48], const float Y[16], float x, float y, float z,
                                            float raw[3], float S[3][3]) {
#pragma unroll
    for (int k = L * L; k < (L + 1) * (L + 1); ++k) {
        float bx, by, bz;
        sh_basis_grad(x, y, z, k, bx, by, bz);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            raw[c] = fmaf(r[3 * k + c], Y[k], raw[c]);
            if (L > 0) {
                S[c][0] = fmaf(r[3 * k + c], bx, S[c][0]);
                S[c][1] = fmaf(r[3 * k + c], by, S[c][1]);
                S[c][2] = fmaf(r[3 * k + c], bz, S[c][2]);
            }
        }
    }
}

// d sh_kc += gr_c Y_k for band L
template <int L>
__device__ __forceinline__ void band_grad(const float gr[3], const float Y[16], float d[48]) {
#pragma unroll
    for (int k = L * L; k < (L + 1) * (L + 1); ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) d[3 * k + c] += gr[c] * Y[k];
}

// Colour chain of one seen Gaussian; vis = mask of the views that see it, g2
// = its 2D gradients in view 0 (those of the next view g2_stride floats on):
// replaces its coefficient row in LDS by the row's gradients, and returns its
// part of the mean's gradient (through the view direction) in dmu and of the
// colour constant's in dcb.  The row stays in LDS and the sum of its gradients
// in registers over the views, so each row is read and written once: adding
// to the row in memory view by view read 17 and wrote 7 GB per step of 12M
// Gaussians in eight views.
template <bool kMulti>
__device__ __forceinline__ void colour_bwd_one(const GaussIn& in, const ViewTable& vt, const OptK& opt,
                                               const float* __restrict__ grad2d, int64_t g2_stride, uint32_t vis,
                                               F4* __restrict__ row, double dmu[3], float dcb[3]) {
    const double mu0 = in.mu[0], mu1 = in.mu[1], mu2 = in.mu[2];
    float d[48];
#pragma unroll
    for (int k = 0; k < 48; ++k) d[k] = 0.0f;
    const int n_views = kMulti ? vt.n_views : 1;
    int v0 = 0;      // opaque: the views' constants are read here, not held in registers from batch to batch
    asm volatile("" : "+s"(v0));
    for (int v = 0; v < n_views; ++v) {
        if (kMulti && !(vis & (1u << v))) continue;
        const ViewK& V = vt.v[v + v0];
        const float* g2 = grad2d + v * g2_stride;
        const float gc[3] = {g2[6], g2[7], g2[8]};
        const double e0d = mu0 - V.campos[0], e1d = mu1 - V.campos[1], e2d = mu2 - V.campos[2];
        const double dn = sqrt(e0d * e0d + e1d * e1d + e2d * e2d);
        const double inv = 1.0 / dn;
        const float d0 = (float)(e0d * inv), d1 = (float)(e1d * inv), d2 = (float)(e2d * inv);
        float Y[16];
        sh_eval_basis<float>(d0, d1, d2, opt.sh_degree, Y);
        // colour: raw = sum_k sh_k Y_k(dhat) + dc, clamped at 0 (SH in FP32).
        // One pass over the coefficient row gives the colour and, per
        // channel c, S_c = sum_k sh_kc grad Y_k, so that the direction
        // gradient is sum_c gr_c S_c (coefficient e of the row is channel
        // e % 3 of basis e / 3)
        float raw[3] = {in.app.x, in.app.y, in.app.z};
        float S[3][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
        float r[48];
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            const F4 t = row[q];
            r[4 * q + 0] = t.x; r[4 * q + 1] = t.y; r[4 * q + 2] = t.z; r[4 * q + 3] = t.w;
        }
        // band by band, so that a degree is one branch
        const int deg = opt.sh_degree;
        band_colour<0>(r, Y, d0, d1, d2, raw, S);
        if (deg > 0) band_colour<1>(r, Y, d0, d1, d2, raw, S);
        if (deg > 1) band_colour<2>(r, Y, d0, d1, d2, raw, S);
        if (deg > 2) band_colour<3>(r, Y, d0, d1, d2, raw, S);
        const float gr[3] = {raw[0] < 0.0f ? 0.0f : gc[0], raw[1] < 0.0f ? 0.0f : gc[1], raw[2] < 0.0f ? 0.0f : gc[2]};
        dcb[0] += gr[0]; dcb[1] += gr[1]; dcb[2] += gr[2];
        const float e0 = gr[0] * S[0][0] + gr[1] * S[1][0] + gr[2] * S[2][0];
        const float e1 = gr[0] * S[0][1] + gr[1] * S[1][1] + gr[2] * S[2][1];
        const float e2 = gr[0] * S[0][2] + gr[1] * S[1][2] + gr[2] * S[2][2];
        // d sh_kc = gr_c Y_k, summed over the views
        band_grad<0>(gr, Y, d);
        if (deg > 0) band_grad<1>(gr, Y, d);
        if (deg > 1) band_grad<2>(gr, Y, d);
        if (deg > 2) band_grad<3>(gr, Y, d);
        const double dd = (double)e0 * d0 + (double)e1 * d1 + (double)e2 * d2;
        dmu[0] += ((double)e0 - d0 * dd) * inv;
        dmu[1] += ((double)e1 - d1 * dd) * inv;
        dmu[2] += ((double)e2 - d2 * dd) * inv;
    }
#pragma unroll
    for (int q = 0; q < 12; ++q) row[q] = F4{d[4 * q + 0], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]};
}

struct Rotation {      // unit quaternion and 1 / |q|
    double w, x, y, z, inv;
    __device__ explicit Rotation(const float q[4]) {
        const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        inv = 1.0 / sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
        w = q0 * inv; x = q1 * inv; y = q2 * inv; z = q3 * inv;
    }
};

// Geometry chain of one seen Gaussian; dmu and dcb hold the colour chain's
// sums.  Writes every gradient but the coefficients', and the per-view
// statistics of the views that see it.
template <bool kZeroed, bool kMulti>
__device__ __forceinline__ void geometry_bwd_one(const GaussIn& in, bool has_app, const ViewTable& vt, const OptK& opt,
                                                 const float* __restrict__ grad2d, int64_t g2_stride, uint32_t vis,
                                                 double dmu[3], const float dcb[3], const GradPtrs& out, int64_t n,
                                                 int64_t g, float* __restrict__ mean2d_norm,
                                                 float* __restrict__ absgrad) {
    const double mu0 = in.mu[0], mu1 = in.mu[1], mu2 = in.mu[2];
    double M[9];   // R(q) diag(s)
    {
        const Rotation R(in.q);
        const double s0 = in.s[0], s1 = in.s[1], s2 = in.s[2];
        M[0] = (1.0 - 2.0 * (R.y * R.y + R.z * R.z)) * s0;
        M[1] = 2.0 * (R.x * R.y - R.w * R.z) * s1;
        M[2] = 2.0 * (R.x * R.z + R.w * R.y) * s2;
        M[3] = 2.0 * (R.x * R.y + R.w * R.z) * s0;
        M[4] = (1.0 - 2.0 * (R.x * R.x + R.z * R.z)) * s1;
        M[5] = 2.0 * (R.y * R.z - R.w * R.x) * s2;
        M[6] = 2.0 * (R.x * R.z - R.w * R.y) * s0;
        M[7] = 2.0 * (R.y * R.z + R.w * R.x) * s1;
        M[8] = (1.0 - 2.0 * (R.x * R.x + R.y * R.y)) * s2;
    }
    // appearance offsets: opacity o (1 - do)
    const double o = has_app ? (double)in.o * (1.0 - (double)in.app.w) : (double)in.o;

    double dM[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    double dop = 0.0;

    const int n_views = kMulti ? vt.n_views : 1;
    int v0 = 0;      // opaque: the views' constants are read here, not held in registers from batch to batch
    asm volatile("" : "+s"(v0));
    for (int v = 0; v < n_views; ++v) {
        if (kMulti && !(vis & (1u << v))) continue;
        const ViewK& V = vt.v[v + v0];
        const float* g2 = grad2d + v * g2_stride;
        if (kMulti) {
            const int64_t slot = v * n + g;
            mean2d_norm[slot] = sqrtf(g2[0] * g2[0] + g2[1] * g2[1]);
            if (absgrad) {
                absgrad[2 * slot] = g2[10];
                absgrad[2 * slot + 1] = g2[11];
            }
        }
        const double gmx = g2[0], gmy = g2[1], gA = g2[2], gB = g2[3], gC = g2[4], gop = g2[5];
        const double gz = g2[9];
        float W[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) W[i] = V.R[i];
        const double tx = W[0] * mu0 + W[1] * mu1 + W[2] * mu2 + (double)V.t[0];
        const double ty = W[3] * mu0 + W[4] * mu1 + W[5] * mu2 + (double)V.t[1];
        const double tz = W[6] * mu0 + W[7] * mu1 + W[8] * mu2 + (double)V.t[2];
        const double fx = V.fx, fy = V.fy;

        // recomputed as in the forward, but with 1 / tz once
        const double itz = 1.0 / tz, itz2 = itz * itz;
        const double u = tx * itz, vv = ty * itz;
        const bool ucl = u < V.ulo || u > V.uhi, vcl = vv < V.vlo || vv > V.vhi;
        const double uc = fmin(fmax(u, V.ulo), V.uhi), vc = fmin(fmax(vv, V.vlo), V.vhi);
        const double j00 = fx * itz, j02 = -j00 * uc, j11 = fy * itz, j12 = -j11 * vc;
        double Tm[6];
        Tm[0] = j00 * W[0] + j02 * W[6]; Tm[1] = j00 * W[1] + j02 * W[7]; Tm[2] = j00 * W[2] + j02 * W[8];
        Tm[3] = j11 * W[3] + j12 * W[6]; Tm[4] = j11 * W[4] + j12 * W[7]; Tm[5] = j11 * W[5] + j12 * W[8];
        double Vm[6];   // Tm M; Sigma_2D = Vm Vm^T
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 3; ++c)
                Vm[3 * r + c] = Tm[3 * r] * M[c] + Tm[3 * r + 1] * M[3 + c] + Tm[3 * r + 2] * M[6 + c];
        const double ca = Vm[0] * Vm[0] + Vm[1] * Vm[1] + Vm[2] * Vm[2];
        const double cb = Vm[0] * Vm[3] + Vm[1] * Vm[4] + Vm[2] * Vm[5];
        const double cc = Vm[3] * Vm[3] + Vm[4] * Vm[4] + Vm[5] * Vm[5];
        const double x0 = Vm[1] * Vm[5] - Vm[2] * Vm[4], x1 = Vm[2] * Vm[3] - Vm[0] * Vm[5],
                     x2 = Vm[0] * Vm[4] - Vm[1] * Vm[3];
        const double det2 = x0 * x0 + x1 * x1 + x2 * x2;
        const double dil = (double)opt.dilation;
        const double ad = ca + dil, cd = cc + dil;
        const double detd = det2 + dil * (ca + cc) + dil * dil;
        const double invd = 1.0 / detd;
        const double A = cd * invd, B = -cb * invd, C = ad * invd;
        const double rho = opt.aa ? (det2 > 0.0 ? sqrt(det2 * invd) : 0.0) : 1.0;

        double dt0 = 0.0, dt1 = 0.0, dt2 = 0.0;
        // mean2d = (fx tx/tz + cx, fy ty/tz + cy), depth = tz
        dt0 += gmx * j00;
        dt2 -= gmx * j00 * u;
        dt1 += gmy * j11;
        dt2 -= gmy * j11 * vv;
        dt2 += gz;
        // conic = inverse of [[ad, cb], [cb, cd]]
        double ga = gA * (-A * A) + gB * (-A * B) + gC * (-B * B);
        double gb = gA * (-2.0 * A * B) + gB * (-(A * C + B * B)) + gC * (-2.0 * B * C);
        double gc = gA * (-B * B) + gB * (-B * C) + gC * (-C * C);
        // opacity' = o rho, rho = sqrt(det2 / detd)
        dop += gop * rho;
        if (opt.aa && rho > 0.0) {
            const double k = gop * o / (2.0 * rho) * invd * invd;
            ga += k * (cc * detd - det2 * cd);
            gc += k * (ca * detd - det2 * ad);
            gb += k * (-2.0 * cb * detd + 2.0 * cb * det2);
        }
        // Sigma_2D = Vm Vm^T with the symmetric gradient G = [[ga, gb/2], [gb/2, gc]]
        const double G01 = 0.5 * gb;
        double dVm[6];
        for (int c = 0; c < 3; ++c) {
            dVm[c] = 2.0 * (ga * Vm[c] + G01 * Vm[3 + c]);
            dVm[3 + c] = 2.0 * (G01 * Vm[c] + gc * Vm[3 + c]);
        }
        // Vm = Tm M: dM += Tm^T dVm, dTm = dVm M^T
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) dM[3 * r + c] += Tm[r] * dVm[c] + Tm[3 + r] * dVm[3 + c];
        double dTm[6];
        for (int r = 0; r < 2; ++r)
            for (int c = 0; c < 3; ++c)
                dTm[3 * r + c] = dVm[3 * r] * M[3 * c] + dVm[3 * r + 1] * M[3 * c + 1] + dVm[3 * r + 2] * M[3 * c + 2];
        // dJ = dTm W^T; J has entries (0,0), (0,2), (1,1), (1,2)
        const double dJ00 = dTm[0] * W[0] + dTm[1] * W[1] + dTm[2] * W[2];
        const double dJ02 = dTm[0] * W[6] + dTm[1] * W[7] + dTm[2] * W[8];
        const double dJ11 = dTm[3] * W[3] + dTm[4] * W[4] + dTm[5] * W[5];
        const double dJ12 = dTm[3] * W[6] + dTm[4] * W[7] + dTm[5] * W[8];
        const double fxz2 = fx * itz2, fyz2 = fy * itz2;
        dt2 -= dJ00 * fxz2 + dJ11 * fyz2;
        if (!ucl) {
            dt0 -= dJ02 * fxz2;
            dt2 += dJ02 * (2.0 * fxz2 * u);
        } else {
            dt2 += dJ02 * (fxz2 * uc);
        }
        if (!vcl) {
            dt1 -= dJ12 * fyz2;
            dt2 += dJ12 * (2.0 * fyz2 * vv);
        } else {
            dt2 += dJ12 * (fyz2 * vc);
        }
        // t = W mu + t_w
        dmu[0] += W[0] * dt0 + W[3] * dt1 + W[6] * dt2;
        dmu[1] += W[1] * dt0 + W[4] * dt1 + W[7] * dt2;
        dmu[2] += W[2] * dt0 + W[5] * dt1 + W[8] * dt2;
    }

    // (opaque copies, so that the quaternion's and the scales' doubles are
    // computed again here and not held over the views)
    float qf[4], sf[3];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        qf[c] = in.q[c];
        asm volatile("" : "+v"(qf[c]));
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        sf[c] = in.s[c];
        asm volatile("" : "+v"(sf[c]));
    }
    const Rotation R(qf);
    const double w = R.w, x = R.x, y = R.y, z = R.z, iqn = R.inv;
    // M = R(q) diag(s): ds_c = sum_r dM[r][c] R[r][c], dR[r][c] = dM[r][c] s_c
    const double sc[3] = {sf[0], sf[1], sf[2]};
    double dR[9], ds[3] = {0.0, 0.0, 0.0};
    for (int c = 0; c < 3; ++c) {
        for (int r = 0; r < 3; ++r) {
            ds[c] += dM[3 * r + c] * M[3 * r + c];
            dR[3 * r + c] = dM[3 * r + c] * sc[c];
        }
        ds[c] /= sc[c];
    }
    // rotation of the unit quaternion (w, x, y, z)
    double dq[4];
    dq[0] = 2.0 * (-z * dR[1] + y * dR[2] + z * dR[3] - x * dR[5] - y * dR[6] + x * dR[7]);
    dq[1] = 2.0 * (y * dR[1] + z * dR[2] + y * dR[3] - 2.0 * x * dR[4] - w * dR[5] + z * dR[6] + w * dR[7] - 2.0 * x * dR[8]);
    dq[2] = 2.0 * (-2.0 * y * dR[0] + x * dR[1] + w * dR[2] + x * dR[3] + z * dR[5] - w * dR[6] + z * dR[7] - 2.0 * y * dR[8]);
    dq[3] = 2.0 * (-2.0 * z * dR[0] - w * dR[1] + x * dR[2] + w * dR[3] - 2.0 * z * dR[4] + y * dR[5] + x * dR[6] + y * dR[7]);
    // normalisation q / |q|
    const double dot = dq[0] * w + dq[1] * x + dq[2] * y + dq[3] * z;
    const double qh[4] = {w, x, y, z};
    const auto put = [&](int c, float v) {
        float* p = grad_row(out, n, g, c);
        // plain stores meet in L2: with the zeros that the scan wrote to the
        // line, or, with several views, with those of other batches
        if (kZeroed && !kMulti) __builtin_nontemporal_store(v, p);
        else *p = v;
    };
    for (int c = 0; c < 3; ++c) put(c, (float)dmu[c]);
    for (int c = 0; c < 3; ++c) put(3 + c, (float)ds[c]);
    for (int c = 0; c < 4; ++c) put(6 + c, (float)((dq[c] - qh[c] * dot) * iqn));
    // dop is the gradient with respect to o (1 - do)
    put(10, (float)(has_app ? dop * (1.0 - (double)in.app.w) : dop));
    if (out.app) {
        put(kRowApp + 0, dcb[0]);
        put(kRowApp + 1, dcb[1]);
        put(kRowApp + 2, dcb[2]);
        put(kRowApp + 3, (float)(-dop * (double)in.o));
    }
}


// kZeroed: the gradient outputs already hold zeros (gs_grads_zero, run
// beside the compositing backward), so only the entries of Gaussians some
// view sees are written.  One wave per workgroup; chunk k of the wave is
// chunk blockIdx.x + k gridDim.x of 64 * per Gaussians (per <= kChunkPer, at
// most 256 chunks per wave).
template <bool kZeroed, bool kMulti>
__global__ __launch_bounds__(64, 2) void k_project_bwd(GaussPtrs gp, uint32_t n, ViewTable vt, OptK opt, Projected proj,
                                                       const float* __restrict__ grad2d, GradPtrs out,
                                                       float* __restrict__ mean2d_norm, float* __restrict__ absgrad,
                                                       int per) {
    constexpr uint32_t kCap = 64 * (1 + kChunkPer);
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
    // one view: the next chunk's tile counts are read ahead of the chain
    uint32_t ahead[kChunkPer];
    const auto read_ahead = [&](uint32_t c) {
#pragma unroll
        for (int i = 0; i < kChunkPer; ++i) {
            const uint64_t g = (uint64_t)c * span + 64 * i + lane;
            ahead[i] = i < per && g < n ? proj.tiles[g] : 0u;
        }
    };
    if (!kMulti) read_ahead(chunk);
    for (;;) {
        // scan: list the seen Gaussians; zeros for the others
        while (cnt < 64 && chunk < n_chunks) {
            const uint32_t g0 = chunk * span;
            uint32_t ln = lane;      // opaque: no address is held over the chain
            asm volatile("" : "+v"(ln));
            uint32_t vis[kChunkPer];
            if (kMulti) {
                uint32_t t[GS_MAX_VIEWS][kChunkPer];
#pragma unroll
                for (int v = 0; v < GS_MAX_VIEWS; ++v)
#pragma unroll
                    for (int i = 0; i < kChunkPer; ++i) {
                        const uint64_t g = (uint64_t)g0 + 64 * i + ln;
                        t[v][i] = v < n_views && i < per && g < n ? proj.tiles[(int64_t)v * n + g] : 0u;
                    }
#pragma unroll
                for (int i = 0; i < kChunkPer; ++i) {
                    vis[i] = 0;
#pragma unroll
                    for (int v = 0; v < GS_MAX_VIEWS; ++v) vis[i] |= t[v][i] ? 1u << v : 0u;
                }
            } else {
#pragma unroll
                for (int i = 0; i < kChunkPer; ++i) vis[i] = ahead[i] ? 1u : 0u;
            }
            uint64_t seen[kChunkPer];
#pragma unroll
            for (int i = 0; i < kChunkPer; ++i) {
                const uint32_t loc = 64 * i + ln;
                const bool in = i < per && (uint64_t)g0 + loc < n;
                seen[i] = __ballot(vis[i] != 0);
                if (vis[i]) {
                    const uint32_t m = __builtin_amdgcn_mbcnt_hi((uint32_t)(seen[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)seen[i], 0));
                    s_list[cnt + m] = loc | k << 8 | vis[i] << 16;
                }
                cnt += (uint32_t)__popcll(seen[i]);
                // statistics: of every Gaussian, a whole line at a time, with
                // one view; with several the chain writes the seen ones'
                for (int v = 0; v < n_views; ++v)
                    if (in && (!kMulti || !(vis[i] & (1u << v)))) {
                        const int64_t slot = (int64_t)v * n + g0 + loc;
                        const bool read = !kMulti && vis[i];
                        const float* g2 = grad2d + slot * kG2;
                        const float gx = read ? g2[0] : 0.0f, gy = read ? g2[1] : 0.0f;
                        const float ax = read && absgrad ? g2[10] : 0.0f, ay = read && absgrad ? g2[11] : 0.0f;
                        if (kMulti) {
                            mean2d_norm[slot] = 0.0f;
                            if (absgrad) absgrad[2 * slot] = absgrad[2 * slot + 1] = 0.0f;
                        } else {
                            __builtin_nontemporal_store(sqrtf(gx * gx + gy * gy), mean2d_norm + slot);
                            if (absgrad) {
                                __builtin_nontemporal_store(ax, absgrad + 2 * slot);
                                __builtin_nontemporal_store(ay, absgrad + 2 * slot + 1);
                            }
                        }
                    }
                if (!kZeroed && in && !vis[i]) {
#pragma unroll
                    for (int c = 0; c < 11; ++c) *grad_row(out, n, g0 + loc, c) = 0.0f;
                    if (out.app) reinterpret_cast<float4*>(out.app)[g0 + loc] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
            }
            if (!kZeroed) {
                // zero coefficient rows, twelve neighbouring lanes to a row
                F4* dsh = reinterpret_cast<F4*>(out.sh) + (int64_t)12 * g0 + ln;
#pragma unroll
                for (int i = 0; i < kChunkPer; ++i)
                    for (int a = 0; a < 4 && i < per; ++a)
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const int r = 16 * a + rl.rc[c];
                            if ((uint64_t)g0 + 64 * i + r < n && !((seen[i] >> r) & 1))
                                __builtin_nontemporal_store(F4{0.0f, 0.0f, 0.0f, 0.0f}, dsh + 768 * i + 192 * a + 64 * c);
                        }
            }
            chunk += gridDim.x;
            ++k;
            if (!kMulti) read_ahead(chunk);
        }
        wave_sync();
        const bool last = chunk >= n_chunks;
        const uint32_t* lst = s_list;
        if (kMulti) {
            group_by_views(s_list, cnt, s_group, s_hist);
            lst = s_group;
        }
        // the chain, 64 listed Gaussians at a time (with several views,
        // those seen by the same views side by side); lanes past the end
        // work on the last one and write nothing
        uint32_t b = 0;
        for (; b + 64 <= cnt || (last && b < cnt); b += 64) {
            const int m = cnt - b < 64u ? (int)(cnt - b) : 64;
            const uint32_t e = lst[b + (lane < m ? lane : m - 1)];
            uint32_t g = (((e >> 8) & 255u) * gridDim.x + blockIdx.x) * span + (e & 255u);
            const GaussIn in = load_gauss(gp, n, g);
            double dmu[3] = {0.0, 0.0, 0.0};
            float dcb[3] = {0.0f, 0.0f, 0.0f};
            load_rows(gp.sh, g, nq, rl, s_rows);
            colour_bwd_one<kMulti>(in, vt, opt, grad2d + (int64_t)g * kG2, (int64_t)n * kG2, e >> 16,
                                   s_rows + lane * kRowF4, dmu, dcb);
            store_rows(out.sh, g, m, rl, s_rows);
            // (opaque, so that no address of the geometry's outputs is held
            // over the colour chain)
            asm volatile("" : "+v"(g) : : "memory");
            if (lane < m)
                geometry_bwd_one<kZeroed, kMulti>(in, gp.app != nullptr, vt, opt, grad2d + (int64_t)g * kG2, (int64_t)n * kG2,
                                         e >> 16, dmu, dcb, out, n, g, mean2d_norm, absgrad);
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

}  // namespace

hipError_t launch_project_bwd(const GaussPtrs& g, int64_t n, const ViewTable& vt, const OptK& opt,
                              const Projected& proj, const float* grad2d, const GradPtrs& out, float* mean2d_norm,
                              float* absgrad, hipStream_t s, bool grads_zeroed) {
    if (n > 0xFFFFFFFFLL) return hipErrorInvalidValue;     // Gaussians are kept as 32-bit indices
    if (!n) return hipSuccess;
    // chunks of 256 Gaussians when that leaves every wave several, else of 64
    const int per = n >= (int64_t)kMaxWaves * 64 * kChunkPer ? kChunkPer : 1;
    const int64_t chunks = (n + 64 * per - 1) / (64 * per);
    int64_t blocks = chunks < kMaxWaves ? chunks : kMaxWaves;
    if (blocks * 256 < chunks) blocks = (chunks + 255) / 256;
    const hipEvent_t timed_ = timer_begin(GS_KERNEL_PROJECT_BWD, s);
    const auto kernel = grads_zeroed ? (vt.n_views > 1 ? k_project_bwd<true, true> : k_project_bwd<true, false>)
                                     : (vt.n_views > 1 ? k_project_bwd<false, true> : k_project_bwd<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64), 0, s, g, (uint32_t)n, vt, opt, proj, grad2d, out, mean2d_norm,
                       absgrad, per);
    timer_end(timed_, s);
    return hipGetLastError();
}

namespace {

// Zeroes n floats with 16-byte streaming stores from a grid of at most
// kZeroGrid workgroups (grid-stride).  It runs beside the issue-bound
// compositing backward, which it should neither outlast nor slow: a training
// step over 6M Gaussians took 1797, 1770, 1759 and 1775 us with 64, 96, 128
// and 192 workgroups.
constexpr unsigned kZeroGrid = 128;
__global__ __launch_bounds__(256) void k_zero_floats(float* __restrict__ p, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t head = (int64_t)(((16 - ((uintptr_t)p & 15)) & 15) / 4);     // floats before the first 16-byte boundary
    const int64_t h = head < n ? head : n;
    const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i0 < h) p[i0] = 0.0f;
    F4* q = reinterpret_cast<F4*>(p + h);
    const int64_t n4 = (n - h) / 4;
    for (int64_t i = i0; i < n4; i += stride) __builtin_nontemporal_store(F4{0.0f, 0.0f, 0.0f, 0.0f}, q + i);
    const int64_t t = h + 4 * n4 + i0;
    if (t < n) p[t] = 0.0f;
}

}  // namespace

hipError_t launch_zero_grads(const GradPtrs& out, int64_t n, hipStream_t s) {
    const struct {
        float* p;
        int64_t count;
    } parts[] = {{out.means, 3 * n}, {out.scales, 3 * n}, {out.quats, 4 * n}, {out.opac, n}, {out.sh, 48 * n},
                 {out.app, out.app ? 4 * n : 0}};
    for (const auto& a : parts) {
        if (!a.p || a.count <= 0) continue;
        const int64_t need = (a.count / 4 + 255) / 256 + 1;
        const unsigned grid = (unsigned)(need < (int64_t)kZeroGrid ? need : (int64_t)kZeroGrid);
        hipLaunchKernelGGL(k_zero_floats, dim3(grid), dim3(256), 0, s, a.p, a.count);
    }
    return hipGetLastError();
}

}  // namespace gs
