// EWA projection of 3D Gaussians and its backward (one thread per Gaussian).
//
// PocketGS composites "depth-sorted visible Gaussians" (Sec. "Explicit
// Computation Graph") and inherits the projection from 3D Gaussian Splatting.
// Reading used: near plane 0.2, Sigma2D = (J W) Sigma (J W)^T + 0.3 I,
// J clamped at 1.3x the half field of view, radius ceil(3 sqrt(lambda_max))
// with lambda_max = m + sqrt(max(0.1, m^2 - det)), inclusive tile rectangle
// [floor((u-r)/TW), floor((u+r)/TW)] clipped to the image, real SH colour
// + 1/2 clamped at 0, sigmoid opacity.
//
// All per-Gaussian maths runs in float64 and is rounded once to float32.
// The work is bound by the canonical-parameter reads (56 B/Gaussian at SH
// degree 0, 236 B at degree 3), so the float64 ALU cost is hidden; in
// exchange every integer decision (culling, radius, rectangle, depth-key
// bits) is taken on values accurate to ~1e-16 relative.
#include <math.h>

#include "common.hpp"

namespace {

using pgs::CamD;

// Real SH normalisation constants (textbook values, Condon-Shortley phase):
constexpr double kY00 = 0.28209479177387814;   // 1/(2 sqrt(pi))
constexpr double kY1 = 0.4886025119029199;     // sqrt(3/(4 pi))
constexpr double kY2a = 1.0925484305920792;    // sqrt(15/(4 pi))
constexpr double kY2b = 0.31539156525252005;   // sqrt(5/(16 pi))
constexpr double kY2c = 0.5462742152960396;    // sqrt(15/(16 pi))
constexpr double kY3a = 0.5900435899266435;    // sqrt(35/(32 pi))
constexpr double kY3b = 2.890611442640554;     // sqrt(105/(4 pi))
constexpr double kY3c = 0.4570457994644658;    // sqrt(21/(32 pi))
constexpr double kY3d = 0.3731763325901154;    // sqrt(7/(16 pi))
constexpr double kY3e = 1.445305721320277;     // sqrt(105/(16 pi))

// Basis values Y[k], k = l*l + l + m, at unit direction (x, y, z).
template <int D>
__device__ __forceinline__ void sh_eval(double x, double y, double z, double* Y) {
    Y[0] = kY00;
    if (D >= 1) {
        Y[1] = -kY1 * y;
        Y[2] = kY1 * z;
        Y[3] = -kY1 * x;
    }
    if (D >= 2) {
        Y[4] = kY2a * x * y;
        Y[5] = -kY2a * y * z;
        Y[6] = kY2b * (3.0 * z * z - 1.0);
        Y[7] = -kY2a * x * z;
        Y[8] = kY2c * (x * x - y * y);
    }
    if (D >= 3) {
        Y[9] = -kY3a * y * (3.0 * x * x - y * y);
        Y[10] = kY3b * x * y * z;
        Y[11] = -kY3c * y * (5.0 * z * z - 1.0);
        Y[12] = kY3d * z * (5.0 * z * z - 3.0);
        Y[13] = -kY3c * x * (5.0 * z * z - 1.0);
        Y[14] = kY3e * z * (x * x - y * y);
        Y[15] = -kY3a * x * (x * x - 3.0 * y * y);
    }
}

// Gradient of polynomial Y[k] with respect to (x, y, z) (any extension off
// the sphere works: the chain through normalisation removes the radial
// part); k is a constant wherever this is called, so the switch folds away.
__device__ __forceinline__ void sh_grad_k(int k, double x, double y, double z, double& gx, double& gy,
                                          double& gz) {
    switch (k) {
        case 1: gx = 0.0; gy = -kY1; gz = 0.0; break;
        case 2: gx = 0.0; gy = 0.0; gz = kY1; break;
        case 3: gx = -kY1; gy = 0.0; gz = 0.0; break;
        case 4: gx = kY2a * y; gy = kY2a * x; gz = 0.0; break;
        case 5: gx = 0.0; gy = -kY2a * z; gz = -kY2a * y; break;
        case 6: gx = 0.0; gy = 0.0; gz = 6.0 * kY2b * z; break;
        case 7: gx = -kY2a * z; gy = 0.0; gz = -kY2a * x; break;
        case 8: gx = 2.0 * kY2c * x; gy = -2.0 * kY2c * y; gz = 0.0; break;
        case 9: gx = -6.0 * kY3a * x * y; gy = -3.0 * kY3a * (x * x - y * y); gz = 0.0; break;
        case 10: gx = kY3b * y * z; gy = kY3b * x * z; gz = kY3b * x * y; break;
        case 11: gx = 0.0; gy = -kY3c * (5.0 * z * z - 1.0); gz = -10.0 * kY3c * y * z; break;
        case 12: gx = 0.0; gy = 0.0; gz = kY3d * (15.0 * z * z - 3.0); break;
        case 13: gx = -kY3c * (5.0 * z * z - 1.0); gy = 0.0; gz = -10.0 * kY3c * x * z; break;
        case 14: gx = 2.0 * kY3e * x * z; gy = -2.0 * kY3e * y * z; gz = kY3e * (x * x - y * y); break;
        case 15: gx = -3.0 * kY3a * (x * x - y * y); gy = 6.0 * kY3a * x * y; gz = 0.0; break;
        default: gx = gy = gz = 0.0; break;
    }
}

// Geometry shared by the forward and the backward kernels: the part that
// does not depend on the view (rotation, scales, 3D covariance) and the
// per-view part (camera-space mean, Jacobian, 2D covariance).
struct Shape {
    double qn[4], qlen;      // normalised quaternion and |q|
    double R[9];             // rotation of the Gaussian
    double s[3];             // exp(log-scale)
    double Sig[6];           // 3D covariance xx, xy, xz, yy, yz, zz
};

struct Geo {
    double x, y, z;          // camera-space mean
    double tx, ty;           // clamped x/z, y/z
    bool clx, cly;           // J clamp active
    double T0[3], T1[3];     // rows of J W
    double a, b, c, det;     // Sigma2D with dilation
};

__device__ __forceinline__ double prow(const float* P, int r, int n, int i) {
    return (double)P[(size_t)r * n + i];
}

__device__ __forceinline__ void shape_of(const float* __restrict__ P, int n, int i, Shape& S3) {
    const double qw = prow(P, 6, n, i), qx = prow(P, 7, n, i), qy = prow(P, 8, n, i),
                 qz = prow(P, 9, n, i);
    S3.qlen = sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    const double w = qw / S3.qlen, x = qx / S3.qlen, y = qy / S3.qlen, z = qz / S3.qlen;
    S3.qn[0] = w; S3.qn[1] = x; S3.qn[2] = y; S3.qn[3] = z;
    double* R = S3.R;
    R[0] = 1.0 - 2.0 * (y * y + z * z); R[1] = 2.0 * (x * y - w * z); R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z); R[4] = 1.0 - 2.0 * (x * x + z * z); R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y); R[7] = 2.0 * (y * z + w * x); R[8] = 1.0 - 2.0 * (x * x + y * y);
    for (int k = 0; k < 3; ++k) S3.s[k] = exp(prow(P, 3 + k, n, i));
    // Sigma = R diag(s^2) R^T
    const double s0 = S3.s[0] * S3.s[0], s1 = S3.s[1] * S3.s[1], s2 = S3.s[2] * S3.s[2];
    auto sig = [&](int r, int c) { return R[3 * r] * R[3 * c] * s0 + R[3 * r + 1] * R[3 * c + 1] * s1 + R[3 * r + 2] * R[3 * c + 2] * s2; };
    S3.Sig[0] = sig(0, 0); S3.Sig[1] = sig(0, 1); S3.Sig[2] = sig(0, 2);
    S3.Sig[3] = sig(1, 1); S3.Sig[4] = sig(1, 2); S3.Sig[5] = sig(2, 2);
}

__device__ __forceinline__ void view_geometry(const double (&mu)[3], const Shape& S3, const CamD& cam, Geo& G) {
    const double mx = mu[0], my = mu[1], mz = mu[2];
    G.x = cam.R[0] * mx + cam.R[1] * my + cam.R[2] * mz + cam.t[0];
    G.y = cam.R[3] * mx + cam.R[4] * my + cam.R[5] * mz + cam.t[1];
    G.z = cam.R[6] * mx + cam.R[7] * my + cam.R[8] * mz + cam.t[2];
    const double xz = G.x / G.z, yz = G.y / G.z;
    G.clx = (xz < -cam.lim_x) || (xz > cam.lim_x);
    G.cly = (yz < -cam.lim_y) || (yz > cam.lim_y);
    G.tx = fmin(cam.lim_x, fmax(-cam.lim_x, xz));
    G.ty = fmin(cam.lim_y, fmax(-cam.lim_y, yz));
    const double j00 = cam.fx / G.z, j02 = -cam.fx * G.tx / G.z;
    const double j11 = cam.fy / G.z, j12 = -cam.fy * G.ty / G.z;
    for (int k = 0; k < 3; ++k) {
        G.T0[k] = j00 * cam.R[k] + j02 * cam.R[6 + k];
        G.T1[k] = j11 * cam.R[3 + k] + j12 * cam.R[6 + k];
    }
    const double* S = S3.Sig;
    const double U0 = S[0] * G.T0[0] + S[1] * G.T0[1] + S[2] * G.T0[2];
    const double U1 = S[1] * G.T0[0] + S[3] * G.T0[1] + S[4] * G.T0[2];
    const double U2 = S[2] * G.T0[0] + S[4] * G.T0[1] + S[5] * G.T0[2];
    const double V0 = S[0] * G.T1[0] + S[1] * G.T1[1] + S[2] * G.T1[2];
    const double V1 = S[1] * G.T1[0] + S[3] * G.T1[1] + S[4] * G.T1[2];
    const double V2 = S[2] * G.T1[0] + S[4] * G.T1[1] + S[5] * G.T1[2];
    G.a = G.T0[0] * U0 + G.T0[1] * U1 + G.T0[2] * U2 + 0.3;
    G.b = G.T0[0] * V0 + G.T0[1] * V1 + G.T0[2] * V2;
    G.c = G.T1[0] * V0 + G.T1[1] * V1 + G.T1[2] * V2 + 0.3;
    G.det = G.a * G.c - G.b * G.b;
}

// Half-extents (x, y) of the pixel region where the compositing kernels can
// find alpha >= 1/255 for a splat with the float32 conic (A, B, C) and
// opacity o that they read.  The region is the ellipse
// A dx^2 + 2B dx dy + C dy^2 <= tau, tau = 2 ln(255 o), enlarged so that it
// also covers the float32 evaluation of the quadratic form (relative error
// below 20 * 2^-24 / (1 - rho), rho = |B| / sqrt(AC)) and of exp (1e-3 added
// to tau).  (-1, -1) when o is below the threshold (no pixel qualifies);
// (inf, inf) when the conic is too close to degenerate (1 - rho < 1e-3) for
// the bound, so that nothing is skipped.  The extents are part of the record
// for its readers outside; the compositing kernels test each wave's rows
// against the conic itself, which keeps fewer splats.
__device__ __forceinline__ double alpha_tau(float o) { return 2.0 * log(255.0 * fmax((double)o, 1.0 / 255.0)); }

__device__ __forceinline__ void alpha_extent(float A, float B, float C, float o, double tau, float& hx, float& hy) {
    if (o < pgs::kAlphaMin * (1.0f - 1e-6f)) {
        hx = hy = -1.f;
        return;
    }
    const double a = A, b = B, c = C;
    const double det = a * c - b * b;
    const double one_m_rho = 1.0 - fabs(b) / sqrt(a * c);
    if (!(det > 0.0) || !(a > 0.0) || !(c > 0.0) || !(one_m_rho >= 1e-3)) {
        hx = hy = INFINITY;
        return;
    }
    const double eta = 20.0 * 0x1p-24 / one_m_rho;
    const double t = (tau + 1e-3) / (1.0 - eta);
    hx = (float)(sqrt(t * c / det) * (1.0 + 1e-5) + 1e-2);
    hy = (float)(sqrt(t * a / det) * (1.0 + 1e-5) + 1e-2);
}

__device__ __forceinline__ float opacity_of(const float* __restrict__ P, int n, int i) {
    return (float)(1.0 / (1.0 + exp(-prow(P, 10, n, i))));
}

// Projection of Gaussian i into one view: its record's first 12 words in rec
// (the last four are zero; all zero where it is culled), radius, rectangle and
// tile count at index i of that view's arrays.  coef(k, ch): SH coefficient;
// o32, tau: its opacity and alpha_tau of it.
template <int D, class Coef>
__device__ __forceinline__ void project_view(const double (&mu)[3], int n, int i, const Shape& S3, float o32, double tau,
                                             Coef&& coef, const CamD& cam, int tw, int th, int TX, int TY,
                                             float4 (&rec)[3], int* __restrict__ radius,
                                             uint32_t* __restrict__ rect, uint32_t* __restrict__ touched) {
    constexpr int K = (D + 1) * (D + 1);
    Geo G;
    view_geometry(mu, S3, cam, G);
    bool ok = G.z > 0.2 && G.det > 0.0;
    double u = 0, v = 0, r = 0, x0 = 0, x1 = -1, y0 = 0, y1 = -1;
    if (ok) {
        u = cam.fx * G.x / G.z + cam.cx;
        v = cam.fy * G.y / G.z + cam.cy;
        const double mid = 0.5 * (G.a + G.c);
        const double lam = mid + sqrt(fmax(0.1, mid * mid - G.det));
        r = ceil(3.0 * sqrt(lam));
        x0 = fmin(fmax(floor((u - r) / tw), 0.0), (double)TX);
        x1 = fmin(fmax(floor((u + r) / tw), -1.0), (double)(TX - 1));
        y0 = fmin(fmax(floor((v - r) / th), 0.0), (double)TY);
        y1 = fmin(fmax(floor((v + r) / th), -1.0), (double)(TY - 1));
        ok = isfinite(u) && isfinite(v) && x0 <= x1 && y0 <= y1;
    }
    if (!ok) {
        rec[0] = rec[1] = rec[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        radius[i] = 0;
        rect[i] = 0;
        rect[(size_t)n + i] = 0;
        touched[i] = 0;
        return;
    }
    // colour from the view direction
    double d0 = mu[0] - cam.campos[0];
    double d1 = mu[1] - cam.campos[1];
    double d2 = mu[2] - cam.campos[2];
    const double dl = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
    d0 /= dl; d1 /= dl; d2 /= dl;
    double Y[K];
    sh_eval<D>(d0, d1, d2, Y);
    double col[3];
    for (int ch = 0; ch < 3; ++ch) {
        double acc = 0.5;
        for (int k = 0; k < K; ++k) acc += Y[k] * coef(k, ch);
        col[ch] = fmax(acc, 0.0);
    }
    static_assert(PGS_PROJ_U == 0 && PGS_PROJ_V == 1 && PGS_PROJ_DEPTH == 2 && PGS_PROJ_A == 3 &&
                      PGS_PROJ_B == 4 && PGS_PROJ_C == 5 && PGS_PROJ_OPACITY == 6 && PGS_PROJ_R == 7 &&
                      PGS_PROJ_G == 8 && PGS_PROJ_BLUE == 9 && PGS_PROJ_STRIDE == 16,
                  "record layout");
    const float A32 = (float)(G.c / G.det), B32 = (float)(-G.b / G.det), C32 = (float)(G.a / G.det);
    float hx, hy;
    alpha_extent(A32, B32, C32, o32, tau, hx, hy);
    rec[0] = make_float4((float)u, (float)v, (float)G.z, A32);
    rec[1] = make_float4(B32, C32, o32, (float)col[0]);
    rec[2] = make_float4((float)col[1], (float)col[2], hx, hy);
    radius[i] = (int)r;
    const uint32_t ix0 = (uint32_t)x0, ix1 = (uint32_t)x1, iy0 = (uint32_t)y0, iy1 = (uint32_t)y1;
    rect[i] = ix0 | (iy0 << 16);
    rect[(size_t)n + i] = ix1 | (iy1 << 16);
    touched[i] = (ix1 - ix0 + 1) * (iy1 - iy0 + 1);
}

template <int D>
__global__ __launch_bounds__(256) void k_project(const float* __restrict__ P, int n, CamD cam,
                                                 int tw, int th, int TX, int TY,
                                                 float* __restrict__ out, int* __restrict__ radius,
                                                 uint32_t* __restrict__ rect,
                                                 uint32_t* __restrict__ touched) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Shape S3;
    shape_of(P, n, i, S3);
    const float o = opacity_of(P, n, i);
    const double mu[3] = {prow(P, 0, n, i), prow(P, 1, n, i), prow(P, 2, n, i)};
    float4 rec[3];
    project_view<D>(mu, n, i, S3, o, alpha_tau(o),
                    [&](int k, int ch) { return prow(P, 11 + 3 * k + ch, n, i); }, cam, tw, th, TX, TY, rec, radius,
                    rect, touched);
    float4* dst = reinterpret_cast<float4*>(out + (size_t)i * PGS_PROJ_STRIDE);
    dst[0] = rec[0];
    dst[1] = rec[1];
    dst[2] = rec[2];
    dst[3] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Up to kLaunchViews views per multi-view launch, cameras by value.
constexpr int kLaunchViews = 8;
struct LaunchViews {
    int nv, v0;  // views in this launch, index of the first
    CamD cam[kLaunchViews];
    int TX[kLaunchViews], TY[kLaunchViews];
};

// Start of row r at a wave's first Gaussian, kept a scalar: left to itself the
// compiler steps a 64-bit address per lane from row to row and holds all of
// them until the stores.
template <class T>
__device__ __forceinline__ T* row_start(T* base, int r, int n) {
    size_t off = (size_t)r * n;
    asm volatile("" : "+s"(off));
    return base + off;
}

// Every view of a launch for one Gaussian: shape and opacity once, the SH
// coefficients read once and kept in LDS (a column per lane, no barrier).
// Re-read from cache by every view, they and their addresses left room for
// one wave per SIMD at SH degree 3: eight views of 1M Gaussians 422 us, now
// 361, bound by the store of their records and by float64 arithmetic.
// Up to degree 1 a view's 64 records, 4 KB in a row, turn in LDS (chunks
// swizzled over the banks) and leave as whole lines: 300k at degree 0 60 us
// stored lane by lane, 53 turned.  From degree 2 on the LDS for it costs more
// waves than it gains (degree 2 74 against 84 us, degree 3 361 against 393).
template <int D>
__global__ __launch_bounds__(64, 3) void k_project_views(const float* __restrict__ P, int n, LaunchViews lv,
                                                         int tw, int th, float* __restrict__ out_all,
                                                         int* __restrict__ radius_all,
                                                         uint32_t* __restrict__ rect_all,
                                                         uint32_t* __restrict__ touched_all) {
    constexpr int K = (D + 1) * (D + 1);
    __shared__ float sh[3 * K][64];
    __shared__ float4 turn[D < 2 ? 64 * 4 : 1];
    const int i0 = blockIdx.x * 64, lane = threadIdx.x;
    if (i0 + lane >= n) return;
    const int chunks = 4 * min(64, n - i0);
#pragma unroll
    for (int r = 0; r < 3 * K; ++r) sh[r][lane] = row_start(P + i0, 11 + r, n)[lane];
    Shape S3;
    shape_of(P + i0, n, lane, S3);
    const double mu[3] = {prow(P + i0, 0, n, lane), prow(P + i0, 1, n, lane), prow(P + i0, 2, n, lane)};
    const float o = opacity_of(P + i0, n, lane);
    const double tau = alpha_tau(o);
#pragma unroll 1
    for (int k = 0; k < lv.nv; ++k) {
        const size_t at = (size_t)(lv.v0 + k) * n + i0;
        int l = lane;  // opaque per view: the coefficients stay in LDS
        asm volatile("" : "+v"(l));
        float4 rec[3];
        project_view<D>(mu, n, lane, S3, o, tau, [&](int q, int ch) { return (double)sh[3 * q + ch][l]; },
                        lv.cam[k], tw, th, lv.TX[k], lv.TY[k], rec, radius_all + at,
                        rect_all + at + (size_t)(lv.v0 + k) * n, touched_all + at);
        float4* dst = reinterpret_cast<float4*>(out_all + at * PGS_PROJ_STRIDE);
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (D < 2) {
            const auto slot = [](int record, int c) { return 4 * record + (c ^ ((record >> 2) & 3)); };
#pragma unroll
            for (int c = 0; c < 4; ++c) turn[slot(lane, c)] = c < 3 ? rec[c] : zero;
            wave_fence();
            for (int q = lane; q < chunks; q += min(64, n - i0)) dst[q] = turn[slot(q >> 2, q & 3)];
            wave_fence();
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) dst[4 * lane + c] = c < 3 ? rec[c] : zero;
        }
    }
}

// Backward: exact derivative of k_project's outputs (u, v, A, B, C, o, rgb)
// with every discrete decision frozen, accumulated into the canonical
// gradient rows: each view adds in float64 and rounds to float32, in view
// order, whether the views share a launch or not.
//
// One thread walks the views twice.  The first walk keeps the eleven rows of
// mean, scale, rotation and opacity in registers and decides which colour
// channels are clamped; the second keeps the SH rows, with the direction and
// the basis formed again.  The SH coefficients, which the first walk reads
// twice in every view, wait in LDS (a column per lane, no barrier).  One walk
// with all rows and coefficients in registers left room for a single wave per
// SIMD at SH degree 3, whose memory accesses nothing hid: eight views of 1M
// Gaussians 1335 us, now 388; one view of 100k 39, now 25.

// Unit vector from the camera to the mean and its length's reciprocal.
__device__ __forceinline__ double view_direction(const double (&mu)[3], const CamD& cam, double (&d)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = mu[k] - cam.campos[k];
    const double inv = 1.0 / sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] *= inv;
    return inv;
}

// What one view adds to a Gaussian's rows 0..9 (mean, log-scales,
// quaternion), without the mean's part through the colour.
__device__ __forceinline__ void bwd_geometry(const double (&mu)[3], const Shape& S3, const CamD& cam, double gu,
                                             double gv, double gA, double gB, double gC, double (&gmu)[3],
                                             double (&glog)[3], double (&gqraw)[4]) {
    Geo G;
    view_geometry(mu, S3, cam, G);
    const double a = G.a, b = G.b, c = G.c, idet2 = 1.0 / (G.det * G.det);
    // conic (A, B, C) = (c, -b, a) / det  ->  Sigma2D entries
    const double ga = (-c * c * gA + b * c * gB - b * b * gC) * idet2;
    const double gb = (2.0 * b * c * gA - (a * c + b * b) * gB + 2.0 * a * b * gC) * idet2;
    const double gc = (-b * b * gA + a * b * gB - a * a * gC) * idet2;
    // symmetric 2x2 gradient of Sigma2D
    const double G00 = ga, G01 = 0.5 * gb, G11 = gc;
    const double* S = S3.Sig;
    double Sm[3][3] = {{S[0], S[1], S[2]}, {S[1], S[3], S[4]}, {S[2], S[4], S[5]}};
    // dL/dSigma = T^T G2 T (3x3 symmetric)
    double GS[3][3];
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q)
            GS[r][q] = G.T0[r] * (G00 * G.T0[q] + G01 * G.T1[q]) +
                       G.T1[r] * (G01 * G.T0[q] + G11 * G.T1[q]);
    // dL/dT = 2 G2 T Sigma (2x3)
    double TS0[3], TS1[3];
    for (int q = 0; q < 3; ++q) {
        TS0[q] = G.T0[0] * Sm[0][q] + G.T0[1] * Sm[1][q] + G.T0[2] * Sm[2][q];
        TS1[q] = G.T1[0] * Sm[0][q] + G.T1[1] * Sm[1][q] + G.T1[2] * Sm[2][q];
    }
    double dT0[3], dT1[3];
    for (int q = 0; q < 3; ++q) {
        dT0[q] = 2.0 * (G00 * TS0[q] + G01 * TS1[q]);
        dT1[q] = 2.0 * (G01 * TS0[q] + G11 * TS1[q]);
    }
    // T = J W: dL/dJ = dL/dT W^T; only J00, J02, J11, J12 are non-zero
    const double* W = cam.R;
    const double gJ00 = dT0[0] * W[0] + dT0[1] * W[1] + dT0[2] * W[2];
    const double gJ02 = dT0[0] * W[6] + dT0[1] * W[7] + dT0[2] * W[8];
    const double gJ11 = dT1[0] * W[3] + dT1[1] * W[4] + dT1[2] * W[5];
    const double gJ12 = dT1[0] * W[6] + dT1[1] * W[7] + dT1[2] * W[8];
    const double iz = 1.0 / G.z, iz2 = iz * iz;
    double gx = 0, gy = 0, gz = 0;
    // J00 = fx/z, J02 = -fx tx/z (tx = x/z unless clamped), same in y
    gz -= iz2 * (cam.fx * gJ00 + cam.fy * gJ11);
    gz += iz2 * (cam.fx * G.tx * gJ02 + cam.fy * G.ty * gJ12);
    if (!G.clx) {
        gx -= cam.fx * iz2 * gJ02;
        gz += cam.fx * G.x * (iz2 * iz) * gJ02;
    }
    if (!G.cly) {
        gy -= cam.fy * iz2 * gJ12;
        gz += cam.fy * G.y * (iz2 * iz) * gJ12;
    }
    // pixel mean
    gx += gu * cam.fx * iz;
    gy += gv * cam.fy * iz;
    gz -= iz2 * (gu * cam.fx * G.x + gv * cam.fy * G.y);
    // x_c = W mu + t
    for (int k = 0; k < 3; ++k) gmu[k] = W[k] * gx + W[3 + k] * gy + W[6 + k] * gz;

    // Sigma = M M^T, M = R diag(s): dL/dM = 2 dL/dSigma M
    double M[3][3], gM[3][3];
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q) M[r][q] = S3.R[3 * r + q] * S3.s[q];
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q)
            gM[r][q] = 2.0 * (GS[r][0] * M[0][q] + GS[r][1] * M[1][q] + GS[r][2] * M[2][q]);
    double gR[9];
    for (int q = 0; q < 3; ++q) {
        double a_ = 0.0;
        for (int r = 0; r < 3; ++r) {
            a_ += gM[r][q] * S3.R[3 * r + q];
            gR[3 * r + q] = gM[r][q] * S3.s[q];
        }
        glog[q] = a_ * S3.s[q];
    }
    const double w = S3.qn[0], x = S3.qn[1], y = S3.qn[2], zq = S3.qn[3];
    double gq[4];
    gq[0] = 2.0 * (-zq * gR[1] + y * gR[2] + zq * gR[3] - x * gR[5] - y * gR[6] + x * gR[7]);
    gq[1] = 2.0 * (y * gR[1] + zq * gR[2] + y * gR[3] - 2.0 * x * gR[4] - w * gR[5] +
                   zq * gR[6] + w * gR[7] - 2.0 * x * gR[8]);
    gq[2] = 2.0 * (-2.0 * y * gR[0] + x * gR[1] + w * gR[2] + x * gR[3] + zq * gR[5] -
                   w * gR[6] + zq * gR[7] - 2.0 * y * gR[8]);
    gq[3] = 2.0 * (-2.0 * zq * gR[0] - w * gR[1] + x * gR[2] + w * gR[3] - 2.0 * zq * gR[4] +
                   y * gR[5] + x * gR[6] + y * gR[7]);
    const double dotq = gq[0] * w + gq[1] * x + gq[2] * y + gq[3] * zq;
    for (int k = 0; k < 4; ++k) gqraw[k] = (gq[k] - S3.qn[k] * dotq) / S3.qlen;
}

// Four words of a 2D-gradient record, of which a float's alignment is asked.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Lane's Gaussian of a wave; P and grads point at the wave's first Gaussian, so
// that a row's address is a scalar and the lane's offset.  Bit k of seen: view k
// holds the Gaussian.  view(k, rec) gives view k's camera and where its 2D
// gradients of the wave begin; they are loaded one view ahead.
template <int D, class View>
__device__ __forceinline__ void project_bwd_rows(const float* __restrict__ P, int n, int lane, int nv, uint32_t seen, View&& view,
                                                 float* __restrict__ grads, float (*sh)[64]) {
    constexpr int K = (D + 1) * (D + 1);
#pragma unroll
    for (int r = 0; r < 3 * K; ++r) sh[r][lane] = row_start(P, 11 + r, n)[lane];
    double mu[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) mu[k] = prow(P, k, n, lane);
    Shape S3;
    shape_of(P, n, lane, S3);
    const double o = 1.0 / (1.0 + exp(-prow(P, 10, n, lane))), go_do = o * (1.0 - o);
    uint32_t open = 0u;  // bits 3k..3k+2: unclamped channels of view k
    {
        float acc[11];
#pragma unroll
        for (int r = 0; r < 11; ++r) acc[r] = row_start(grads, r, n)[lane];
        const auto add = [&](int r, double g) { acc[r] = (float)((double)acc[r] + g); };
        f32x4u n0, n1;
        float n2;
        const auto fetch = [&](int k) {
            if (!((seen >> k) & 1u)) return;  // also past the last view
            const float* rec;
            view(k, rec);
            rec += lane * PGS_GRAD2D_STRIDE;
            n0 = reinterpret_cast<const f32x4u*>(rec)[0];
            n1 = reinterpret_cast<const f32x4u*>(rec)[1];
            n2 = rec[8];
        };
        fetch(0);
#pragma unroll 1
        for (int k = 0; k < nv; ++k) {
            const float* rec;
            const CamD& cam = view(k, rec);
            const f32x4u r0 = n0, r1 = n1;
            const float gcol[3] = {r1.z, r1.w, n2};
            fetch(k + 1);
            if (!((seen >> k) & 1u)) continue;
            // opaque per view: the coefficients stay in LDS, and products of
            // scales and rotation are formed again, instead of being held in
            // registers across the loop
            int l = lane;
            asm volatile("" : "+v"(l), "+v"(S3.s[0]), "+v"(S3.s[1]), "+v"(S3.s[2]));
            asm volatile("" : "+v"(S3.qn[0]), "+v"(S3.qn[1]), "+v"(S3.qn[2]), "+v"(S3.qn[3]));
            // colour: c = max(0, sum_k Y_k(d) f_k + 1/2), d = unit(mu - campos)
            double gd[3] = {0.0, 0.0, 0.0};
            {
                double d[3], Y[K], graw[3];
                const double inv = view_direction(mu, cam, d);
                sh_eval<D>(d[0], d[1], d[2], Y);
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) {
                    double c_ = 0.5;
#pragma unroll
                    for (int q = 0; q < K; ++q) c_ += Y[q] * (double)sh[3 * q + ch][l];
                    graw[ch] = c_ >= 0.0 ? (double)gcol[ch] : 0.0;
                    open |= c_ >= 0.0 ? 1u << (3 * k + ch) : 0u;
                }
                if (D >= 1) {
                    asm volatile("" : "+v"(l));  // read again, not kept
#pragma unroll
                    for (int q = 1; q < K; ++q) {
                        const double g = (double)sh[3 * q][l] * graw[0] + (double)sh[3 * q + 1][l] * graw[1] +
                                         (double)sh[3 * q + 2][l] * graw[2];
                        double dx, dy, dz;
                        sh_grad_k(q, d[0], d[1], d[2], dx, dy, dz);
                        gd[0] += g * dx;
                        gd[1] += g * dy;
                        gd[2] += g * dz;
                    }
                    const double dd = gd[0] * d[0] + gd[1] * d[1] + gd[2] * d[2];
#pragma unroll
                    for (int q = 0; q < 3; ++q) gd[q] = (gd[q] - d[q] * dd) * inv;
                }
            }
            double gmu[3], glog[3], gqraw[4];
            bwd_geometry(mu, S3, cam, r0.x, r0.y, r0.z, r0.w, r1.x, gmu, glog, gqraw);
#pragma unroll
            for (int q = 0; q < 3; ++q) add(q, gmu[q] + gd[q]);
#pragma unroll
            for (int q = 0; q < 3; ++q) add(3 + q, glog[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) add(6 + q, gqraw[q]);
            add(10, (double)r1.y * go_do);
        }
#pragma unroll
        for (int r = 0; r < 11; ++r) row_start(grads, r, n)[lane] = acc[r];
    }
    __builtin_amdgcn_sched_barrier(0);  // one view: the SH rows are not loaded ahead of the first walk
    float acc[3 * K];
#pragma unroll
    for (int r = 0; r < 3 * K; ++r) acc[r] = row_start(grads, 11 + r, n)[lane];
    float ahead[3];
    const auto fetch = [&](int k) {
        if (!((seen >> k) & 1u)) return;
        const float* rec;
        view(k, rec);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) ahead[ch] = rec[lane * PGS_GRAD2D_STRIDE + 6 + ch];
    };
    fetch(0);
#pragma unroll 1
    for (int k = 0; k < nv; ++k) {
        const float* rec;
        const CamD& cam = view(k, rec);
        double d[3], Y[K], graw[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) graw[ch] = (open >> (3 * k + ch)) & 1u ? (double)ahead[ch] : 0.0;
        fetch(k + 1);
        if (!((seen >> k) & 1u)) continue;
        view_direction(mu, cam, d);
        sh_eval<D>(d[0], d[1], d[2], Y);
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) acc[3 * q + ch] = (float)((double)acc[3 * q + ch] + Y[q] * graw[ch]);
    }
#pragma unroll
    for (int r = 0; r < 3 * K; ++r) row_start(grads, 11 + r, n)[lane] = acc[r];
}

template <int D>
__global__ __launch_bounds__(64, D == 3 ? 2 : 3) void k_project_bwd(const float* __restrict__ P, int n, CamD cam,
                                                       const int* __restrict__ radius,
                                                       const float* __restrict__ g2d, float* __restrict__ grads) {
    __shared__ float sh[3 * (D + 1) * (D + 1)][64];
    const int i0 = blockIdx.x * 64, lane = threadIdx.x;
    if (i0 + lane >= n || radius[i0 + lane] == 0) return;
    project_bwd_rows<D>(P + i0, n, lane, 1, 1u,
                        [&](int, const float*& rec) -> const CamD& {
                            rec = g2d + (size_t)i0 * PGS_GRAD2D_STRIDE;
                            return cam;
                        },
                        grads + i0, sh);
}

template <int D>
__global__ __launch_bounds__(64, 3) void k_project_bwd_views(const float* __restrict__ P, int n, LaunchViews lv,
                                                             const int* __restrict__ radius_all,
                                                             const float* __restrict__ g2d_all,
                                                             float* __restrict__ grads) {
    static_assert(3 * kLaunchViews <= 32, "a bit per view and channel");
    __shared__ float sh[3 * (D + 1) * (D + 1)][64];
    const int i0 = blockIdx.x * 64, lane = threadIdx.x;
    if (i0 + lane >= n) return;
    uint32_t seen = 0u;
#pragma unroll
    for (int k = 0; k < kLaunchViews; ++k)
        if (k < lv.nv && radius_all[(size_t)(lv.v0 + k) * n + i0 + lane] != 0) seen |= 1u << k;
    if (seen == 0u) return;
    project_bwd_rows<D>(P + i0, n, lane, lv.nv, seen,
                        [&](int k, const float*& rec) -> const CamD& {
                            rec = g2d_all + ((size_t)(lv.v0 + k) * n + i0) * PGS_GRAD2D_STRIDE;
                            return lv.cam[k];
                        },
                        grads + i0, sh);
}

}  // namespace

extern "C" pgs_status pgs_project(const float* params_dev, int32_t n, int32_t sh_degree,
                                  const pgs_camera* cam_host, int32_t tile_w, int32_t tile_h,
                                  float* proj_dev, int32_t* radius_dev, uint32_t* rect_dev,
                                  uint32_t* touched_dev, void* stream) {
    PGS_REQUIRE(n >= 0, "pgs_project: n < 0");
    PGS_REQUIRE(sh_degree >= 0 && sh_degree <= 3, "pgs_project: sh_degree %d", sh_degree);
    PGS_REQUIRE(cam_host != nullptr, "pgs_project: null camera");
    PGS_REQUIRE(cam_host->width > 0 && cam_host->height > 0 && tile_w > 0 && tile_h > 0,
                "pgs_project: bad image/tile size");
    const int TX = (cam_host->width + tile_w - 1) / tile_w;
    const int TY = (cam_host->height + tile_h - 1) / tile_h;
    PGS_REQUIRE(TX <= 65535 && TY <= 65535, "pgs_project: too many tiles");
    if (n == 0) return PGS_OK;
    PGS_REQUIRE(params_dev && proj_dev && radius_dev && rect_dev && touched_dev,
                "pgs_project: null pointer");
    const pgs::CamD cam = pgs::make_cam(*cam_host);
    const dim3 grid((n + 255) / 256), block(256);
    hipStream_t s = pgs::as_stream(stream);
    switch (sh_degree) {
        case 0: k_project<0><<<grid, block, 0, s>>>(params_dev, n, cam, tile_w, tile_h, TX, TY, proj_dev, radius_dev, rect_dev, touched_dev); break;
        case 1: k_project<1><<<grid, block, 0, s>>>(params_dev, n, cam, tile_w, tile_h, TX, TY, proj_dev, radius_dev, rect_dev, touched_dev); break;
        case 2: k_project<2><<<grid, block, 0, s>>>(params_dev, n, cam, tile_w, tile_h, TX, TY, proj_dev, radius_dev, rect_dev, touched_dev); break;
        default: k_project<3><<<grid, block, 0, s>>>(params_dev, n, cam, tile_w, tile_h, TX, TY, proj_dev, radius_dev, rect_dev, touched_dev); break;
    }
    PGS_CHECK_LAUNCH("pgs_project");
    return PGS_OK;
}

extern "C" pgs_status pgs_project_bwd(const float* params_dev, int32_t n, int32_t sh_degree,
                                      const pgs_camera* cam_host, const int32_t* radius_dev,
                                      const float* grad2d_dev, float* grads_dev, void* stream) {
    PGS_REQUIRE(n >= 0, "pgs_project_bwd: n < 0");
    PGS_REQUIRE(sh_degree >= 0 && sh_degree <= 3, "pgs_project_bwd: sh_degree %d", sh_degree);
    PGS_REQUIRE(cam_host != nullptr, "pgs_project_bwd: null camera");
    if (n == 0) return PGS_OK;
    PGS_REQUIRE(params_dev && radius_dev && grad2d_dev && grads_dev, "pgs_project_bwd: null pointer");
    const pgs::CamD cam = pgs::make_cam(*cam_host);
    const dim3 grid((n + 63) / 64), block(64);
    hipStream_t s = pgs::as_stream(stream);
    switch (sh_degree) {
        case 0: k_project_bwd<0><<<grid, block, 0, s>>>(params_dev, n, cam, radius_dev, grad2d_dev, grads_dev); break;
        case 1: k_project_bwd<1><<<grid, block, 0, s>>>(params_dev, n, cam, radius_dev, grad2d_dev, grads_dev); break;
        case 2: k_project_bwd<2><<<grid, block, 0, s>>>(params_dev, n, cam, radius_dev, grad2d_dev, grads_dev); break;
        default: k_project_bwd<3><<<grid, block, 0, s>>>(params_dev, n, cam, radius_dev, grad2d_dev, grads_dev); break;
    }
    PGS_CHECK_LAUNCH("pgs_project_bwd");
    return PGS_OK;
}

namespace {

// Cameras of views [v0, v0 + nv) of a batch, for one multi-view launch.
LaunchViews launch_views(const pgs_view_batch& vb, int v0, int nv) {
    LaunchViews lv{};
    lv.nv = nv;
    lv.v0 = v0;
    for (int k = 0; k < nv; ++k) {
        const pgs_camera& c = vb.cams[v0 + k];
        lv.cam[k] = pgs::make_cam(c);
        lv.TX[k] = (c.width + vb.tile_w - 1) / vb.tile_w;
        lv.TY[k] = (c.height + vb.tile_h - 1) / vb.tile_h;
    }
    return lv;
}

}  // namespace

extern "C" pgs_status pgs_project_views(const pgs_view_batch* views, const float* params_dev, int32_t n,
                                        int32_t sh_degree, float* proj_all_dev, int32_t* radius_all_dev,
                                        uint32_t* rect_all_dev, uint32_t* touched_all_dev, void* stream) {
    if (pgs_status st = pgs::check_views(views, "pgs_project_views")) return st;
    PGS_REQUIRE(n >= 0, "pgs_project_views: n < 0");
    PGS_REQUIRE(sh_degree >= 0 && sh_degree <= 3, "pgs_project_views: sh_degree %d", sh_degree);
    if (n == 0) return PGS_OK;
    PGS_REQUIRE(params_dev && proj_all_dev && radius_all_dev && rect_all_dev && touched_all_dev,
                "pgs_project_views: null pointer");
    const dim3 grid((n + 63) / 64), block(64);
    hipStream_t s = pgs::as_stream(stream);
    const int tw = views->tile_w, th = views->tile_h;
    for (int v0 = 0; v0 < views->n_views; v0 += kLaunchViews) {
        const LaunchViews lv = launch_views(*views, v0, min(kLaunchViews, views->n_views - v0));
        switch (sh_degree) {
            case 0: k_project_views<0><<<grid, block, 0, s>>>(params_dev, n, lv, tw, th, proj_all_dev, radius_all_dev, rect_all_dev, touched_all_dev); break;
            case 1: k_project_views<1><<<grid, block, 0, s>>>(params_dev, n, lv, tw, th, proj_all_dev, radius_all_dev, rect_all_dev, touched_all_dev); break;
            case 2: k_project_views<2><<<grid, block, 0, s>>>(params_dev, n, lv, tw, th, proj_all_dev, radius_all_dev, rect_all_dev, touched_all_dev); break;
            default: k_project_views<3><<<grid, block, 0, s>>>(params_dev, n, lv, tw, th, proj_all_dev, radius_all_dev, rect_all_dev, touched_all_dev); break;
        }
    }
    PGS_CHECK_LAUNCH("pgs_project_views");
    return PGS_OK;
}

extern "C" pgs_status pgs_project_bwd_views(const pgs_view_batch* views, const float* params_dev, int32_t n,
                                            int32_t sh_degree, const int32_t* radius_all_dev,
                                            const float* grad2d_all_dev, float* grads_dev, void* stream) {
    if (pgs_status st = pgs::check_views(views, "pgs_project_bwd_views")) return st;
    PGS_REQUIRE(n >= 0, "pgs_project_bwd_views: n < 0");
    PGS_REQUIRE(sh_degree >= 0 && sh_degree <= 3, "pgs_project_bwd_views: sh_degree %d", sh_degree);
    if (n == 0) return PGS_OK;
    PGS_REQUIRE(params_dev && radius_all_dev && grad2d_all_dev && grads_dev, "pgs_project_bwd_views: null pointer");
    const dim3 grid((n + 63) / 64), block(64);
    hipStream_t s = pgs::as_stream(stream);
    for (int v0 = 0; v0 < views->n_views; v0 += kLaunchViews) {
        const LaunchViews lv = launch_views(*views, v0, min(kLaunchViews, views->n_views - v0));
        switch (sh_degree) {
            case 0: k_project_bwd_views<0><<<grid, block, 0, s>>>(params_dev, n, lv, radius_all_dev, grad2d_all_dev, grads_dev); break;
            case 1: k_project_bwd_views<1><<<grid, block, 0, s>>>(params_dev, n, lv, radius_all_dev, grad2d_all_dev, grads_dev); break;
            case 2: k_project_bwd_views<2><<<grid, block, 0, s>>>(params_dev, n, lv, radius_all_dev, grad2d_all_dev, grads_dev); break;
            default: k_project_bwd_views<3><<<grid, block, 0, s>>>(params_dev, n, lv, radius_all_dev, grad2d_all_dev, grads_dev); break;
        }
    }
    PGS_CHECK_LAUNCH("pgs_project_bwd_views");
    return PGS_OK;
}
