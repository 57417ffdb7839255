// Photometric loss L = (1 - lambda) L1 + lambda (1 - SSIM) and dL/dx.
//
// The paper does not state its loss; this is the 3D Gaussian Splatting form.
// SSIM (Wang et al. 2004): 11x11 Gaussian window (sigma 1.5), C1 = 1e-4,
// C2 = 9e-4, zero padding, mean over pixels and channels.
//
// Forward: the windowed sums mu_x, mu_y, E[x^2], E[y^2], E[xy] -> the SSIM map's
// partial derivatives m1 = dS/dmu_x, m2 = dS/dE[x^2], m3 = dS/dE[xy] and the
// sum of the map.  Backward: the same windowed pass over (m1, m2, m3) gives
//     dSSIM/dx_p = (1/N) (w*m1 + 2 x_p w*m2 + y_p w*m3)(p),
// the adjoint of the zero-padded blur being the zero-padded blur.
//
// Both walk a strip of 128 columns, two neighbouring ones a lane, down some
// rows with a workgroup of one wave.  Each input row (with a 5-column halo),
// loaded two rows ahead, passes through LDS and is blurred horizontally; the
// results of the last 11 rows sit in a register ring, from which the vertical
// pass forms the 11 x 11 window sums.  Where the image is flat the gradient is a
// difference of terms a thousand times its size, so every sum is taken in the
// order of its taps, with the roundings of the plain formula.
//
// The forward spends 55% of its time issuing vector instructions and a third
// waiting, the backward 32% and over half (its loads).  With one column
// a lane, 22 (33) single LDS reads a pixel, addresses and bounds in vector
// registers and 32 rows a wave whatever the image, 1920 x 1440 took 125 us with
// the final sum, now 119; 1024 x 1024 77, now 60; 317 x 243 55, now 26.  (One
// kernel for both, with the denominators from the blurred squared difference,
// took 93 for the largest but changed flat gradients by 1e-4 of themselves.)
#include <math.h>

#include "common.hpp"

namespace {

constexpr int kHalo = 5;
constexpr int kSW = 128;                // output columns of a strip, two per lane
constexpr int kRowW = kSW + 2 * kHalo;  // 138 input columns
constexpr float kC1 = 1e-4f, kC2 = 9e-4f;

struct Win {
    float w[11];
};

inline Win gaussian_window() {
    Win win;
    double g[11], s = 0;
    for (int i = 0; i < 11; ++i) {
        const double d = i - 5;
        g[i] = exp(-d * d / (2.0 * 1.5 * 1.5));
        s += g[i];
    }
    for (int i = 0; i < 11; ++i) win.w[i] = (float)(g[i] / s);
    return win;
}

__device__ __forceinline__ float block_sum(float v, float* red) {
    // wave sums to lane 63, then the 4 wave totals
    const float w = wave_sum_to_lane63(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 63) red[wv] = w;
    __syncthreads();
    float tot = 0.f;
    if (threadIdx.x == 0) tot = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    return tot;
}

__global__ __launch_bounds__(256) void k_l1(const float* __restrict__ x, const float* __restrict__ y,
                                            size_t N, float scale, float* __restrict__ dl,
                                            float* __restrict__ part) {
    __shared__ float red[4];
    float s = 0.f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        const float d = x[i] - y[i];
        s += fabsf(d);
        dl[i] = d > 0.f ? scale : (d < 0.f ? -scale : 0.f);
    }
    const float tot = block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// One row of a plane as a buffer resource: loads outside [0, W) return zero
// and stores there are dropped, without a comparison or an address in vector
// registers.  Rows outside the image have no extent at all; kNoByte lies past
// the end of every row.
constexpr int kNoByte = 0x7ffffff0;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const float* plane, int gy, int W, int H) {
    const bool in = gy >= 0 && gy < H;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(plane + (in ? (size_t)gy * W : (size_t)0)), 0,
                                             in ? W * 4 : 0, 0x00027000);
}

__device__ __forceinline__ float row_load(__amdgpu_buffer_rsrc_t row, int byte) {
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(row, byte, 0, 0));
}

__device__ __forceinline__ void row_store(__amdgpu_buffer_rsrc_t row, int byte, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), row, byte, 0, 0);
}

// Input row r0 - 5 + ii of a strip of NQ planes: lane l takes columns l, l + 64
// and (for l < 10) l + 128.
template <int NQ>
struct RowLoad {
    float v[NQ][3];
    __device__ __forceinline__ void load(const float* const* planes, int W, int H, int c0, int gy, int l) {
        const int byte = (c0 - kHalo + l) * 4;
#pragma unroll
        for (int f = 0; f < NQ; ++f) {
            const auto row = row_buffer(planes[f], gy, W, H);
#pragma unroll
            for (int h = 0; h < 3; ++h) v[f][h] = row_load(row, byte + 256 * h >= 0 ? byte + 256 * h : kNoByte);
        }
    }
    __device__ __forceinline__ void store(float (*lds)[kRowW + 2], int l) const {
#pragma unroll
        for (int h = 0; h < 3; ++h)
            if (h < 2 || l < kRowW - 128) {
#pragma unroll
                for (int f = 0; f < NQ; ++f) lds[f][l + 64 * h] = v[f][h];
            }
    }
};

// The 12 values of two neighbouring windows.
__device__ __forceinline__ void read_windows(const float* p, float (&v)[12]) {
#pragma unroll
    for (int u = 0; u < 6; ++u) {
        const float2 q = *reinterpret_cast<const float2*>(p + 2 * u);
        v[2 * u] = q.x;
        v[2 * u + 1] = q.y;
    }
}

template <int NF>
__device__ __forceinline__ void vertical(const Win& win, const float (&ring)[11][NF][2], int k, int c, float (&q)[NF]) {
#pragma unroll
    for (int f = 0; f < NF; ++f) q[f] = win.w[0] * ring[(k + 1) % 11][f][c];
#pragma unroll
    for (int t = 1; t < 11; ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f) q[f] = fmaf(win.w[t], ring[(k + 1 + t) % 11][f][c], q[f]);
}

__global__ __launch_bounds__(64, 2) void k_ssim_fwd(const float* __restrict__ x, const float* __restrict__ y, int W,
                                                    int H, int rows, Win win, float* __restrict__ m,
                                                    float* __restrict__ part) {
    __shared__ __align__(8) float lds[2][2][kRowW + 2];
    const int l = threadIdx.x, ch = blockIdx.z, c0 = blockIdx.x * kSW, r0 = blockIdx.y * rows;
    const size_t plane = (size_t)W * H;
    const float* planes[2] = {x + ch * plane, y + ch * plane};
    m += 3 * ch * plane;
    const int col = c0 + 2 * l, rows_in = min(rows, H - r0) + 2 * kHalo;
    float ring[11][5][2];
    float ssum = 0.f;
    RowLoad<2> a1, a2;
    a1.load(planes, W, H, c0, r0 - kHalo, l);
    a2.load(planes, W, H, c0, r0 - kHalo + 1, l);
    for (int base = 0; base < rows_in; base += 11) {
#pragma unroll
        for (int k = 0; k < 11; ++k) {
            const int ii = base + k;
            if (ii < rows_in) {
                float(*row)[kRowW + 2] = lds[ii & 1];
                a1.store(row, l);
                a1 = a2;
                a2.load(planes, W, H, c0, r0 - kHalo + ii + 2, l);
                wave_fence();
                float xv[12], yv[12];
                read_windows(&row[0][2 * l], xv);
                read_windows(&row[1][2 * l], yv);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    float a[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < 11; ++t) {
                        const float w = win.w[t], xe = xv[t + c], ye = yv[t + c], wx = w * xe, wy = w * ye;
                        if (t == 0) {
                            a[0] = wx;
                            a[1] = wy;
                            a[2] = wx * xe;
                            a[3] = wy * ye;
                            a[4] = wx * ye;
                        } else {
                            a[0] = fmaf(w, xe, a[0]);
                            a[1] = fmaf(w, ye, a[1]);
                            a[2] = fmaf(wx, xe, a[2]);
                            a[3] = fmaf(wy, ye, a[3]);
                            a[4] = fmaf(wx, ye, a[4]);
                        }
                    }
#pragma unroll
                    for (int f = 0; f < 5; ++f) ring[k][f][c] = a[f];
                }
                if (ii >= 2 * kHalo) {
                    const int o = r0 + ii - 2 * kHalo;  // output row
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float q[5];
                        vertical<5>(win, ring, k, c, q);
                        const float mx = q[0], my = q[1];
                        const float vx = q[2] - mx * mx, vy = q[3] - my * my, cxy = q[4] - mx * my;
                        const float N1 = 2.f * mx * my + kC1, N2 = 2.f * cxy + kC2;
                        const float D1 = mx * mx + my * my + kC1, D2 = vx + vy + kC2;
                        const float inv = 1.f / (D1 * D2);
                        const float S = N1 * N2 * inv;
                        const float m1 = (2.f * my * N2 - 2.f * my * N1) * inv - S * (2.f * mx / D1 - 2.f * mx / D2);
                        const float m2 = -S / D2;
                        const float m3 = 2.f * N1 * inv;
                        row_store(row_buffer(m, o, W, H), (col + c) * 4, m1);
                        row_store(row_buffer(m + plane, o, W, H), (col + c) * 4, m2);
                        row_store(row_buffer(m + 2 * plane, o, W, H), (col + c) * 4, m3);
                        ssum += col + c < W ? S : 0.f;
                    }
                }
            }
        }
    }
    const float tot = wave_sum_to_lane63(ssum);
    if (l == 63) part[(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = tot;
}

__global__ __launch_bounds__(64, 3) void k_ssim_bwd(const float* __restrict__ x, const float* __restrict__ y, int W,
                                                    int H, int rows, Win win, const float* __restrict__ m,
                                                    float l1_scale, float ssim_scale, float* __restrict__ dl,
                                                    float* __restrict__ part) {
    __shared__ __align__(8) float lds[2][3][kRowW + 2];
    const int l = threadIdx.x, ch = blockIdx.z, c0 = blockIdx.x * kSW, r0 = blockIdx.y * rows;
    const size_t plane = (size_t)W * H;
    const float* planes[3] = {m + 3 * ch * plane, m + (3 * ch + 1) * plane, m + (3 * ch + 2) * plane};
    x += ch * plane;
    y += ch * plane;
    dl += ch * plane;
    const int byte = (c0 + 2 * l) * 4, rows_in = min(rows, H - r0) + 2 * kHalo;
    float ring[11][3][2];
    float l1sum = 0.f;
    RowLoad<3> a1, a2;
    a1.load(planes, W, H, c0, r0 - kHalo, l);
    a2.load(planes, W, H, c0, r0 - kHalo + 1, l);
    for (int base = 0; base < rows_in; base += 11) {
#pragma unroll
        for (int k = 0; k < 11; ++k) {
            const int ii = base + k;
            if (ii < rows_in) {
                float(*row)[kRowW + 2] = lds[ii & 1];
                a1.store(row, l);
                a1 = a2;
                a2.load(planes, W, H, c0, r0 - kHalo + ii + 2, l);
                const int o = r0 + ii - 2 * kHalo;  // output row, from ii = 10 on
                const auto xr = row_buffer(x, o, W, H), yr = row_buffer(y, o, W, H);
                float xv[2], yv[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    xv[c] = row_load(xr, byte + 4 * c);
                    yv[c] = row_load(yr, byte + 4 * c);
                }
                wave_fence();
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    float v[12];
                    read_windows(&row[f][2 * l], v);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float a = win.w[0] * v[c];
#pragma unroll
                        for (int t = 1; t < 11; ++t) a = fmaf(win.w[t], v[t + c], a);
                        ring[k][f][c] = a;
                    }
                }
                if (ii >= 2 * kHalo) {
                    const auto dr = row_buffer(dl, o, W, H);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float b[3];
                        vertical<3>(win, ring, k, c, b);
                        const float d = xv[c] - yv[c];  // zero outside the image
                        l1sum += fabsf(d);
                        const float sgn = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
                        row_store(dr, byte + 4 * c,
                                  l1_scale * sgn - ssim_scale * (b[0] + 2.f * xv[c] * b[1] + yv[c] * b[2]));
                    }
                }
            }
        }
    }
    const float tot = wave_sum_to_lane63(l1sum);
    if (l == 63) part[(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = tot;
}

// Sums the per-block partials in a fixed order (deterministic, no atomics):
// 1024 lanes, eight independent accumulators each so the loads overlap.
constexpr int kFinalThreads = 1024;

__device__ __forceinline__ float strided_sum(const float* __restrict__ p, int n) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int base = threadIdx.x; base < n; base += 8 * kFinalThreads) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kFinalThreads;
            if (i < n) acc[u] += p[i];
        }
    }
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
}

__device__ __forceinline__ float block_sum_1024(float v, float* red) {
    const float w = wave_sum_to_lane63(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 63) red[wv] = w;
    __syncthreads();
    float tot = 0.f;
    if (threadIdx.x == 0)
        for (int k = 0; k < kFinalThreads / 64; ++k) tot += red[k];
    __syncthreads();
    return tot;
}

__global__ __launch_bounds__(kFinalThreads) void k_loss_final(const float* __restrict__ part_l1, int nl,
                                                              const float* __restrict__ part_s, int ns,
                                                              float lambda, float invN,
                                                              float* __restrict__ out) {
    __shared__ float red[kFinalThreads / 64];
    const float l1 = block_sum_1024(strided_sum(part_l1, nl), red) * invN;
    const float ss = block_sum_1024(strided_sum(part_s, ns), red) * invN;
    if (threadIdx.x == 0) out[0] = lambda > 0.f ? (1.f - lambda) * l1 + lambda * (1.f - ss) : l1;
}

constexpr int kL1Blocks = 1024;

// Squared error of the two images clamped to [0, 1], per-block partials.
__global__ __launch_bounds__(256) void k_sq_err(const float* __restrict__ x, const float* __restrict__ y,
                                                size_t N, float* __restrict__ part) {
    __shared__ float red[4];
    float s = 0.f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x) {
        const float d = fminf(fmaxf(x[i], 0.f), 1.f) - fminf(fmaxf(y[i], 0.f), 1.f);
        s += d * d;
    }
    const float tot = block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// out[0] = MSE, out[1] = 10 log10(1 / MSE) (infinite for identical images).
__global__ __launch_bounds__(kFinalThreads) void k_psnr_final(const float* __restrict__ part, int np,
                                                              double invN, float* __restrict__ out) {
    __shared__ float red[kFinalThreads / 64];
    const float sse = block_sum_1024(strided_sum(part, np), red);
    if (threadIdx.x == 0) {
        const double mse = (double)sse * invN;
        out[0] = (float)mse;
        out[1] = mse > 0.0 ? (float)(10.0 * log10(1.0 / mse)) : INFINITY;
    }
}

// Output rows of a wave.  A wave lasts about rows + 8 row times (the first 10
// input rows skip the later stages); two waves on one of the card's 1024 SIMDs
// take about 1.25 times as long as one.  Hence few rows where the image has
// little work (317 x 243 with 4 rows 26 us, with 32 58) and waves just below
// a multiple of 2048 elsewhere.
inline int ssim_rows(int W, int H) {
    const long strips = 3L * ((W + kSW - 1) / kSW);
    int best = 4;
    long best_cost = -1;
    for (int rows = 4; rows <= 64; ++rows) {
        const long per_simd = (strips * ((H + rows - 1) / rows) + 1023) / 1024;
        const long cost = (5 * (per_simd / 2) + 4 * (per_simd % 2)) * (rows + 8);
        if (best_cost < 0 || cost < best_cost) {
            best = rows;
            best_cost = cost;
        }
    }
    return best;
}

inline int ssim_blocks(int W, int H) {
    const int rows = ssim_rows(W, H);
    return 3 * ((W + kSW - 1) / kSW) * ((H + rows - 1) / rows);
}

inline size_t part_bytes(int W, int H) {
    const int nb = ssim_blocks(W, H) > kL1Blocks ? ssim_blocks(W, H) : kL1Blocks;
    return (((size_t)2 * nb * sizeof(float)) + 255) & ~(size_t)255;
}

}  // namespace

extern "C" pgs_status pgs_psnr(const float* x_dev, const float* y_dev, int32_t width, int32_t height,
                               float* out_dev, void* workspace_dev, size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(width > 0 && height > 0, "pgs_psnr: bad size");
    PGS_REQUIRE(x_dev && y_dev && out_dev && workspace_dev, "pgs_psnr: null pointer");
    PGS_REQUIRE(workspace_bytes >= kL1Blocks * sizeof(float), "pgs_psnr: workspace too small");
    hipStream_t s = pgs::as_stream(stream);
    const size_t N = (size_t)3 * width * height;
    float* part = static_cast<float*>(workspace_dev);
    k_sq_err<<<kL1Blocks, 256, 0, s>>>(x_dev, y_dev, N, part);
    k_psnr_final<<<1, kFinalThreads, 0, s>>>(part, kL1Blocks, 1.0 / (double)N, out_dev);
    PGS_CHECK_LAUNCH("pgs_psnr");
    return PGS_OK;
}

extern "C" size_t pgs_loss_workspace(int32_t width, int32_t height) {
    if (width <= 0 || height <= 0) return 256;
    return part_bytes(width, height) + (size_t)9 * width * height * sizeof(float);
}

extern "C" pgs_status pgs_loss_l1_dssim(const float* x_dev, const float* y_dev, int32_t width,
                                        int32_t height, float lambda, float* loss_dev, float* dl_dx_dev,
                                        void* workspace_dev, size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(width > 0 && height > 0, "pgs_loss_l1_dssim: bad size");
    PGS_REQUIRE(lambda >= 0.f && lambda <= 1.f, "pgs_loss_l1_dssim: lambda %g", (double)lambda);
    PGS_REQUIRE(x_dev && y_dev && loss_dev && dl_dx_dev && workspace_dev, "pgs_loss_l1_dssim: null pointer");
    const size_t need = lambda > 0.f ? pgs_loss_workspace(width, height) : part_bytes(width, height);
    PGS_REQUIRE(workspace_bytes >= need, "pgs_loss_l1_dssim: workspace %zu < %zu", workspace_bytes, need);
    hipStream_t s = pgs::as_stream(stream);
    const int npart = (int)(part_bytes(width, height) / (2 * sizeof(float)));
    float* part_l1 = static_cast<float*>(workspace_dev);
    float* part_s = part_l1 + npart;
    const size_t N = (size_t)3 * width * height;
    const float invN = (float)(1.0 / (double)N);
    int nl = kL1Blocks, ns = 0;
    if (lambda == 0.f) {
        k_l1<<<kL1Blocks, 256, 0, s>>>(x_dev, y_dev, N, invN, dl_dx_dev, part_l1);
    } else {
        static const Win win = gaussian_window();
        const int rows = ssim_rows(width, height);
        const dim3 grid((width + kSW - 1) / kSW, (height + rows - 1) / rows, 3);
        nl = ns = ssim_blocks(width, height);
        float* m = reinterpret_cast<float*>(static_cast<char*>(workspace_dev) + part_bytes(width, height));
        k_ssim_fwd<<<grid, 64, 0, s>>>(x_dev, y_dev, width, height, rows, win, m, part_s);
        k_ssim_bwd<<<grid, 64, 0, s>>>(x_dev, y_dev, width, height, rows, win, m, (1.f - lambda) * invN,
                                       lambda * invN, dl_dx_dev, part_l1);
    }
    k_loss_final<<<1, kFinalThreads, 0, s>>>(part_l1, nl, part_s, ns, lambda, invN, loss_dev);
    PGS_CHECK_LAUNCH("pgs_loss_l1_dssim");
    return PGS_OK;
}
