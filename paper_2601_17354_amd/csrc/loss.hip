// Photometric loss L = (1 - lambda) L1 + lambda (1 - SSIM) and dL/dx.
//
// The paper does not state its loss; this is the 3D Gaussian Splatting form.
// SSIM (Wang et al. 2004): 11x11 Gaussian window (sigma 1.5), C1 = 1e-4,
// C2 = 9e-4, zero padding, mean over pixels and channels.
//
// One kernel of one-wave workgroups does all of it: the windowed sums mu_x,
// mu_y, E[(x - y)^2], E[xy] (the denominators need the squares only as the
// sums mu_x^2 + mu_y^2 = 2 mu_x mu_y + (mu_x - mu_y)^2 and var_x + var_y =
// 2 cov + var(x - y), and so equal the numerators where x equals y), the
// SSIM map's partial derivatives m1 = dS/dmu_x, m2 = dS/dE[x^2],
// m3 = dS/dE[xy], and
//     dSSIM/dx_p = (1/N) (w*m1 + 2 x_p w*m2 + y_p w*m3)(p),
// the adjoint of the zero-padded blur being the zero-padded blur (m is zero
// outside the image).
#include <math.h>

#include "common.hpp"

namespace {

constexpr int kHalo = 5;
constexpr int kMW = 128;                // columns of a strip whose m a wave forms, two per lane
constexpr int kSW = kMW - 2 * kHalo;    // 118 output columns
constexpr int kRowW = kMW + 2 * kHalo;  // 138 input columns
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

// Horizontal blur of the two windows that begin at p[0] and p[1].
__device__ __forceinline__ void blur_pair(const Win& win, const float* p, float (&out)[2]) {
    float2 v[6];
#pragma unroll
    for (int u = 0; u < 6; ++u) v[u] = *reinterpret_cast<const float2*>(p + 2 * u);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        float a = win.w[0] * (c ? v[0].y : v[0].x);
#pragma unroll
        for (int t = 1; t < 11; ++t) a = fmaf(win.w[t], (t + c) & 1 ? v[(t + c) / 2].y : v[(t + c) / 2].x, a);
        out[c] = a;
    }
}

// A wave walks a strip of 118 output columns down `rows` output rows.  Each
// input row (10 columns of halo on either side, loaded two rows ahead) passes
// through LDS and is blurred horizontally, two neighbouring columns a lane, so
// that a product x y is formed once for both windows and the LDS is read in
// pairs; the results of the last 11 rows sit in a register ring, from which
// the vertical pass forms the window sums of row i - 5 and the lane's two m
// triples.  These take the same way again, LDS, horizontal, ring, vertical,
// to the gradient of row i - 10.
//
// Bound by the vector units (about 300 instructions a pixel, the 20 halo rows
// of a strip included).  Two kernels with the nine planes of m in memory
// between them moved 3.7 times the bytes and spent 11 x 3 products and 22
// single LDS reads a pixel on each window: 1920 x 1440 125 us with the final sum, now 93;
// 317 x 243 55 us, now 26.
__global__ __launch_bounds__(64, 2) void k_ssim(const float* __restrict__ x, const float* __restrict__ y, int W, int H,
                                                int rows, Win win, float l1_scale, float ssim_scale,
                                                float* __restrict__ dl, float* __restrict__ part_l1,
                                                float* __restrict__ part_s) {
    __shared__ __align__(8) float s_in[2][4][kRowW + 6];
    __shared__ __align__(8) float s_m[2][3][kRowW + 2];
    const int l = threadIdx.x, ch = blockIdx.z, c0 = blockIdx.x * kSW, r0 = blockIdx.y * rows;
    const size_t plane = (size_t)W * H;
    x += ch * plane;
    y += ch * plane;
    dl += ch * plane;
    const int rows_out = min(rows, H - r0), rows_in = rows_out + 4 * kHalo;
    const int mcol = c0 - kHalo + 2 * l;  // this lane's columns of m
    const bool m_in[2] = {mcol >= 0 && mcol < W, mcol + 1 >= 0 && mcol + 1 < W};
    const bool own[2] = {m_in[0] && mcol >= c0 && mcol < c0 + kSW, m_in[1] && mcol + 1 >= c0 && mcol + 1 < c0 + kSW};
    const int in_byte = (c0 - 2 * kHalo + l) * 4;
    const int in_first = in_byte >= 0 ? in_byte : kNoByte;
    const int out_byte = l < kSW / 2 ? (c0 + 2 * l) * 4 : kNoByte;  // lanes 59..63 have no output column
    float ring[11][4][2], mring[11][3][2];
    float ssum = 0.f, l1sum = 0.f;
    float ahead[2][2][3];  // [rows ahead][plane][column group]
    const auto fetch = [&](int ii, float (&v)[2][3]) {
        const int gy = r0 - 2 * kHalo + ii;
        const auto xr = row_buffer(x, gy, W, H), yr = row_buffer(y, gy, W, H);
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            v[0][h] = row_load(xr, h ? in_byte + 256 * h : in_first);
            v[1][h] = row_load(yr, h ? in_byte + 256 * h : in_first);
        }
    };
    fetch(0, ahead[0]);
    fetch(1, ahead[1]);
    for (int base = 0; base < rows_in; base += 11) {
#pragma unroll
        for (int k = 0; k < 11; ++k) {
            const int ii = base + k;
            if (ii < rows_in) {
                float(*row)[kRowW + 6] = s_in[ii & 1];
#pragma unroll
                for (int h = 0; h < 3; ++h) {
                    const float xe = ahead[0][0][h], ye = ahead[0][1][h], d = xe - ye;
                    if (h < 2 || l < kRowW - 128) {
                        row[0][l + 64 * h] = xe;
                        row[1][l + 64 * h] = ye;
                        row[2][l + 64 * h] = d * d;
                        row[3][l + 64 * h] = xe * ye;
                    }
#pragma unroll
                    for (int f = 0; f < 2; ++f) ahead[0][f][h] = ahead[1][f][h];
                }
                fetch(ii + 2, ahead[1]);
                wave_fence();
#pragma unroll
                for (int f = 0; f < 4; ++f) blur_pair(win, &row[f][2 * l], ring[k][f]);
                if (ii >= 2 * kHalo) {
                    const int gm = r0 - 3 * kHalo + ii;  // row of m
                    const bool row_in = gm >= 0 && gm < H, own_row = gm >= r0 && gm < r0 + rows_out;
                    float m[3][2];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float q[4];
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            q[f] = win.w[0] * ring[(k + 1) % 11][f][c];
#pragma unroll
                            for (int t = 1; t < 11; ++t) q[f] = fmaf(win.w[t], ring[(k + 1 + t) % 11][f][c], q[f]);
                        }
                        const float mx = q[0], my = q[1];
                        const float N1 = 2.f * mx * my + kC1, N2 = 2.f * (q[3] - mx * my) + kC2;
                        const float md = mx - my, md2 = md * md;
                        const float D1 = N1 + md2, D2 = N2 + (q[2] - md2);
                        const float inv = 1.f / (D1 * D2), i1 = D2 * inv, i2 = D1 * inv;
                        const float S = N1 * N2 * inv;
                        const bool in = row_in && m_in[c];
                        m[0][c] = in ? 2.f * (my * (N2 - N1) * inv - S * mx * (i1 - i2)) : 0.f;
                        m[1][c] = in ? -S * i2 : 0.f;
                        m[2][c] = in ? 2.f * N1 * inv : 0.f;
                        ssum += own_row && own[c] ? S : 0.f;
                    }
                    float(*mrow)[kRowW + 2] = s_m[ii & 1];
#pragma unroll
                    for (int f = 0; f < 3; ++f)
                        *reinterpret_cast<float2*>(&mrow[f][2 * l]) = make_float2(m[f][0], m[f][1]);
                    wave_fence();
#pragma unroll
                    for (int f = 0; f < 3; ++f) blur_pair(win, &mrow[f][2 * l], mring[k][f]);
                }
                if (ii >= 4 * kHalo) {
                    const int o = r0 + ii - 4 * kHalo;
                    const auto xr = row_buffer(x, o, W, H), yr = row_buffer(y, o, W, H), dr = row_buffer(dl, o, W, H);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const float xv = row_load(xr, out_byte + 4 * c), yv = row_load(yr, out_byte + 4 * c);
                        float b[3];
#pragma unroll
                        for (int f = 0; f < 3; ++f) {
                            b[f] = win.w[0] * mring[(k + 1) % 11][f][c];
#pragma unroll
                            for (int t = 1; t < 11; ++t) b[f] = fmaf(win.w[t], mring[(k + 1 + t) % 11][f][c], b[f]);
                        }
                        const float d = xv - yv;  // zero outside the image
                        l1sum += fabsf(d);
                        const float sgn = d > 0.f ? l1_scale : (d < 0.f ? -l1_scale : 0.f);
                        const float g = sgn - ssim_scale * (b[0] + 2.f * xv * b[1] + yv * b[2]);
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(g), dr, out_byte + 4 * c, 0, 0);
                    }
                }
            }
        }
    }
    const float tot_s = wave_sum_to_lane63(ssum), tot_l1 = wave_sum_to_lane63(l1sum);
    if (l == 63) {
        const int b = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        part_s[b] = tot_s;
        part_l1[b] = tot_l1;
    }
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

__global__ __launch_bounds__(256) void k_copy(const float* __restrict__ from, float* __restrict__ to, size_t N) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
        to[i] = from[i];
}

inline bool overlap(const float* a, const float* b, size_t N) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b), bytes = N * sizeof(float);
    return p < q + bytes && q < p + bytes;
}

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

// Output rows of a wave.  Two waves fit on each of the card's 1024 SIMDs, and
// two take about 1.25 times as long as one; a wave lasts about rows + 12 row
// times (the 20 halo rows skip the later stages).  Hence few rows where the
// image has little work, and waves just below a multiple of 1024 elsewhere.
inline int ssim_rows(int W, int H) {
    const long strips = 3L * ((W + kSW - 1) / kSW);
    int best = 4;
    long best_cost = -1;
    for (int rows = 4; rows <= 64; ++rows) {
        const long per_simd = (strips * ((H + rows - 1) / rows) + 1023) / 1024;
        const long cost = (5 * (per_simd / 2) + 4 * (per_simd % 2)) * (rows + 12);
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
    return part_bytes(width, height) + (size_t)3 * width * height * sizeof(float);
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
        // a wave reads its neighbours' columns and rows of x and y while they
        // write their gradients: written in place, these go to the workspace first
        const bool in_place = overlap(dl_dx_dev, x_dev, N) || overlap(dl_dx_dev, y_dev, N);
        float* out = in_place ? reinterpret_cast<float*>(static_cast<char*>(workspace_dev) + part_bytes(width, height))
                              : dl_dx_dev;
        k_ssim<<<grid, 64, 0, s>>>(x_dev, y_dev, width, height, rows, win, (1.f - lambda) * invN, lambda * invN, out,
                                   part_l1, part_s);
        if (in_place) k_copy<<<kL1Blocks, 256, 0, s>>>(out, dl_dx_dev, N);
    }
    k_loss_final<<<1, kFinalThreads, 0, s>>>(part_l1, nl, part_s, ns, lambda, invN, loss_dev);
    PGS_CHECK_LAUNCH("pgs_loss_l1_dssim");
    return PGS_OK;
}
