// Single-reference cost-volume multi-view stereo on gfx950 (subsection
// "Single-Reference Cost-Volume MVS": probabilistic depth range, reference
// score S_ref, Census plane-sweep cost, SGM aggregation, confidence filter,
// fusion into the dense cloud).
//
// Kernels:
//   k_mvs_depths / k_mvs_range  camera depths of the sparse points that
//       project into each view as float64 bit patterns (all ones for the
//       others), then per view (one workgroup) the ranks that define the 5%
//       and 95% quantiles found by radix selection; range =
//       [0.5 q_.05, 1.5 q_.95];
//   k_mvs_ref     per target view the candidate maximising
//       exp(-(b - b_target)^2 / (2 sigma_b^2)) max(alpha / alpha_min, 1);
//   k_census      7 x 7 Census (48 bits) from a 22 x 22 LDS tile;
//   k_cost<D>     one lane per (pixel, four planes) over 128 pixels per
//       workgroup: the plane-sweep pixel in the
//       reference view from float32 arithmetic in a fixed order without
//       contraction (the nearest-pixel decision is reproducible), Hamming
//       distance of the Census strings; cost volume [y][x][plane] bytes;
//   k_sgm_*<D>    semi-global aggregation, four image lines per wave: 16 lanes
//       hold a line's D planes two to a register (packed 16-bit arithmetic),
//       the least path cost is four rotations of the 16 lanes.  k_sgm_rows
//       sums both row directions, k_sgm_cols adds both column directions and
//       takes winner, confidence test and refined depth; path costs are
//       recomputed from checkpoints instead of stored.  k_sgm_paths stores
//       three directions side by side where few lines would leave the chip
//       idle;
//   k_fuse_*      per-row counts, one scan over rows and the back-projection
//       of the kept pixels in row-major order.

#include <math.h>

#include "common.hpp"

namespace {

constexpr int kCensusR = 3;
constexpr int kCensusBits = (2 * kCensusR + 1) * (2 * kCensusR + 1) - 1;  // 48
constexpr int kCostOut = kCensusBits;
constexpr int kTile = 16;
constexpr int kHalo = kTile + 2 * kCensusR;

struct Cam64 {
    double fx, fy, cx, cy, R[9], t[3];
};

__device__ __forceinline__ Cam64 cam64(const pgs_camera& c) {
    Cam64 d;
    d.fx = c.fx;
    d.fy = c.fy;
    d.cx = c.cx;
    d.cy = c.cy;
    for (int r = 0; r < 3; ++r) {
        for (int k = 0; k < 3; ++k) d.R[3 * r + k] = c.viewmat[4 * r + k];
        d.t[r] = c.viewmat[4 * r + 3];
    }
    return d;
}

// ---------------------------------------------------------------- census

__global__ __launch_bounds__(256) void k_census(const uint8_t* __restrict__ grey, int W, int H,
                                                uint64_t* __restrict__ out) {
    __shared__ int tile[kHalo][kHalo];
    const size_t off = (size_t)blockIdx.z * W * H;
    const int x0 = blockIdx.x * kTile - kCensusR, y0 = blockIdx.y * kTile - kCensusR;
    for (int e = threadIdx.x; e < kHalo * kHalo; e += 256) {
        const int ty = e / kHalo, tx = e - ty * kHalo;
        const int gx = min(max(x0 + tx, 0), W - 1), gy = min(max(y0 + ty, 0), H - 1);
        tile[ty][tx] = grey[off + (size_t)gy * W + gx];
    }
    __syncthreads();
    const int lx = threadIdx.x % kTile, ly = threadIdx.x / kTile;
    const int x = blockIdx.x * kTile + lx, y = blockIdx.y * kTile + ly;
    if (x >= W || y >= H) return;
    const int c = tile[ly + kCensusR][lx + kCensusR];
    uint64_t v = 0;
    int b = 0;
#pragma unroll
    for (int dy = -kCensusR; dy <= kCensusR; ++dy)
#pragma unroll
        for (int dx = -kCensusR; dx <= kCensusR; ++dx) {
            if (dy == 0 && dx == 0) continue;
            v |= (uint64_t)(tile[ly + kCensusR + dy][lx + kCensusR + dx] < c) << b;
            ++b;
        }
    out[off + (size_t)y * W + x] = v;
}

// ---------------------------------------------------------------- range

__global__ __launch_bounds__(256) void k_mvs_clear(uint32_t* __restrict__ p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Key of point j in view v: the float64 bit pattern of its camera depth when
// it projects into the view (positive, so the patterns order like the
// values), all ones otherwise (after every valid key).
__global__ __launch_bounds__(256) void k_mvs_depths(const pgs_camera* __restrict__ cams, int W, int H,
                                                    const double* __restrict__ pts, int M,
                                                    uint64_t* __restrict__ keys) {
#pragma clang fp contract(off)
    const int v = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= M) return;
    const Cam64 c = cam64(cams[v]);
    const double P0 = pts[3 * (size_t)j], P1 = pts[3 * (size_t)j + 1], P2 = pts[3 * (size_t)j + 2];
    const double x = c.R[0] * P0 + c.R[1] * P1 + c.R[2] * P2 + c.t[0];
    const double y = c.R[3] * P0 + c.R[4] * P1 + c.R[5] * P2 + c.t[1];
    const double z = c.R[6] * P0 + c.R[7] * P1 + c.R[8] * P2 + c.t[2];
    const double u = c.fx * (x / z) + c.cx, w = c.fy * (y / z) + c.cy;
    const bool in = z > 0.0 && u >= -0.5 && u < (double)W - 0.5 && w >= -0.5 && w < (double)H - 0.5;
    keys[(size_t)v * M + j] = in ? (uint64_t)__double_as_longlong(z) : ~0ull;
}

struct RangeLds {
    uint32_t hist[256];
    uint32_t wsum[16];
    uint64_t wmin[16];
    uint64_t prefix;
    uint32_t rank;
};

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, RangeLds& L) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) L.wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t s = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += L.wsum[w];
    __syncthreads();
    return s;
}

__device__ __forceinline__ uint64_t block_min_u64(uint64_t v, RangeLds& L) {
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t u = ((uint64_t)(uint32_t)__shfl_xor((int)(v >> 32), o) << 32) |
                           (uint32_t)__shfl_xor((int)(uint32_t)v, o);
        v = u < v ? u : v;
    }
    if ((threadIdx.x & 63) == 0) L.wmin[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t m = ~0ull;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = L.wmin[w] < m ? L.wmin[w] : m;
    __syncthreads();
    return m;
}

// The rank-th smallest of the keys (one workgroup), by radix selection over
// 8-bit digits from the most significant; the digit is found by one wave
// (four bins per lane, a lane prefix sum and a ballot).
__device__ uint64_t select_rank(const uint64_t* __restrict__ keys, uint32_t n, uint32_t rank, RangeLds& L) {
    const int t = threadIdx.x, lane = t & 63;
    uint64_t prefix = 0, mask = 0;
    uint32_t r = rank;
    for (int shift = 56; shift >= 0; shift -= 8) {
        if (t < 256) L.hist[t] = 0u;
        __syncthreads();
        for (uint32_t i = t; i < n; i += blockDim.x) {
            const uint64_t k = keys[i];
            if ((k & mask) == prefix) atomicAdd(&L.hist[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (t < 64) {
            const uint32_t h0 = L.hist[4 * lane], h1 = L.hist[4 * lane + 1], h2 = L.hist[4 * lane + 2],
                           h3 = L.hist[4 * lane + 3];
            const uint32_t own = h0 + h1 + h2 + h3;
            uint32_t inc = own;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(inc, o);
                if (lane >= o) inc += u;
            }
            const uint32_t exc = inc - own;
            const uint64_t hit = __ballot(inc > r);
            const int q = __ffsll((long long)hit) - 1;  // first lane whose bins reach past r
            if (lane == q) {
                uint32_t acc = exc, d = 4 * lane + 3;
                const uint32_t hs[4] = {h0, h1, h2, h3};
                for (int e = 0; e < 4; ++e) {
                    if (acc + hs[e] > r) {
                        d = 4 * lane + e;
                        break;
                    }
                    acc += hs[e];
                }
                L.prefix = prefix | ((uint64_t)d << shift);
                L.rank = r - acc;
            }
        }
        __syncthreads();
        prefix = L.prefix;
        r = L.rank;
        mask |= 255ull << shift;
        __syncthreads();
    }
    return prefix;
}

// q(p) = z_i + (z_{i+1} - z_i)(h - i), h = (n - 1) p: z_i by selection, z_{i+1}
// is z_i when more than i + 1 keys are <= z_i, else the smallest key above.
__device__ double quantile_of(const uint64_t* keys, uint32_t M, uint32_t n, double p, RangeLds& L) {
#pragma clang fp contract(off)
    const double h = (double)(n - 1) * p;
    const uint32_t i = (uint32_t)floor(h);
    const uint64_t ki = select_rank(keys, M, i, L);
    const double zi = __longlong_as_double((long long)ki);
    if (i + 1 >= n) return zi;
    uint32_t le = 0;
    uint64_t above = ~0ull;
    for (uint32_t e = threadIdx.x; e < M; e += blockDim.x) {
        const uint64_t k = keys[e];
        le += k <= ki;
        if (k > ki && k < above) above = k;
    }
    le = block_sum_u32(le, L);
    above = block_min_u64(above, L);
    const double zj = le >= i + 2 ? zi : __longlong_as_double((long long)above);
    return zi + (zj - zi) * (h - (double)i);
}

__global__ __launch_bounds__(1024) void k_mvs_range(int M, const uint64_t* __restrict__ keys,
                                                    double* __restrict__ range) {
#pragma clang fp contract(off)
    __shared__ RangeLds L;
    const int v = blockIdx.x;
    const uint64_t* k = keys + (size_t)v * M;
    uint32_t c = 0;
    for (int e = threadIdx.x; e < M; e += blockDim.x) c += k[e] != ~0ull;
    const uint32_t n = block_sum_u32(c, L);
    double lo = 0.0, hi = 0.0;
    if (n > 0) {
        lo = 0.5 * quantile_of(k, M, n, 0.05, L);
        hi = 1.5 * quantile_of(k, M, n, 0.95, L);
    }
    if (threadIdx.x == 0) {
        range[2 * v] = lo;
        range[2 * v + 1] = hi;
    }
}

// ---------------------------------------------------------------- reference

__global__ __launch_bounds__(64) void k_mvs_ref(const pgs_camera* __restrict__ cams, int V, double b_target,
                                                double sigma_b, double alpha_min, int32_t* __restrict__ ref) {
    const int tv = blockIdx.x * 64 + threadIdx.x;
    if (tv >= V) return;
    const Cam64 a = cam64(cams[tv]);
    double ca[3];
    for (int k = 0; k < 3; ++k) ca[k] = -(a.R[k] * a.t[0] + a.R[3 + k] * a.t[1] + a.R[6 + k] * a.t[2]);
    double best = -1.0;
    int arg = -1;
    for (int c = 0; c < V; ++c) {
        if (c == tv) continue;
        const Cam64 b = cam64(cams[c]);
        double d2 = 0.0, dot = 0.0;
        for (int k = 0; k < 3; ++k) {
            const double cb = -(b.R[k] * b.t[0] + b.R[3 + k] * b.t[1] + b.R[6 + k] * b.t[2]);
            d2 += (cb - ca[k]) * (cb - ca[k]);
            dot += a.R[6 + k] * b.R[6 + k];
        }
        const double base = sqrt(d2), alpha = acos(fmin(1.0, fmax(-1.0, dot)));
        const double s = exp(-(base - b_target) * (base - b_target) / (2.0 * sigma_b * sigma_b)) *
                         fmax(alpha / alpha_min, 1.0);
        if (arg < 0 || s > best) {
            best = s;
            arg = c;
        }
    }
    ref[tv] = arg;
}

// ---------------------------------------------------------------- cost volume

constexpr int kCostPix = 128;  // pixels per cost workgroup
constexpr int kCostLane = 4;   // consecutive planes per lane
// four costs of a volume, of which no alignment beyond a byte's is asked
typedef uint32_t word_u __attribute__((aligned(1)));

// x / z and y / z, correctly rounded, from one reciprocal: the operations of
// the hardware's own divide (reciprocal refined once, each quotient corrected
// twice by its exact remainder) without the scaling that it wraps around them
// for operands whose remainders would leave the exponent range.  The caller
// keeps z within [2^-40, 2^40]; a numerator below 2^-78 gives a quotient below
// 2^-38 whatever its last bits, which no pixel coordinate shows, and one that
// overflows gives infinity or NaN, outside every image like the true quotient.
__device__ __forceinline__ void divide_pair(float x, float y, float z, float& qx_out, float& qy_out) {
    float r = __builtin_amdgcn_rcpf(z);
    r = __builtin_fmaf(__builtin_fmaf(-z, r, 1.0f), r, r);
    float qx = x * r, qy = y * r;
    qx = __builtin_fmaf(__builtin_fmaf(-z, qx, x), r, qx);
    qy = __builtin_fmaf(__builtin_fmaf(-z, qy, y), r, qy);
    qx_out = __builtin_fmaf(__builtin_fmaf(-z, qx, x), r, qx);
    qy_out = __builtin_fmaf(__builtin_fmaf(-z, qy, y), r, qy);
}

// Workgroup: kCostPix consecutive pixels of one target, all D planes; a lane
// takes kCostLane consecutive planes of a pixel, so their costs leave as one
// word, and the pixel's ray and Census string are read once for them.  The
// relative pose, the plane depths d_k and the pixel rays are float64 values
// rounded to float32 (d_k once per lane, the rays once per pixel in LDS); the
// per pixel-plane sweep is unfused float32 in a fixed order.  Bound by vector
// issue.  The two divisions were the sweep's largest part (11 instructions
// each, with a reciprocal of their own); they now share one, and pixel
// coordinates are range-checked and clamped before the gather instead of
// selected after it: 75 -> 57 vector instructions per cell, 1.07 -> 0.82 ms
// for eight 960 x 720 targets of 128 planes (without the gathers 0.80).
// WIDE: an image side of 2^24 or more, or 2^29 pixels (32-bit byte offsets
// and 24-bit products otherwise).
template <int D, bool WIDE>
__global__ __launch_bounds__(256) void k_cost(const pgs_camera* __restrict__ cams, int W, int H,
                                              const uint64_t* __restrict__ census,
                                              const int32_t* __restrict__ targets, const int32_t* __restrict__ refs,
                                              const double* __restrict__ range, uint8_t* __restrict__ cost) {
#pragma clang fp contract(off)
    constexpr int LP = D / kCostLane;  // lanes per pixel
    constexpr int SL = 256 / LP;       // pixels per pass
    __shared__ float s_pose[16];  // M, m, the reference intrinsics
    __shared__ float s_a[kCostPix], s_b[kCostPix];
    __shared__ uint64_t s_cen[kCostPix];
    const int t = threadIdx.x, ti = blockIdx.y, tv = targets[ti], rv = refs[tv];
    const uint32_t npix = (uint32_t)W * (uint32_t)H, base = blockIdx.x * kCostPix;
    // every lane reads the pose below, so it is defined without a reference too
    if (rv < 0 && t < 16) s_pose[t] = 0.0f;
    if (t == 0 && rv >= 0) {
        const Cam64 ct = cam64(cams[tv]), cr = cam64(cams[rv]);
        double M[9];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j)
                M[3 * i + j] = cr.R[3 * i] * ct.R[3 * j] + cr.R[3 * i + 1] * ct.R[3 * j + 1] +
                               cr.R[3 * i + 2] * ct.R[3 * j + 2];
        for (int i = 0; i < 9; ++i) s_pose[i] = (float)M[i];
        for (int i = 0; i < 3; ++i)
            s_pose[9 + i] =
                (float)(cr.t[i] - (M[3 * i] * ct.t[0] + M[3 * i + 1] * ct.t[1] + M[3 * i + 2] * ct.t[2]));
        s_pose[12] = cams[rv].fx;
        s_pose[13] = cams[rv].fy;
        s_pose[14] = cams[rv].cx;
        s_pose[15] = cams[rv].cy;
    }
    for (int q = t; q < kCostPix; q += blockDim.x) {
        if (base + q >= npix) {  // the ragged tail's slots are masked but still read
            s_a[q] = s_b[q] = 0.0f;
            s_cen[q] = 0;
            continue;
        }
        const pgs_camera& c = cams[tv];
        const uint32_t pix = base + q, y = pix / (uint32_t)W, x = pix - y * (uint32_t)W;
        s_a[q] = (float)(((double)x - (double)c.cx) / (double)c.fx);
        s_b[q] = (float)(((double)y - (double)c.cy) / (double)c.fy);
        s_cen[q] = census[(size_t)tv * npix + pix];
    }
    __syncthreads();
    if (t >= SL * LP) return;
    const int k0 = (t % LP) * kCostLane, slot = t / LP;
    const double d_min = range[2 * tv], d_max = range[2 * tv + 1];
    // no reference (a single view) or an empty range: every cost is the out cost
    const bool ranged = rv >= 0 && d_min > 0.0 && d_max > d_min;
    float M[12];
    for (int i = 0; i < 12; ++i) M[i] = s_pose[i];
    const float fx = s_pose[12], fy = s_pose[13], cx = s_pose[14], cy = s_pose[15];
    float d[kCostLane], mx[kCostLane], my[kCostLane], mz[kCostLane];
#pragma unroll
    for (int u = 0; u < kCostLane; ++u) {
        d[u] = 0.0f;
        if (ranged) {
            const double inv_far = 1.0 / d_max;
            const double h = (1.0 / d_min - inv_far) / (double)(D - 1);
            d[u] = (float)(1.0 / (inv_far + (double)(k0 + u) * h));
        }
        mx[u] = M[2] * d[u];
        my[u] = M[5] * d[u];
        mz[u] = M[8] * d[u];
    }
    // a coordinate c is inside when 0 <= floor(c) <= side - 1: c up to the
    // float below side (from 2^23 on every float is whole)
    auto top = [](int side) {
        const float last = (float)(side - 1);
        return last < 8388608.0f ? __uint_as_float(__float_as_uint(last + 1.0f) - 1u) : last;
    };
    const float wtop = top(W), htop = top(H);
    const char* rc = reinterpret_cast<const char*>(census + (size_t)(rv >= 0 ? rv : tv) * npix);
    uint8_t* out = cost + ((size_t)ti * npix + base) * D + k0;
    const int count = (int)min((uint32_t)kCostPix, npix - base);
    for (int i = slot; i < count; i += SL) {
        const float a = s_a[i], b = s_b[i];
        float xr[kCostLane], yr[kCostLane], zr[kCostLane];
#pragma unroll
        for (int u = 0; u < kCostLane; ++u) {
            const float X = d[u] * a, Y = d[u] * b;
            xr[u] = M[0] * X + M[1] * Y + mx[u] + M[9];
            yr[u] = M[3] * X + M[4] * Y + my[u] + M[10];
            zr[u] = M[6] * X + M[7] * Y + mz[u] + M[11];
        }
        // every depth within [2^-40, 2^40] (so in front), else true divisions
        static_assert(kCostLane == 4, "four depths");
        const float zlo = fminf(fminf(zr[0], zr[1]), fminf(zr[2], zr[3]));
        const float zhi = fmaxf(fmaxf(zr[0], zr[1]), fmaxf(zr[2], zr[3]));
        bool front[kCostLane] = {true, true, true, true};
        if (__all(zlo >= 0x1p-40f && zhi <= 0x1p40f)) {
#pragma unroll
            for (int u = 0; u < kCostLane; ++u) divide_pair(xr[u], yr[u], zr[u], xr[u], yr[u]);
        } else {
#pragma unroll
            for (int u = 0; u < kCostLane; ++u) {
                xr[u] = xr[u] / zr[u];
                yr[u] = yr[u] / zr[u];
                front[u] = zr[u] > 0.0f;
            }
        }
        uint64_t g[kCostLane];
        bool ok[kCostLane];
#pragma unroll
        for (int u = 0; u < kCostLane; ++u) {
            const float cu = fx * xr[u] + cx + 0.5f, cv = fy * yr[u] + cy + 0.5f;
            const float ku = __builtin_amdgcn_fmed3f(cu, 0.0f, wtop), kv = __builtin_amdgcn_fmed3f(cv, 0.0f, htop);
            ok[u] = ranged && front[u] && cu == ku && cv == kv;
            // the clamped pixel is gathered whether inside or not
            const uint32_t iu = (uint32_t)ku, iv = (uint32_t)kv;
            if (WIDE) g[u] = *reinterpret_cast<const uint64_t*>(rc + ((size_t)iv * W + iu) * 8);
            else g[u] = *reinterpret_cast<const uint64_t*>(rc + (uint32_t)((__umul24(iv, (uint32_t)W) + iu) * 8u));
        }
        const uint64_t cen = s_cen[i];
        uint32_t word = 0;
#pragma unroll
        for (int u = 0; u < kCostLane; ++u)
            word |= (uint32_t)(ok[u] ? __popcll(cen ^ g[u]) : kCostOut) << (8 * u);
        *reinterpret_cast<word_u*>(out + (size_t)i * D) = word;
    }
}

template <int D>
void launch_cost(dim3 grid, hipStream_t s, const pgs_camera* cams, int W, int H, const uint64_t* census,
                 const int32_t* targets, const int32_t* refs, const double* range, uint8_t* cost) {
    if (W >= (1 << 24) || H >= (1 << 24) || (long long)W * H >= (1ll << 29))
        k_cost<D, true><<<grid, 256, 0, s>>>(cams, W, H, census, targets, refs, range, cost);
    else
        k_cost<D, false><<<grid, 256, 0, s>>>(cams, W, H, census, targets, refs, range, cost);
}

// ---------------------------------------------------------------- SGM

struct SgmArgs {
    const uint8_t* cost;
    // workspace, e = T H W D bytes each: [0] checkpoints (sweeps of whole lines)
    // or left-to-right path costs, [1] row sums (their low bytes) or
    // right-to-left, [2] top-to-bottom
    uint8_t* buf[3];
    uint16_t* agg_out;   // the full sums, if wanted
    uint32_t* over;      // [T][ceil(H / 4)] not 0: a cost of these rows is past byte_cost
    const int32_t* targets;
    const double* range;
    float* depth;        // [T][H][W]
    float* conf;
    int W, H, p1, p2;
    uint32_t byte_cost;  // 127 - p2: up to it two path costs fit a byte, four 9 bits
    double keep_ratio;   // 1 - confidence threshold
};

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <bool V>
struct Const {
    constexpr operator bool() const { return V; }
};

__device__ __forceinline__ u16x2 pair_of(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t word_of(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ u16x2 splat(uint32_t v) { return pair_of(v | (v << 16)); }

// A wave sweeps four image lines at once, one per row of 16 lanes: lane i of
// a row holds the PL = D / 16 consecutive planes PL i .. of its line's pixel
// as NR registers of two 16-bit values (packed 16-bit arithmetic: two planes
// an instruction; the row minimum is four rotations inside the 16 lanes).
// A pixel's costs and path costs are NB words of bytes per lane.  kSeg
// steps are held in registers at a time.
template <int D>
struct Sweep {
    static constexpr int PL = D / 16, NR = PL / 2, NB = PL / 4;
    static constexpr int kSeg = D <= 128 ? 16 : 8;
    struct Bytes {
        uint32_t w[NB];
    };
    typedef uint32_t Any __attribute__((ext_vector_type(NB == 1 ? 2 : NB), aligned(1)));

    __device__ static __forceinline__ Bytes load(const uint8_t* p) {
        Bytes b;
        if constexpr (NB == 1) {
            b.w[0] = *reinterpret_cast<const word_u*>(p);
        } else {
            const Any v = *reinterpret_cast<const Any*>(p);
#pragma unroll
            for (int k = 0; k < NB; ++k) b.w[k] = v[k];
        }
        return b;
    }
    __device__ static __forceinline__ void store(uint8_t* p, const Bytes& b) {
        if constexpr (NB == 1) {
            *reinterpret_cast<word_u*>(p) = b.w[0];
        } else {
            Any v;
#pragma unroll
            for (int k = 0; k < NB; ++k) v[k] = b.w[k];
            *reinterpret_cast<Any*>(p) = v;
        }
    }
    // planes 2 i and 2 i + 1 of packed bytes, as a pair
    __device__ static __forceinline__ u16x2 pair(const Bytes& b, int i) {
        return pair_of(__builtin_amdgcn_perm(0u, b.w[i >> 1], (i & 1) ? 0x0c030c02u : 0x0c010c00u));
    }
    __device__ static __forceinline__ Bytes bytes(const u16x2 (&v)[NR]) {
        Bytes b;
#pragma unroll
        for (int k = 0; k < NB; ++k) b.w[k] = __builtin_amdgcn_perm(word_of(v[2 * k + 1]), word_of(v[2 * k]), 0x06040200u);
        return b;
    }
};

// Minimum over a row's 16 lanes of both halves of v, in both halves of every
// lane.
__device__ __forceinline__ u16x2 row_min(u16x2 v) {
    v = __builtin_elementwise_min(v, __builtin_shufflevector(v, v, 1, 0));
    uint32_t w = word_of(v);  // equal halves: the words order like them
    w = min(w, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x128, 0xf, 0xf, true));
    w = min(w, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x124, 0xf, 0xf, true));
    w = min(w, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x122, 0xf, 0xf, true));
    w = min(w, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x121, 0xf, 0xf, true));
    return pair_of(w);
}

template <int NR>
__device__ __forceinline__ u16x2 least(const u16x2 (&v)[NR]) {
    u16x2 m = v[0];
#pragma unroll
    for (int i = 1; i < NR; ++i) m = __builtin_elementwise_min(m, v[i]);
    return row_min(m);
}

// One step of a path: L(k) = C(k) + min(L(k), L(k +- 1) + P1, m + P2) - m with
// m the least L, over the previous pixel's L; as every L is at least m, the
// minimum less m is min(min(L(k), L(k +- 1) + P1) - m, P2).  A path starts from
// L = 0, which gives its first pixel's costs.
template <int D>
__device__ __forceinline__ void path_step(u16x2 (&L)[Sweep<D>::NR], const typename Sweep<D>::Bytes& c, u16x2 p1,
                                          u16x2 p2) {
    constexpr int NR = Sweep<D>::NR;
    constexpr int kNone = 0x7fff7fff;  // beyond the first and the last plane
    const u16x2 m = least<NR>(L);
    const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)word_of(L[NR - 1]), 0x111, 0xf, 0xf, false);
    const uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp(kNone, (int)word_of(L[0]), 0x101, 0xf, 0xf, false);
    // s[i] = (plane 2 i - 1, plane 2 i): the planes below those of register i,
    // and above those of register i - 1
    u16x2 s[NR + 1];
    s[0] = pair_of(__builtin_amdgcn_alignbit(word_of(L[0]), below, 16));
#pragma unroll
    for (int i = 1; i < NR; ++i) s[i] = pair_of(__builtin_amdgcn_alignbit(word_of(L[i]), word_of(L[i - 1]), 16));
    s[NR] = pair_of(__builtin_amdgcn_alignbit(above, word_of(L[NR - 1]), 16));
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const u16x2 side = __builtin_elementwise_min(s[i], s[i + 1]) + p1;
        const u16x2 best = __builtin_elementwise_min(__builtin_elementwise_min(L[i], side) - m, p2);
        L[i] = Sweep<D>::pair(c, i) + best;
    }
}

// Where a wave's lines lie: line l of a target starts at pixel l (columns) or
// l W (rows) and steps by W or 1.  Lines past the last repeat it: they store
// the same bytes again, so no store is masked and the sweeps' loops know how
// many are in flight when they wait for their loads.
struct Lines {
    size_t first;    // byte of this lane's planes at step 0
    size_t step;     // bytes from a step to the next
    int n, line;     // steps, this lane's line
    bool live;
    __device__ __forceinline__ size_t at(int s) const { return first + (size_t)s * step; }
};

template <int D>
__device__ __forceinline__ Lines lines_of(const SgmArgs& a, bool rows, int wave, int ti) {
    const int lane = threadIdx.x & 63, count = rows ? a.H : a.W;
    Lines q;
    q.n = rows ? a.W : a.H;
    q.line = 4 * wave + (lane >> 4);
    q.live = q.line < count;
    q.line = min(q.line, count - 1);
    const size_t pix = (size_t)ti * a.W * a.H + (rows ? (size_t)q.line * a.W : (size_t)q.line);
    q.first = pix * D + (lane & 15) * Sweep<D>::PL;
    q.step = rows ? (size_t)D : (size_t)a.W * D;
    return q;
}

template <int D>
__device__ __forceinline__ void load_seg(const uint8_t* base, const Lines& q, int seg,
                                         typename Sweep<D>::Bytes (&v)[Sweep<D>::kSeg]) {
    constexpr int S = Sweep<D>::kSeg;
#pragma unroll
    for (int s = 0; s < S; ++s) v[s] = Sweep<D>::load(base + q.at(min(max(seg, 0) * S + s, q.n - 1)));
}

// The bits that any of a segment's costs has, byte by byte.
template <int D>
__device__ __forceinline__ void gather_bits(const typename Sweep<D>::Bytes (&c)[Sweep<D>::kSeg], uint32_t& bits) {
#pragma unroll
    for (int s = 0; s < Sweep<D>::kSeg; ++s)
#pragma unroll
        for (int k = 0; k < Sweep<D>::NB; ++k) bits |= c[s].w[k];
}

// Whether a cost of the wave's lines is above lim (48 to 127), given the bits
// of all of them.  A Census cost is at most 48, so for most limits the bits
// settle it; else the lines are read again and every byte compared (bit 7 of a
// byte: above lim).
template <int D>
__device__ __forceinline__ bool exceeds(uint32_t bits, const uint8_t* cost, const Lines& q, uint32_t lim) {
    constexpr uint32_t kBytes = 0x01010101u;
    const uint32_t within = lim >= 127u ? 0x7fu : lim >= 63u ? 0x3fu : 0x1fu;
    if (__ballot((bits & ~(within * kBytes)) != 0u) == 0ull) return false;
    uint32_t over = 0u;
    for (int s = 0; s < q.n; ++s) {
        const typename Sweep<D>::Bytes c = Sweep<D>::load(cost + q.at(s));
#pragma unroll
        for (int k = 0; k < Sweep<D>::NB; ++k)
            over |= ((c.w[k] & 0x7f7f7f7fu) + (127u - lim) * kBytes) | c.w[k];
    }
    return __ballot((over & 0x80808080u) != 0u) != 0ull;
}

// Forward sweep of whole segments 0 .. nseg - 2 that keeps only the state
// before each segment from 1 on (checkpoints, one per kSeg steps), and with
// BITS the bits of those segments' costs.
template <int D, bool BITS>
__device__ __forceinline__ void checkpoint_sweep(const uint8_t* cost, uint8_t* ck, const Lines& q, u16x2 p1, u16x2 p2,
                                                 uint32_t& bits) {
    typedef Sweep<D> SW;
    constexpr int S = SW::kSeg, NR = SW::NR;
    const int nseg = (q.n + S - 1) / S;
    u16x2 L[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) L[i] = splat(0u);
    typename SW::Bytes c[S], cn[S];
    load_seg<D>(cost, q, 0, c);
    for (int seg = 0; seg + 1 < nseg; ++seg) {
        load_seg<D>(cost, q, seg + 1, cn);
        if constexpr (BITS) gather_bits<D>(c, bits);
#pragma unroll
        for (int s = 0; s < S; ++s) path_step<D>(L, c[s], p1, p2);
        SW::store(ck + q.at((seg + 1) * S), SW::bytes(L));
#pragma unroll
        for (int s = 0; s < S; ++s) c[s] = cn[s];
    }
}

// A segment's forward path costs again, from its checkpoint.
template <int D>
__device__ __forceinline__ void recompute(const typename Sweep<D>::Bytes& ck, bool first,
                                          const typename Sweep<D>::Bytes (&c)[Sweep<D>::kSeg],
                                          typename Sweep<D>::Bytes (&f)[Sweep<D>::kSeg], u16x2 p1, u16x2 p2) {
    typedef Sweep<D> SW;
    u16x2 L[SW::NR];
#pragma unroll
    for (int i = 0; i < SW::NR; ++i) L[i] = first ? splat(0u) : SW::pair(ck, i);
#pragma unroll
    for (int s = 0; s < SW::kSeg; ++s) {
        path_step<D>(L, c[s], p1, p2);
        f[s] = SW::bytes(L);
    }
}

// Both row directions of four rows.  The forward path costs are not stored:
// the forward sweep leaves a checkpoint per segment, and the backward sweep
// recomputes a segment's forward path before walking it back, both from the
// segment's costs in registers.  Per cell the costs are read twice and one
// byte of sum is written (2 (48 + P2) <= 255), where storing the path costs
// and 16-bit sums moved six bytes.  In rows with a cost past 127 - P2, which no
// Census cost is, a sum may pass 255: its low byte is written alone.
template <int D>
__global__ __launch_bounds__(64) void k_sgm_rows(SgmArgs a) {
    typedef Sweep<D> SW;
    constexpr int S = SW::kSeg, NR = SW::NR, NB = SW::NB;
    const Lines q = lines_of<D>(a, true, blockIdx.x, blockIdx.y);
    const u16x2 p1 = splat((uint32_t)a.p1), p2 = splat((uint32_t)a.p2);
    uint32_t bits = 0u;
    checkpoint_sweep<D, true>(a.cost, a.buf[0], q, p1, p2, bits);
    u16x2 L[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) L[i] = splat(0u);
    const int nseg = (q.n + S - 1) / S;
    typename SW::Bytes c[S], cn[S], f[S], ck, ckn;
    load_seg<D>(a.cost, q, nseg - 1, c);
    ck = SW::load(a.buf[0] + q.at((nseg - 1) * S));
    auto back = [&](int seg, auto whole, auto wide) {
        load_seg<D>(a.cost, q, seg - 1, cn);
        ckn = SW::load(a.buf[0] + q.at(max(seg - 1, 0) * S));
        recompute<D>(ck, seg == 0, c, f, p1, p2);
#pragma unroll
        for (int s = S - 1; s >= 0; --s) {
            const int x = seg * S + s;
            if (whole || x < q.n) {
                path_step<D>(L, c[s], p1, p2);
                if constexpr (wide) {
                    u16x2 sum[NR];
#pragma unroll
                    for (int i = 0; i < NR; ++i) sum[i] = L[i] + SW::pair(f[s], i);
                    SW::store(a.buf[1] + q.at(x), SW::bytes(sum));
                } else {
                    typename SW::Bytes b = SW::bytes(L);
#pragma unroll
                    for (int k = 0; k < NB; ++k) b.w[k] += f[s].w[k];  // four sums of bytes, none past 255
                    SW::store(a.buf[1] + q.at(x), b);
                }
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) c[s] = cn[s];
        ck = ckn;
    };
    // only the last segment may be short
    gather_bits<D>(c, bits);
    const bool over = exceeds<D>(bits, a.cost, q, a.byte_cost);
    if (threadIdx.x == 0) a.over[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = over;
    if (q.n % S) back(nseg - 1, Const<false>(), Const<true>());
    for (int seg = q.n / S - 1; seg >= 0; --seg) {
        if (over) back(seg, Const<true>(), Const<true>());
        else back(seg, Const<true>(), Const<false>());
    }
}

// One direction of four lines, its path costs stored: blocks of the grid take
// left to right, right to left and top to bottom side by side.
template <int D>
__global__ __launch_bounds__(64) void k_sgm_paths(SgmArgs a, int row_waves) {
    typedef Sweep<D> SW;
    constexpr int S = SW::kSeg, NR = SW::NR;
    const int dir = (int)blockIdx.x < row_waves ? 0 : (int)blockIdx.x < 2 * row_waves ? 1 : 2;
    const Lines q = lines_of<D>(a, dir < 2, (int)blockIdx.x - dir * row_waves, blockIdx.y);
    const u16x2 p1 = splat((uint32_t)a.p1), p2 = splat((uint32_t)a.p2);
    uint8_t* out = a.buf[dir];
    // step s of a backward path is pixel n - 1 - s
    Lines w = q;
    if (dir == 1) {
        w.first = q.at(q.n - 1);
        w.step = (size_t)0 - q.step;
    }
    u16x2 L[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) L[i] = splat(0u);
    typename SW::Bytes c[S], cn[S];
    load_seg<D>(a.cost, w, 0, c);
    uint32_t bits = 0u;
    auto ahead = [&](int seg, auto whole) {
        load_seg<D>(a.cost, w, seg + 1, cn);
        if constexpr (D == 128) gather_bits<D>(c, bits);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int x = seg * S + s;
            if (whole || x < q.n) {
                path_step<D>(L, c[s], p1, p2);
                SW::store(out + w.at(x), SW::bytes(L));
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) c[s] = cn[s];
    };
    for (int seg = 0; seg < q.n / S; ++seg) ahead(seg, Const<true>());
    if (q.n % S) ahead(q.n / S, Const<false>());
    if (D == 128 && a.over && dir == 0) {
        const bool over = exceeds<D>(bits, a.cost, q, a.byte_cost);
        if (threadIdx.x == 0) a.over[(size_t)blockIdx.y * row_waves + blockIdx.x] = over;
    }
}

// Bottom to top over four columns, added to the other three paths, and each
// pixel's winner.  STAGED: the three are read (buf 0, 1, 2); else the row
// sums are read (buf 1) and top to bottom is swept here first, recomputed by
// segment as in k_sgm_rows.  Per step and row of lanes: the least sum and the
// smallest plane that has it (FUSED, where sum and plane fit 16 bits: one
// minimum of D sum + plane; else one of the sums and one of
// 256 [sum > least] + plane), then the least sum two or more planes away
// (excluded planes raised past every sum); lane s of the row keeps step s,
// and at the segment's end every lane finishes one pixel, taking the winner's
// two neighbours from the segment's sums in LDS.  AGG also stores the sums.
// WIDE: a target with a cost past 127 - P2, whose row sums' low bytes are to be
// completed and whose sums may need ten bits.
template <int D, bool STAGED, bool FUSED, bool AGG, bool WIDE>
__device__ __forceinline__ void cols_lines(const SgmArgs& a, uint32_t (*sums)[4][D / 2]) {
#pragma clang fp contract(off)
    typedef Sweep<D> SW;
    constexpr int S = SW::kSeg, NR = SW::NR;
    const int lane = threadIdx.x & 63, li = lane & 15, row = lane >> 4, ti = blockIdx.y;
    const Lines q = lines_of<D>(a, false, blockIdx.x, ti);
    const u16x2 p1 = splat((uint32_t)a.p1), p2 = splat((uint32_t)a.p2);
    uint32_t bits = 0u;
    if (!STAGED) checkpoint_sweep<D, false>(a.cost, a.buf[0], q, p1, p2, bits);
    const int tv = a.targets[ti];
    const double d_min = a.range[2 * tv], d_max = a.range[2 * tv + 1];
    const double inv_far = 1.0 / d_max, h = (1.0 / d_min - inv_far) / (double)(D - 1);
    u16x2 L[NR], plane[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        L[i] = splat(0u);
        const uint32_t k = (uint32_t)(li * SW::PL + 2 * i);
        plane[i] = pair_of(k | ((k + 1u) << 16));
    }
    const int nseg = (q.n + S - 1) / S;
    typename SW::Bytes c[S], cn[S], r[S], rn[S], f[S], fn[S], ck, ckn;
    typename SW::Bytes r2[STAGED ? S : 1], r2n[STAGED ? S : 1];
    auto fetch = [&](int seg, typename SW::Bytes (&cc)[S], typename SW::Bytes (&rr)[S]) {
        load_seg<D>(a.cost, q, seg, cc);
        load_seg<D>(a.buf[1], q, seg, rr);
    };
    fetch(nseg - 1, c, r);
    if constexpr (STAGED) {
        load_seg<D>(a.buf[2], q, nseg - 1, f);
        load_seg<D>(a.buf[0], q, nseg - 1, r2);
    } else {
        ck = SW::load(a.buf[0] + q.at((nseg - 1) * S));
    }
    auto back = [&](int seg, auto whole) {
        fetch(seg - 1, cn, rn);
        if constexpr (STAGED) {
            load_seg<D>(a.buf[2], q, seg - 1, fn);
            load_seg<D>(a.buf[0], q, seg - 1, r2n);
        } else {
            ckn = SW::load(a.buf[0] + q.at(max(seg - 1, 0) * S));
            recompute<D>(ck, seg == 0, c, f, p1, p2);
        }
        uint32_t my_sums = 0, my_plane = 0;  // (second << 16 | least), winner of step li
#pragma unroll
        for (int s = S - 1; s >= 0; --s) {
            const int y = seg * S + s;
            if (whole || y < q.n) {
                path_step<D>(L, c[s], p1, p2);
                u16x2 T[NR];
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    T[i] = L[i] + SW::pair(f[s], i) + SW::pair(r[s], i);
                    if constexpr (STAGED) T[i] += SW::pair(r2[s], i);
                }
                if constexpr (WIDE && !STAGED) {
                    // a path cost is between C and C + P2, so a row sum lies less
                    // than 256 above 2 C and its low byte tells the rest
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        const u16x2 r0 = SW::pair(r[s], i), c2 = SW::pair(c[s], i) + SW::pair(c[s], i);
                        T[i] += c2 + ((r0 - c2) & splat(0xffu)) - r0;
                    }
                }
                if constexpr (AGG) {
                    typedef uint32_t Half __attribute__((aligned(2)));
                    Half* o = reinterpret_cast<Half*>(a.agg_out + q.at(y));
#pragma unroll
                    for (int i = 0; i < NR; ++i) o[i] = word_of(T[i]);
                }
#pragma unroll
                for (int i = 0; i < NR; ++i) sums[s][row][li * NR + i] = word_of(T[i]);
                u16x2 v[NR], s1, kw;
                if constexpr (FUSED && !(WIDE && D == 128)) {
#pragma unroll
                    for (int i = 0; i < NR; ++i) v[i] = T[i] * splat(D) + plane[i];
                    const u16x2 key = least<NR>(v);
                    s1 = key / splat(D);
                    kw = key & splat(D - 1);
                } else {
                    s1 = least<NR>(T);
#pragma unroll
                    for (int i = 0; i < NR; ++i)  // 256 less where the sum is the least
                        v[i] = __builtin_elementwise_sub_sat(splat(1u), T[i] - s1) * splat(0xff00u) +
                               (plane[i] + splat(256u));
                    kw = least<NR>(v);
                }
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    // 0, 1, 2 for the planes next to and at the winner
                    const u16x2 e = plane[i] + splat(1u) - kw;
                    v[i] = __builtin_elementwise_sub_sat(splat(3u), e) * splat(0x4000u) + T[i];
                }
                const u16x2 s2 = least<NR>(v);
                const uint32_t both = __builtin_amdgcn_perm(word_of(s2), word_of(s1), 0x05040100u);
                my_sums = li == s ? both : my_sums;
                my_plane = li == s ? word_of(kw) & 0xffffu : my_plane;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int y = seg * S + li;
        if (li < S && y < q.n && q.live) {
            const int s1 = (int)(my_sums & 0xffffu), s2 = (int)(my_sums >> 16), kw = (int)my_plane;
            const uint16_t* t = reinterpret_cast<const uint16_t*>(sums[li][row]);
            const int vm = t[kw > 0 ? kw - 1 : 0], vq = t[kw < D - 1 ? kw + 1 : D - 1];
            const bool keep = kw > 0 && kw < D - 1 && s2 > 0 && (double)s1 <= a.keep_ratio * (double)s2;
            float dout = 0.0f;
            if (keep) {
                const int den = vm - 2 * s1 + vq;
                const double delta = den > 0 ? (double)(vm - vq) / (2.0 * (double)den) : 0.0;
                dout = (float)(1.0 / (inv_far + ((double)kw + delta) * h));
            }
            const size_t o = ((size_t)ti * a.H + y) * a.W + q.line;
            a.depth[o] = dout;
            a.conf[o] = s2 > 0 ? (float)(1.0 - (double)s1 / (double)s2) : 0.0f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int s = 0; s < S; ++s) {
            c[s] = cn[s];
            r[s] = rn[s];
            if constexpr (STAGED) {
                f[s] = fn[s];
                r2[s] = r2n[s];
            }
        }
        ck = ckn;
    };
    // only the last segment may be short
    if (q.n % S) back(nseg - 1, Const<false>());
    for (int seg = q.n / S - 1; seg >= 0; --seg) back(seg, Const<true>());
}

// The two bodies side by side, as one that chose per segment cost 6% (eight
// 960 x 720 targets of 128 planes 1229 us, 1300 so; 1228 now).  Two waves a
// SIMD for whole lines, which the second body's registers would make one.
template <int D, bool STAGED, bool FUSED, bool AGG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(STAGED ? 1 : 2))) void k_sgm_cols(SgmArgs a) {
    __shared__ __align__(16) uint32_t sums[Sweep<D>::kSeg][4][D / 2];
    if constexpr (!STAGED || (FUSED && D == 128)) {
        const int rows = (a.H + 3) / 4;
        uint32_t over = 0u;
        for (int k = threadIdx.x; k < rows; k += 64) over |= a.over[(size_t)blockIdx.y * rows + k];
        if (__ballot(over != 0u) != 0ull) {
            cols_lines<D, STAGED, FUSED, AGG, true>(a, sums);
            return;
        }
    }
    cols_lines<D, STAGED, FUSED, AGG, false>(a, sums);
}

// ---------------------------------------------------------------- fusion

__global__ __launch_bounds__(256) void k_fuse_count(const float* __restrict__ depth, int W,
                                                    uint32_t* __restrict__ rowcnt) {
    const size_t row = blockIdx.x;
    const float* d = depth + row * W;
    int c = 0;
    for (int x = threadIdx.x; x < W; x += 256) c += d[x] > 0.0f;
    __shared__ int s[256];
    s[threadIdx.x] = c;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) rowcnt[row] = (uint32_t)s[0];
}

// Exclusive scan of the row counts (one workgroup); total to *total.
__global__ __launch_bounds__(1024) void k_fuse_scan(uint32_t* __restrict__ rows, int n, uint32_t* __restrict__ total) {
    __shared__ uint32_t s[1024];
    uint32_t carry = 0;
    for (int base = 0; base < n; base += 1024) {
        const int i = base + threadIdx.x;
        const uint32_t v = i < n ? rows[i] : 0u;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const uint32_t add = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0u;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < n) rows[i] = carry + s[threadIdx.x] - v;
        carry += s[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// Kept pixel number idx (row-major over the targets) becomes point idx / stride
// when idx is a multiple of stride: world position into out [3][capacity]
// and, with grey given, its intensity / 255 into colour [3][capacity].
__global__ __launch_bounds__(256) void k_fuse_write(const pgs_camera* __restrict__ cams,
                                                    const int32_t* __restrict__ targets, int W, int H,
                                                    const float* __restrict__ depth,
                                                    const uint32_t* __restrict__ rowoff, const uint8_t* __restrict__ grey,
                                                    uint32_t stride, float* __restrict__ out,
                                                    float* __restrict__ colour, uint32_t capacity) {
    __shared__ uint32_t wcnt[4];
    const size_t row = blockIdx.x;
    const int ti = (int)(row / H), y = (int)(row - (size_t)ti * H);
    const Cam64 c = cam64(cams[targets[ti]]);
    const float* d = depth + row * W;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t base = rowoff[row];
    for (int x0 = 0; x0 < W; x0 += 256) {
        const int x = x0 + threadIdx.x;
        const float z = x < W ? d[x] : 0.0f;
        const bool keep = z > 0.0f;
        const uint64_t b = __ballot(keep);
        if (lane == 0) wcnt[wv] = (uint32_t)__popcll(b);
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (int w = 0; w < 4; ++w) {
            before += w < wv ? wcnt[w] : 0u;
            all += wcnt[w];
        }
        const uint32_t idx = base + before + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
        const uint32_t o = idx / stride;
        if (keep && idx == o * stride && o < capacity) {
            const double zz = z;
            const double X = zz * (((double)x - c.cx) / c.fx) - c.t[0];
            const double Y = zz * (((double)y - c.cy) / c.fy) - c.t[1];
            const double Z = zz - c.t[2];
            for (int k = 0; k < 3; ++k)
                out[(size_t)k * capacity + o] = (float)(c.R[k] * X + c.R[3 + k] * Y + c.R[6 + k] * Z);
            if (colour) {
                const float v = (float)grey[((size_t)targets[ti] * H + y) * W + x] / 255.0f;
                for (int k = 0; k < 3; ++k) colour[(size_t)k * capacity + o] = v;
            }
        }
        base += all;
        __syncthreads();
    }
}

inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

pgs_status check_params(const pgs_mvs_params* p, const char* who) {
    PGS_REQUIRE(p, "%s: null params", who);
    PGS_REQUIRE(p->n_planes == 64 || p->n_planes == 128 || p->n_planes == 192 || p->n_planes == 256,
                "%s: n_planes %d not 64, 128, 192 or 256", who, p->n_planes);
    PGS_REQUIRE(p->p1 >= 0 && p->p2 >= 0 && p->p1 <= 1000 && p->p2 <= 1000, "%s: penalties %d, %d not in 0..1000",
                who, p->p1, p->p2);
    PGS_REQUIRE(p->conf_min >= 0.0 && p->conf_min <= 1.0, "%s: conf_min not in [0, 1]", who);
    return PGS_OK;
}

// Large batches sweep whole lines twice (rows, then columns; six bytes moved
// per cell, three forward steps for two).  Small ones, whose few lines leave
// the chip waiting for each step's chain, run three of the four directions
// side by side with their path costs stored (ten bytes per cell), which
// halves the steps that follow one another.  The line lies where the two
// measured even, by waves of four rows (whole lines / side by side): 640x480
// of 64 planes 402 / 372 us at 960 waves; 960x720 of 128 658 / 366 us at 180,
// 680 / 552 at 540, 701 / 725 at 720; 640x480 of 256 818 / 673 at 480,
// 1177 / 1501 at 960.  Sums of two rows that pass a byte, and calls that want
// the sums, run side by side too.  Before, one line per wave with 32-bit
// planes, path costs stored as bytes and row sums in 16 bits: twelve bytes per
// cell and about 50 vector instructions a pixel-step against 11; eight
// 960x720 targets of 128 planes 2.12 -> 1.19 ms, one 0.70 -> 0.37 ms.
template <int D>
constexpr long long kSgmWaves = D == 64 ? 1024 : 640;

template <int D>
pgs_status launch_sgm(SgmArgs a, int n_targets, hipStream_t s) {
    const int rows = (a.H + 3) / 4, cols = (a.W + 3) / 4;
    const bool wide = 2 * (kCostOut + a.p2) > 255;
    if ((long long)rows * n_targets <= kSgmWaves<D> || wide || a.agg_out) {
        // four path costs below 256, or below 128 in a segment without costs
        // past 127 - P2 (Census costs where 4 (48 + P2) < 512), and log2 D
        // bits of plane in 16
        constexpr bool kFits = D == 64;
        const bool fused = kFits || (D == 128 && 4 * (kCostOut + a.p2) < 512);
        const dim3 grid(cols, n_targets);
        if (kFits || !fused) a.over = nullptr;  // right for every cost
        k_sgm_paths<D><<<dim3(2 * rows + cols, n_targets), 64, 0, s>>>(a, rows);
        if (fused) {
            if constexpr (D <= 128) {
                if (a.agg_out) k_sgm_cols<D, true, true, true><<<grid, 64, 0, s>>>(a);
                else k_sgm_cols<D, true, true, false><<<grid, 64, 0, s>>>(a);
            }
        } else if constexpr (!kFits) {
            if (a.agg_out) k_sgm_cols<D, true, false, true><<<grid, 64, 0, s>>>(a);
            else k_sgm_cols<D, true, false, false><<<grid, 64, 0, s>>>(a);
        }
    } else {
        k_sgm_rows<D><<<dim3(rows, n_targets), 64, 0, s>>>(a);
        k_sgm_cols<D, false, (D <= 128), false><<<dim3(cols, n_targets), 64, 0, s>>>(a);
    }
    PGS_CHECK_LAUNCH("pgs_mvs_sgm");
    return PGS_OK;
}

}  // namespace

extern "C" pgs_status pgs_mvs_census(const uint8_t* grey_dev, int32_t n_views, int32_t width, int32_t height,
                                     uint64_t* census_dev, void* stream) {
    PGS_REQUIRE(n_views >= 0 && width >= 0 && height >= 0, "pgs_mvs_census: negative size");
    if (n_views == 0 || width == 0 || height == 0) return PGS_OK;
    PGS_REQUIRE(grey_dev && census_dev, "pgs_mvs_census: null pointer");
    PGS_REQUIRE(n_views <= 65535, "pgs_mvs_census: more than 65535 views");
    const dim3 grid((width + kTile - 1) / kTile, (height + kTile - 1) / kTile, n_views);
    k_census<<<grid, 256, 0, pgs::as_stream(stream)>>>(grey_dev, width, height, census_dev);
    PGS_CHECK_LAUNCH("pgs_mvs_census");
    return PGS_OK;
}

extern "C" size_t pgs_mvs_range_workspace(int32_t n_views, int32_t n_points) {
    if (n_views <= 0 || n_points < 0) return 0;
    return al256((size_t)n_views * n_points * 8);
}

extern "C" pgs_status pgs_mvs_depth_range(const pgs_camera* cams_dev, int32_t n_views, int32_t width, int32_t height,
                                          const double* points_dev, int32_t n_points, double* range_dev,
                                          void* workspace_dev, size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(n_views >= 0 && n_points >= 0 && width > 0 && height > 0, "pgs_mvs_depth_range: bad size");
    if (n_views == 0) return PGS_OK;
    PGS_REQUIRE(n_views <= 65535, "pgs_mvs_depth_range: more than 65535 views");
    PGS_REQUIRE(cams_dev && range_dev && (points_dev || n_points == 0) && workspace_dev,
                "pgs_mvs_depth_range: null pointer");
    PGS_REQUIRE(workspace_bytes >= pgs_mvs_range_workspace(n_views, n_points),
                "pgs_mvs_depth_range: workspace %zu < %zu", workspace_bytes,
                pgs_mvs_range_workspace(n_views, n_points));
    hipStream_t s = pgs::as_stream(stream);
    uint64_t* keys = static_cast<uint64_t*>(workspace_dev);
    if (n_points > 0)
        k_mvs_depths<<<dim3((n_points + 255) / 256, n_views), 256, 0, s>>>(cams_dev, width, height, points_dev,
                                                                           n_points, keys);
    k_mvs_range<<<n_views, 1024, 0, s>>>(n_points, keys, range_dev);
    PGS_CHECK_LAUNCH("pgs_mvs_depth_range");
    return PGS_OK;
}

extern "C" pgs_status pgs_mvs_select_ref(const pgs_camera* cams_dev, int32_t n_views, const pgs_mvs_params* params,
                                         int32_t* ref_dev, void* stream) {
    PGS_REQUIRE(n_views >= 0, "pgs_mvs_select_ref: negative size");
    if (n_views == 0) return PGS_OK;
    PGS_REQUIRE(cams_dev && ref_dev && params, "pgs_mvs_select_ref: null pointer");
    PGS_REQUIRE(params->sigma_b > 0.0 && params->alpha_min > 0.0, "pgs_mvs_select_ref: sigma_b, alpha_min must be > 0");
    k_mvs_ref<<<(n_views + 63) / 64, 64, 0, pgs::as_stream(stream)>>>(cams_dev, n_views, params->b_target,
                                                                      params->sigma_b, params->alpha_min, ref_dev);
    PGS_CHECK_LAUNCH("pgs_mvs_select_ref");
    return PGS_OK;
}

extern "C" pgs_status pgs_mvs_cost(const pgs_camera* cams_dev, int32_t width, int32_t height,
                                   const uint64_t* census_dev, const int32_t* targets_dev, int32_t n_targets,
                                   const int32_t* ref_dev, const double* range_dev, const pgs_mvs_params* params,
                                   uint8_t* cost_dev, void* stream) {
    if (pgs_status st = check_params(params, "pgs_mvs_cost")) return st;
    PGS_REQUIRE(n_targets >= 0 && width > 0 && height > 0, "pgs_mvs_cost: bad size");
    if (n_targets == 0) return PGS_OK;
    PGS_REQUIRE(n_targets <= 65535, "pgs_mvs_cost: more than 65535 targets");
    PGS_REQUIRE(cams_dev && census_dev && targets_dev && ref_dev && range_dev && cost_dev, "pgs_mvs_cost: null pointer");
    const int D = params->n_planes;
    const long long npix = (long long)width * height;
    PGS_REQUIRE(npix < (1ll << 31), "pgs_mvs_cost: image too large");
    hipStream_t s = pgs::as_stream(stream);
    const dim3 grid((unsigned)((npix + kCostPix - 1) / kCostPix), n_targets);
    switch (D) {
        case 64: launch_cost<64>(grid, s, cams_dev, width, height, census_dev, targets_dev, ref_dev, range_dev, cost_dev); break;
        case 128: launch_cost<128>(grid, s, cams_dev, width, height, census_dev, targets_dev, ref_dev, range_dev, cost_dev); break;
        case 192: launch_cost<192>(grid, s, cams_dev, width, height, census_dev, targets_dev, ref_dev, range_dev, cost_dev); break;
        default: launch_cost<256>(grid, s, cams_dev, width, height, census_dev, targets_dev, ref_dev, range_dev, cost_dev); break;
    }
    PGS_CHECK_LAUNCH("pgs_mvs_cost");
    return PGS_OK;
}

extern "C" size_t pgs_mvs_sgm_workspace(int32_t n_targets, int32_t width, int32_t height, int32_t n_planes) {
    if (n_targets <= 0 || width <= 0 || height <= 0 || n_planes <= 0) return 0;
    const size_t e = (size_t)n_targets * width * height * n_planes;
    return al256(e) + al256(e * 2) + al256((size_t)n_targets * ((height + 3) / 4) * 4);
}

extern "C" pgs_status pgs_mvs_sgm(const uint8_t* cost_dev, int32_t width, int32_t height, const int32_t* targets_dev,
                                  int32_t n_targets, const double* range_dev, const pgs_mvs_params* params,
                                  float* depth_dev, float* conf_dev, uint16_t* agg_out_dev, void* workspace_dev,
                                  size_t workspace_bytes, void* stream) {
    if (pgs_status st = check_params(params, "pgs_mvs_sgm")) return st;
    PGS_REQUIRE(n_targets >= 0 && width > 0 && height > 0, "pgs_mvs_sgm: bad size");
    if (n_targets == 0) return PGS_OK;
    PGS_REQUIRE(n_targets <= 65535, "pgs_mvs_sgm: more than 65535 targets");
    PGS_REQUIRE(cost_dev && targets_dev && range_dev && depth_dev && conf_dev, "pgs_mvs_sgm: null pointer");
    PGS_REQUIRE(workspace_dev && workspace_bytes >= pgs_mvs_sgm_workspace(n_targets, width, height,
                                                                           params->n_planes),
                "pgs_mvs_sgm: workspace too small");
    PGS_REQUIRE(48 + params->p2 <= 255, "pgs_mvs_sgm: path costs up to %d do not fit a byte", 48 + params->p2);
    const size_t e = (size_t)n_targets * width * height * params->n_planes;
    SgmArgs a{};
    a.cost = cost_dev;
    char* ws = static_cast<char*>(workspace_dev);
    a.buf[0] = reinterpret_cast<uint8_t*>(ws);
    a.buf[1] = reinterpret_cast<uint8_t*>(ws + al256(e));
    a.buf[2] = a.buf[1] + e;
    a.over = reinterpret_cast<uint32_t*>(ws + al256(e) + al256(e * 2));
    a.agg_out = agg_out_dev;
    a.targets = targets_dev;
    a.range = range_dev;
    a.depth = depth_dev;
    a.conf = conf_dev;
    a.W = width;
    a.H = height;
    a.p1 = params->p1;
    a.p2 = params->p2;
    a.byte_cost = (uint32_t)max(127 - params->p2, 0);
    a.keep_ratio = 1.0 - params->conf_min;
    hipStream_t s = pgs::as_stream(stream);
    switch (params->n_planes) {
        case 64: return launch_sgm<64>(a, n_targets, s);
        case 128: return launch_sgm<128>(a, n_targets, s);
        case 192: return launch_sgm<192>(a, n_targets, s);
        default: return launch_sgm<256>(a, n_targets, s);
    }
}

extern "C" size_t pgs_mvs_fuse_workspace(int32_t n_targets, int32_t height) {
    if (n_targets <= 0 || height <= 0) return 0;
    return al256((size_t)n_targets * height * 4);
}

extern "C" pgs_status pgs_mvs_fuse(const pgs_camera* cams_dev, const int32_t* targets_dev, int32_t n_targets,
                                   int32_t width, int32_t height, const float* depth_dev, const uint8_t* grey_dev,
                                   uint32_t stride, float* points_dev, float* colour_dev, uint32_t capacity,
                                   uint32_t* count_dev, void* workspace_dev, size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(n_targets >= 0 && width > 0 && height > 0 && stride >= 1, "pgs_mvs_fuse: bad size or stride");
    PGS_REQUIRE(count_dev, "pgs_mvs_fuse: null count");
    PGS_REQUIRE(!colour_dev || grey_dev, "pgs_mvs_fuse: colours need the grey images");
    hipStream_t s = pgs::as_stream(stream);
    if (n_targets == 0) {
        k_mvs_clear<<<1, 256, 0, s>>>(count_dev, 1);
        PGS_CHECK_LAUNCH("pgs_mvs_fuse");
        return PGS_OK;
    }
    PGS_REQUIRE(cams_dev && targets_dev && depth_dev && (points_dev || capacity == 0) && workspace_dev,
                "pgs_mvs_fuse: null pointer");
    PGS_REQUIRE(workspace_bytes >= pgs_mvs_fuse_workspace(n_targets, height), "pgs_mvs_fuse: workspace too small");
    const long long rows = (long long)n_targets * height;
    PGS_REQUIRE(rows < (1ll << 31), "pgs_mvs_fuse: too many rows");
    uint32_t* rowcnt = static_cast<uint32_t*>(workspace_dev);
    k_fuse_count<<<(unsigned)rows, 256, 0, s>>>(depth_dev, width, rowcnt);
    k_fuse_scan<<<1, 1024, 0, s>>>(rowcnt, (int)rows, count_dev);
    k_fuse_write<<<(unsigned)rows, 256, 0, s>>>(cams_dev, targets_dev, width, height, depth_dev, rowcnt, grey_dev,
                                                stride, points_dev, colour_dev, capacity);
    PGS_CHECK_LAUNCH("pgs_mvs_fuse");
    return PGS_OK;
}
