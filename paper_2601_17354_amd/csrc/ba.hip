// Robust bundle adjustment with the reduced camera system (PocketGS
// subsection "GPU-Native Global BA as Mobile MAP Refinement": the robustified
// reprojection objective of equation ba_obj, scale-aware gauge fixing, and
// the Schur complement over the block-diagonal point blocks).
//
// Everything is float64.  One Levenberg-Marquardt step (pgs_ba_step):
//   k_ba_points   one thread per point, over its observations: residual,
//                 Huber weight, Jacobians; the point block H_pp + lambda
//                 diag(H_pp) inverted in place (3x3, adjugate), v = H_pp^-1 b_p.
//                 The observations' own blocks are not stored: every kernel
//                 that needs one linearises the observation again (about 150
//                 instructions; its 45 stored values made 360 bytes per
//                 observation out and several times back);
//   k_ba_cameras  16 workgroups per camera, each over a slice of its
//                 observations: the camera's pose block and gradient, and
//                 partial row blocks of the reduced system
//                 S = H_tt - H_tp H_pp^-1 H_pt (its blocks (i, k), k <= i:
//                 the solve reads the lower triangle) and g = b_t - H_tp v,
//                 accumulated in LDS over every pair of observations that
//                 share a point (float64 LDS atomics); k_ba_rows sums the
//                 slices in order, damps, and writes the gauge-free lower
//                 triangle (camera 0's six parameters and camera 1's centre
//                 coordinate along the gauge axis left out);
//   k_ba_first /  a Cholesky in 32-column panels, one launch per panel, the
//   k_ba_panel    right-hand side carried as an extra row so the forward
//                 substitution comes with the factor, and k_ba_back, the
//                 back substitution -> the pose step;
//   k_ba_backsub  one thread per point: dP = v - H_pp^-1 sum H_tp^T dt.
// The cost (sum of Huber terms) is reduced per block in a fixed order.
#include <math.h>

#include "common.hpp"

namespace {

constexpr int kCamThreads = 256;
constexpr int kCostThreads = 256;
constexpr int kPointThreads = 64;

// Per-point record: damped H_pp^-1 (3x3 row-major) and v (3).
constexpr int kPtRec = 12;

// A camera in LDS: rotation (9, row-major) and centre (3), padded so that
// different cameras' words fall in different banks.
constexpr int kCamRec = 13;

struct Obs {
    double r[2];        // residual
    double w;           // Huber weight
    double Jt[2][6];    // d r / d(dphi, dc)
    double Jp[2][3];    // d r / dP
};

__device__ __forceinline__ void load_cams(const pgs_ba_problem& pb, const double* __restrict__ rot,
                                          const double* __restrict__ centre, double* cam) {
    for (int e = threadIdx.x; e < pb.n_cams * 12; e += blockDim.x) {
        const int i = e / 12, k = e - i * 12;
        cam[i * kCamRec + k] = k < 9 ? rot[9 * (size_t)i + k] : centre[3 * (size_t)i + k - 9];
    }
}

// The observation (u, v) of point P by the camera record cam.
__device__ __forceinline__ void observe(const pgs_ba_problem& pb, const double* cam, const double (&P)[3], double u,
                                        double v, Obs& ob) {
    double R[9];
    for (int k = 0; k < 9; ++k) R[k] = cam[k];
    const double d0 = P[0] - cam[9], d1 = P[1] - cam[10], d2 = P[2] - cam[11];
    const double x0 = R[0] * d0 + R[1] * d1 + R[2] * d2;
    const double x1 = R[3] * d0 + R[4] * d1 + R[5] * d2;
    const double x2 = R[6] * d0 + R[7] * d1 + R[8] * d2;
    const double iz = 1.0 / x2;
    ob.r[0] = pb.fx * x0 * iz + pb.cx - u;
    ob.r[1] = pb.fy * x1 * iz + pb.cy - v;
    const double s = ob.r[0] * ob.r[0] + ob.r[1] * ob.r[1];
    const double nrm = sqrt(s);
    ob.w = nrm <= pb.huber_delta ? 1.0 : pb.huber_delta / nrm;
    // d pi / d x
    const double a00 = pb.fx * iz, a02 = -pb.fx * x0 * iz * iz;
    const double a11 = pb.fy * iz, a12 = -pb.fy * x1 * iz * iz;
    // A R (2x3): d r / dP; d r / dc = -A R; d r / ddphi = -A R [d]x
    double AR[2][3];
    for (int k = 0; k < 3; ++k) {
        AR[0][k] = a00 * R[k] + a02 * R[6 + k];
        AR[1][k] = a11 * R[3 + k] + a12 * R[6 + k];
    }
    for (int r = 0; r < 2; ++r) {
        // (A R) [d]x with [d]x = [[0,-d2,d1],[d2,0,-d0],[-d1,d0,0]]
        const double m0 = AR[r][1] * d2 - AR[r][2] * d1;
        const double m1 = -AR[r][0] * d2 + AR[r][2] * d0;
        const double m2 = AR[r][0] * d1 - AR[r][1] * d0;
        ob.Jt[r][0] = -m0;
        ob.Jt[r][1] = -m1;
        ob.Jt[r][2] = -m2;
        for (int k = 0; k < 3; ++k) {
            ob.Jt[r][3 + k] = -AR[r][k];
            ob.Jp[r][k] = AR[r][k];
        }
    }
}

__device__ __forceinline__ void load_point(const double* __restrict__ pts, size_t j, double (&P)[3]) {
    for (int a = 0; a < 3; ++a) P[a] = pts[3 * j + a];
}

__device__ __forceinline__ int tri6(int a, int b) {  // index of (a, b), a <= b, in the 6x6 upper triangle
    return a * 6 - a * (a - 1) / 2 + (b - a);
}

__global__ __launch_bounds__(kPointThreads) void k_ba_points(pgs_ba_problem pb, const double* __restrict__ rot,
                                                             const double* __restrict__ centre,
                                                             const double* __restrict__ pts, double lam,
                                                             double* __restrict__ pt_rec) {
    extern __shared__ double cam[];
    load_cams(pb, rot, centre, cam);
    __syncthreads();
    const int j = blockIdx.x * kPointThreads + threadIdx.x;
    if (j >= pb.n_points) return;
    double P[3];
    load_point(pts, j, P);
    double Hp[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, bp[3] = {0, 0, 0};
    const uint32_t o0 = pb.point_start_dev[j], o1 = pb.point_start_dev[j + 1];
    for (uint32_t o = o0; o < o1; ++o) {
        Obs ob;
        observe(pb, cam + pb.obs_cam_dev[o] * kCamRec, P, pb.obs_uv_dev[2 * (size_t)o],
                pb.obs_uv_dev[2 * (size_t)o + 1], ob);
        for (int a = 0; a < 3; ++a) {
            for (int b = 0; b < 3; ++b) Hp[a][b] += ob.w * (ob.Jp[0][a] * ob.Jp[0][b] + ob.Jp[1][a] * ob.Jp[1][b]);
            bp[a] -= ob.w * (ob.Jp[0][a] * ob.r[0] + ob.Jp[1][a] * ob.r[1]);
        }
    }
    // damped point block and its inverse (adjugate / determinant)
    for (int a = 0; a < 3; ++a) Hp[a][a] += lam * Hp[a][a];
    const double c00 = Hp[1][1] * Hp[2][2] - Hp[1][2] * Hp[2][1];
    const double c01 = Hp[1][2] * Hp[2][0] - Hp[1][0] * Hp[2][2];
    const double c02 = Hp[1][0] * Hp[2][1] - Hp[1][1] * Hp[2][0];
    const double det = Hp[0][0] * c00 + Hp[0][1] * c01 + Hp[0][2] * c02;
    const double id = 1.0 / det;
    double Ai[3][3];
    Ai[0][0] = c00 * id;
    Ai[1][0] = c01 * id;
    Ai[2][0] = c02 * id;
    Ai[0][1] = (Hp[0][2] * Hp[2][1] - Hp[0][1] * Hp[2][2]) * id;
    Ai[1][1] = (Hp[0][0] * Hp[2][2] - Hp[0][2] * Hp[2][0]) * id;
    Ai[2][1] = (Hp[0][1] * Hp[2][0] - Hp[0][0] * Hp[2][1]) * id;
    Ai[0][2] = (Hp[0][1] * Hp[1][2] - Hp[0][2] * Hp[1][1]) * id;
    Ai[1][2] = (Hp[0][2] * Hp[1][0] - Hp[0][0] * Hp[1][2]) * id;
    Ai[2][2] = (Hp[0][0] * Hp[1][1] - Hp[0][1] * Hp[1][0]) * id;
    double* pr = pt_rec + (size_t)j * kPtRec;
    for (int a = 0; a < 3; ++a) {
        for (int b = 0; b < 3; ++b) pr[3 * a + b] = Ai[a][b];
        pr[9 + a] = Ai[a][0] * bp[0] + Ai[a][1] * bp[1] + Ai[a][2] * bp[2];
    }
}

__device__ __forceinline__ double wave_sum_f64(double v) {
    for (int k = 32; k > 0; k >>= 1) {
        const long long b = __double_as_longlong(v);
        const int lo = __shfl_xor((int)(b & 0xffffffffll), k), hi = __shfl_xor((int)(b >> 32), k);
        v += __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    }
    return v;
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup (i, s): slice s of camera i's observations, 64 to a wave.  First
// each lane linearises one observation of camera i: its pose block and
// gradient, its share of - H_tp v, and T = H_tp H_pp^-1 with the point's
// coordinates into the wave's LDS slots.  Then the pairs (observation, member
// k <= i of its point's track) are listed, eight members of every track at a
// time, and taken one per lane whichever observation they belong to: the
// lane linearises the member and adds - T H_tp(k)^T, 36 float64 LDS atomics.
// The lane's own track in lockstep (half of its members past i) and each
// member's block read from memory took 0.55 ms for 60 cameras and 786k
// observations, 0.21 ms now, of which the LDS is busy 0.09 ms with the adds
// (two workgroups per CU is what its size allows).  Blocks of 37 values
// put different cameras' terms in different banks.
// An observation's pair with itself, which would put as many adds on one
// block as the wave has tracks, is taken off the pose block in registers (its
// product is symmetric too).
// Partials go to part[i][s][36 n_cams + 33]: row blocks k <= i, then pose
// block less own pairs (21), the pose block's diagonal (6, for the damping)
// and gradient less H_tp v (6).
constexpr int kCamSplit = 16;
constexpr int kBlk = 37;               // 36 values of a row block, padded
constexpr int kSlot = 21;              // T (18) and the point (3)
constexpr int kMembers = 8;            // members of a track listed at a time
constexpr int kPose = 33;

constexpr size_t cameras_lds(int n_cams) {
    return (size_t)(kCamRec + kBlk) * n_cams * 8 + (kCamThreads / 64) * (64 * kSlot * 8 + 64 * kMembers * 4 + 64 * 4);
}

__global__ __launch_bounds__(kCamThreads) void k_ba_cameras(pgs_ba_problem pb, const double* __restrict__ rot,
                                                            const double* __restrict__ centre,
                                                            const double* __restrict__ pts,
                                                            const double* __restrict__ pt_rec,
                                                            double* __restrict__ part) {
    extern __shared__ double lds[];
    constexpr int NW = kCamThreads / 64;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, C = pb.n_cams, split = blockIdx.y;
    const int i = C - 1 - (int)blockIdx.x;  // the last cameras have the most pairs and go first
    double* cam = lds;                            // [C][kCamRec]
    double* acc = cam + (size_t)C * kCamRec;      // [C][kBlk]
    double* slots = acc + (size_t)C * kBlk + (size_t)wv * 64 * kSlot;
    uint32_t* lists = reinterpret_cast<uint32_t*>(acc + (size_t)C * kBlk + (size_t)NW * 64 * kSlot);
    uint32_t* list = lists + wv * 64 * (kMembers + 1);
    uint32_t* starts = list + 64 * kMembers;      // first observation of each slot's track
    load_cams(pb, rot, centre, cam);
    for (int e = t; e < (i + 1) * kBlk; e += kCamThreads) acc[e] = 0.0;
    __syncthreads();
    const uint32_t c0 = pb.cam_start_dev[i], c1 = pb.cam_start_dev[i + 1];
    const uint32_t chunk = (c1 - c0 + kCamSplit - 1) / kCamSplit;
    const uint32_t q0 = c0 + split * chunk, q1 = min(c1, q0 + chunk);
    double pose[kPose];
#pragma unroll
    for (int k = 0; k < kPose; ++k) pose[k] = 0.0;
    for (uint32_t qb = q0 + wv * 64; qb < q1; qb += kCamThreads) {
        const bool has = qb + lane < q1;
        uint32_t s0 = 0, n = 0, own = 0;
        if (has) {
            const uint32_t o = pb.cam_obs_dev[qb + lane], j = pb.obs_pt_dev[o];
            own = o;
            s0 = pb.point_start_dev[j];
            n = pb.point_start_dev[j + 1] - s0;
            double P[3];
            load_point(pts, j, P);
            Obs ob;
            observe(pb, cam + i * kCamRec, P, pb.obs_uv_dev[2 * (size_t)o], pb.obs_uv_dev[2 * (size_t)o + 1], ob);
            const double* pr = pt_rec + (size_t)j * kPtRec;
            double h0[3], h1[3];  // w Jp H_pp^-1
            double v0 = 0.0, v1 = 0.0;
            for (int b = 0; b < 3; ++b) {
                h0[b] = ob.w * (ob.Jp[0][0] * pr[b] + ob.Jp[0][1] * pr[3 + b] + ob.Jp[0][2] * pr[6 + b]);
                h1[b] = ob.w * (ob.Jp[1][0] * pr[b] + ob.Jp[1][1] * pr[3 + b] + ob.Jp[1][2] * pr[6 + b]);
                v0 += ob.w * ob.Jp[0][b] * pr[9 + b];
                v1 += ob.w * ob.Jp[1][b] * pr[9 + b];
            }
            double* slot = slots + lane * kSlot;
            // H_tp H_pp^-1 H_pt of the observation itself: Jt^T G Jt
            double g00 = 0.0, g01 = 0.0, g11 = 0.0;
            for (int b = 0; b < 3; ++b) {
                g00 += ob.w * h0[b] * ob.Jp[0][b];
                g01 += ob.w * h0[b] * ob.Jp[1][b];
                g11 += ob.w * h1[b] * ob.Jp[1][b];
            }
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                const double w0 = ob.w * ob.Jt[0][a], w1 = ob.w * ob.Jt[1][a];
                const double u0 = w0 - (g00 * ob.Jt[0][a] + g01 * ob.Jt[1][a]);
                const double u1 = w1 - (g01 * ob.Jt[0][a] + g11 * ob.Jt[1][a]);
#pragma unroll
                for (int b = a; b < 6; ++b) pose[tri6(a, b)] += u0 * ob.Jt[0][b] + u1 * ob.Jt[1][b];
                pose[21 + a] += w0 * ob.Jt[0][a] + w1 * ob.Jt[1][a];
                pose[27 + a] -= ob.Jt[0][a] * (ob.w * ob.r[0] + v0) + ob.Jt[1][a] * (ob.w * ob.r[1] + v1);
                for (int b = 0; b < 3; ++b) slot[3 * a + b] = ob.Jt[0][a] * h0[b] + ob.Jt[1][a] * h1[b];
            }
            for (int a = 0; a < 3; ++a) slot[18 + a] = P[a];
            starts[lane] = s0;
        }
        for (uint32_t m = 0; __any(m < n); m += kMembers) {
            uint32_t mine = 0;
#pragma unroll
            for (int u = 0; u < kMembers; ++u)
                if (m + u < n && s0 + m + u != own && (int)pb.obs_cam_dev[s0 + m + u] <= i) mine |= 1u << u;
            const int cnt = __popc(mine);
            int inc = cnt;
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(inc, o);
                if (lane >= o) inc += up;
            }
            const int total = __shfl(inc, 63);
            int at = inc - cnt;
            for (uint32_t w = mine; w; w &= w - 1) list[at++] = ((uint32_t)lane << 3) | (uint32_t)(__ffs(w) - 1);
            wave_sync();
            for (int f = lane; f < total; f += 64) {
                const uint32_t en = list[f], sl = en >> 3, o2 = starts[sl] + m + (en & 7u);
                const int k = (int)pb.obs_cam_dev[o2];
                const double* slot = slots + sl * kSlot;
                double P[3];
                for (int a = 0; a < 3; ++a) P[a] = slot[18 + a];
                Obs ob;
                observe(pb, cam + k * kCamRec, P, pb.obs_uv_dev[2 * (size_t)o2], pb.obs_uv_dev[2 * (size_t)o2 + 1],
                        ob);
                double* out = acc + (size_t)k * kBlk;
                for (int a = 0; a < 6; ++a) {
                    const double t0 = slot[3 * a], t1 = slot[3 * a + 1], t2 = slot[3 * a + 2];
                    const double u0 = -ob.w * (t0 * ob.Jp[0][0] + t1 * ob.Jp[0][1] + t2 * ob.Jp[0][2]);
                    const double u1 = -ob.w * (t0 * ob.Jp[1][0] + t1 * ob.Jp[1][1] + t2 * ob.Jp[1][2]);
                    for (int b = 0; b < 6; ++b) atomicAdd(&out[6 * a + b], u0 * ob.Jt[0][b] + u1 * ob.Jt[1][b]);
                }
            }
            wave_sync();  // the list is read before it is written again
        }
    }
    __syncthreads();
    double* out = part + ((size_t)i * kCamSplit + split) * (36 * (size_t)C + kPose);
    for (int e = t; e < (i + 1) * 36; e += kCamThreads) out[e] = acc[(e / 36) * kBlk + e % 36];
    // the waves' pose sums, added in order (the slots are free again)
    double* wsum = acc + (size_t)C * kBlk;  // [NW][kPose]
#pragma unroll
    for (int k = 0; k < kPose; ++k) {
        const double v = wave_sum_f64(pose[k]);
        if (lane == 0) wsum[wv * kPose + k] = v;
    }
    __syncthreads();
    if (t < kPose) {
        double h = 0.0;
        for (int w = 0; w < NW; ++w) h += wsum[w * kPose + t];
        out[36 * (size_t)C + t] = h;
    }
}

// Number of pose parameter p among the free (moving) ones, or -1: camera 0's six
// and camera 1's centre coordinate along the gauge axis are fixed.
__device__ __forceinline__ int free_index(int p, int gauge_axis) {
    if (p < 6 || p == 9 + gauge_axis) return -1;
    return p - 6 - (p > 9 + gauge_axis ? 1 : 0);
}

// The gauge-free reduced system from the camera slices' partials, summed in
// slice order: thread (i, k, a, b) of the lower triangle's row blocks, the
// damped pose block added at k = i; the right-hand side becomes row nf of A.
__global__ __launch_bounds__(256) void k_ba_rows(int n_cams, int gauge_axis, double lam,
                                                 const double* __restrict__ part, double* __restrict__ A) {
    const int nf = 6 * n_cams - 7, per = 36 * n_cams + kPose;
    const int i = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x;
    if (e >= 36 * (i + 1) + 6) return;
    const double* p = part + (size_t)i * kCamSplit * per;
    auto slices = [&](int at) {
        double acc = 0.0;
        for (int sp = 0; sp < kCamSplit; ++sp) acc += p[(size_t)sp * per + at];
        return acc;
    };
    if (e >= 36 * (i + 1)) {
        const int a = e - 36 * (i + 1), r = free_index(6 * i + a, gauge_axis);
        if (r >= 0) A[(size_t)nf * nf + r] = slices(36 * n_cams + 27 + a);
        return;
    }
    const int k = e / 36, ab = e - 36 * k, a = ab / 6, b = ab - 6 * a;
    const int r = free_index(6 * i + a, gauge_axis), c = free_index(6 * k + b, gauge_axis);
    if (r < 0 || c < 0 || c > r) return;
    double v = slices(e);
    if (k == i) {
        v += slices(36 * n_cams + (a <= b ? tri6(a, b) : tri6(b, a)));
        if (a == b) v += lam * slices(36 * n_cams + 21 + a);
    }
    A[(size_t)r * nf + c] = v;
}

// ---------------------------------------------------------------- solve
//
// A holds nf + 1 rows of nf: the lower triangle of the system, then the
// right-hand side as an extra row, so that the Cholesky factorisation
// A = L L^T of the rows computes the forward substitution L y = g as that
// row's entries of L.  Right-looking, in panels of 32 columns with one launch
// each (k_ba_panel): a workgroup per 32 x 32 tile of the trailing triangle
// turns its own two row blocks of the panel into L (rows x of A solved for
// x L11^T, with the diagonal block's factor that the launch before left) and
// subtracts their product; the workgroup of the next panel's diagonal block
// then factors it.  Nothing but that block's chain is serial.  Both triangular
// solves are substitutions: products with the diagonal blocks' inverses, which
// took as long, left 20 to 100 times the backward error on views so narrow that
// turning and moving a camera hardly differ.  One workgroup factoring a panel,
// another launch updating the
// trailing triangle and a triangular solve per row of the panel took 505 + 74
// us at 60 cameras (nf = 353), 12 launches of 13.3 us and 39 + 10 us for the
// back substitution and the first block now (products with inverses: 12.3 and
// 30): each launch's fixed 4 us, its substitution and the 5 us of its 32 pivots
// are what is left.
constexpr int kPW = 32;
constexpr int kPS = kPW + 1;
constexpr int kSolveThreads = 1024;

__device__ __forceinline__ double read_lane_f64(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// 1 / sqrt(d) to the last place or two: the hardware's estimate and one
// third-order correction.
__device__ __forceinline__ double inv_sqrt(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Cholesky factor of the 32 x 32 block D (lower triangle, row stride kPS, in
// LDS), by one wave in registers: lane r < 32 eliminates row r (the other
// lanes repeat them).  The next pivot's entry goes from lane to lane through
// scalar registers, so that the chain of pivots is a reciprocal root and three
// products a step; the rest of the column is read back from LDS (col, 32 x 32)
// in its shadow.  Column-major to out, what lies above the diagonal arbitrary.
__device__ __forceinline__ void factor_block(const double* D, double* col, double* __restrict__ out, int lane) {
    double v[kPW];
    const int r = lane & 31;
#pragma unroll
    for (int c = 0; c < kPW; ++c) v[c] = D[r * kPS + c];
    double pivot = read_lane_f64(v[0], 0);
#pragma unroll
    for (int p = 0; p < kPW; ++p) {
        const double m = v[p] * inv_sqrt(pivot);
        v[p] = m;
        if (p + 1 < kPW) {
            v[p + 1] = fma(-m, read_lane_f64(m, p + 1), v[p + 1]);
            pivot = read_lane_f64(v[p + 1], p + 1);
        }
        if (p + 2 < kPW) {
            if (lane < 32) col[p * kPW + r] = m;
            wave_sync();
#pragma unroll
            for (int c = p + 2; c < kPW; ++c) v[c] = fma(-m, col[p * kPW + c], v[c]);
        }
    }
    if (lane < 32) {
#pragma unroll
        for (int c = 0; c < kPW; ++c) out[c * kPW + r] = v[c];
    }
}

// The first panel's diagonal block (identity past nf).
__global__ __launch_bounds__(64) void k_ba_first(int nf, const double* __restrict__ A, double* __restrict__ fac) {
    __shared__ __align__(16) double D[kPW * kPS], col[kPW * kPW];
    for (int e = threadIdx.x; e < kPW * kPW; e += 64) {
        const int r = e / kPW, c = e % kPW;
        D[r * kPS + c] = r < nf && c <= r ? A[(size_t)r * nf + c] : (r == c ? 1.0 : 0.0);
    }
    __syncthreads();
    factor_block(D, col, fac, threadIdx.x);
}

// Thread (ty, tx) of a 16 x 16 grid: rows 2 ty, 2 ty + 1 of X times rows
// 2 tx, 2 tx + 1 of Y (32 columns each).
__device__ __forceinline__ void tile_product(const double* X, const double* Y, int ty, int tx, double (&o)[2][2]) {
    o[0][0] = o[0][1] = o[1][0] = o[1][1] = 0.0;
#pragma unroll 8
    for (int p = 0; p < kPW; ++p) {
        const double a0 = X[2 * ty * kPS + p], a1 = X[(2 * ty + 1) * kPS + p];
        const double b0 = Y[2 * tx * kPS + p], b1 = Y[(2 * tx + 1) * kPS + p];
        o[0][0] = fma(a0, b0, o[0][0]);
        o[0][1] = fma(a0, b1, o[0][1]);
        o[1][0] = fma(a1, b0, o[1][0]);
        o[1][1] = fma(a1, b1, o[1][1]);
    }
}

template <int V>
struct Int {
    static constexpr int value = V;
};

// The value of lane LANE of each four.
template <int LANE>
__device__ __forceinline__ double quad_lane_f64(double v) {
    const long long b = __double_as_longlong(v);
    constexpr int kCtrl = LANE * 0x55;
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Panel k0: tile e of the lower triangle of rows k0 + 32 .. nf (the
// right-hand side last).  L gets the panel's rows below its diagonal block.
// Four lanes solve a row of each block, lane l its columns 4 i + l: what the
// factor's words cost from LDS is shared by two rows.  (One row a lane, the
// whole factor read by every lane, took 1.5 us more a launch.)
__global__ __launch_bounds__(256) void k_ba_panel(int nf, int k0, double* __restrict__ A, double* __restrict__ L,
                                                  double* __restrict__ facs) {
    __shared__ __align__(16) double F[kPW * kPW], X[kPW * kPS], Y[kPW * kPS], D[kPW * kPS], rd[kPW];
    const int t = threadIdx.x, nb = min(kPW, nf - k0), r0 = k0 + nb;
    const int mt = nf + 1 - r0, mc = nf - r0;  // rows and columns left
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    const int tj = (int)blockIdx.x - ti * (ti + 1) / 2, i0 = ti * kPW, j0 = tj * kPW;
    if (tj > 0 && j0 >= mc) return;
    const double* fac = facs + (size_t)(k0 / kPW) * kPW * kPW;
    for (int q = t; q < kPW * kPW; q += 256) {
        const int r = q / kPW, p = q % kPW;
        F[q] = p > r ? fac[q] : 0.0;  // column r, row p, below the diagonal
        X[r * kPS + p] = i0 + r < mt && p < nb ? A[(size_t)(r0 + i0 + r) * nf + k0 + p] : 0.0;
        Y[r * kPS + p] = j0 + r < mc && p < nb ? A[(size_t)(r0 + j0 + r) * nf + k0 + p] : 0.0;
        if (r == p) rd[r] = 1.0 / fac[q];
    }
    __syncthreads();
    if (t < 4 * kPW) {
        const int l = t & 3;
        double *xr = X + (t >> 2) * kPS + l, *yr = Y + (t >> 2) * kPS + l;
        const double* fl = F + l;
        double x[kPW / 4], y[kPW / 4];
#pragma unroll
        for (int i = 0; i < kPW / 4; ++i) {
            x[i] = xr[4 * i];
            y[i] = yr[4 * i];
        }
        auto quad = [&](auto k) {  // columns 4 k .. 4 k + 3
            constexpr int K = decltype(k)::value;
            auto column = [&](auto c) {
                constexpr int C = decltype(c)::value, P = 4 * K + C;
                const double xp = quad_lane_f64<C>(x[K] * rd[P]), yp = quad_lane_f64<C>(y[K] * rd[P]);
#pragma unroll
                for (int i = K; i < kPW / 4; ++i) {
                    const double f = fl[P * kPW + 4 * i];  // zero up to the column itself
                    x[i] = fma(-xp, f, x[i]);
                    y[i] = fma(-yp, f, y[i]);
                }
                x[K] = l == C ? xp : x[K];
                y[K] = l == C ? yp : y[K];
            };
            column(Int<0>());
            column(Int<1>());
            column(Int<2>());
            column(Int<3>());
        };
        quad(Int<0>());
        quad(Int<1>());
        quad(Int<2>());
        quad(Int<3>());
        quad(Int<4>());
        quad(Int<5>());
        quad(Int<6>());
        quad(Int<7>());
        static_assert(kPW == 32, "eight quads of columns");
#pragma unroll
        for (int i = 0; i < kPW / 4; ++i) {
            xr[4 * i] = x[i];
            yr[4 * i] = y[i];
        }
    }
    __syncthreads();
    const int ty = t >> 4, tx = t & 15;
    if (tj == 0) {
        for (int q = t; q < kPW * kPW; q += 256) {
            const int r = q / kPW, p = q % kPW;
            if (i0 + r < mt && p < nb) L[(size_t)(r0 + i0 + r) * nf + k0 + p] = X[r * kPS + p];
        }
    }
    if (mc == 0) return;  // the last panel: only the right-hand side's row is left
    double o[2][2];
    tile_product(X, Y, ty, tx, o);
    const bool next = blockIdx.x == 0;  // the next panel's diagonal block
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int r = 2 * ty + u, c = 2 * tx + v, ii = i0 + r, jj = j0 + c;
            double w = 0.0;
            if (ii < mt && jj < mc && jj <= ii) {
                double* at = A + (size_t)(r0 + ii) * nf + r0 + jj;
                w = *at - o[u][v];
                *at = w;
            }
            if (next) D[r * kPS + c] = ii < mc && jj <= ii ? w : (r == c ? 1.0 : 0.0);
        }
    if (!next) return;
    __syncthreads();
    if (t < 64) factor_block(D, F, facs + (size_t)(k0 / kPW + 1) * kPW * kPW, t);
}

// Sum over each half of the wave, in every lane of the half.
template <int CTRL>
__device__ __forceinline__ double dpp_add_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double half_sum(double v) {
    v = dpp_add_f64<0x128>(v);  // rotations inside a row of 16 lanes
    v = dpp_add_f64<0x124>(v);
    v = dpp_add_f64<0x122>(v);
    v = dpp_add_f64<0x121>(v);
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)(b & 0xffffffffll), hi = (uint32_t)(b >> 32);
    // rows 0 and 1, and 2 and 3, meet
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __longlong_as_double(((long long)h[0] << 32) | l[0]) + __longlong_as_double(((long long)h[1] << 32) | l[1]);
}

// Back substitution L^T x = y, y = row nf of L, by one workgroup, panels last
// to first: x_p = L11^-T (y_p - sum over the rows below of L^T x).  Thread
// (slice, column) sums the column's products with the solved entries over
// every 32nd row below the panel, whose factors are loaded a panel ahead (they
// do not depend on x); the slices meet through LDS, each half wave adding one
// column's; one wave then substitutes through the panel's factor, whose entries
// were loaded a panel ahead too.  The step is scattered to the free pose
// entries; the fixed ones are 0.
constexpr int kBackRows = (6 * PGS_BA_MAX_CAMS + kPW - 1) / kPW;  // rows per slice at most

__global__ __launch_bounds__(kSolveThreads) void k_ba_back(int n_cams, int gauge_axis, const double* __restrict__ L,
                                                           const double* __restrict__ facs,
                                                           double* __restrict__ dpose) {
    __shared__ double red[kPW][kPS], F[kPW][kPS], xs[6 * PGS_BA_MAX_CAMS], z[kPW];
    const int n6 = 6 * n_cams, nf = n6 - 7, t = threadIdx.x, cc = t % kPW, sl = t / kPW;
    const int last = (nf - 1) / kPW, rows = (nf + kPW - 1) / kPW;
    double f[kBackRows], fe, y;
    auto fetch = [&](int pn) {
        const int k0 = pn * kPW, nb = min(kPW, nf - k0), r0 = k0 + nb;
        fe = y = 0.0;
        if (pn < 0) return;  // uniform
#pragma unroll
        for (int q = 0; q < kBackRows; ++q)
            if (q < rows) {
                const int r = r0 + sl + q * kPW;
                f[q] = cc < nb && r < nf ? L[(size_t)r * nf + k0 + cc] : 0.0;
            }
        // row cc, column sl of the factor; the right-hand side's entry sl
        fe = facs[(size_t)pn * kPW * kPW + sl * kPW + cc];
        y = sl < nb ? L[(size_t)nf * nf + k0 + sl] : 0.0;
    };
    for (int e = t; e < 6 * PGS_BA_MAX_CAMS; e += kSolveThreads) xs[e] = 0.0;
    fetch(last);
    __syncthreads();
    for (int pn = last; pn >= 0; --pn) {
        const int k0 = pn * kPW, r0 = min(k0 + kPW, nf);
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < kBackRows; ++q)
            if (q < rows) {
                const int r = r0 + sl + q * kPW;
                if (r < nf) v = fma(f[q], xs[r], v);
            }
        red[sl][cc] = v;
        F[sl][cc] = fe;
        const double yy = y;
        fetch(pn - 1);
        __syncthreads();
        // column sl: its slices' sums, one per lane of the half
        const double w = yy - half_sum(red[cc][sl]);
        if (cc == 0) z[sl] = w;
        __syncthreads();
        if (t < 64) {  // lane cc: entry cc (both halves alike)
            double left = z[cc], x = 0.0;
            const double rd = 1.0 / F[cc][cc];
#pragma unroll 8
            for (int q = kPW - 1; q >= 0; --q) {
                const double own = left * rd, xq = read_lane_f64(own, q);
                if (cc == q) x = own;
                left = fma(-xq, F[cc][q], left);  // of no use to lanes past q
            }
            if (t < kPW && k0 + cc < nf) xs[k0 + cc] = x;
        }
        __syncthreads();
    }
    for (int e = t; e < n6; e += kSolveThreads) {
        const int r = free_index(e, gauge_axis);
        dpose[e] = r >= 0 ? xs[r] : 0.0;
    }
}

__global__ __launch_bounds__(kPointThreads) void k_ba_backsub(pgs_ba_problem pb, const double* __restrict__ rot,
                                                              const double* __restrict__ centre,
                                                              const double* __restrict__ pts,
                                                              const double* __restrict__ pt_rec,
                                                              const double* __restrict__ dpose,
                                                              double* __restrict__ dpoint) {
    extern __shared__ double cam[];
    load_cams(pb, rot, centre, cam);
    __syncthreads();
    const int j = blockIdx.x * kPointThreads + threadIdx.x;
    if (j >= pb.n_points) return;
    double P[3], s[3] = {0, 0, 0};
    load_point(pts, j, P);
    for (uint32_t o = pb.point_start_dev[j]; o < pb.point_start_dev[j + 1]; ++o) {
        const uint32_t i = pb.obs_cam_dev[o];
        Obs ob;
        observe(pb, cam + i * kCamRec, P, pb.obs_uv_dev[2 * (size_t)o], pb.obs_uv_dev[2 * (size_t)o + 1], ob);
        const double* dt = dpose + 6 * (size_t)i;
        double d0 = 0.0, d1 = 0.0;  // Jt dt
        for (int a = 0; a < 6; ++a) {
            d0 += ob.Jt[0][a] * dt[a];
            d1 += ob.Jt[1][a] * dt[a];
        }
        for (int b = 0; b < 3; ++b) s[b] += ob.w * (ob.Jp[0][b] * d0 + ob.Jp[1][b] * d1);
    }
    const double* pr = pt_rec + (size_t)j * kPtRec;
    for (int a = 0; a < 3; ++a)
        dpoint[3 * (size_t)j + a] = pr[9 + a] - (pr[3 * a] * s[0] + pr[3 * a + 1] * s[1] + pr[3 * a + 2] * s[2]);
}

// Robust cost: per-block partial sums of rho over the observations.
__global__ __launch_bounds__(kCostThreads) void k_ba_cost(pgs_ba_problem pb, const double* __restrict__ rot,
                                                          const double* __restrict__ centre,
                                                          const double* __restrict__ pts,
                                                          double* __restrict__ part) {
    __shared__ double s[kCostThreads];
    extern __shared__ double cam[];
    load_cams(pb, rot, centre, cam);
    __syncthreads();
    double acc = 0.0;
    for (int j = blockIdx.x * kCostThreads + threadIdx.x; j < pb.n_points; j += gridDim.x * kCostThreads) {
        double P[3];
        load_point(pts, j, P);
        for (uint32_t o = pb.point_start_dev[j]; o < pb.point_start_dev[j + 1]; ++o) {
            Obs ob;
            observe(pb, cam + pb.obs_cam_dev[o] * kCamRec, P, pb.obs_uv_dev[2 * (size_t)o],
                    pb.obs_uv_dev[2 * (size_t)o + 1], ob);
            const double q = ob.r[0] * ob.r[0] + ob.r[1] * ob.r[1];
            const double n = sqrt(q);
            acc += n <= pb.huber_delta ? q : 2.0 * pb.huber_delta * n - pb.huber_delta * pb.huber_delta;
        }
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int k = kCostThreads / 2; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// The blocks' sums, added in a fixed order (one thread alone took 20 us over
// 386 of them).
__global__ __launch_bounds__(kCostThreads) void k_ba_cost_final(const double* __restrict__ part, int n,
                                                                double* __restrict__ out) {
    __shared__ double s[kCostThreads];
    double acc = 0.0;
    for (int k = threadIdx.x; k < n; k += kCostThreads) acc += part[k];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int k = kCostThreads / 2; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

__global__ __launch_bounds__(256) void k_ba_apply(int n_cams, int n_points, const double* __restrict__ rot,
                                                  const double* __restrict__ centre,
                                                  const double* __restrict__ pts, const double* __restrict__ dpose,
                                                  const double* __restrict__ dpoint, double* __restrict__ rot_out,
                                                  double* __restrict__ centre_out, double* __restrict__ pts_out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n_points)
        for (int a = 0; a < 3; ++a) pts_out[3 * (size_t)k + a] = pts[3 * (size_t)k + a] + dpoint[3 * (size_t)k + a];
    if (k < n_cams) {
        const double* w = dpose + 6 * k;
        const double th = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        // exp([w]x) = I + a [w]x + b [w]x^2 (Rodrigues; series below 1e-8)
        const double a = th < 1e-8 ? 1.0 - th * th / 6.0 : sin(th) / th;
        const double b = th < 1e-8 ? 0.5 - th * th / 24.0 : (1.0 - cos(th)) / (th * th);
        const double K[9] = {0, -w[2], w[1], w[2], 0, -w[0], -w[1], w[0], 0};
        double E[9];
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) {
                double kk = 0.0;
                for (int m = 0; m < 3; ++m) kk += K[3 * r + m] * K[3 * m + c];
                E[3 * r + c] = (r == c ? 1.0 : 0.0) + a * K[3 * r + c] + b * kk;
            }
        const double* R = rot + 9 * k;
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c)
                rot_out[9 * k + 3 * r + c] = R[3 * r] * E[c] + R[3 * r + 1] * E[3 + c] + R[3 * r + 2] * E[6 + c];
        for (int a2 = 0; a2 < 3; ++a2) centre_out[3 * k + a2] = centre[3 * k + a2] + w[3 + a2];
    }
}

// ------------------------------------------------------------ refinement

// Thread per point: the least-squares intersection of its observation rays
// (sum (I - d d^T) P = sum (I - d d^T) c, d the unit world ray of the
// measured pixel, solved by the adjugate when det > 1e-12 trace^3), then
// over its observations in front of their cameras the mean reprojection
// error and the smallest cosine between two camera-to-point rays; the point
// is kept with >= 2 such observations, mean error <= max_err and smallest
// cosine <= cos_min; an observation is kept when its point is and it lies
// in front of its camera.
__global__ __launch_bounds__(256) void k_ba_refine(pgs_ba_problem pb, const double* __restrict__ rot,
                                                   const double* __restrict__ centre, double max_err,
                                                   double cos_min, double* __restrict__ pts_out,
                                                   uint8_t* __restrict__ keep_pt, uint8_t* __restrict__ keep_obs) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= pb.n_points) return;
    const uint32_t o0 = pb.point_start_dev[j], o1 = pb.point_start_dev[j + 1];
    double A[6] = {0, 0, 0, 0, 0, 0}, b[3] = {0, 0, 0};  // A00 A01 A02 A11 A12 A22
    for (uint32_t o = o0; o < o1; ++o) {
        const int i = (int)pb.obs_cam_dev[o];
        const double* R = rot + 9 * (size_t)i;
        const double* c = centre + 3 * (size_t)i;
        const double q0 = (pb.obs_uv_dev[2 * (size_t)o] - pb.cx) / pb.fx;
        const double q1 = (pb.obs_uv_dev[2 * (size_t)o + 1] - pb.cy) / pb.fy;
        double d[3];
        for (int a = 0; a < 3; ++a) d[a] = R[a] * q0 + R[3 + a] * q1 + R[6 + a];  // R^T (q0, q1, 1)
        const double inv = 1.0 / sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        for (int a = 0; a < 3; ++a) d[a] *= inv;
        const double dc = d[0] * c[0] + d[1] * c[1] + d[2] * c[2];
        A[0] += 1.0 - d[0] * d[0];
        A[1] -= d[0] * d[1];
        A[2] -= d[0] * d[2];
        A[3] += 1.0 - d[1] * d[1];
        A[4] -= d[1] * d[2];
        A[5] += 1.0 - d[2] * d[2];
        for (int a = 0; a < 3; ++a) b[a] += c[a] - d[a] * dc;
    }
    const double c00 = A[3] * A[5] - A[4] * A[4], c01 = A[2] * A[4] - A[1] * A[5], c02 = A[1] * A[4] - A[2] * A[3];
    const double c11 = A[0] * A[5] - A[2] * A[2], c12 = A[1] * A[2] - A[0] * A[4], c22 = A[0] * A[3] - A[1] * A[1];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    const double tr = A[0] + A[3] + A[5];
    const bool solvable = det > 1e-12 * tr * tr * tr;
    double P[3] = {0.0, 0.0, 0.0};
    if (solvable) {
        const double id = 1.0 / det;
        P[0] = (c00 * b[0] + c01 * b[1] + c02 * b[2]) * id;
        P[1] = (c01 * b[0] + c11 * b[1] + c12 * b[2]) * id;
        P[2] = (c02 * b[0] + c12 * b[1] + c22 * b[2]) * id;
    }
    int cnt = 0;
    double esum = 0.0, mincos = 2.0;
    for (uint32_t o = o0; o < o1 && solvable; ++o) {
        const int i = (int)pb.obs_cam_dev[o];
        const double* R = rot + 9 * (size_t)i;
        const double* c = centre + 3 * (size_t)i;
        const double v0 = P[0] - c[0], v1 = P[1] - c[1], v2 = P[2] - c[2];
        const double x0 = R[0] * v0 + R[1] * v1 + R[2] * v2, x1 = R[3] * v0 + R[4] * v1 + R[5] * v2,
                     x2 = R[6] * v0 + R[7] * v1 + R[8] * v2;
        if (!(x2 > 0.0)) continue;
        const double du = pb.fx * x0 / x2 + pb.cx - pb.obs_uv_dev[2 * (size_t)o];
        const double dv = pb.fy * x1 / x2 + pb.cy - pb.obs_uv_dev[2 * (size_t)o + 1];
        esum += sqrt(du * du + dv * dv);
        ++cnt;
        const double n0 = 1.0 / sqrt(v0 * v0 + v1 * v1 + v2 * v2);
        for (uint32_t o2 = o + 1; o2 < o1; ++o2) {
            const int k = (int)pb.obs_cam_dev[o2];
            const double* R2 = rot + 9 * (size_t)k;
            const double* c2 = centre + 3 * (size_t)k;
            const double w0 = P[0] - c2[0], w1 = P[1] - c2[1], w2 = P[2] - c2[2];
            if (!(R2[6] * w0 + R2[7] * w1 + R2[8] * w2 > 0.0)) continue;
            const double cs = (v0 * w0 + v1 * w1 + v2 * w2) * n0 / sqrt(w0 * w0 + w1 * w1 + w2 * w2);
            mincos = fmin(mincos, cs);
        }
    }
    const bool keep = solvable && cnt >= 2 && esum / (double)(cnt > 0 ? cnt : 1) <= max_err && mincos <= cos_min;
    for (int a = 0; a < 3; ++a) pts_out[3 * (size_t)j + a] = P[a];
    keep_pt[j] = keep ? 1 : 0;
    for (uint32_t o = o0; o < o1; ++o) {
        bool front = false;
        if (keep) {
            const int i = (int)pb.obs_cam_dev[o];
            const double* R = rot + 9 * (size_t)i;
            const double* c = centre + 3 * (size_t)i;
            front = R[6] * (P[0] - c[0]) + R[7] * (P[1] - c[1]) + R[8] * (P[2] - c[2]) > 0.0;
        }
        keep_obs[o] = front ? 1 : 0;
    }
}

// Exclusive scan of 0/1 flags (optionally read through a permutation) into
// idx[0..n] (idx[n] = total): per-block sums, one workgroup over the block
// sums, then per-block prefixes.
constexpr int kFlagBlock = 1024;

__device__ __forceinline__ uint32_t flag_at(const uint8_t* f, const uint32_t* perm, uint32_t i) {
    return f[perm ? perm[i] : i] ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_flag_sums(const uint8_t* __restrict__ f, const uint32_t* __restrict__ perm,
                                                   uint32_t n, uint32_t* __restrict__ bsum) {
    __shared__ uint32_t s[4];
    const uint32_t base = blockIdx.x * kFlagBlock;
    uint32_t c = 0;
    for (uint32_t i = base + threadIdx.x; i < min(n, base + kFlagBlock); i += 256) c += flag_at(f, perm, i);
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) bsum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(1024) void k_flag_top(uint32_t* __restrict__ bsum, uint32_t nb) {
    __shared__ uint32_t s[1024];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nb; base += 1024) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t v = i < nb ? bsum[i] : 0u;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const uint32_t add = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0u;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nb) bsum[i] = carry + s[threadIdx.x] - v;
        carry += s[1023];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_flag_apply(const uint8_t* __restrict__ f, const uint32_t* __restrict__ perm,
                                                    uint32_t n, const uint32_t* __restrict__ bsum,
                                                    uint32_t* __restrict__ idx) {
    __shared__ uint32_t s[4];
    const uint32_t base = blockIdx.x * kFlagBlock;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t run = bsum[blockIdx.x];
    for (uint32_t c0 = base; c0 < min(n, base + kFlagBlock); c0 += 256) {
        const uint32_t i = c0 + threadIdx.x;
        const uint32_t v = i < n ? flag_at(f, perm, i) : 0u;
        const uint64_t bal = __ballot(v != 0u);
        if (lane == 0) s[wv] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (int w = 0; w < 4; ++w) {
            before += w < wv ? s[w] : 0u;
            all += s[w];
        }
        if (i < n) idx[i] = run + before + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        run += all;
        __syncthreads();
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) idx[n] = run;
}

pgs_status flag_scan(const uint8_t* f, const uint32_t* perm, uint32_t n, uint32_t* idx, uint32_t* bsum,
                     hipStream_t s) {
    const uint32_t nb = (n + kFlagBlock - 1) / kFlagBlock;
    if (nb == 0) return PGS_OK;
    k_flag_sums<<<nb, 256, 0, s>>>(f, perm, n, bsum);
    k_flag_top<<<1, 1024, 0, s>>>(bsum, nb);
    k_flag_apply<<<nb, 256, 0, s>>>(f, perm, n, bsum, idx);
    return PGS_OK;
}

// Points: kept ones renumbered, their first observation's new index.
__global__ __launch_bounds__(256) void k_compact_points(int M, const uint8_t* __restrict__ keep_pt,
                                                        const uint32_t* __restrict__ pidx,
                                                        const uint32_t* __restrict__ oidx,
                                                        const uint32_t* __restrict__ point_start,
                                                        const double* __restrict__ pts, double* __restrict__ pts_out,
                                                        uint32_t* __restrict__ point_start_out, int O,
                                                        uint32_t* __restrict__ counts) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < M && keep_pt[j]) {
        const uint32_t n = pidx[j];
        for (int a = 0; a < 3; ++a) pts_out[3 * (size_t)n + a] = pts[3 * (size_t)j + a];
        point_start_out[n] = oidx[point_start[j]];
    }
    if (j == 0) {
        point_start_out[pidx[M]] = oidx[point_start[M]];
        counts[0] = pidx[M];
        counts[1] = oidx[O];
    }
}

__global__ __launch_bounds__(256) void k_compact_obs(pgs_ba_problem pb, const uint8_t* __restrict__ keep_obs,
                                                     const uint32_t* __restrict__ oidx,
                                                     const uint32_t* __restrict__ pidx, const uint32_t* __restrict__ qidx,
                                                     uint32_t* __restrict__ cam_out, uint32_t* __restrict__ pt_out,
                                                     double* __restrict__ uv_out, uint32_t* __restrict__ cam_obs_out,
                                                     uint32_t* __restrict__ cam_start_out) {
    const uint32_t o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o < (uint32_t)pb.n_obs) {
        if (keep_obs[o]) {
            const uint32_t n = oidx[o];
            cam_out[n] = pb.obs_cam_dev[o];
            pt_out[n] = pidx[pb.obs_pt_dev[o]];
            uv_out[2 * (size_t)n] = pb.obs_uv_dev[2 * (size_t)o];
            uv_out[2 * (size_t)n + 1] = pb.obs_uv_dev[2 * (size_t)o + 1];
        }
        // o is a position in the by-camera list here
        const uint32_t ob = pb.cam_obs_dev[o];
        if (keep_obs[ob]) cam_obs_out[qidx[o]] = oidx[ob];
    }
    if (o <= (uint32_t)pb.n_cams) cam_start_out[o] = qidx[pb.cam_start_dev[o]];
}

// Workspace layout of one problem size.
struct BaWs {
    double *pt_rec, *cam_part, *A, *L, *facs, *part;
    size_t bytes;
};

inline size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr int kCostBlocks = 1024;

BaWs ba_layout(void* base, int C, int M, int O) {
    (void)O;
    BaWs w{};
    char* p = static_cast<char*>(base);
    size_t off = 0;
    const size_t n6 = 6 * (size_t)C, nf = n6 > 7 ? n6 - 7 : 0;
    auto take = [&](size_t n) { double* q = reinterpret_cast<double*>(p + off); off += al(n * 8); return q; };
    w.pt_rec = take((size_t)M * kPtRec);
    w.cam_part = take((size_t)C * kCamSplit * (36 * (size_t)C + kPose));
    w.A = take((nf + 1) * nf);
    w.L = take((nf + 1) * nf);
    w.facs = take(((nf + kPW - 1) / kPW) * kPW * kPW);
    w.part = take(kCostBlocks);
    w.bytes = off;
    return w;
}

inline size_t cams_lds(int C) { return (size_t)C * kCamRec * sizeof(double); }

bool cameras_lds_reserved() {
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(k_ba_cameras),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)cameras_lds(PGS_BA_MAX_CAMS)) == hipSuccess;
    return ok;
}

// The solve as a chain of launches, one per panel.
void solve_panels(int C, int gauge_axis, const BaWs& w, double* dpose, hipStream_t s) {
    const int nf = 6 * C - 7;
    k_ba_first<<<1, 64, 0, s>>>(nf, w.A, w.facs);
    for (int k0 = 0; k0 < nf; k0 += kPW) {
        const int mt = nf + 1 - min(k0 + kPW, nf), tiles = (mt + kPW - 1) / kPW;
        k_ba_panel<<<tiles * (tiles + 1) / 2, 256, 0, s>>>(nf, k0, w.A, w.L, w.facs);
    }
    k_ba_back<<<1, kSolveThreads, 0, s>>>(C, gauge_axis, w.L, w.facs, dpose);
}

pgs_status check_problem(const pgs_ba_problem* pb, const char* who) {
    PGS_REQUIRE(pb != nullptr, "%s: null problem", who);
    PGS_REQUIRE(pb->n_cams >= 2 && pb->n_cams <= PGS_BA_MAX_CAMS, "%s: n_cams %d not in 2..%d", who, pb->n_cams,
                PGS_BA_MAX_CAMS);
    PGS_REQUIRE(pb->n_points >= 1 && pb->n_obs >= 1, "%s: empty problem", who);
    PGS_REQUIRE(pb->gauge_axis >= 0 && pb->gauge_axis <= 2, "%s: gauge_axis %d", who, pb->gauge_axis);
    PGS_REQUIRE(pb->huber_delta > 0.0, "%s: huber_delta must be > 0", who);
    PGS_REQUIRE(pb->obs_cam_dev && pb->obs_pt_dev && pb->obs_uv_dev && pb->point_start_dev && pb->cam_obs_dev &&
                    pb->cam_start_dev, "%s: null pointer in the problem", who);
    return PGS_OK;
}

}  // namespace

extern "C" size_t pgs_ba_workspace(int32_t n_cams, int32_t n_points, int32_t n_obs) {
    if (n_cams < 0 || n_points < 0 || n_obs < 0) return 0;
    return ba_layout(nullptr, n_cams, n_points, n_obs).bytes;
}

extern "C" pgs_status pgs_ba_cost(const pgs_ba_problem* problem, const double* rot_dev, const double* centre_dev,
                                  const double* points_dev, double* cost_dev, void* workspace_dev,
                                  size_t workspace_bytes, void* stream) {
    if (pgs_status st = check_problem(problem, "pgs_ba_cost")) return st;
    PGS_REQUIRE(rot_dev && centre_dev && points_dev && cost_dev && workspace_dev, "pgs_ba_cost: null pointer");
    const BaWs w = ba_layout(workspace_dev, problem->n_cams, problem->n_points, problem->n_obs);
    PGS_REQUIRE(workspace_bytes >= w.bytes, "pgs_ba_cost: workspace %zu < %zu", workspace_bytes, w.bytes);
    hipStream_t s = pgs::as_stream(stream);
    const int blocks = min(kCostBlocks, (problem->n_points + kCostThreads - 1) / kCostThreads);
    k_ba_cost<<<blocks, kCostThreads, cams_lds(problem->n_cams), s>>>(*problem, rot_dev, centre_dev, points_dev,
                                                                     w.part);
    k_ba_cost_final<<<1, kCostThreads, 0, s>>>(w.part, blocks, cost_dev);
    PGS_CHECK_LAUNCH("pgs_ba_cost");
    return PGS_OK;
}

extern "C" pgs_status pgs_ba_step(const pgs_ba_problem* problem, const double* rot_dev, const double* centre_dev,
                                  const double* points_dev, double lambda, double* dpose_dev, double* dpoint_dev,
                                  void* workspace_dev, size_t workspace_bytes, void* stream) {
    if (pgs_status st = check_problem(problem, "pgs_ba_step")) return st;
    PGS_REQUIRE(lambda >= 0.0, "pgs_ba_step: lambda < 0");
    PGS_REQUIRE(rot_dev && centre_dev && points_dev && dpose_dev && dpoint_dev && workspace_dev,
                "pgs_ba_step: null pointer");
    const int C = problem->n_cams, M = problem->n_points;
    const BaWs w = ba_layout(workspace_dev, C, M, problem->n_obs);
    PGS_REQUIRE(workspace_bytes >= w.bytes, "pgs_ba_step: workspace %zu < %zu", workspace_bytes, w.bytes);
    hipStream_t s = pgs::as_stream(stream);
    PGS_REQUIRE(cameras_lds_reserved(), "pgs_ba_step: cannot reserve LDS for the camera rows");
    const int pblocks = (M + kPointThreads - 1) / kPointThreads;
    k_ba_points<<<pblocks, kPointThreads, cams_lds(C), s>>>(*problem, rot_dev, centre_dev, points_dev, lambda,
                                                            w.pt_rec);
    k_ba_cameras<<<dim3(C, kCamSplit), kCamThreads, cameras_lds(C), s>>>(*problem, rot_dev, centre_dev, points_dev,
                                                                         w.pt_rec, w.cam_part);
    k_ba_rows<<<dim3((36 * C + 6 + 255) / 256, C), 256, 0, s>>>(C, problem->gauge_axis, lambda, w.cam_part, w.A);
    solve_panels(C, problem->gauge_axis, w, dpose_dev, s);
    k_ba_backsub<<<pblocks, kPointThreads, cams_lds(C), s>>>(*problem, rot_dev, centre_dev, points_dev, w.pt_rec,
                                                             dpose_dev, dpoint_dev);
    PGS_CHECK_LAUNCH("pgs_ba_step");
    return PGS_OK;
}

extern "C" pgs_status pgs_ba_apply(int32_t n_cams, int32_t n_points, const double* rot_dev,
                                   const double* centre_dev, const double* points_dev, const double* dpose_dev,
                                   const double* dpoint_dev, double* rot_out_dev, double* centre_out_dev,
                                   double* points_out_dev, void* stream) {
    PGS_REQUIRE(n_cams >= 0 && n_points >= 0, "pgs_ba_apply: negative size");
    PGS_REQUIRE(rot_dev && centre_dev && points_dev && dpose_dev && dpoint_dev && rot_out_dev && centre_out_dev &&
                    points_out_dev, "pgs_ba_apply: null pointer");
    const int n = max(n_cams, n_points);
    if (n == 0) return PGS_OK;
    k_ba_apply<<<(n + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(n_cams, n_points, rot_dev, centre_dev,
                                                                   points_dev, dpose_dev, dpoint_dev, rot_out_dev,
                                                                   centre_out_dev, points_out_dev);
    PGS_CHECK_LAUNCH("pgs_ba_apply");
    return PGS_OK;
}

extern "C" pgs_status pgs_ba_refine(const pgs_ba_problem* problem, const double* rot_dev, const double* centre_dev,
                                    double max_err, double min_angle, double* points_out_dev,
                                    uint8_t* keep_point_dev, uint8_t* keep_obs_dev, void* stream) {
    if (pgs_status st = check_problem(problem, "pgs_ba_refine")) return st;
    PGS_REQUIRE(rot_dev && centre_dev && points_out_dev && keep_point_dev && keep_obs_dev,
                "pgs_ba_refine: null pointer");
    PGS_REQUIRE(max_err >= 0.0 && min_angle >= 0.0, "pgs_ba_refine: negative threshold");
    const int M = problem->n_points;
    k_ba_refine<<<(M + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(*problem, rot_dev, centre_dev, max_err,
                                                                     cos(min_angle), points_out_dev, keep_point_dev,
                                                                     keep_obs_dev);
    PGS_CHECK_LAUNCH("pgs_ba_refine");
    return PGS_OK;
}

extern "C" size_t pgs_ba_compact_workspace(int32_t n_points, int32_t n_obs) {
    if (n_points < 0 || n_obs < 0) return 0;
    const size_t nb = ((size_t)(n_points > n_obs ? n_points : n_obs) + kFlagBlock - 1) / kFlagBlock + 1;
    return al(((size_t)n_points + 1) * 4) + 2 * al(((size_t)n_obs + 1) * 4) + 3 * al(nb * 4);
}

extern "C" pgs_status pgs_ba_compact(const pgs_ba_problem* problem, const uint8_t* keep_point_dev,
                                     const uint8_t* keep_obs_dev, const double* points_dev,
                                     uint32_t* obs_cam_out_dev, uint32_t* obs_pt_out_dev, double* obs_uv_out_dev,
                                     uint32_t* point_start_out_dev, uint32_t* cam_obs_out_dev,
                                     uint32_t* cam_start_out_dev, double* points_out_dev, uint32_t* counts_out_dev,
                                     void* workspace_dev, size_t workspace_bytes, void* stream) {
    if (pgs_status st = check_problem(problem, "pgs_ba_compact")) return st;
    PGS_REQUIRE(keep_point_dev && keep_obs_dev && points_dev && obs_cam_out_dev && obs_pt_out_dev &&
                    obs_uv_out_dev && point_start_out_dev && cam_obs_out_dev && cam_start_out_dev &&
                    points_out_dev && counts_out_dev && workspace_dev, "pgs_ba_compact: null pointer");
    const int M = problem->n_points, O = problem->n_obs;
    PGS_REQUIRE(workspace_bytes >= pgs_ba_compact_workspace(M, O), "pgs_ba_compact: workspace %zu < %zu",
                workspace_bytes, pgs_ba_compact_workspace(M, O));
    hipStream_t s = pgs::as_stream(stream);
    char* p = static_cast<char*>(workspace_dev);
    const size_t nb = ((size_t)(M > O ? M : O) + kFlagBlock - 1) / kFlagBlock + 1;
    uint32_t* pidx = reinterpret_cast<uint32_t*>(p);
    p += al(((size_t)M + 1) * 4);
    uint32_t* oidx = reinterpret_cast<uint32_t*>(p);
    p += al(((size_t)O + 1) * 4);
    uint32_t* qidx = reinterpret_cast<uint32_t*>(p);
    p += al(((size_t)O + 1) * 4);
    uint32_t* b0 = reinterpret_cast<uint32_t*>(p);
    p += al(nb * 4);
    uint32_t* b1 = reinterpret_cast<uint32_t*>(p);
    p += al(nb * 4);
    uint32_t* b2 = reinterpret_cast<uint32_t*>(p);
    flag_scan(keep_point_dev, nullptr, (uint32_t)M, pidx, b0, s);
    flag_scan(keep_obs_dev, nullptr, (uint32_t)O, oidx, b1, s);
    flag_scan(keep_obs_dev, problem->cam_obs_dev, (uint32_t)O, qidx, b2, s);
    k_compact_points<<<(M + 255) / 256, 256, 0, s>>>(M, keep_point_dev, pidx, oidx, problem->point_start_dev,
                                                     points_dev, points_out_dev, point_start_out_dev, O,
                                                     counts_out_dev);
    const int n = (O > problem->n_cams + 1 ? O : problem->n_cams + 1);
    k_compact_obs<<<(n + 255) / 256, 256, 0, s>>>(*problem, keep_obs_dev, oidx, pidx, qidx, obs_cam_out_dev,
                                                  obs_pt_out_dev, obs_uv_out_dev, cam_obs_out_dev,
                                                  cam_start_out_dev);
    PGS_CHECK_LAUNCH("pgs_ba_compact");
    return PGS_OK;
}
