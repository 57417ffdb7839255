// KNN local surface statistics and disc-like covariance seeding (PocketGS
// Sec. "Prior-Conditioned Gaussian Parameterization").
//
// pgs_knn: exact k nearest neighbours through a uniform grid.  The points'
// bounding box is cut into cubic cells (1 to 128 along its longest side, the
// count chosen from how a sample of the points shares cells, k_grid_choose);
// points are counted per cell, the counts scanned into cell starts and the
// points' coordinates and indices gathered in cell order.  One lane per query
// (queries in cell order, so a wave searches neighbouring cells) visits the
// cells within one cell of its own, then shells of growing Chebyshev distance
// r.  A row of cells along x is one run of points, so the first block is nine
// runs.  Every point of a cell r + 1 or more cells away is farther than
// r cell widths (plus the query's distance to its own cell's nearest face),
// so the search stops once the k-th distance is within that reach: no
// unvisited point can enter or tie.  Squared distances are
// ((dx*dx) + (dy*dy)) + (dz*dz) in float64 with contraction off, which fixes
// every rounding, so the neighbour sets and their order equal a brute-force
// search with ties broken by the smaller index, bit for bit, whatever order
// the cells are visited in.
//
// The search keeps its candidates as 64-bit keys, the float32 rounding of the
// distance above the point's position in cell order.  Such a key is ordered
// like the positive double it spells, so a sorted list takes a new key with
// one v_max_f64 and one v_min_f64 per slot and no index moves (the lists of
// (double, index) pairs that this replaces took about ten instructions per
// slot, and one lane's insertion holds up its wave).  The list holds two keys
// more than k; its entries' exact distances and indices are then formed again
// and sorted.  Rounding is monotone, so every point left out has an exact
// distance above the k-th whenever the k-th's rounding is below the list's
// last key.  Where it is not (many points at one distance), the points that
// round to the k-th's float32 are gone through again with keys of their exact
// distances (knn_ties).  On 300k points of a
// scene's surfaces with k = 16 the search went from 0.93 to 0.20 ms (41M vector
// instructions, 314 MB of writes scattered to the queries' own order) and the
// whole call from 1.06 to 0.27 ms; on 2000 points from 7.8 to 0.17 ms.
//
// pgs_pca_seed: per point, in float64: covariance of the 16 neighbours about
// their centroid, cyclic Jacobi eigen-decomposition of the 3x3 matrix,
// normal = eigenvector of the smallest eigenvalue, s_t = mean distance to
// the 3 nearest, s_n = r_normal s_t; rotation [t1 t2 n] with the tangent
// basis of Duff et al. (2017) and its quaternion by Shepperd's method.
#include <math.h>

#include "common.hpp"

namespace {

constexpr int kKnnThreads = 256;
constexpr int kMaxK = 32;

__device__ __forceinline__ double sqdist(double qx, double qy, double qz, double px, double py, double pz) {
#pragma clang fp contract(off)
    const double dx = px - qx, dy = py - qy, dz = pz - qz;
    return (dx * dx + dy * dy) + dz * dz;
}

// Grid of a KNN search: cubic cells of width h from the box corner lo,
// dims[3] cells per axis (at most kGridMax).
constexpr int kGridMax = 128;
constexpr int kBoxBlocks = 256;
constexpr uint32_t kGridCells = (uint32_t)kGridMax * kGridMax * kGridMax;

struct GridDesc {
    double lo[3];
    double h;
    int dims[3];
    uint32_t cells;  // dims[0] dims[1] dims[2]
};

__device__ __forceinline__ int cell_axis(double v, double lo, double h, int dim) {
    int c = (int)floor((v - lo) / h);
    return c < 0 ? 0 : (c >= dim ? dim - 1 : c);
}

// Per-block partial bounding boxes: part[b][0..2] minima, [3..5] maxima.
// Also clears the cell counts.
__global__ __launch_bounds__(256) void k_box_partial(const float* __restrict__ pts, int m, float* __restrict__ part,
                                                     uint32_t* __restrict__ counts) {
    __shared__ float red[6][256];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < kGridCells / 4; i += gridDim.x * 256)
        reinterpret_cast<uint4*>(counts)[i] = make_uint4(0u, 0u, 0u, 0u);
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x)
        for (int a = 0; a < 3; ++a) {
            const float v = pts[(size_t)a * m + i];
            mn[a] = fminf(mn[a], v);
            mx[a] = fmaxf(mx[a], v);
        }
    for (int a = 0; a < 3; ++a) {
        red[a][threadIdx.x] = mn[a];
        red[3 + a][threadIdx.x] = mx[a];
    }
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off)
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + off]);
                red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + off]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = red[threadIdx.x][0];
}

// A grid of `cells` cells along the longest side of the box [mn, mx].
__device__ __forceinline__ GridDesc make_grid(const float* mn, const float* mx, double cells) {
    GridDesc g;
    double ext = 0.0;
    for (int a = 0; a < 3; ++a) ext = fmax(ext, (double)mx[a] - (double)mn[a]);
    g.h = ext > 0.0 ? ext / cells : 1.0;
    for (int a = 0; a < 3; ++a) {
        g.lo[a] = mn[a];
        const int d = (int)floor(((double)mx[a] - (double)mn[a]) / g.h) + 1;
        g.dims[a] = d < 1 ? 1 : (d > kGridMax ? kGridMax : d);
    }
    g.cells = (uint32_t)g.dims[0] * g.dims[1] * g.dims[2];
    return g;
}

// The grid (one workgroup).  The search costs what the points of the 27
// cells around a query cost as long as k neighbours lie within one cell
// width, and far more when shells of empty cells have to be walked: with 128
// cells a side whatever the cloud, 2000 points took 9 ms where 300k took
// 0.9 ms.  So the cells are sized for `want` other points in the cell of a
// point, which on a surface puts about pi want within one cell width; the
// caller's max(4, 0.7 k) measured best or close to it for each k (surface
// clouds of 20k and 300k points, wanted shares 5 to 20).
// A sample of the points is dropped into grids of 64, 32, 16, 8 and 4 cells a
// side (each the halved coordinates of the one before); the pairs that share
// a cell, scaled from the sample to m points, are each grid's share, and the
// wanted share lies between two of them (or beyond the finest) with the
// dimension that the two show.  Only the cost of the search depends on the
// choice, never its result.  One point per thread and the three coarse grids
// in LDS: with four points and every grid counted by atomics in memory the
// kernel took 150 us of queueing on the coarse grids' few cells, 18 us now.
constexpr int kChooseThreads = 1024;
constexpr int kLevels = 5;              // 64 >> level cells a side
constexpr int kLdsCells = 17 * 17 * 17 + 9 * 9 * 9 + 5 * 5 * 5;

__global__ __launch_bounds__(kChooseThreads) void k_grid_choose(const float* __restrict__ pts, int m,
                                                                const float* __restrict__ part,
                                                                uint32_t* __restrict__ counts, float want,
                                                                GridDesc* __restrict__ desc) {
    __shared__ float box[6];
    __shared__ uint32_t pairs[kLevels];
    __shared__ uint32_t coarse[kLdsCells];
    const int t = threadIdx.x;
    const int s = min(m, kChooseThreads);
    float p[3] = {0.f, 0.f, 0.f};
    if (t < s) {
        const int i = (int)((long long)t * m / s);
        for (int a = 0; a < 3; ++a) p[a] = pts[(size_t)a * m + i];
    }
    if (t < 6 * 64) {  // one wave per box bound
        const int a = t >> 6, l = t & 63;
        float v = part[l * 6 + a];
        for (int b = l + 64; b < kBoxBlocks; b += 64) {
            const float u = part[b * 6 + a];
            v = a < 3 ? fminf(v, u) : fmaxf(v, u);
        }
        for (int o = 32; o > 0; o >>= 1) {
            const float u = __shfl_xor(v, o);
            v = a < 3 ? fminf(v, u) : fmaxf(v, u);
        }
        if (l == 0) box[a] = v;
    }
    if (t < kLevels) pairs[t] = 0u;
    for (int e = t; e < kLdsCells; e += kChooseThreads) coarse[e] = 0u;
    __syncthreads();
    uint32_t at[2] = {0u, 0u};
    if (t < s) {
        const GridDesc g = make_grid(box, box + 3, 64.0);
        int c[3], d[3];
        for (int a = 0; a < 3; ++a) {
            c[a] = cell_axis(p[a], g.lo[a], g.h, g.dims[a]);
            d[a] = g.dims[a];  // at most 65
        }
        uint32_t old[kLevels], base = 0;
        for (int l = 0; l < kLevels; ++l) {
            const uint32_t cell = base + ((uint32_t)c[2] * d[1] + c[1]) * d[0] + c[0];
            if (l < 2) {
                at[l] = cell;
                old[l] = atomicAdd(&counts[cell], 1u);
            } else {
                old[l] = atomicAdd(&coarse[cell], 1u);
            }
            base = l == 1 ? 0u : base + (uint32_t)d[0] * d[1] * d[2];
            for (int a = 0; a < 3; ++a) {
                c[a] >>= 1;
                d[a] = (d[a] + 1) >> 1;
            }
        }
        for (int l = 0; l < kLevels; ++l)
            if (old[l]) atomicAdd(&pairs[l], old[l]);
    }
    __syncthreads();  // every count has returned
    if (t < s) {
        counts[at[0]] = 0u;
        counts[at[1]] = 0u;
    }
    if (t == 0) {
        // mean number of other points in a point's cell, at m points
        float share[kLevels];
        const float up = 2.0f / (float)s * ((float)(m - 1) / (float)max(s - 1, 1));
        for (int l = 0; l < kLevels; ++l) share[l] = fmaxf((float)pairs[l] * up, 0.1f);
        // the finest grid that holds the wanted share, or the coarsest
        int l = 0;
        while (l + 1 < kLevels && share[l] < want) ++l;
        // share ~ side^-dimension between this grid and its finer (or, from
        // the finest, coarser) neighbour, the dimension kept between 1 and 3
        const int n = l > 0 ? l : 1;
        const float dim = fminf(3.0f, fmaxf(1.0f, log2f(share[n] / share[n - 1])));
        const float side = (float)(64 >> l) * exp2f(log2f(share[l] / want) / dim);
        *desc = make_grid(box, box + 3, (double)fminf((float)kGridMax, fmaxf(1.0f, floorf(side))));
    }
}

// Cell of every point and its rank among the cell's points.
__global__ __launch_bounds__(256) void k_cell_count(const float* __restrict__ pts, int m,
                                                    const GridDesc* __restrict__ desc, uint32_t* __restrict__ counts,
                                                    uint32_t* __restrict__ cell_of, uint32_t* __restrict__ rank_of) {
    const GridDesc g = *desc;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x) {
        const int cx = cell_axis(pts[i], g.lo[0], g.h, g.dims[0]);
        const int cy = cell_axis(pts[(size_t)m + i], g.lo[1], g.h, g.dims[1]);
        const int cz = cell_axis(pts[2 * (size_t)m + i], g.lo[2], g.h, g.dims[2]);
        const uint32_t c = ((uint32_t)cz * g.dims[1] + cy) * g.dims[0] + cx;
        cell_of[i] = c;
        rank_of[i] = atomicAdd(&counts[c], 1u);
    }
}

// Exclusive scan of the cell counts into starts, starts[cells] = m (one chunk
// of 4096 per workgroup, chunks past the last cell empty; the chunk totals
// are added up by each workgroup itself).
constexpr int kCellScanItems = 4096;

__device__ __forceinline__ uint32_t block_sum_256(uint32_t v, uint32_t* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void k_cell_total(const uint32_t* __restrict__ counts,
                                                    const GridDesc* __restrict__ desc,
                                                    uint32_t* __restrict__ totals) {
    __shared__ uint32_t red[4];
    const uint32_t n = desc->cells;
    if (blockIdx.x * kCellScanItems >= n) return;
    // counts past the last cell are zero, and the array holds whole chunks
    const uint4* c = reinterpret_cast<const uint4*>(counts + (size_t)blockIdx.x * kCellScanItems);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kCellScanItems / 1024; ++k) {
        const uint4 v = c[k * 256 + threadIdx.x];
        s += v.x + v.y + v.z + v.w;
    }
    s = block_sum_256(s, red);
    if (threadIdx.x == 0) totals[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_cell_starts(const uint32_t* __restrict__ counts, int m,
                                                     const GridDesc* __restrict__ desc,
                                                     const uint32_t* __restrict__ totals,
                                                     uint32_t* __restrict__ starts) {
    __shared__ uint32_t red[4], wsum[4];
    const uint32_t n = desc->cells, base = blockIdx.x * kCellScanItems;
    if (base >= n) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t run = 0;
    for (uint32_t k = t; k < blockIdx.x; k += 256) run += totals[k];
    run = block_sum_256(run, red);
    // four cells per thread and round
    for (int k = 0; k < kCellScanItems / 1024; ++k) {
        const uint32_t at = base + k * 1024 + t * 4;
        const uint4 v = *reinterpret_cast<const uint4*>(counts + at);
        const uint32_t own = v.x + v.y + v.z + v.w;
        uint32_t inc = own;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(inc, o);
            if (lane >= o) inc += u;
        }
        if (lane == 63) wsum[wv] = inc;
        __syncthreads();
        uint32_t before = run;
        for (int w = 0; w < 4; ++w) {
            if (w < wv) before += wsum[w];
            run += wsum[w];
        }
        const uint32_t e = before + inc - own;
        *reinterpret_cast<uint4*>(starts + at) = make_uint4(e, e + v.x, e + v.x + v.y, e + v.x + v.y + v.z);
        __syncthreads();
    }
    // a chunk that ends on the last cell leaves its end to be written
    if (t == 0 && base + kCellScanItems >= n) starts[n] = (uint32_t)m;
}

// Points in cell order (order inside a cell is arbitrary: the search's
// tie rule does not depend on it).
__global__ __launch_bounds__(256) void k_cell_scatter(const float* __restrict__ pts, int m,
                                                      const uint32_t* __restrict__ cell_of,
                                                      const uint32_t* __restrict__ rank_of,
                                                      const uint32_t* __restrict__ starts,
                                                      float4* __restrict__ sorted) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x)
        sorted[starts[cell_of[i]] + rank_of[i]] =
            make_float4(pts[i], pts[(size_t)m + i], pts[2 * (size_t)m + i], __int_as_float(i));
}

template <int K>
__device__ __forceinline__ void knn_insert(double d, int idx, double (&bd)[K], int (&bi)[K]) {
    // (d, idx) enters when it precedes the last entry in (distance, index)
    // order; entries it precedes shift down one slot
    if (!(d < bd[K - 1] || (d == bd[K - 1] && idx < bi[K - 1]))) return;
    bool placed = false;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        if (!placed) {
            if (k > 0 && (bd[k - 1] > d || (bd[k - 1] == d && bi[k - 1] > idx))) {
                bd[k] = bd[k - 1];
                bi[k] = bi[k - 1];
            } else {
                bd[k] = d;
                bi[k] = idx;
                placed = true;
            }
        }
    }
}

// Search of one query with exact comparisons throughout (the general path:
// distances outside float32's normal numbers, coordinates that are not finite).
template <int K>
__device__ __noinline__ void knn_exact(const float4* __restrict__ sorted, int m, const GridDesc& g,
                                       const uint32_t* __restrict__ starts, float4 qp, int* __restrict__ nbr,
                                       double* __restrict__ d2out) {
    const int q = __float_as_int(qp.w);
    const double qx = qp.x, qy = qp.y, qz = qp.z;
    const int cx = cell_axis(qx, g.lo[0], g.h, g.dims[0]);
    const int cy = cell_axis(qy, g.lo[1], g.h, g.dims[1]);
    const int cz = cell_axis(qz, g.lo[2], g.h, g.dims[2]);
    double bd[K];
    int bi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        bd[k] = INFINITY;
        bi[k] = 0x7fffffff;
    }
    const int rmax = max(g.dims[0], max(g.dims[1], g.dims[2]));
    for (int r = 0; r <= rmax; ++r) {
        for (int dz = -r; dz <= r; ++dz) {
            const int z = cz + dz;
            if (z < 0 || z >= g.dims[2]) continue;
            for (int dy = -r; dy <= r; ++dy) {
                const int y = cy + dy;
                if (y < 0 || y >= g.dims[1]) continue;
                const bool face = dz == -r || dz == r || dy == -r || dy == r;
                // on the shell: every x of a face row, else only x = -r and x = +r
                for (int dx = -r; dx <= r; dx += (face || r == 0) ? 1 : 2 * r) {
                    const int x = cx + dx;
                    if (x < 0 || x >= g.dims[0]) continue;
                    const uint32_t c = ((uint32_t)z * g.dims[1] + y) * g.dims[0] + x;
                    const uint32_t e = starts[c + 1];
                    for (uint32_t t = starts[c]; t < e; ++t) {
                        const float4 p = sorted[t];
                        const int idx = __float_as_int(p.w);
                        if (idx == q) continue;
                        knn_insert<K>(sqdist(qx, qy, qz, p.x, p.y, p.z), idx, bd, bi);
                    }
                }
            }
        }
        // cells r + 1 or more away hold only points farther than r h
        const double reach = (double)r * g.h;
        if (bi[K - 1] != 0x7fffffff && bd[K - 1] <= reach * reach * (1.0 - 1e-12)) break;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        nbr[(size_t)k * m + q] = bi[k];
        d2out[(size_t)k * m + q] = bd[k];
    }
}

// Key of a candidate: the float32 rounding of its squared distance above its
// position, as a double.  The patterns up to float32's infinity spell positive
// finite doubles, ordered like the pairs (rounded distance, position); those
// of NaN (sign cleared) lie above them or spell NaN and are never taken.
constexpr uint32_t kInfBits = 0x7f800000u;
__device__ __forceinline__ double knn_key(uint32_t hi, uint32_t lo) { return __hiloint2double((int)hi, (int)lo); }

// The smaller and the larger of two keys, one instruction each (the compiler's
// fmin and fmax first quiet each operand, which doubles the list's cost).
__device__ __forceinline__ double key_min(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double key_max(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Takes key x into the sorted list a, dropping its last.
template <int N>
__device__ __forceinline__ void key_insert(double (&a)[N], double x) {
#pragma unroll
    for (int k = N - 1; k > 0; --k) a[k] = key_min(a[k], key_max(a[k - 1], x));
    a[0] = key_min(a[0], x);
}

// Entries from..K-1 of a query: the nearest points whose distance rounds to the
// float32 r (a normal number, or zero), sorted by keys of (exact distance,
// index).  The doubles that round to one float32 follow one another, 2^29 or so
// of them, so a distance's place among them takes the upper half of a key.  The
// points lie in the cells between the query's coordinates less and plus the root
// of r (a cell number does not fall as a coordinate grows).  False where a
// distance rounds to zero without being zero.  Searched from nothing with exact
// comparisons, a lattice of 300k points took 993 us and 10k points 30 times each
// 366, more than before there were lists (856 and 240); 455 and 190 now.
template <int K>
__device__ __forceinline__ bool knn_ties(const float4* __restrict__ sorted, int m, const GridDesc& g,
                                         const uint32_t* __restrict__ starts, const float4& qp, float r, int from,
                                         int* __restrict__ nbr, double* __restrict__ d2out) {
    const double c[3] = {qp.x, qp.y, qp.z};
    const double rad = sqrt((double)r * (1.0 + 1e-6) + 0x1p-149);  // what rounds to r is nearer
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double w = rad + fabs(c[a]) * 1e-15;  // the sums' rounding
        lo[a] = cell_axis(c[a] - w, g.lo[a], g.h, g.dims[a]);
        hi[a] = cell_axis(c[a] + w, g.lo[a], g.h, g.dims[a]);
    }
    // the least double that rounds to r, or the one that ties below it
    const double least =
        r > 0.0f ? 0.5 * ((double)r + (double)__uint_as_float(__float_as_uint(r) - 1u)) : 0.0;
    const long long first = __double_as_longlong(least);
    bool exact = true;
    double b[K];
#pragma unroll
    for (int k = 0; k < K; ++k) b[k] = knn_key(kInfBits, 0xffffffffu);
    for (int z = lo[2]; z <= hi[2]; ++z)
        for (int y = lo[1]; y <= hi[1]; ++y) {
            const uint32_t row = ((uint32_t)z * g.dims[1] + y) * g.dims[0];
            const uint32_t e = starts[row + hi[0] + 1];
            for (uint32_t t0 = starts[row + lo[0]]; t0 < e; t0 += 4) {
                float4 p[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) p[u] = sorted[min(t0 + u, e - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double d = sqdist(c[0], c[1], c[2], p[u].x, p[u].y, p[u].z);
                    if ((float)d == r && t0 + u < e && __float_as_int(p[u].w) != __float_as_int(qp.w)) {
                        const uint32_t place = (uint32_t)(__double_as_longlong(d) - first);
                        exact = exact && (r > 0.0f || d == 0.0);
                        const double x = knn_key(place, __float_as_uint(p[u].w));
                        if (x < b[K - 1]) key_insert<K>(b, x);
                    }
                }
            }
        }
    const int q = __float_as_int(qp.w);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (from + k < K) {
            nbr[(size_t)(from + k) * m + q] = __double2loint(b[k]);
            d2out[(size_t)(from + k) * m + q] = __longlong_as_double(first + (long long)(uint32_t)__double2hiint(b[k]));
        }
    return exact;
}

// About 15 vector instructions per candidate and, whenever one of the wave's
// lanes takes it, two per slot of the list, most of them float64: at 300k points
// a third of the waves' time waits for an issue slot, 43% for the candidates'
// loads (three waves a SIMD, what the list's registers leave).
template <int K>
__global__ __launch_bounds__(kKnnThreads) void k_knn_grid(const float4* __restrict__ sorted, int m,
                                                          const GridDesc* __restrict__ desc,
                                                          const uint32_t* __restrict__ starts,
                                                          int* __restrict__ nbr, double* __restrict__ d2out) {
    constexpr int KE = K + 2;
    const GridDesc& g = *desc;
    const int j = blockIdx.x * kKnnThreads + threadIdx.x;
    if (j >= m) return;
    const float4 qp = sorted[j];
    const double qx = qp.x, qy = qp.y, qz = qp.z;
    const int nx = g.dims[0], ny = g.dims[1], nz = g.dims[2];
    const double h = g.h;
    const int cx = cell_axis(qx, g.lo[0], h, nx);
    const int cy = cell_axis(qy, g.lo[1], h, ny);
    const int cz = cell_axis(qz, g.lo[2], h, nz);
    // distance from the query to its own cell's nearest face, in cells, less
    // a margin for the rounding of the cell decisions
    auto face_gap = [&](double v, double lo, int c) {
        const double f = (v - lo) / h - c;
        return fmin(f, 1.0 - f);
    };
    double gap = fmin(face_gap(qx, g.lo[0], cx), fmin(face_gap(qy, g.lo[1], cy), face_gap(qz, g.lo[2], cz)));
    gap = fmax(gap, 0.0) - 1e-9;
    double a[KE];
#pragma unroll
    for (int k = 0; k < KE; ++k) a[k] = knn_key(kInfBits, 0xffffffffu);
    auto take = [&](uint32_t s, uint32_t e) {
        for (uint32_t t0 = s; t0 < e; t0 += 4) {
            float4 p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = sorted[min(t0 + u, e - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t t = t0 + u;
                const float d = (float)sqdist(qx, qy, qz, p[u].x, p[u].y, p[u].z);
                const double x = knn_key(__float_as_uint(d) & 0x7fffffffu, t);
                if (t < e && t != (uint32_t)j && x < a[KE - 1]) key_insert<KE>(a, x);
            }
        }
    };
    auto run_of = [&](int y, int z, int x0, int x1) {
        if (y < 0 || y >= ny || z < 0 || z >= nz) return;
        x0 = max(x0, 0);
        x1 = min(x1, nx - 1);
        if (x0 > x1) return;
        const uint32_t c = ((uint32_t)z * ny + y) * nx;
        take(starts[c + x0], starts[c + x1 + 1]);
    };
    // whether no point farther than `reach` can enter or tie: the k-th distance
    // is at most its rounded key's value and a unit of rounding more (relative,
    // or among the subnormal numbers their spacing)
    auto within = [&](double reach) {
        const uint32_t kth = (uint32_t)__double2hiint(a[K - 1]);
        const double most = (double)__uint_as_float(kth) * (1.0 + 1e-6) + 0x1p-149;
        return kth < kInfBits && most <= reach * reach * (1.0 - 1e-12);
    };
    // the 3 x 3 x 3 block, the query's own row first (enough where a point is
    // repeated more than K times)
    run_of(cy, cz, cx - 1, cx + 1);
    const bool at_once = gap > 0.0 && within(gap * h);
    for (int i = at_once ? 9 : 0; i < 9; ++i)
        if (i != 4) run_of(cy + i % 3 - 1, cz + i / 3 - 1, cx - 1, cx + 1);
    const int rmax = at_once ? 0 : max(nx, max(ny, nz));
    for (int r = 2; r <= rmax; ++r) {
        // visited: every cell within r - 1
        if (within(((double)(r - 1) + gap) * h)) break;
        for (int dz = -r; dz <= r; ++dz)
            for (int dy = -r; dy <= r; ++dy) {
                if (dz == -r || dz == r || dy == -r || dy == r) {
                    run_of(cy + dy, cz + dz, cx - r, cx + r);
                } else {
                    run_of(cy + dy, cz + dz, cx - r, cx - r);
                    run_of(cy + dy, cz + dz, cx + r, cx + r);
                }
            }
    }
    // exact distances and indices of the list, sorted (they are in the order
    // of their roundings already, so usually nothing moves)
    double bd[KE];
    int bi[KE];
#pragma unroll
    for (int k = 0; k < KE; ++k) {
        const uint32_t t = (uint32_t)__double2loint(a[k]);
        const bool has = t != 0xffffffffu;
        const float4 p = sorted[has ? t : (uint32_t)j];
        bd[k] = has ? sqdist(qx, qy, qz, p.x, p.y, p.z) : INFINITY;
        bi[k] = has ? __float_as_int(p.w) : 0x7fffffff;
    }
    for (bool moved = true; moved;) {
        moved = false;
#pragma unroll
        for (int k = 0; k + 1 < KE; ++k) {
            const bool sw = bd[k + 1] < bd[k] || (bd[k + 1] == bd[k] && bi[k + 1] < bi[k]);
            const double d0 = bd[k], d1 = bd[k + 1];
            const int i0 = bi[k], i1 = bi[k + 1];
            bd[k] = sw ? d1 : d0;
            bd[k + 1] = sw ? d0 : d1;
            bi[k] = sw ? i1 : i0;
            bi[k + 1] = sw ? i0 : i1;
            moved |= sw;
        }
    }
    // every point left out rounds to the last key's distance or more
    const float r = (float)bd[K - 1];
    const bool sure = __float_as_uint(r) < (uint32_t)__double2hiint(a[KE - 1]);
    const int q = __float_as_int(qp.w);
    int below = 0;  // entries that round to less than the k-th
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (sure || (float)bd[k] < r) {
            nbr[(size_t)k * m + q] = bi[k];
            d2out[(size_t)k * m + q] = bd[k];
            below = k + 1;
        }
    }
    if (sure) return;
    if (!(__float_as_uint(r) < kInfBits && (r == 0.0f || r >= 0x1p-126f)) ||
        !knn_ties<K>(sorted, m, g, starts, qp, r, below, nbr, d2out))
        knn_exact<K>(sorted, m, g, starts, qp, nbr, d2out);
}

// Workspace of pgs_knn for m points.
struct KnnWs {
    float* part;
    GridDesc* desc;
    uint32_t* counts;
    uint32_t* starts;
    uint32_t* totals;
    uint32_t* cell_of;
    uint32_t* rank_of;
    float4* sorted;
    size_t bytes;
};

KnnWs knn_layout(void* base, int m) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    KnnWs w{};
    char* p = static_cast<char*>(base);
    size_t off = 0;
    w.part = reinterpret_cast<float*>(p + off); off += up((size_t)kBoxBlocks * 6 * 4);
    w.desc = reinterpret_cast<GridDesc*>(p + off); off += up(sizeof(GridDesc));
    w.counts = reinterpret_cast<uint32_t*>(p + off); off += up((size_t)kGridCells * 4);
    w.starts = reinterpret_cast<uint32_t*>(p + off); off += up(((size_t)kGridCells + 1) * 4);
    w.totals = reinterpret_cast<uint32_t*>(p + off); off += up((size_t)(kGridCells / kCellScanItems + 1) * 4);
    w.cell_of = reinterpret_cast<uint32_t*>(p + off); off += up((size_t)m * 4);
    w.rank_of = reinterpret_cast<uint32_t*>(p + off); off += up((size_t)m * 4);
    w.sorted = reinterpret_cast<float4*>(p + off); off += up((size_t)m * 16);
    w.bytes = off;
    return w;
}

// One Jacobi rotation that zeroes the off-diagonal entry apq of a symmetric 3x3
// matrix with diagonal app, aqq and the third row's entries akp, akq; vp, vq are
// the vectors' columns.
__device__ __forceinline__ void jacobi_rotate(double& app, double& aqq, double& apq, double& akp, double& akq,
                                              double (&vp)[3], double (&vq)[3]) {
    if (apq == 0.0) return;
    const double d = aqq - app;
    // tan of the angle: sign(d) 2 apq / (|d| + sqrt(d^2 + 4 apq^2))
    const double den = fabs(d) + sqrt(d * d + 4.0 * apq * apq);
    const double t = d == 0.0 ? 1.0 : (d > 0.0 ? 2.0 : -2.0) * apq / den;
    const double c = rsqrt(t * t + 1.0), s = t * c;
    app -= t * apq;
    aqq += t * apq;
    apq = 0.0;
    const double kp = akp, kq = akq;
    akp = c * kp - s * kq;
    akq = s * kp + c * kq;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a = vp[k], b = vq[k];
        vp[k] = c * a - s * b;
        vq[k] = s * a + c * b;
    }
}

// Eigen-decomposition of a symmetric 3x3 matrix (xx, xy, xz, yy, yz, zz) by
// cyclic Jacobi rotations: w[c] the eigenvalue of vector V[c].  A rotation
// updates only what it changes, with one division and no indexed arrays; the
// matrix products in full took the plain seed of 300k points 80 us, now 76, and
// the features of 200k 91, now 86 (both wait for the neighbours' gathers).
__device__ __forceinline__ void jacobi3(const double (&A)[6], double (&w)[3], double (&V)[3][3]) {
    double xx = A[0], xy = A[1], xz = A[2], yy = A[3], yz = A[4], zz = A[5];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) V[r][c] = r == c ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 30; ++sweep) {
        const double off = fabs(xy) + fabs(xz) + fabs(yz);
        const double scale = fabs(xx) + fabs(yy) + fabs(zz);
        if (off <= 1e-300 || off <= 1e-18 * scale) break;
        jacobi_rotate(xx, yy, xy, xz, yz, V[0], V[1]);
        jacobi_rotate(xx, zz, xz, xy, yz, V[0], V[2]);
        jacobi_rotate(yy, zz, yz, xy, xz, V[1], V[2]);
    }
    w[0] = xx;
    w[1] = yy;
    w[2] = zz;
}

// Unit vector along v.
__device__ __forceinline__ void unit(const double (&v)[3], double (&u)[3]) {
    const double inv = 1.0 / sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] = v[a] * inv;
}

constexpr int kKn = 16;

// The 16 neighbours of point i in float64 and their covariance about the
// neighbourhood centroid (PocketGS, equation for C_i).
__device__ __forceinline__ void neighbourhood(const float* __restrict__ pts, int m, const int* __restrict__ nbr, int i,
                              double (&P)[kKn][3], double (&A)[6]) {
    double cen[3] = {0, 0, 0};
    for (int j = 0; j < kKn; ++j) {
        const int id = nbr[(size_t)j * m + i];
        for (int a = 0; a < 3; ++a) {
            P[j][a] = pts[(size_t)a * m + id];
            cen[a] += P[j][a];
        }
    }
    for (int a = 0; a < 3; ++a) cen[a] /= kKn;
    for (int a = 0; a < 6; ++a) A[a] = 0.0;
    for (int j = 0; j < kKn; ++j) {
        const double x = P[j][0] - cen[0], y = P[j][1] - cen[1], z = P[j][2] - cen[2];
        A[0] += x * x;
        A[1] += x * y;
        A[2] += x * z;
        A[3] += y * y;
        A[4] += y * z;
        A[5] += z * z;
    }
    for (int a = 0; a < 6; ++a) A[a] /= kKn;
}

// Unit quaternion (w, x, y, z) of a rotation matrix, Shepperd's method: the
// branch follows the largest of the trace and the three diagonal entries.
__device__ void quat_of_rot(const double R[3][3], double q[4]) {
    const double tr = R[0][0] + R[1][1] + R[2][2];
    if (tr >= R[0][0] && tr >= R[1][1] && tr >= R[2][2]) {
        q[0] = 0.5 * sqrt(1.0 + tr);
        const double inv = 0.25 / q[0];
        q[1] = (R[2][1] - R[1][2]) * inv;
        q[2] = (R[0][2] - R[2][0]) * inv;
        q[3] = (R[1][0] - R[0][1]) * inv;
    } else if (R[0][0] >= R[1][1] && R[0][0] >= R[2][2]) {
        q[1] = 0.5 * sqrt(1.0 + R[0][0] - R[1][1] - R[2][2]);
        const double inv = 0.25 / q[1];
        q[0] = (R[2][1] - R[1][2]) * inv;
        q[2] = (R[0][1] + R[1][0]) * inv;
        q[3] = (R[0][2] + R[2][0]) * inv;
    } else if (R[1][1] >= R[2][2]) {
        q[2] = 0.5 * sqrt(1.0 - R[0][0] + R[1][1] - R[2][2]);
        const double inv = 0.25 / q[2];
        q[0] = (R[0][2] - R[2][0]) * inv;
        q[1] = (R[0][1] + R[1][0]) * inv;
        q[3] = (R[1][2] + R[2][1]) * inv;
    } else {
        q[3] = 0.5 * sqrt(1.0 - R[0][0] - R[1][1] + R[2][2]);
        const double inv = 0.25 / q[3];
        q[0] = (R[1][0] - R[0][1]) * inv;
        q[1] = (R[0][2] + R[2][0]) * inv;
        q[2] = (R[1][2] + R[2][1]) * inv;
    }
}

__device__ void rot_of_quat(const double qin[4], double R[3][3]) {
    const double n = sqrt(qin[0] * qin[0] + qin[1] * qin[1] + qin[2] * qin[2] + qin[3] * qin[3]);
    const double w = qin[0] / n, x = qin[1] / n, y = qin[2] / n, z = qin[3] / n;
    R[0][0] = 1 - 2 * (y * y + z * z); R[0][1] = 2 * (x * y - w * z); R[0][2] = 2 * (x * z + w * y);
    R[1][0] = 2 * (x * y + w * z); R[1][1] = 1 - 2 * (x * x + z * z); R[1][2] = 2 * (y * z - w * x);
    R[2][0] = 2 * (x * z - w * y); R[2][1] = 2 * (y * z + w * x); R[2][2] = 1 - 2 * (x * x + y * y);
}

__global__ __launch_bounds__(256) void k_pca_seed(const float* __restrict__ pts, const float* __restrict__ col,
                                                  int m, const int* __restrict__ nbr,
                                                  const double* __restrict__ d2, int k, double r_normal,
                                                  float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    constexpr int KS = 3;
    double P[kKn][3], A[6], ev[3], V[3][3], nrm[3];
    neighbourhood(pts, m, nbr, i, P, A);
    jacobi3(A, ev, V);
    // the vector of the smallest eigenvalue, the first of equal ones
    const bool second = ev[1] < ev[0], third = ev[2] < (second ? ev[1] : ev[0]);
    for (int c = 0; c < 3; ++c) nrm[c] = third ? V[2][c] : (second ? V[1][c] : V[0][c]);
    unit(nrm, nrm);
    const double nx = nrm[0], ny = nrm[1], nz = nrm[2];
    double st = 0.0;
    for (int j = 0; j < KS; ++j) st += sqrt(d2[(size_t)j * m + i]);
    st /= KS;
    const double sn = r_normal * st;
    // right-handed tangent frame (t1, t2, n), Duff et al. 2017
    const double sg = nz >= 0.0 ? 1.0 : -1.0;
    const double a = -1.0 / (sg + nz), b = nx * ny * a;
    const double t1[3] = {1.0 + sg * nx * nx * a, sg * b, -sg * nx};
    const double t2[3] = {b, sg + ny * ny * a, -ny};
    const double R[3][3] = {{t1[0], t2[0], nx}, {t1[1], t2[1], ny}, {t1[2], t2[2], nz}};
    double q[4];
    quat_of_rot(R, q);
    const double y00 = 0.28209479177387814;  // 1/(2 sqrt(pi))
    float vals[14];
    for (int a2 = 0; a2 < 3; ++a2) vals[a2] = pts[(size_t)a2 * m + i];
    vals[3] = (float)log(st);
    vals[4] = (float)log(st);
    vals[5] = (float)log(sn);
    for (int c = 0; c < 4; ++c) vals[6 + c] = (float)q[c];
    vals[10] = (float)log(0.1 / 0.9);
    for (int c = 0; c < 3; ++c) vals[11 + c] = (float)(((double)col[(size_t)c * m + i] - 0.5) / y00);
    for (int r = 0; r < 14; ++r) out[(size_t)r * m + i] = vals[r];
}

// Features of the seeding network for point i.  Frame R = [e1 e2 e3]:
// eigenvectors of C_i for the largest and middle eigenvalue, each signed so
// that the third moment of the offsets p_k - p_i along it is >= 0, and
// e3 = e1 x e2.  x = offsets in the frame / s_t (16 x 3), R^T C_i R / s_t^2
// (3 x 3), seven zeros.  base = R (row-major), plain-seed log-scales,
// quaternion of R.
__global__ __launch_bounds__(256) void k_mlp_features(const float* __restrict__ pts, int m,
                                                      const int* __restrict__ nbr,
                                                      const double* __restrict__ d2, double r_normal,
                                                      float* __restrict__ x, float* __restrict__ base) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    double P[kKn][3], A[6], ev[3], V[3][3];
    neighbourhood(pts, m, nbr, i, P, A);
    jacobi3(A, ev, V);
    // vectors by eigenvalue, largest first, equal ones in place
    const auto order = [&](int a, int b) {
        const bool swap = ev[b] > ev[a];
        const double e = ev[a];
        ev[a] = swap ? ev[b] : e;
        ev[b] = swap ? e : ev[b];
        for (int c = 0; c < 3; ++c) {
            const double v = V[a][c];
            V[a][c] = swap ? V[b][c] : v;
            V[b][c] = swap ? v : V[b][c];
        }
    };
    order(0, 1);
    order(1, 2);
    order(0, 1);
    const double C[3][3] = {{A[0], A[1], A[2]}, {A[1], A[3], A[4]}, {A[2], A[4], A[5]}};
    const double p[3] = {pts[i], pts[(size_t)m + i], pts[2 * (size_t)m + i]};
    for (int j = 0; j < kKn; ++j)
        for (int a = 0; a < 3; ++a) P[j][a] -= p[a];   // offsets from the point
    double e[3][3];
    for (int c = 0; c < 2; ++c) {
        double v[3];
        unit(V[c], v);
        double m3 = 0.0;
        for (int j = 0; j < kKn; ++j) {
            const double d = P[j][0] * v[0] + P[j][1] * v[1] + P[j][2] * v[2];
            m3 += d * d * d;
        }
        const double sg = m3 < 0.0 ? -1.0 : 1.0;
        for (int a = 0; a < 3; ++a) e[c][a] = sg * v[a];
    }
    e[2][0] = e[0][1] * e[1][2] - e[0][2] * e[1][1];
    e[2][1] = e[0][2] * e[1][0] - e[0][0] * e[1][2];
    e[2][2] = e[0][0] * e[1][1] - e[0][1] * e[1][0];
    double st = 0.0;
    for (int j = 0; j < 3; ++j) st += sqrt(d2[(size_t)j * m + i]);
    st /= 3.0;
    const double inv_st = 1.0 / st, inv_st2 = inv_st * inv_st;
    float* xr = x + (size_t)i * 64;
    for (int j = 0; j < kKn; ++j)
        for (int c = 0; c < 3; ++c)
            xr[3 * j + c] = (float)((P[j][0] * e[c][0] + P[j][1] * e[c][1] + P[j][2] * e[c][2]) * inv_st);
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            double v = 0.0;
            for (int u = 0; u < 3; ++u)
                for (int w = 0; w < 3; ++w) v += e[a][u] * C[u][w] * e[b][w];
            xr[48 + 3 * a + b] = (float)(v * inv_st2);
        }
    for (int k = 57; k < 64; ++k) xr[k] = 0.f;
    double R[3][3];
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) R[a][c] = e[c][a];
    double q[4];
    quat_of_rot(R, q);
    float* br = base + (size_t)i * 16;
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) br[3 * a + c] = (float)R[a][c];
    br[9] = (float)log(st);
    br[10] = (float)log(st);
    br[11] = (float)log(r_normal * st);
    for (int c = 0; c < 4; ++c) br[12 + c] = (float)q[c];
}

// Training target of Gaussian i: log S = R diag(2 s) R^T (6 entries), logit.
__global__ __launch_bounds__(256) void k_seed_targets(const float* __restrict__ params, int n,
                                                      float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double q[4], R[3][3], s2[3];
    for (int c = 0; c < 4; ++c) q[c] = params[(size_t)(6 + c) * n + i];
    for (int c = 0; c < 3; ++c) s2[c] = 2.0 * (double)params[(size_t)(3 + c) * n + i];
    rot_of_quat(q, R);
    auto M = [&](int a, int b) { return R[a][0] * s2[0] * R[b][0] + R[a][1] * s2[1] * R[b][1] + R[a][2] * s2[2] * R[b][2]; };
    float* o = out + (size_t)i * 8;
    o[0] = (float)M(0, 0);
    o[1] = (float)M(1, 1);
    o[2] = (float)M(2, 2);
    o[3] = (float)M(0, 1);
    o[4] = (float)M(0, 2);
    o[5] = (float)M(1, 2);
    o[6] = params[(size_t)10 * n + i];
    o[7] = 0.f;
}

// Seed from network outputs y with the fall back to the plain seed (pca
// columns): y not finite, |q_out| < 1e-6, a |d log-scale| > 2, or the axis
// of the smallest predicted scale more than 60 degrees from the plain
// normal (e3).  `pca` and `out` may be the same buffer.
__global__ __launch_bounds__(256) void k_seed_apply(const float* __restrict__ y, const float* __restrict__ base,
                                                    const float* pca, int m, float* out,
                                                    uint8_t* __restrict__ flags, uint32_t* __restrict__ count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool fb = false;
    if (i < m) {
        float vals[14];
        for (int r = 0; r < 14; ++r) vals[r] = pca[(size_t)r * m + i];
        double Y[8];
        for (int k = 0; k < 8; ++k) {
            const float v = y[(size_t)i * 8 + k];
            fb = fb || !isfinite(v);
            Y[k] = v;
        }
        const double qn = fb ? 0.0 : sqrt(Y[3] * Y[3] + Y[4] * Y[4] + Y[5] * Y[5] + Y[6] * Y[6]);
        fb = fb || qn < 1e-6;
        if (!fb) {
            double dl = 0.0;
            for (int k = 0; k < 3; ++k) dl = fmax(dl, fabs(Y[k]));
            double Ro[3][3], s[3];
            const double qo[4] = {Y[3] / qn, Y[4] / qn, Y[5] / qn, Y[6] / qn};
            rot_of_quat(qo, Ro);
            for (int k = 0; k < 3; ++k) s[k] = (double)base[(size_t)i * 16 + 9 + k] + Y[k];
            int kmin = 0;
            if (s[1] < s[kmin]) kmin = 1;
            if (s[2] < s[kmin]) kmin = 2;
            // (Rb Ro e_kmin) . (Rb e3) = (Ro e_kmin) . e3 = Ro[2][kmin]
            const double c = fabs(Ro[2][kmin]);
            fb = dl > 2.0 || c < 0.5;
            if (!fb) {
                double qb[4];
                for (int k = 0; k < 4; ++k) qb[k] = base[(size_t)i * 16 + 12 + k];
                const double w = qb[0] * qo[0] - qb[1] * qo[1] - qb[2] * qo[2] - qb[3] * qo[3];
                const double qx = qb[0] * qo[1] + qo[0] * qb[1] + qb[2] * qo[3] - qb[3] * qo[2];
                const double qy = qb[0] * qo[2] + qo[0] * qb[2] + qb[3] * qo[1] - qb[1] * qo[3];
                const double qz = qb[0] * qo[3] + qo[0] * qb[3] + qb[1] * qo[2] - qb[2] * qo[1];
                for (int k = 0; k < 3; ++k) vals[3 + k] = (float)s[k];
                vals[6] = (float)w;
                vals[7] = (float)qx;
                vals[8] = (float)qy;
                vals[9] = (float)qz;
                vals[10] = (float)(log(1.0 / 9.0) + Y[7]);
            }
        }
        for (int r = 0; r < 14; ++r) out[(size_t)r * m + i] = vals[r];
        if (flags) flags[i] = fb ? 1 : 0;
    }
    const unsigned long long b = __ballot(fb);
    if (count && (threadIdx.x & 63) == 0 && b) atomicAdd(count, (uint32_t)__popcll(b));
}

}  // namespace

extern "C" size_t pgs_knn_workspace(int32_t m) { return knn_layout(nullptr, m > 0 ? m : 0).bytes; }

extern "C" pgs_status pgs_knn(const float* points_dev, int32_t m, int32_t k, int32_t* nbr_dev,
                              double* d2_dev, void* workspace_dev, size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(k == 4 || k == 8 || k == 16 || k == kMaxK, "pgs_knn: k must be 4, 8, 16 or 32 (k=%d)", k);
    PGS_REQUIRE(m > k, "pgs_knn: need m > k (k=%d m=%d)", k, m);
    PGS_REQUIRE(points_dev && nbr_dev && d2_dev && workspace_dev, "pgs_knn: null pointer");
    const KnnWs w = knn_layout(workspace_dev, m);
    PGS_REQUIRE(workspace_bytes >= w.bytes, "pgs_knn: workspace %zu < %zu", workspace_bytes, w.bytes);
    hipStream_t s = pgs::as_stream(stream);
    const int gm = (m + 255) / 256 < 4096 ? (m + 255) / 256 : 4096;
    k_box_partial<<<kBoxBlocks, 256, 0, s>>>(points_dev, m, w.part, w.counts);
    k_grid_choose<<<1, kChooseThreads, 0, s>>>(points_dev, m, w.part, w.counts, fmaxf(4.0f, 0.7f * (float)k), w.desc);
    k_cell_count<<<gm, 256, 0, s>>>(points_dev, m, w.desc, w.counts, w.cell_of, w.rank_of);
    const uint32_t chunks = kGridCells / kCellScanItems;
    k_cell_total<<<chunks, 256, 0, s>>>(w.counts, w.desc, w.totals);
    k_cell_starts<<<chunks, 256, 0, s>>>(w.counts, m, w.desc, w.totals, w.starts);
    k_cell_scatter<<<gm, 256, 0, s>>>(points_dev, m, w.cell_of, w.rank_of, w.starts, w.sorted);
    const dim3 grid((m + kKnnThreads - 1) / kKnnThreads), block(kKnnThreads);
    switch (k) {
        case 4: k_knn_grid<4><<<grid, block, 0, s>>>(w.sorted, m, w.desc, w.starts, nbr_dev, d2_dev); break;
        case 8: k_knn_grid<8><<<grid, block, 0, s>>>(w.sorted, m, w.desc, w.starts, nbr_dev, d2_dev); break;
        case 16: k_knn_grid<16><<<grid, block, 0, s>>>(w.sorted, m, w.desc, w.starts, nbr_dev, d2_dev); break;
        default: k_knn_grid<kMaxK><<<grid, block, 0, s>>>(w.sorted, m, w.desc, w.starts, nbr_dev, d2_dev); break;
    }
    PGS_CHECK_LAUNCH("pgs_knn");
    return PGS_OK;
}

extern "C" pgs_status pgs_pca_seed(const float* points_dev, const float* colours_dev, int32_t m,
                                   const int32_t* nbr_dev, const double* d2_dev, int32_t k, float r_normal,
                                   float* params_dev, void* stream) {
    PGS_REQUIRE(m > 16 && k >= 16, "pgs_pca_seed: need m > 16 and k >= 16");
    PGS_REQUIRE(r_normal > 0.f, "pgs_pca_seed: r_normal must be positive");
    PGS_REQUIRE(points_dev && colours_dev && nbr_dev && d2_dev && params_dev, "pgs_pca_seed: null pointer");
    k_pca_seed<<<(m + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(points_dev, colours_dev, m, nbr_dev, d2_dev,
                                                                  k, (double)r_normal, params_dev);
    PGS_CHECK_LAUNCH("pgs_pca_seed");
    return PGS_OK;
}

extern "C" pgs_status pgs_mlp_features(const float* points_dev, int32_t m, const int32_t* nbr_dev,
                                       const double* d2_dev, int32_t k, float r_normal, float* x_dev,
                                       float* base_dev, void* stream) {
    PGS_REQUIRE(m > 16 && k >= 16, "pgs_mlp_features: need m > 16 and k >= 16");
    PGS_REQUIRE(r_normal > 0.f, "pgs_mlp_features: r_normal must be positive");
    PGS_REQUIRE(points_dev && nbr_dev && d2_dev && x_dev && base_dev, "pgs_mlp_features: null pointer");
    k_mlp_features<<<(m + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(points_dev, m, nbr_dev, d2_dev,
                                                                      (double)r_normal, x_dev, base_dev);
    PGS_CHECK_LAUNCH("pgs_mlp_features");
    return PGS_OK;
}

extern "C" pgs_status pgs_seed_targets(const float* params_dev, int32_t n, float* targets_dev, void* stream) {
    PGS_REQUIRE(n >= 0, "pgs_seed_targets: n must be >= 0");
    if (n == 0) return PGS_OK;
    PGS_REQUIRE(params_dev && targets_dev, "pgs_seed_targets: null pointer");
    k_seed_targets<<<(n + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(params_dev, n, targets_dev);
    PGS_CHECK_LAUNCH("pgs_seed_targets");
    return PGS_OK;
}

extern "C" pgs_status pgs_seed_apply(const float* y_dev, const float* base_dev, const float* pca_params_dev,
                                     int32_t m, float* params_dev, uint8_t* fallback_dev,
                                     uint32_t* fallback_count_dev, void* stream) {
    PGS_REQUIRE(m >= 0, "pgs_seed_apply: m must be >= 0");
    if (m == 0) return PGS_OK;
    PGS_REQUIRE(y_dev && base_dev && pca_params_dev && params_dev, "pgs_seed_apply: null pointer");
    k_seed_apply<<<(m + 255) / 256, 256, 0, pgs::as_stream(stream)>>>(y_dev, base_dev, pca_params_dev, m,
                                                                    params_dev, fallback_dev, fallback_count_dev);
    PGS_CHECK_LAUNCH("pgs_seed_apply");
    return PGS_OK;
}
