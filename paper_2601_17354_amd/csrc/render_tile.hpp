// Per-tile compositing forward and backward, shared by the single-view
// kernels (one workgroup per tile) and the multi-view persistent kernels
// (workgroups pull (view, tile) items from a queue).
//
// Forward (PocketGS Sec. "Explicit Computation Graph", "Bandwidth-Efficient
// Forward Replay Cache"): one lane per pixel of a TW x TH tile.  The tile's
// sorted splat list is staged through LDS in batches of BG splats (36 B of
// 2D attributes each) and every wave steps through the batch in lockstep,
// each lane compositing its pixel front to back.  A barrier with a live-lane
// count ends the tile once every pixel terminated.
//
// Replay trace.  S = {id, C_in, alpha} is recorded per wave of 64 pixels as
// groups, one per sorted splat id that at least one of the wave's pixels
// composited: a 64-bit ballot mask of those pixels (stored at the id's slot)
// followed by their entries in lane order.  The id of an entry is thus the
// slot of its group, its pixel the lane of its mask bit, and a pixel's
// entries in group order are its contributors front to back.  After the
// front to back pass each wave knows how many entries it recorded and takes
// a region of exactly that size from a device-wide bump counter (one 64-bit
// atomic per tile, split among its waves in order); a wave whose region does
// not fit the entry capacity is left unrecorded and the overflow flag is
// raised, the counter then holding the demand the caller needs.  A per-wave
// step counter bounds the valid groups, so masks of earlier iterations are
// never read and nothing is cleared between iterations.  The tile's groups
// are then walked back to front with the splats re-staged in LDS, and each
// entry is written once, one coalesced run per group: C_in (12 bytes; the
// backward recomputes alpha) or (C_in, alpha) (16 bytes), C_in being the
// colour of everything behind the splat, the over-recursion
// C_out = C_in (1 - alpha) + alpha c run from the background.
//
// Backward (equation "backward_chain"), two variants:
//   cached     steps through each wave's groups front to back, visiting only
//              non-empty masks, four groups at a time with the next four's
//              entries in flight; a lane with a bit set reads its entry, takes
//              dL/dC_out (starts at dL/dC, times (1 - alpha) after each own
//              entry), dL/dalpha = <dL/dC_out, c - C_in> and dL/dc =
//              alpha dL/dC_out, forms the per-pixel terms that the splat's 2D
//              gradients are linear in, and the wave reduces the four groups'
//              terms together (DPP and lane swaps).
//   recompute  walks the list back to front from n_contrib, re-evaluates
//              alpha with the forward's exact arithmetic, recovers
//              T_k = T_{k+1} / (1 - alpha_k) from T_final and accumulates the
//              colour behind as it goes (the 3D Gaussian Splatting backward).
// Per-wave partial sums meet in LDS; once per batch the splat's conic and
// opacity turn them into its nine 2D gradients, which leave with one float
// atomic per field and (tile, splat), scattered to the canonical index
// values[id] (index-mapping equation).
#pragma once

#include "common.hpp"

// Splats a wave composites between two termination checks.  Four leave room for
// eight waves a SIMD with their colours at hand (untraced, 300k Gaussians at
// 1920 x 1440: six took 1.05 times as long, eight 1.09 times).
#ifndef FWD_UNROLL
#define FWD_UNROLL 4
#endif

namespace pgs {

// A splat as staged in LDS: mean (u, v), the conic (A, B, C) held as
// hA = -A/2, nB = -B, hC = -C/2 (scalings by powers of two and a sign, so
// exact), opacity and colour.
struct Splat {
    float u, v, hA, nB, hC, o, r, g, b;
};

// Alpha of a splat at pixel centre (px, py).  Evaluated with contraction off
// so that the forward and the recompute backward produce identical bits.
__device__ __forceinline__ bool splat_alpha(const Splat& s, float px, float py, float& alpha,
                                            float& gauss, float& dx, float& dy, bool& positive) {
#pragma clang fp contract(off)
    dx = s.u - px;
    dy = s.v - py;
    // power = -(A dx^2 + 2 B dx dy + C dy^2) / 2 = (hA dx + nB dy) dx + hC dy^2
    const float power = __builtin_fmaf(__builtin_fmaf(s.hA, dx, s.nB * dy), dx, s.hC * dy * dy);
    gauss = __expf(power);
    alpha = fminf(kAlphaMax, s.o * gauss);
    positive = power > 0.f;
    return alpha >= kAlphaMin;
}
__device__ __forceinline__ bool splat_alpha(const Splat& s, float px, float py, float& alpha, float& gauss, float& dx,
                                            float& dy) {
    bool positive;
    const bool seen = splat_alpha(s, px, py, alpha, gauss, dx, dy, positive);
    return seen && !positive;
}

// One splat's record (u, v, depth, A | B, C, o, r | g, b, ex, ey) is one
// 64-byte line: three 16-byte loads.  (The compositing kernels decide which
// waves a splat can reach from its conic instead of the half-extents
// (ex, ey).)
__device__ __forceinline__ void stage_splat(const float* __restrict__ proj, int n, uint32_t g,
                                            float4* sa, float4* sb, float* sc, int slot) {
    (void)n;
    const float4* rec = reinterpret_cast<const float4*>(proj + (size_t)g * PGS_PROJ_STRIDE);
    const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
    sa[slot] = make_float4(r0.x, r0.y, -0.5f * r0.w, -r1.x);   // u, v, hA, nB
    sb[slot] = make_float4(-0.5f * r1.y, r1.z, r1.w, r2.x);    // hC, o, r, g
    sc[slot] = r2.y;                                  // b
}

__device__ __forceinline__ Splat load_splat(const float4* sa, const float4* sb, const float* sc, int k) {
    const float4 a = sa[k], b = sb[k];
    return Splat{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, sc[k]};
}

// Mean, conic and opacity of a staged splat (colour left zero).
__device__ __forceinline__ Splat load_shape(const float4* sa, const float4* sb, int k) {
    const float4 a = sa[k];
    const float2 b = *reinterpret_cast<const float2*>(&sb[k]);
    return Splat{a.x, a.y, a.z, a.w, b.x, b.y, 0.f, 0.f, 0.f};
}

// first + the set bits of m below this lane: its rank among the lanes of m.
__device__ __forceinline__ uint32_t lane_rank(uint64_t m, uint32_t first = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, first));
}

// Whether this lane's bit is set in the wave-uniform mask m (the mask
// becomes the execution mask directly).
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// A wave's trace entries are addressed through a buffer resource on the
// start of its region (kept in scalar registers) with 32-bit byte offsets:
// a run's start as the scalar offset and the lane's rank in it as the vector
// one, so an access takes no 64-bit per-lane address arithmetic.  A region
// stays far below 4 GiB: a pixel composites at most ln(1e-4) / ln(1 - 1/255)
// < 2400 splats before its transmittance ends it, so a wave's region holds
// fewer than 64 * 2400 entries.  Word 3 of the resource selects the 32-bit
// data format (value 4 in bits 15-18), which untyped buffer access on this
// GPU family expects; the record count is left at its maximum.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t region_rsrc(const void* region) {
    const uint64_t a = reinterpret_cast<uint64_t>(region);
    const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0, -1, 0x00020000);
}

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Entries are read once, so loads pass the caches as streams (the non-temporal
// bit): the backward of 300k Gaussians at 1920 x 1440 441 -> 417 us.  Stores do
// so only where several views record one trace of many gigabytes (eight views of
// 1M Gaussians 2.56 -> 2.34 ms); for one view they lose as much or more than they
// gain (300k Gaussians at 1920 x 1440: 488 us streamed, 486 not; a scene with half
// as many pairs again: 725 and 647).
constexpr int kStream = 2;

// Entry `rank` (< 64) of the run of EW-word entries that starts `first`
// entries into the region.
template <int EW>
__device__ __forceinline__ float4 load_entry(__amdgpu_buffer_rsrc_t rs, uint32_t first, uint32_t rank) {
    // first is the same in every lane; saying so keeps the offset scalar
    const uint32_t voff = __umul24(rank, 4u * EW),
                   soff = (uint32_t)__builtin_amdgcn_readfirstlane((int)(first * (4u * EW)));
    if constexpr (EW == 4) {
        const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, kStream);
        return make_float4(__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w));
    } else {
        const u32x3 r = __builtin_amdgcn_raw_buffer_load_b96(rs, voff, soff, kStream);
        return make_float4(__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), 0.f);
    }
}

// Stores take the whole offset in the vector operand and a zero scalar
// offset: the compiler inserts the wait that a store of more than 8 bytes
// needs before its data registers are overwritten only for that form, and
// with a register scalar offset the store was measured to pick up the next
// value of its data registers.
template <int EW, bool STREAM>
__device__ __forceinline__ void store_entry(__amdgpu_buffer_rsrc_t rs, uint32_t first, uint64_t lanes, float c0,
                                            float c1, float c2, float alpha) {
    const uint32_t voff = __umul24(lane_rank(lanes, first), 4u * EW);  // a region: far below 2^24 entries
    if constexpr (EW == 4) {
        u32x4 d = {__float_as_uint(c0), __float_as_uint(c1), __float_as_uint(c2), __float_as_uint(alpha)};
        __builtin_amdgcn_raw_buffer_store_b128(d, rs, voff, 0, STREAM ? kStream : 0);
    } else {
        u32x3 d = {__float_as_uint(c0), __float_as_uint(c1), __float_as_uint(c2)};
        __builtin_amdgcn_raw_buffer_store_b96(d, rs, voff, 0, STREAM ? kStream : 0);
        (void)alpha;
    }
}

__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Lanes that composite a step: those it hits, less the terminated ones and the
// ones that it ends (whose transmittance would fall below the threshold), which
// leave live.  In assembly because the compiler turned this wave-uniform chain
// into vector instructions.
__device__ __forceinline__ uint64_t step_lanes(uint64_t hit, uint64_t below, uint64_t& live) {
    uint64_t took;
    asm("s_and_b64 %0, %2, %3\n"
        "s_andn2_b64 %1, %1, %0\n"
        "s_and_b64 %0, %2, %1"
        : "=&s"(took), "+s"(live)
        : "s"(hit), "s"(below)
        : "scc");
    return took;
}

// v_writelane_b32, for which this compiler has no builtin, by the intrinsic's
// name (the instruction in assembly needs m0, which an asm block must not take).
extern "C" __device__ __attribute__((const)) uint32_t pgs_writelane(uint32_t v, uint32_t lane,
                                                                    uint32_t old) __asm("llvm.amdgcn.writelane.i32");

// Puts the wave-uniform v into lane `lane` of (lo, hi).
__device__ __forceinline__ void write_lane64(uint32_t& lo, uint32_t& hi, uint64_t v, int lane) {
    lo = pgs_writelane((uint32_t)v, (uint32_t)lane, lo);
    hi = pgs_writelane((uint32_t)(v >> 32), (uint32_t)lane, hi);
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int j = 32; j > 0; j >>= 1) v += (uint32_t)__shfl_xor((int)v, j);
    return v;
}

struct Trace {
    uint64_t* mask;             // [NW][pair_cap]
    uint32_t* steps;            // [n_tiles][NW]
    uint32_t* base;             // [n_tiles][NW] first entry of the wave's region
    unsigned long long* used;   // entries handed out in this forward
    float* entry;               // [entry_cap][EW]: (C_in r, g, b[, alpha])
    uint32_t* count;            // [pixels]
    size_t entry_cap;
    uint32_t pair_cap;
    int words;                  // EW of the launch: 4 with alpha, 3 without
};

// A trace entry holds EW words: (C_in r, g, b, alpha) as one 16-byte record,
// or (C_in r, g, b) as one 12-byte record when the backward recomputes alpha
// from the staged splat with the forward's arithmetic (same bits).

// One tile of one view.  Pixel arrays (image planes, t_final, n_contrib,
// count) are the view's own; gt is the tile's global index in the ranges.
struct TileJob {
    int W, H, tx, ty, gt;
    const float* proj;
    float* image;
    float* t_final;
    uint32_t* n_contrib;
    uint32_t* count;
};

// LDS of a tile pass: one batch of BG staged splats (forward), plus their
// canonical ids and the gradient accumulator (backward); declared by each
// kernel and handed to the tile functions.
template <int BG>
struct FwdLds {
    float4 a[BG];
    float4 b[BG];
    float c[BG];
    uint8_t reach[BG];  // bit w: the splat can reach a pixel of wave w
    uint32_t steps;
    // per wave of the tile: entries, steps, fit flag and region start
    uint32_t wcur[4], wsteps[4], wfit[4];
    unsigned long long wbase[4];
};

// The four waves' partial sums of a splat meet in two accumulators, two waves in
// each: a sum of two does not depend on which comes first, so a tile's sums
// are the same in every run (added to one accumulator by all four, they varied
// with the order, by as much as the order of the tiles makes the totals vary).
// Batches of the single-view backward then hold 224 splats at most, which keeps
// six workgroups on a CU, as many as their registers allow (with 256 five:
// 1920 x 1440 447 us, with 224 427); those of the multi-view backward 192 (with
// 224 its registers spill, 2279 us against 2166).
template <int NW>
constexpr int kAccs = NW > 2 ? 2 : 1;
template <int BG, int NW, int MOST = 224>
constexpr int kBwdBatch = NW > 2 && BG > MOST ? MOST : BG;

template <int BG, int NA = 1>
struct TileLds {
    float4 a[BG];
    float4 b[BG];
    float c[BG];
    uint32_t g[BG];
    float io[BG];  // 1 / opacity
    uint8_t reach[BG];  // bit w: the splat can reach a pixel of wave w (recompute backward)
    float acc[NA][9][BG + 1];  // one word of padding per row: a splat's nine terms fall in nine banks
    uint32_t steps;
};

// Stages splats base .. base+nb-1 of the sorted list into LDS slots 0..nb-1.
template <int NT, bool KEEP_IDS, class Lds>
__device__ __forceinline__ void stage_batch(Lds& L, const float* __restrict__ proj, int n,
                                            const uint32_t* __restrict__ values, uint32_t base, int nb,
                                            int t) {
    for (int q = t; q < nb; q += NT) {
        const uint32_t g = values[base + q];
        stage_splat(proj, n, g, L.a, L.b, L.c, q);
        if constexpr (KEEP_IDS) {
            L.g[q] = g;
            L.io[q] = 1.f / L.b[q].y;
        }
    }
}

// Which waves of a TW x TH tile a splat can reach: bit w is cleared only if
// splat_alpha gives alpha < 1/255 at every pixel centre of wave w's rows
// (the wave's pixel-centre rectangle R_w).  Alpha reaches 1/255 only where
// q = A dx^2 + 2 B dx dy + C dy^2 <= 2 ln(255 o).  The minimum of q over R_w
// is zero if the centre lies inside R_w, else the least of the four edge
// minima, each the minimum of a convex quadratic in one variable, clamped to
// the edge.  Rounding: with rho = |B| / sqrt(A C), the magnitudes of q's
// three terms sum to at most q (1 + rho) / (1 - rho), and each term carries
// a relative error of a few units of roundoff u in float32, both in
// splat_alpha and here (an error in the position of an edge minimum changes q
// only to second order), so both evaluations are within
// kappa = 64 u (1 + rho) / (1 - rho) of q relative to it.  A wave is dropped
// when the computed minimum, shrunk by 2 kappa, still exceeds 2 ln(255 o) by
// 1e-4, which also covers the rounding of the exponential, the opacity
// product and the threshold; and never when kappa >= 1/8.
template <int TW, int TH>
__device__ __forceinline__ uint32_t reach_waves(float u, float v, float A, float B, float C, float o, int tx,
                                                int ty) {
    constexpr int NW = TW * TH / 64;
    constexpr int R = 64 / TW;  // pixel rows per wave
    constexpr uint32_t kAll = (1u << NW) - 1u;
    if (!(o > kAlphaMin * 0.5f)) return 0u;  // alpha = o e^power <= o < 1/255 everywhere
    if (!(A > 0.f && C > 0.f)) return kAll;
    const float ac = A * C;
    const float rho = fabsf(B) * __frsqrt_rn(ac);
    // 1 - rho = (A C - B^2) / (A C (1 + rho)), the determinant taken with one rounding
    const float det = __builtin_fmaf(A, C, -B * B);
    const float omr = det / (ac * (1.f + rho));
    const float kappa = 64.f * 0x1p-24f * (1.f + rho) / omr;
    if (!(omr > 0.f && kappa < 0.125f)) return kAll;
    const float thr = 2.f * __logf(255.f * o) + 1e-4f;
    const float shrink = 1.f - 2.f * kappa;
    const float ra = 1.f / A, rc = 1.f / C;
    const float xlo = (float)(tx * TW) + 0.5f, xhi = xlo + (float)(TW - 1);
    // dx over the rectangle's columns, dy over its rows (d = centre - pixel)
    const float dxa = u - xhi, dxb = u - xlo;
    const float ma = -B * dxa * rc, mb = -B * dxb * rc;  // best dy on the columns x = xhi, xlo
    auto q = [&](float dx, float dy) { return A * dx * dx + 2.f * B * dx * dy + C * dy * dy; };
    uint32_t bits = 0u;
#pragma unroll 1
    for (int w = 0; w < NW; ++w) {
        const float ylo = (float)(ty * TH + w * R) + 0.5f, yhi = ylo + (float)(R - 1);
        const float dya = v - yhi, dyb = v - ylo;
        float m = 0.f;
        if (!(dxa <= 0.f && dxb >= 0.f && dya <= 0.f && dyb >= 0.f)) {
            m = fminf(q(dxa, fminf(fmaxf(ma, dya), dyb)), q(dxb, fminf(fmaxf(mb, dya), dyb)));
            // rows y = yhi, ylo: dx minimising q at fixed dy is -B dy / A
            m = fminf(m, q(fminf(fmaxf(-B * dya * ra, dxa), dxb), dya));
            m = fminf(m, q(fminf(fmaxf(-B * dyb * ra, dxa), dxb), dyb));
        }
        if (!(m * shrink > thr)) bits |= 1u << w;
    }
    return bits;
}

// Stages splats base .. base+nb-1 of the sorted list into LDS slots 0..nb-1
// with the waves each can reach (and, for the backward, their canonical ids
// and 1 / opacity).
template <int TW, int TH, int NT, bool KEEP_IDS, class Lds>
__device__ __forceinline__ void stage_batch_reach(Lds& L, const float* __restrict__ proj,
                                                  const uint32_t* __restrict__ values, uint32_t base, int nb,
                                                  int t, int tx, int ty) {
    for (int q = t; q < nb; q += NT) {
        const uint32_t g = values[base + q];
        const float4* rec = reinterpret_cast<const float4*>(proj + (size_t)g * PGS_PROJ_STRIDE);
        const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
        L.a[q] = make_float4(r0.x, r0.y, -0.5f * r0.w, -r1.x);   // u, v, hA, nB
        L.b[q] = make_float4(-0.5f * r1.y, r1.z, r1.w, r2.x);    // hC, o, r, g
        L.c[q] = r2.y;                                           // b
        L.reach[q] = (uint8_t)reach_waves<TW, TH>(r0.x, r0.y, r0.w, r1.x, r1.y, r1.z, tx, ty);
        if constexpr (KEEP_IDS) {
            L.g[q] = g;
            L.io[q] = 1.f / r1.z;
        }
    }
}

template <int TW, int TH, int BG, bool CACHED, int EW = 4, bool STREAM = false>
__device__ __forceinline__ void fwd_tile(const TileJob& j, int n_tiles_total, int n,
                                         const uint32_t* __restrict__ values,
                                         const uint32_t* __restrict__ ranges, float bg0, float bg1,
                                         float bg2, const Trace& tr, uint32_t* __restrict__ flags,
                                         FwdLds<BG>& L) {
    constexpr int NT = TW * TH;
    constexpr int NW = NT / 64;
    static_assert((BG & (BG - 1)) == 0 && BG >= 32, "batch: a power of two, at least half a window");
    static_assert(NW <= 4, "at most four waves per tile");
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int px = j.tx * TW + (t % TW), py = j.ty * TH + (t / TW);
    const bool inside = px < j.W && py < j.H;
    const uint32_t start = ranges[j.gt], end = ranges[n_tiles_total + j.gt];
    const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;

    // the trace is recorded only if this tile's pairs fit the trace buffers
    const bool rec = CACHED && end <= tr.pair_cap;
    if (CACHED && !rec && t == 0) atomicOr(flags, PGS_FLAG_CACHE_OVERFLOW);
    // Lane s keeps the mask of step s of the current window of 64 (the pixels
    // that composited it); a window is written as one coalesced 512-byte run
    // (wave-major mask layout).
    uint64_t* wmask = tr.mask + (size_t)wv * tr.pair_cap + start;
    uint32_t mask_lo = 0, mask_hi = 0;
    uint32_t steps = 0, cnt = 0, last = 0;

    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
    uint64_t live = __ballot(inside);  // lanes whose pixel has not terminated

    for (uint32_t base = start; base < end; base += BG) {
        if (__syncthreads_or(live != 0ull) == 0) break;
        const int nb = (int)min((uint32_t)BG, end - base);
        stage_batch_reach<TW, TH, NT, false>(L, j.proj, values, base, nb, t, j.tx, j.ty);
        __syncthreads();
        // Windows of 64 steps.  Of a window the wave visits only the steps
        // whose splat can reach one of its pixels (a wave-uniform bit set,
        // walked with scalar bit scans), FWD_UNROLL at a time: their LDS
        // loads and alphas first, straight-line, then the steps in order,
        // with a termination check per group.  Every step it skips has alpha
        // < 1/255 at all of its pixels, so its mask bits are zero as if it
        // had been visited.  Bound by vector issue, 22 instructions a step;
        // with the alphas and colours fetched between the steps' branches, lane
        // masks in vector registers and a 64 x 64 bit transpose a window for
        // the trace, 300k Gaussians at 1920 x 1440 took 227 us untraced, now
        // 187 (95% of its issue slots), traced 510, now 477 (80%: the entry
        // pass issues as many vector instructions again, 102M to the 98M here,
        // beside 1.5 GB of writes that take 260 alone).
        for (int c0 = 0; c0 < nb; c0 += 64) {
            if (live == 0ull) break;  // the whole wave has terminated
            const int cn = min(64, nb - c0);
            const uint32_t rel0 = base + (uint32_t)c0 - start;
            uint64_t todo = __ballot(lane < cn && ((L.reach[c0 + lane] >> wv) & 1u) != 0u);
            while (todo) {
                if (live == 0ull) break;
                const int left = __popc((uint32_t)todo) + __popc((uint32_t)(todo >> 32));
                int kq[FWD_UNROLL];
                Splat sp[FWD_UNROLL];
#pragma unroll
                for (int u = 0; u < FWD_UNROLL; ++u) {
                    // past the last step: some slot of the batch, not used
                    kq[u] = __builtin_ctzll(todo | (1ull << (BG < 64 ? 31 : 63)));
                    todo &= ~(1ull << kq[u]);
                    sp[u] = load_splat(L.a, L.b, L.c, c0 + kq[u]);
                }
                // alphas and the lanes that reach 1/255 (a wave-uniform mask)
                // are complete before the steps' branches
                float al[FWD_UNROLL];
                uint64_t hit[FWD_UNROLL];
#pragma unroll
                for (int u = 0; u < FWD_UNROLL; ++u) {
                    float gauss, dx, dy;
                    bool pos;
                    const bool seen = splat_alpha(sp[u], fpx, fpy, al[u], gauss, dx, dy, pos);
                    const uint64_t real = (uint64_t)(int64_t)((u - left) >> 31);  // all ones where u < left
                    hit[u] = __ballot(seen) & ~__ballot(pos) & real;
                    asm volatile("" : "+v"(al[u]), "+s"(hit[u]));
                }
#pragma unroll
                for (int u = 0; u < FWD_UNROLL; ++u) {
                    const float alpha = al[u];
                    const float test_T = T * (1.f - alpha);
                    const uint64_t took = step_lanes(hit[u], __ballot(test_T < kTMin), live);
                    if (took == 0ull) continue;  // uniform
                    if constexpr (CACHED) write_lane64(mask_lo, mask_hi, took, kq[u]);
                    if (lane_in(took)) {
                        const float w = alpha * T;
                        C0 += w * sp[u].r;
                        C1 += w * sp[u].g;
                        C2 += w * sp[u].b;
                        T = test_T;
                        last = rel0 + (uint32_t)kq[u] + 1u;
                        if constexpr (CACHED) ++cnt;
                    }
                }
            }
            if constexpr (CACHED) {
                if (rec && lane < cn) wmask[rel0 + lane] = ((uint64_t)mask_hi << 32) | mask_lo;
                mask_lo = mask_hi = 0u;
            }
            steps = rel0 + (uint32_t)cn;
        }
    }
    uint32_t cursor = 0;
    if (rec) cursor = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_sum_u32(cnt));  // the same in every lane
    // Entry regions: one bump-counter atomic per tile (a single device-wide
    // address, so per-wave atomics would queue there), split among the
    // waves in order.  A wave whose region does not fit the entry capacity
    // is left unrecorded (its step count becomes 0, so the backward reads
    // nothing of it) and the overflow flag is raised; the counter keeps the
    // demand either way.
    size_t ebase = 0;
    bool wrec = rec;
    uint32_t smax = 0;
    if (rec) {  // uniform for the block
        if (lane == 0) {
            L.wcur[wv] = cursor;
            L.wsteps[wv] = steps;
        }
        __syncthreads();
        if (t == 0) {
            unsigned long long total = 0;
            for (int w = 0; w < NW; ++w) total += L.wcur[w];
            unsigned long long b = total ? atomicAdd(tr.used, total) : 0ull;
            uint32_t sm = 0;
            bool lost = false;
            for (int w = 0; w < NW; ++w) {
                const bool fit = L.wcur[w] == 0 || b + L.wcur[w] <= tr.entry_cap;
                L.wfit[w] = fit;
                L.wbase[w] = fit ? b : 0ull;
                if (fit) sm = max(sm, L.wsteps[w]);
                lost |= !fit;
                b += L.wcur[w];
            }
            if (lost) atomicOr(flags, PGS_FLAG_CACHE_OVERFLOW);
            L.steps = sm;
        }
        __syncthreads();
        wrec = L.wfit[wv] != 0;
        ebase = (size_t)L.wbase[wv];
        smax = L.steps;
        if (!wrec) steps = 0;
    }
    if (inside) {
        const size_t pix = (size_t)py * j.W + px, plane = (size_t)j.W * j.H;
        j.image[pix] = C0 + T * bg0;
        j.image[plane + pix] = C1 + T * bg1;
        j.image[2 * plane + pix] = C2 + T * bg2;
        j.t_final[pix] = T;
        j.n_contrib[pix] = last;
        if (CACHED) j.count[pix] = wrec ? cnt : 0u;
    }
    if (!rec) return;  // uniform for the block
    if (lane == 0) {
        tr.steps[(size_t)j.gt * NW + wv] = steps;
        tr.base[(size_t)j.gt * NW + wv] = (uint32_t)ebase;
    }

    // Entry pass: back to front over each wave's groups with the splats
    // re-staged in LDS batch by batch (the forward batches in reverse).  Each
    // set lane re-evaluates alpha with the same arithmetic as above (same
    // bits) and writes its entry (C_in, alpha) once, C_in being the colour
    // accumulated behind the splat so far.
    float a0 = bg0, a1 = bg1, a2 = bg2;
    uint32_t cur = cursor;
    if (smax == 0) return;
    const int64_t top = (int64_t)((smax - 1) / BG) * BG;  // first position of the last batch
    // Windows of 64 steps per batch.  A batch's masks are loaded together
    // with its splats: a wait on a vector load also waits for the entry
    // stores issued before it, so this costs one such wait per batch rather
    // than one per window.
    constexpr int kWin = BG >= 64 ? BG / 64 : 1;
    const uint64_t* wm = tr.mask + (size_t)wv * tr.pair_cap + start;
    const __amdgpu_buffer_rsrc_t went = region_rsrc(tr.entry + ebase * EW);
    for (int64_t lo = top; lo >= 0; lo -= BG) {
        const uint32_t hi = min((uint32_t)lo + BG, smax);
        __syncthreads();
        stage_batch<NT, false>(L, j.proj, n, values, start + (uint32_t)lo, (int)(hi - (uint32_t)lo), t);
        const uint32_t whi = min(hi, steps);
        uint64_t mw[kWin];
#pragma unroll
        for (int w = 0; w < kWin; ++w) {
            const uint32_t c0 = (uint32_t)lo + 64u * w;
            mw[w] = c0 + (uint32_t)lane < whi ? wm[c0 + lane] : 0ull;
        }
        __syncthreads();
        // windows last to first; the non-empty groups of a window are taken
        // last to first, four at a time: their splats' loads and alphas
        // first, then each set lane writes its entries in order
#pragma unroll
        for (int w = kWin - 1; w >= 0; --w) {
            const uint32_t c0 = (uint32_t)lo + 64u * w;
            if (c0 >= whi) continue;  // uniform
            const uint64_t mv = mw[w];
            uint64_t any = __ballot(mv != 0ull);
            while (any) {
                int gi[4];
                uint64_t gm[4];
                uint32_t gc[4];
                Splat sq[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // past the first group: any lane's mask, cleared
                    const uint64_t real = (uint64_t)((int64_t)(any ? -1 : 0));
                    gi[q] = 63 - __builtin_clzll(any | 1ull);
                    any &= ~(1ull << gi[q]);
                    gm[q] = read_lane64(mv, gi[q]) & real;
                    cur -= __popc((uint32_t)gm[q]) + __popc((uint32_t)(gm[q] >> 32));
                    gc[q] = cur;
                    sq[q] = load_splat(L.a, L.b, L.c, 64 * w + gi[q]);
                }
                float al[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float gauss, dx, dy;
                    splat_alpha(sq[q], fpx, fpy, al[q], gauss, dx, dy);
                    asm volatile("" : "+v"(al[q]));  // ahead of the groups' branches
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (lane_in(gm[q])) {
                        const float a = al[q], om = 1.f - a;
                        store_entry<EW, STREAM>(went, gc[q], gm[q], a0, a1, a2, a);
                        // blended in place after the store, without copies
                        asm volatile("" : "+v"(a0), "+v"(a1), "+v"(a2));
                        a0 = a * sq[q].r + om * a0;
                        a1 = a * sq[q].g + om * a1;
                        a2 = a * sq[q].b + om * a2;
                    }
                }
            }
        }
    }
}

// Per-pixel terms of one splat's nine 2D gradients, all linear in what the
// wave and the tile sum: with p = dL/dpower = alpha dL/dalpha (0 where alpha
// is clamped) and d = (dx, dy) the offset from the pixel to the mean, the
// terms are p dx, p dy, p dx^2, p dx dy, p dy^2, p and dL/dc = alpha dL/dC_out.
// The splat's conic and opacity, the same for every pixel, are applied once
// per splat and tile to the sums (grad2d_from_sums).  Where 16 lanes lie in one
// pixel row (tiles at least 16 wide) dy is the same in all of them: a lane then
// forms p, p dx, p dx^2 and dL/dc (six terms), and the three with dy come from
// the row's sums.
template <int TW>
constexpr int kTerms = TW >= 16 ? 6 : 9;

template <int NT>
__device__ __forceinline__ void raw_terms(float dx, float dy, float alpha, bool clamped, float dl_dalpha,
                                          float dc0, float dc1, float dc2, float* v) {
    const float p = clamped ? 0.f : alpha * dl_dalpha;
    const float px = p * dx;
    if constexpr (NT == 6) {
        v[0] = p;
        v[1] = px;
        v[2] = px * dx;
    } else {
        const float py = p * dy;
        v[0] = px;
        v[1] = py;
        v[2] = px * dx;
        v[3] = px * dy;
        v[4] = py * dy;
        v[5] = p;
    }
    v[NT - 3] = dc0;
    v[NT - 2] = dc1;
    v[NT - 1] = dc2;
}

// The nine 2D gradients from the summed terms of raw_terms.  With
// power = hA dx^2 + nB dx dy + hC dy^2 (hA = -A/2, nB = -B, hC = -C/2) and
// alpha = o e^power: dL/du = 2 hA S(p dx) + nB S(p dy),
// dL/dv = nB S(p dx) + 2 hC S(p dy), dL/dA = -S(p dx^2) / 2,
// dL/dB = -S(p dx dy), dL/dC = -S(p dy^2) / 2, dL/do = S(p) / o (the
// derivative of o e^power by o is alpha / o), dL/dc unchanged.
__device__ __forceinline__ void grad2d_from_sums(float hA, float nB, float hC, float inv_o, float* f) {
    const float spx = f[0], spy = f[1];
    f[0] = __builtin_fmaf(2.f * hA, spx, nB * spy);
    f[1] = __builtin_fmaf(2.f * hC, spy, nB * spx);
    f[2] = -0.5f * f[2];
    f[3] = -f[3];
    f[4] = -0.5f * f[4];
    f[5] = f[5] * inv_o;
}

// x + y taken from the lane that the DPP control CTRL names inside a 16-lane
// row (every control used here names a lane of the same row).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x, float y) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), CTRL, 0xf, 0xf, false));
}

// One transposing step for two values a and b with the partner lane that CTRL
// names: lanes with lo set keep the sum of a over the pair of lanes, the
// others the sum of b.
template <int CTRL>
__device__ __forceinline__ float fold_pair(float a, float b, bool lo) {
    return dpp_add<CTRL>(lo ? a : b, lo ? b : a);
}

// The same step for NT pairs, the result in a, where the lanes that take b are
// whole quads: an add over all lanes and one whose bank mask admits only those
// quads, two instructions a pair instead of two selects and an add.  Written
// as blocks because the compiler does not form the masked add; the waits cover
// a vector write just before a cross-lane read on either side.
#define PGS_FOLD1(CTRL, MASK, A, B)                                           \
    "v_add_f32_dpp " A ", " A ", " A " " CTRL " row_mask:0xf bank_mask:0xf\n" \
    "v_add_f32_dpp " A ", " B ", " B " " CTRL " row_mask:0xf bank_mask:" MASK "\n"
#define PGS_FOLD3(CTRL, MASK, a, b)                                                                        \
    asm("s_nop 1\n" PGS_FOLD1(CTRL, MASK, "%0", "%3") PGS_FOLD1(CTRL, MASK, "%1", "%4")                    \
            PGS_FOLD1(CTRL, MASK, "%2", "%5") "s_nop 1"                                                    \
        : "+v"((a)[0]), "+v"((a)[1]), "+v"((a)[2])                                                         \
        : "v"((b)[0]), "v"((b)[1]), "v"((b)[2]))
#define PGS_FOLD6(CTRL, MASK, a, b)                                                                        \
    asm("s_nop 1\n" PGS_FOLD1(CTRL, MASK, "%0", "%6") PGS_FOLD1(CTRL, MASK, "%1", "%7")                    \
            PGS_FOLD1(CTRL, MASK, "%2", "%8") PGS_FOLD1(CTRL, MASK, "%3", "%9")                            \
                PGS_FOLD1(CTRL, MASK, "%4", "%10") PGS_FOLD1(CTRL, MASK, "%5", "%11") "s_nop 1"            \
        : "+v"((a)[0]), "+v"((a)[1]), "+v"((a)[2]), "+v"((a)[3]), "+v"((a)[4]), "+v"((a)[5])               \
        : "v"((b)[0]), "v"((b)[1]), "v"((b)[2]), "v"((b)[3]), "v"((b)[4]), "v"((b)[5]))
template <int NT>
__device__ __forceinline__ void fold_ror8(float* a, const float* b) {
    PGS_FOLD6("row_ror:8", "0xc", a, b);
    if constexpr (NT == 9) PGS_FOLD3("row_ror:8", "0xc", a + 6, b + 6);
}
template <int NT>
__device__ __forceinline__ void fold_half_mirror(float* a, const float* b) {
    PGS_FOLD6("row_half_mirror", "0xa", a, b);
    if constexpr (NT == 9) PGS_FOLD3("row_half_mirror", "0xa", a + 6, b + 6);
}

// Where the wave's sums are after wave_reduce: quad k of every row holds
// group k; in even lanes of row r term (0, 2, 1, 3)[r], plus 4 where bit 1 of
// the lane is set; in odd lanes term 8.
__device__ __forceinline__ int term_of_lane(int lane) {
    if (lane & 1) return 8;
    return ((lane >> 3) & 2) + (lane >> 5) + ((lane & 2) << 1);
}
__device__ __forceinline__ bool lane_adds(int lane) { return (lane & 1) == 0 || (lane & 0x33) == 1; }

// Sums the terms of each of four groups over the wave (u[NT q + f] is term f
// of group q at this lane, overwritten; dy[q] the group's offset).  Every step
// meets two values across two lanes, leaving each lane a sum of one of them,
// so that it halves the values and doubles the lanes a value covers.  The
// steps inside a row come first, while there are most values: lane i ^ 8 by a
// rotation for groups q and q + 2, the mirror lane of each half for q and
// q + 1; six terms become nine there, with the dy of the quad's group.  Then
// v_permlane32_swap and v_permlane16_swap across the rows, which cost two issue
// slots each, and i ^ 2 and i ^ 1 inside the quads.  67 instructions and 8 of
// the swaps for six terms, where nine terms that swapped first took 93 with
// their products and 27 swaps: the traced backward of 300k Gaussians at
// 1920 x 1440 477 us, now 434.
template <int NT>
__device__ __forceinline__ float wave_reduce(float* u, const float* dy, int lane) {
    fold_ror8<NT>(u, u + 2 * NT);
    fold_ror8<NT>(u + NT, u + 3 * NT);
    fold_half_mirror<NT>(u, u + NT);
    float v[9];
    if constexpr (NT == 9) {
#pragma unroll
        for (int f = 0; f < 9; ++f) v[f] = u[f];
    } else {
        const float d0 = dy[0], d1 = dy[1], d2 = dy[2], d3 = dy[3];
        const float d01 = (lane & 4) ? d1 : d0, d23 = (lane & 4) ? d3 : d2;
        const float d = (lane & 8) ? d23 : d01;
        v[0] = u[1];
        v[1] = u[0] * d;
        v[2] = u[2];
        v[3] = u[1] * d;
        v[4] = v[1] * d;
        v[5] = u[0];
        v[6] = u[3];
        v[7] = u[4];
        v[8] = u[5];
    }
    const auto across32 = [](float a, float b) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const auto across16 = [](float a, float b) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const float w0 = across32(v[0], v[1]), w1 = across32(v[2], v[3]);
    const float w2 = across32(v[4], v[5]), w3 = across32(v[6], v[7]);
    float t8 = across32(v[8], v[8]);
    const float x0 = across16(w0, w1), x1 = across16(w2, w3);
    t8 = across16(t8, t8);
    constexpr int kSwap2 = 0x4e, kSwap1 = 0xb1;
    const float r0 = fold_pair<kSwap2>(x0, x1, (lane & 2) == 0);
    t8 = dpp_add<kSwap2>(t8, t8);
    // the whole row; kept outside the adding lanes' branch, where the shifted
    // move folds into the add
    const float total = fold_pair<kSwap1>(r0, t8, (lane & 1) == 0);
    asm volatile("" : : "v"(total));
    return total;
}

// Adds the wave's gradient terms of each of four groups (splat slots
// slot0 + gi[q]; an empty group, whose mask is 0, adds nothing) into the LDS
// accumulator: one combined reduction, then one LDS add by the lanes that hold
// the sums.
template <int BG, int NT>
__device__ __forceinline__ void accumulate_groups(float* v, const float* dy, float (*acc)[BG + 1], int lane,
                                                  uint32_t slot0, const int* gi, const uint64_t* gm) {
    const float x = wave_reduce<NT>(v, dy, lane);
    // quad k takes group k's slot, or -1 for an empty group (lane selects
    // of the uniform values, no branch)
    int sq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) sq[q] = gm[q] != 0ull ? (int)slot0 + gi[q] : -1;
    const int s01 = (lane & 4) ? sq[1] : sq[0];
    const int s23 = (lane & 4) ? sq[3] : sq[2];
    const int slot = (lane & 8) ? s23 : s01;
    if (lane_adds(lane) && slot >= 0) atomicAdd(&acc[term_of_lane(lane)][slot], x);
}

// The batch's summed terms become its splats' 2D gradients (one thread per
// splat), then one float atomic per field and splat goes into the canonical
// 2D-gradient records (index map values[id]); the nine fields of a splat
// share one 64-byte record, so consecutive lanes hit the same line.  Each
// accumulator word is cleared as it is read, so the next batch starts from
// zeros (slots past nb are never written).
template <int BG, int NA>
__device__ __forceinline__ void flush_batch(TileLds<BG, NA>& L, int nb, int n, float* __restrict__ grad2d, int t,
                                            int NT) {
    (void)n;
    float (*acc)[BG + 1] = L.acc[0];
    const uint32_t* gid = L.g;
    for (int jj = t; jj < nb; jj += NT) {
        float f[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            f[k] = acc[k][jj];
            if constexpr (NA == 2) {
                f[k] += L.acc[1][k][jj];
                L.acc[1][k][jj] = 0.f;
            }
        }
        grad2d_from_sums(L.a[jj].z, L.a[jj].w, L.b[jj].x, L.io[jj], f);
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[k][jj] = f[k];
    }
    __syncthreads();
    for (int idx = t; idx < nb * 9; idx += NT) {
        const int jj = idx / 9, f = idx - jj * 9;
        float s = acc[f][jj];
        acc[f][jj] = 0.f;
        if constexpr (NA == 2) {
            s += L.acc[1][f][jj];
            L.acc[1][f][jj] = 0.f;
        }
        if (s != 0.f) unsafeAtomicAdd(&grad2d[(size_t)gid[jj] * PGS_GRAD2D_STRIDE + f], s);
    }
}

template <int BG, int NA>
__device__ __forceinline__ void zero_acc(float (&acc)[NA][9][BG + 1], int t, int NT) {
    for (int idx = t; idx < NA * 9 * (BG + 1); idx += NT) (&acc[0][0][0])[idx] = 0.f;
}

// The first step of a 64-step window that `any` marks.  None left: step 0,
// whose splat every window has staged (a batch of 224 or 32 splats ends inside
// a window, so step 63 may lie past its arrays).
__host__ __device__ constexpr int first_step(uint64_t any) { return any ? __builtin_ctzll(any) : 0; }
static_assert(first_step(0) == 0 && first_step(1ull << 63) == 63 && first_step(0x50) == 4, "steps");

// Up to four non-empty groups of a 64-step window, front to back: the
// step within the window, the lane mask and the first entry (relative to the
// wave's region) of each; an unused slot has an empty mask.
struct TraceGroups {
    int gi[4];
    uint64_t gm[4];
    uint32_t gc[4];
};

__device__ __forceinline__ void take_groups(uint64_t& any, uint64_t mv, uint32_t& cursor, TraceGroups& g) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t real = (uint64_t)((int64_t)(any ? -1 : 0));
        g.gi[q] = first_step(any);
        g.gm[q] = read_lane64(mv, g.gi[q]) & real;
        g.gc[q] = cursor;
        any &= any - 1;
        // uniform
        cursor = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)(cursor + __popc((uint32_t)g.gm[q]) + __popc((uint32_t)(g.gm[q] >> 32))));
    }
}

// Every lane loads: its own entry where it has one, else the wave's first
// entry (the region is not empty when a group exists); alpha is taken as 0
// for the latter in bwd_groups.
template <int EW>
__device__ __forceinline__ void load_groups(__amdgpu_buffer_rsrc_t went, const TraceGroups& g, float4* e) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // an empty group (unused slot) reads the region's first entry
        e[q] = load_entry<EW>(went, g.gm[q] != 0ull ? g.gc[q] : 0u, lane_in(g.gm[q]) ? lane_rank(g.gm[q]) : 0u);
    }
}

// Gradients of four groups at this lane's pixel, reduced over the wave into
// the batch accumulator; a lane without an entry in a group contributes
// zeros there (or what a splat that is not finite makes of zero) and keeps its
// dL/dC_out.  An unused slot's terms are formed from some staged splat and
// entry: they stay in the quads of its own group, which add nothing.
template <int BG, int EW, int NT, class Lds>
__device__ __forceinline__ void bwd_groups(const TraceGroups& g, const float4* e, Lds& L, uint32_t slot0, float fpx,
                                           float fpy, int lane, int half, float& g0, float& g1, float& g2) {
    float v[4 * NT], dys[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int jj = (int)slot0 + g.gi[q];
        const Splat s = load_splat(L.a, L.b, L.c, jj);
        float dx = s.u - fpx, dy = s.v - fpy;
        float a;
        if constexpr (EW == 4) {
            a = lane_in(g.gm[q]) ? e[q].w : 0.f;
        } else {
            // the entry's alpha, recomputed with the forward's arithmetic
            float ar, gauss;
            splat_alpha(s, fpx, fpy, ar, gauss, dx, dy);
            a = lane_in(g.gm[q]) ? ar : 0.f;
        }
        // dL/dalpha = <dL/dC_out, c - C_in>, dL/dc = alpha dL/dC_out
        const float dla = g0 * (s.r - e[q].x) + g1 * (s.g - e[q].y) + g2 * (s.b - e[q].z);
        const bool clamped = a >= kAlphaMax;
        raw_terms<NT>(dx, dy, a, clamped, dla, a * g0, a * g1, a * g2, &v[q * NT]);
        dys[q] = dy;
        // dL/dC_in = dL/dC_out (1 - alpha): the next entry's dL/dC_out
        const float om = 1.f - a;
        g0 *= om;
        g1 *= om;
        g2 *= om;
    }
    accumulate_groups<BG, NT>(v, dys, L.acc[half], lane, slot0, g.gi, g.gm);
}

template <int TW, int TH, int BG, int EW = 4>
__device__ __forceinline__ void bwd_cached_tile(const TileJob& j, int n_tiles_total, int n,
                                                const uint32_t* __restrict__ values,
                                                const uint32_t* __restrict__ ranges, const Trace& tr,
                                                const float* __restrict__ dl_dimage,
                                                float* __restrict__ grad2d, TileLds<BG, kAccs<TW * TH / 64>>& L) {
    constexpr int NT = TW * TH;
    constexpr int NW = NT / 64;
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int half = kAccs<NW> == 2 ? wv >> 1 : 0;
    const int px = j.tx * TW + (t % TW), py = j.ty * TH + (t / TW);
    const bool inside = px < j.W && py < j.H;
    const uint32_t start = ranges[j.gt], end = ranges[n_tiles_total + j.gt];
    if (end > tr.pair_cap) return;  // no trace was recorded for this tile (uniform)
    const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
    const size_t pix = (size_t)py * j.W + px, plane = (size_t)j.W * j.H;
    const size_t ebase = tr.base[(size_t)j.gt * NW + wv];
    const __amdgpu_buffer_rsrc_t went = region_rsrc(tr.entry + ebase * EW);

    float g0 = 0.f, g1 = 0.f, g2 = 0.f;  // dL/dC_out of this pixel's next entry
    if (inside) {
        g0 = dl_dimage[pix];
        g1 = dl_dimage[plane + pix];
        g2 = dl_dimage[2 * plane + pix];
    }
    const uint32_t steps = tr.steps[(size_t)j.gt * NW + wv];
    __syncthreads();
    if (t == 0) L.steps = 0;
    __syncthreads();
    if (lane == 0) atomicMax(&L.steps, steps);
    __syncthreads();
    const uint32_t smax = L.steps;
    uint32_t cursor = 0;
    zero_acc<BG>(L.acc, t, NT);  // once: each flush leaves the accumulator cleared

    for (uint32_t base = 0; base < smax; base += BG) {
        const int nb = (int)min((uint32_t)BG, smax - base);
        stage_batch<NT, true>(L, j.proj, n, values, start + base, nb, t);
        __syncthreads();
        const uint32_t whi = min(base + (uint32_t)nb, steps);
        for (uint32_t c0 = base; c0 < whi; c0 += 64) {
            const uint32_t cn = min(64u, whi - c0);
            const uint64_t mv = (uint32_t)lane < cn ? tr.mask[(size_t)wv * tr.pair_cap + start + c0 + lane] : 0ull;
            uint64_t any = __ballot(mv != 0ull);
            if (!any) continue;  // uniform
            // Groups are taken four at a time and software-pipelined: the
            // next four groups' trace entries are loaded while the current
            // four are reduced.  Every lane loads (a lane without an entry in
            // a group reads the wave's first entry and takes alpha = 0 there),
            // so the count of loads in flight is fixed and the wait for the
            // current four leaves the next four outstanding.
            TraceGroups ga, gb;
            float4 ea[4], eb[4];
            take_groups(any, mv, cursor, ga);
            load_groups<EW>(went, ga, ea);
            for (;;) {
                if (!any) {
                    bwd_groups<BG, EW, kTerms<TW>>(ga, ea, L, c0 - base, fpx, fpy, lane, half, g0, g1, g2);
                    break;
                }
                take_groups(any, mv, cursor, gb);
                load_groups<EW>(went, gb, eb);
                bwd_groups<BG, EW, kTerms<TW>>(ga, ea, L, c0 - base, fpx, fpy, lane, half, g0, g1, g2);
                if (!any) {
                    bwd_groups<BG, EW, kTerms<TW>>(gb, eb, L, c0 - base, fpx, fpy, lane, half, g0, g1, g2);
                    break;
                }
                take_groups(any, mv, cursor, ga);
                load_groups<EW>(went, ga, ea);
                bwd_groups<BG, EW, kTerms<TW>>(gb, eb, L, c0 - base, fpx, fpy, lane, half, g0, g1, g2);
            }
        }
        __syncthreads();
        flush_batch<BG>(L, nb, n, grad2d, t, NT);
        __syncthreads();
    }
}

template <int TW, int TH, int BG>
__device__ __forceinline__ void bwd_recompute_tile(const TileJob& j, int n,
                                                   const uint32_t* __restrict__ values,
                                                   const uint32_t* __restrict__ ranges, float bg0,
                                                   float bg1, float bg2, const float* __restrict__ dl_dimage,
                                                   float* __restrict__ grad2d, TileLds<BG, kAccs<TW * TH / 64>>& L) {
    constexpr int NT = TW * TH;
    const int t = threadIdx.x, lane = t & 63;
    const int px = j.tx * TW + (t % TW), py = j.ty * TH + (t / TW);
    const bool inside = px < j.W && py < j.H;
    const uint32_t start = ranges[j.gt];
    const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
    const size_t pix = (size_t)py * j.W + px, plane = (size_t)j.W * j.H;

    uint32_t last = 0;
    float T = 1.f, G0 = 0.f, G1 = 0.f, G2 = 0.f;
    if (inside) {
        last = j.n_contrib[pix];
        T = j.t_final[pix];
        G0 = dl_dimage[pix];
        G1 = dl_dimage[plane + pix];
        G2 = dl_dimage[2 * plane + pix];
    }
    float a0 = bg0, a1 = bg1, a2 = bg2;  // colour behind the current splat
    __syncthreads();
    if (t == 0) L.steps = 0;
    __syncthreads();
    if (last) atomicMax(&L.steps, last);
    __syncthreads();
    const uint32_t top = L.steps;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), half = kAccs<NT / 64> == 2 ? wv >> 1 : 0;
    zero_acc<BG>(L.acc, t, NT);  // once: each flush leaves the accumulator cleared
    uint32_t wlast = last;  // the wave's last contributing step
#pragma unroll
    for (int j2 = 32; j2 > 0; j2 >>= 1) wlast = max(wlast, (uint32_t)__shfl_xor((int)wlast, j2));
    wlast = (uint32_t)__builtin_amdgcn_readfirstlane((int)wlast);

    for (uint32_t hi = top; hi > 0;) {
        const uint32_t lo = hi > (uint32_t)BG ? hi - BG : 0u;
        const int nb = (int)(hi - lo);
        stage_batch_reach<TW, TH, NT, true>(L, j.proj, values, start + lo, nb, t, j.tx, j.ty);
        __syncthreads();
        // back to front over the steps up to the wave's last whose splat can
        // reach one of its pixels (windows of 64 last to first, scalar bit
        // scans), four at a time: their loads and alphas first, straight-line,
        // then the pixels' states step by step, then the four gradients'
        // reduction over the wave.  Step by step up to the alphas, each waited
        // for its LDS loads and branches: 100k Gaussians at 1024 x 768 187 us,
        // now 155.
        const int wn = wlast > lo ? min(nb, (int)(wlast - lo)) : 0;
        int cw = (wn + 63) >> 6;
        uint64_t todo = 0ull;
        for (;;) {
            constexpr int kT = kTerms<TW>;
            int gi[4];
            uint64_t gm[4];
            float al[4], dxs[4], dys[4];
            bool ok[4], clamped[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                while (todo == 0ull && cw > 0) {
                    --cw;
                    const int k = 64 * cw + lane;
                    todo = __ballot(k < wn && ((L.reach[k] >> wv) & 1u) != 0u);
                }
                const int bit = todo ? 63 - __clzll((long long)todo) : 0;
                gi[q] = 64 * cw + bit;
                gm[q] = todo;  // for now: whether there is a step
                todo &= ~(1ull << bit);
            }
            if (gm[0] == 0ull) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const Splat sq = load_shape(L.a, L.b, gi[q]);
                float gauss;
                ok[q] = splat_alpha(sq, fpx, fpy, al[q], gauss, dxs[q], dys[q]) && gm[q] != 0ull &&
                        lo + (uint32_t)gi[q] < last;
                clamped[q] = sq.o * gauss > kAlphaMax;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) gm[q] = __ballot(ok[q]);
            if ((gm[0] | gm[1] | gm[2] | gm[3]) == 0ull) continue;
            float v[4 * kT];
#pragma unroll
            for (int f = 0; f < 4 * kT; ++f) v[f] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (ok[q]) {
                    const float2 rg = *reinterpret_cast<const float2*>(&L.b[gi[q]].z);
                    const float cb = L.c[gi[q]], alpha = al[q], om = 1.f - alpha;
                    // T_k = T_{k+1} / (1 - alpha_k), with the hardware reciprocal
                    // (about one unit of roundoff, the size of the product's own)
                    T *= __builtin_amdgcn_rcpf(om);
                    const float q0 = T * G0, q1 = T * G1, q2 = T * G2;
                    const float dla = q0 * (rg.x - a0) + q1 * (rg.y - a1) + q2 * (cb - a2);
                    raw_terms<kT>(dxs[q], dys[q], alpha, clamped[q], dla, alpha * q0, alpha * q1, alpha * q2,
                                  &v[q * kT]);
                    a0 = alpha * rg.x + om * a0;
                    a1 = alpha * rg.y + om * a1;
                    a2 = alpha * cb + om * a2;
                }
            }
            accumulate_groups<BG, kT>(v, dys, L.acc[half], lane, 0u, gi, gm);
        }
        __syncthreads();
        flush_batch<BG>(L, nb, n, grad2d, t, NT);
        __syncthreads();
        hi = lo;
    }
}

// Checks a replay-trace descriptor and wraps it.
pgs_status make_trace(const pgs_replay* c, Trace& tr, const char* who);

// Zeroes the trace's entry counter ahead of a forward (a kernel, so that the
// call can be captured in a graph).
void reset_trace_counter(const Trace& tr, hipStream_t s);

// Tile shapes the kernels are built for (one lane per pixel, whole waves).
inline bool tile_shape_ok(int tw, int th) {
    return (tw == 16 && th == 16) || (tw == 8 && th == 8) || (tw == 16 && th == 8) ||
           (tw == 32 && th == 8) || (tw == 8 && th == 32);
}

}  // namespace pgs
