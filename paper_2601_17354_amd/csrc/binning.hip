// Tile binning and the (tile, depth) key sort that yields the permutation pi
// of PocketGS's index-mapping subsection.
//
// The pairs are ordered by (tile, depth bits, canonical id).  Instead of
// sorting all 46 significant key bits of every pair, the Gaussians are
// sorted once by depth and the pairs emitted in that order, so that a stable
// sort on the tile bits alone finishes the order:
//   depth    stable LSD sort of the (depth bits, item) of every Gaussian of
//            every view (4 passes over n items instead of 4 over the pairs)
//   scan     exclusive prefix sum of tiles_touched in depth order -> pair
//            offsets + count
//   emit     one (key, canonical id) pair per Gaussian x rectangle tile,
//            key = tile << 32 | bits(float32 depth), each workgroup filling
//            an equal range of pairs (binary search over the offsets), so
//            large Gaussians do not serialise
//   sort     stable LSD radix sort on the tile bits only, 8-bit digits;
//            every pass is histogram -> stable scatter, sorts of more than
//            2^20 keys with a device scan of the histogram in between
//   ranges   per-tile [start, end)
//
// Every kernel reads the item and pair counts from device memory and is
// launched on a grid sized for the capacity, so nothing travels to the host
// and the whole sequence can be captured in a HIP graph.
#include <mutex>

#include "common.hpp"

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanIpt = 8;
constexpr int kScanItems = kScanThreads * kScanIpt;  // 2048 per block

// Workgroups of a sort: 4096 keys on 1024 threads.  Up to kSmallSort keys at
// most 256 workgroups exist and each sums the histograms of the others itself
// (k_radix_scatter); a pass is two launches, where the scan between histogram
// and scatter made it four of about 4.5 us each whatever they move.  Beyond, the
// scan.  2048 keys on 256 threads gave a digit's run 64 bytes and scans of
// twice the size: the sorts of eight views of 1M Gaussians 1100 us, with 4096
// keys 940, with 8192 1010.
constexpr uint32_t kSmallSort = 1u << 20;
template <bool DIRECT>
struct SortShape {
    static constexpr int kThreads = 1024, kRounds = 4, kKeys = kThreads * kRounds;
    static constexpr bool kDirect = DIRECT;
};
using SmallSort = SortShape<true>;
using LargeSort = SortShape<false>;
// Gaussians that one workgroup sorts and scans by itself.
constexpr uint32_t kBlockSort = 4096;
constexpr int kRadix = 256;

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
inline uint32_t div_up(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Block-wide exclusive scan of one value per thread (Hillis-Steele in LDS).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s, uint32_t& total) {
    const int t = threadIdx.x;
    s[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        uint32_t add = t >= off ? s[t - off] : 0u;
        __syncthreads();
        s[t] += add;
        __syncthreads();
    }
    total = s[kScanThreads - 1];
    const uint32_t incl = s[t];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* __restrict__ in,
                                                              uint32_t n, uint32_t* __restrict__ partial) {
    __shared__ uint32_t s[kScanThreads];
    const uint32_t base = blockIdx.x * kScanItems + threadIdx.x * kScanIpt;
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k)
        if (base + k < n) sum += in[base + k];
    uint32_t total;
    block_exclusive_scan(sum, s, total);
    if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// Per-block exclusive scan of `in` offset by the sum of the preceding
// blocks' partial sums (each block adds those up itself, so the partials
// need no scan launch of their own); the last block writes the grand total
// to *total_out (if not null).  `out` may alias `in`.
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t* in, uint32_t n,
                                                             const uint32_t* __restrict__ partial,
                                                             uint32_t* out,
                                                             uint32_t* __restrict__ total_out) {
    __shared__ uint32_t s[kScanThreads];
    uint32_t before = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanThreads) before += partial[i];
    uint32_t offset;
    block_exclusive_scan(before, s, offset);
    const uint32_t base = blockIdx.x * kScanItems + threadIdx.x * kScanIpt;
    uint32_t loc[kScanIpt];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
        loc[k] = (base + k < n) ? in[base + k] : 0u;
        sum += loc[k];
    }
    uint32_t total;
    uint32_t run = offset + block_exclusive_scan(sum, s, total);
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
        if (base + k < n) out[base + k] = run;
        run += loc[k];
    }
    if (total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = offset + total;
}

size_t scan_workspace(uint32_t n) { return align_up((size_t)div_up(n, kScanItems) * 4); }

// Exclusive scan in -> out (may alias), total to total_out (device, may be null).
pgs_status scan_u32(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total_out,
                    uint32_t* partial, hipStream_t s) {
    const uint32_t nb = div_up(n, kScanItems);
    if (nb == 0) return PGS_OK;
    k_scan_reduce<<<nb, kScanThreads, 0, s>>>(in, n, partial);
    k_scan_apply<<<nb, kScanThreads, 0, s>>>(in, n, partial, out, total_out);
    PGS_CHECK_LAUNCH("scan");
    return PGS_OK;
}

// Items of a bin/sort: item i = v * n + g is Gaussian g in view v (one view:
// v = 0), keyed with view v's global tile numbers; values hold the id g.
struct EmitViews {
    int n_views;
    int TX[PGS_MAX_VIEWS];
    int tile_off[PGS_MAX_VIEWS];
};

__device__ __forceinline__ void view_tiles(const EmitViews& ev, int v, int& TX, int& off) {
    TX = ev.TX[0];
    off = ev.tile_off[0];
    for (int u = 1; u < ev.n_views; ++u)
        if (u == v) {
            TX = ev.TX[u];
            off = ev.tile_off[u];
        }
}

__global__ void k_clear_u32(uint32_t* __restrict__ p, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// Where the histogram of digit d in workgroup b goes: block-major (a row of 256
// per workgroup) for sorts that sum rows themselves, else digit-major, so that
// one exclusive scan yields every workgroup's output offset for every digit.
template <class G>
__device__ __forceinline__ size_t hist_at(uint32_t d, uint32_t b, uint32_t nb) {
    return G::kDirect ? (size_t)b * kRadix + d : (size_t)d * nb + b;
}

__device__ __forceinline__ uint32_t depth_key(const float* __restrict__ proj_all,
                                              const uint32_t* __restrict__ touched_all, uint32_t i) {
    // the record's depth is read only for items with pairs (one 4-byte read
    // per 64-byte record, so culled items cost a line)
    return touched_all[i] ? __float_as_uint(proj_all[(size_t)i * PGS_PROJ_STRIDE + PGS_PROJ_DEPTH]) : 0xffffffffu;
}

// Depth keys of every item (float32 depth bits; culled items sort last),
// values = item index, the item count for the depth sort, and the first
// radix pass's digit histogram: workgroup b takes the same items as the
// sort's workgroup b.  Also clears the tile ranges and the pair count.
template <class G>
__global__ __launch_bounds__(G::kThreads) void k_depth_keys(uint32_t items, const float* __restrict__ proj_all,
                                                            const uint32_t* __restrict__ touched_all,
                                                            uint32_t* __restrict__ dkeys,
                                                            uint32_t* __restrict__ dvals,
                                                            uint32_t* __restrict__ count, uint32_t nb,
                                                            uint32_t* __restrict__ hist,
                                                            uint32_t* __restrict__ ranges, uint32_t n_ranges,
                                                            uint32_t* __restrict__ num_pairs) {
    constexpr int NT = G::kThreads;
    __shared__ uint32_t h[kRadix];
    const int t = threadIdx.x;
    if (blockIdx.x == 0 && t == 0) {
        *count = items;
        *num_pairs = 0u;
    }
    for (uint32_t i = blockIdx.x * NT + t; i < n_ranges; i += gridDim.x * NT) ranges[i] = 0u;
    if (t < kRadix) h[t] = 0u;
    __syncthreads();
    const uint32_t base = blockIdx.x * G::kKeys;
#pragma unroll
    for (int r = 0; r < G::kRounds; ++r) {
        const uint32_t i = base + r * NT + t;
        if (i < items) {
            const uint32_t key = depth_key(proj_all, touched_all, i);
            dkeys[i] = key;
            dvals[i] = i;
            atomicAdd(&h[key & 0xffu], 1u);
        }
    }
    __syncthreads();
    if (t < kRadix) hist[hist_at<G>(t, blockIdx.x, nb)] = h[t];
}

// Pairs of the items in depth order.  Workgroup b fills pairs
// [G::kKeys b, G::kKeys (b + 1)), the range of the pair sort's workgroup b: a
// search over the scanned counts finds the item of its first pair (one wave,
// 64 probes a step: a binary search's 19 dependent reads were a third of the
// kernel at 300k items); every item of the range has at least one pair (empty
// items share their successor's offset), so the range spans at most G::kKeys
// items, whose offsets go to LDS; each thread then finds its pairs' items
// there.  The work per workgroup is even however unevenly the rectangles are
// sized.  Each workgroup also writes its part of the pair sort's first
// histogram (the tile's low 8 bits), zeros past the pair count.

__device__ __forceinline__ uint32_t last_le(const uint32_t* off, uint32_t n, uint32_t p) {
    uint32_t lo = 0, hi = n - 1;  // last j with off[j] <= p (off[0] <= p)
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The same by a whole wave: each step probes 64 evenly spaced positions of
// [lo, lo + n) and keeps the stretch from the last one not past p.
__device__ __forceinline__ uint32_t wave_last_le(const uint32_t* __restrict__ off, uint32_t n, uint32_t p, int lane) {
    uint32_t lo = 0;
    while (n > 1) {
        const uint32_t step = (n + 63) >> 6, at = lane * step;
        const uint64_t le = __ballot(at < n && off[lo + (at < n ? at : 0u)] <= p);
        const uint32_t k = 63u - (uint32_t)__clzll((long long)le);  // lane 0 always holds
        lo += k * step;
        n = min(step, n - k * step);
    }
    return lo;
}

template <class G>
__global__ __launch_bounds__(G::kThreads) void k_emit_sorted(uint32_t items, int n, EmitViews ev,
                                                             const uint32_t* __restrict__ dkeys,
                                                             const uint32_t* __restrict__ rect_all,
                                                             const uint32_t* __restrict__ dvals,
                                                             const uint32_t* __restrict__ off,
                                                             const uint32_t* __restrict__ num_pairs,
                                                             uint32_t capacity, uint64_t* __restrict__ keys,
                                                             uint32_t* __restrict__ values,
                                                             uint32_t* __restrict__ flags, uint32_t nb,
                                                             uint32_t* __restrict__ hist) {
    constexpr uint32_t kPairs = G::kKeys;
    constexpr int NT = G::kThreads;
    __shared__ uint32_t s_off[kPairs + 1];
    __shared__ uint32_t s_first;
    __shared__ uint32_t h[kRadix];
    const int t = threadIdx.x;
    const uint32_t total = *num_pairs;
    if (blockIdx.x == 0 && t == 0 && total > capacity) atomicOr(flags, PGS_FLAG_PAIR_OVERFLOW);
    const uint32_t count = min(total, capacity);
    const uint32_t p0 = blockIdx.x * kPairs;
    if (t < kRadix) h[t] = 0u;
    if (p0 < count) {  // uniform for the block
        const uint32_t p1 = min(p0 + kPairs, count);
        if (t < 64) {
            const uint32_t j = wave_last_le(off, items, p0, t);
            if (t == 0) s_first = j;
        }
        __syncthreads();
        const uint32_t i0 = s_first;
        const uint32_t span = min(kPairs + 1, items - i0);
        for (uint32_t q = t; q < span; q += NT) s_off[q] = off[i0 + q];
        __syncthreads();
        for (uint32_t p = p0 + t; p < p1; p += NT) {
            const uint32_t j = last_le(s_off, span, p);
            const uint32_t item = dvals[i0 + j], local = p - s_off[j];
            const uint32_t v = item / (uint32_t)n, g = item - v * (uint32_t)n;
            int TX, toff;
            view_tiles(ev, (int)v, TX, toff);
            const uint32_t r0 = rect_all[(size_t)v * 2 * n + g], r1 = rect_all[(size_t)v * 2 * n + n + g];
            const uint32_t x0 = r0 & 0xffff, y0 = r0 >> 16, x1 = r1 & 0xffff;
            const uint32_t w = x1 - x0 + 1;
            const uint32_t ty = y0 + local / w, tx = x0 + local % w;
            const uint64_t tile = (uint64_t)((uint32_t)toff + ty * (uint32_t)TX + tx);
            // the depth bits are the sorted key itself (no read of the record)
            const uint32_t dbits = dkeys[i0 + j];
            keys[p] = (tile << 32) | (uint64_t)dbits;
            values[p] = g;
            atomicAdd(&h[(uint32_t)tile & 0xffu], 1u);
        }
    }
    __syncthreads();
    if (blockIdx.x < nb && t < kRadix) hist[hist_at<G>(t, blockIdx.x, nb)] = h[t];
}

__device__ __forceinline__ uint32_t clamp_count(const uint32_t* num, uint32_t capacity) {
    const uint32_t c = *num;
    return c < capacity ? c : capacity;
}

// Digit histogram of each workgroup's chunk of keys.
template <class G, class K>
__global__ __launch_bounds__(G::kThreads) void k_radix_hist(const K* __restrict__ keys,
                                                            const uint32_t* __restrict__ num, uint32_t capacity,
                                                            int shift, uint32_t nb, uint32_t* __restrict__ hist) {
    constexpr int NT = G::kThreads, R = G::kRounds;
    __shared__ uint32_t h[kRadix];
    const uint32_t count = clamp_count(num, capacity);
    const uint32_t base = blockIdx.x * G::kKeys;
    if (G::kDirect && base >= count) return;  // rows past the last key are not read
    if (threadIdx.x < kRadix) h[threadIdx.x] = 0;
    __syncthreads();
    if (base < count) {
        uint32_t d[R];  // every load in flight before the first atomic
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t idx = base + r * NT + threadIdx.x;
            d[r] = idx < count ? (uint32_t)(keys[idx] >> shift) & 0xffu : kRadix;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (d[r] < kRadix) atomicAdd(&h[d[r]], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kRadix) hist[hist_at<G>(threadIdx.x, blockIdx.x, nb)] = h[threadIdx.x];
}

// Ranks of a wave's R 64-key rounds: rank[r] = keys of the same digit that come
// before lane's key of round r in the wave, cnt[d] the wave's count of digit d
// so far (LDS, zero at the start).  Same-digit lanes are found by matching the
// 8 digit bits with wave ballots; every lane reads its digit's count before
// the first lane of the digit raises it.
template <int R>
__device__ __forceinline__ void wave_ranks(const uint32_t (&digit)[R], const bool (&valid)[R], uint32_t* cnt,
                                           uint32_t (&rank)[R], int lane) {
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint64_t peers = __ballot(valid[r]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (digit[r] >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t below = __popcll(peers & lt_mask);
        const uint32_t before = valid[r] ? cnt[digit[r]] : 0u;
        rank[r] = before + below;
        wave_fence();
        if (valid[r] && below == 0) cnt[digit[r]] = before + __popcll(peers);
        wave_fence();
    }
}

// Exclusive scan over threads 0..255 of v (wave shuffles, the four wave totals
// through s_wave); the workgroup's other threads only pass the barriers.
__device__ __forceinline__ uint32_t scan_256(uint32_t v, uint32_t* s_wave) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o);
        if (lane >= o) inc += u;
    }
    if (t < kRadix && lane == 63) s_wave[wv] = inc;
    __syncthreads();
    uint32_t before = 0;
    if (t < kRadix)
        for (int w = 0; w < wv; ++w) before += s_wave[w];
    __syncthreads();
    return before + inc - v;
}

// Stable scatter through LDS.  Each wave ranks its own contiguous run of the
// chunk (64 R keys) without waiting for the others; the waves' digit counts
// then give every (digit, wave) its place in the workgroup, the keys go to
// LDS in that order and leave as one contiguous run per digit, so the global
// writes coalesce.  Three barriers around the ranking, where ranking 256 keys
// at a time across the workgroup took two for every round.  The digits'
// places in the output: DIRECT sums the other workgroups' histograms here
// (thread (q, d): every fourth row of digit d), else the scanned digit-major
// histogram.  With gdst, the pass also writes gdst[pos] = gsrc[value] (a
// gather in the output order).
template <class G, class K>
__global__ __launch_bounds__(G::kThreads) void k_radix_scatter(
    const K* __restrict__ kin, const uint32_t* __restrict__ vin, K* __restrict__ kout, uint32_t* __restrict__ vout,
    const uint32_t* __restrict__ num, uint32_t capacity, int shift, uint32_t nb, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ gsrc, uint32_t* __restrict__ gdst) {
    constexpr int NT = G::kThreads, R = G::kRounds, NW = NT / 64;
    __shared__ K s_key[G::kKeys];
    __shared__ uint32_t s_val[G::kKeys];
    __shared__ uint32_t s_cnt[NW][kRadix];  // per-wave digit counts, then each wave's places
    __shared__ uint32_t s_lbase[kRadix];    // digit start inside the block
    __shared__ uint32_t s_gbase[kRadix];    // digit start in the output
    __shared__ uint32_t s_wave[4];
    const uint32_t count = clamp_count(num, capacity);
    const uint32_t base = blockIdx.x * G::kKeys;
    if (base >= count) return;  // uniform for the block
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // the block's loads are all issued before anything waits
    K kreg[R];
    uint32_t vreg[R], digit[R], rank[R];
    bool valid[R];
    const uint32_t first = base + (uint32_t)wv * 64 * R + lane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t idx = first + r * 64;
        valid[r] = idx < count;
        kreg[r] = valid[r] ? kin[idx] : (K)0;
        vreg[r] = valid[r] ? vin[idx] : 0u;
    }
    uint32_t g_total = 0, g_before = 0;  // this thread's share of digit t % 256
    if constexpr (G::kDirect) {
        const uint32_t blocks = (count + G::kKeys - 1) / G::kKeys, d = t & (kRadix - 1);
        for (uint32_t b0 = t / kRadix; b0 < blocks; b0 += 8 * (NT / kRadix)) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t b = b0 + u * (NT / kRadix);
                v[u] = b < blocks ? hist[(size_t)b * kRadix + d] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                g_total += v[u];
                if (b0 + u * (NT / kRadix) < blockIdx.x) g_before += v[u];
            }
        }
    } else {
        if (t < kRadix) g_before = hist[(size_t)t * nb + blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < kRadix / 64; ++k) s_cnt[wv][64 * k + lane] = 0u;
    wave_fence();
#pragma unroll
    for (int r = 0; r < R; ++r) digit[r] = (uint32_t)(kreg[r] >> shift) & 0xffu;
    wave_ranks<R>(digit, valid, s_cnt[wv], rank, lane);
    if constexpr (G::kDirect) {  // shares of the four threads of a digit, in LDS words that are free until the keys come
        s_val[t] = g_total;
        s_val[NT + t] = g_before;
    }
    __syncthreads();
    uint32_t here = 0, total = 0;
    if (t < kRadix) {
        for (int w = 0; w < NW; ++w) here += s_cnt[w][t];
        if constexpr (G::kDirect) {
            g_before = 0;
            for (int q = 0; q < NT / kRadix; ++q) {
                total += s_val[q * kRadix + t];
                g_before += s_val[NT + q * kRadix + t];
            }
        }
    }
    if constexpr (G::kDirect) g_before += scan_256(total, s_wave);
    const uint32_t lb = scan_256(here, s_wave);
    if (t < kRadix) {
        s_lbase[t] = lb;
        s_gbase[t] = g_before;
        uint32_t run = lb;
        for (int w = 0; w < NW; ++w) {
            const uint32_t c = s_cnt[w][t];
            s_cnt[w][t] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (valid[r]) {
            const uint32_t pos = s_cnt[wv][digit[r]] + rank[r];
            s_key[pos] = kreg[r];
            s_val[pos] = vreg[r];
        }
    __syncthreads();
    const uint32_t mine = min((uint32_t)G::kKeys, count - base);
    for (uint32_t i = t; i < mine; i += NT) {
        const K key = s_key[i];
        const uint32_t d = (uint32_t)(key >> shift) & 0xffu;
        const uint32_t pos = s_gbase[d] + (i - s_lbase[d]);
        kout[pos] = key;
        vout[pos] = s_val[i];
        if (gdst) gdst[pos] = gsrc[s_val[i]];
    }
}

// The whole depth order of at most kBlockSort items by one workgroup: keys,
// four passes in LDS, and the pair offsets (the scan of tiles_touched in depth
// order) with their total.  Also clears the tile ranges.  1000 items: one
// launch of 18 us, where the launches it replaces took about 75.
__global__ __launch_bounds__(1024) void k_depth_order(uint32_t items, const float* __restrict__ proj_all,
                                                      const uint32_t* __restrict__ touched_all,
                                                      uint32_t* __restrict__ dkeys, uint32_t* __restrict__ dvals,
                                                      uint32_t* __restrict__ off, uint32_t* __restrict__ ranges,
                                                      uint32_t n_ranges, uint32_t* __restrict__ num_pairs) {
    constexpr int NT = 1024, NW = NT / 64, R = kBlockSort / NT;
    __shared__ uint32_t s_key[kBlockSort], s_val[kBlockSort], s_cnt[NW][kRadix], s_wave[NW];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    for (uint32_t i = t; i < n_ranges; i += NT) ranges[i] = 0u;
    uint32_t key[R], val[R], digit[R], rank[R];
    bool valid[R];
    const uint32_t first = (uint32_t)wv * 64 * R + lane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t i = first + r * 64;
        valid[r] = i < items;
        val[r] = i;
        key[r] = valid[r] ? depth_key(proj_all, touched_all, i) : 0u;
    }
    for (int shift = 0; shift < 32; shift += 8) {
#pragma unroll
        for (int k = 0; k < kRadix / 64; ++k) s_cnt[wv][64 * k + lane] = 0u;
        wave_fence();
#pragma unroll
        for (int r = 0; r < R; ++r) digit[r] = (key[r] >> shift) & 0xffu;
        wave_ranks<R>(digit, valid, s_cnt[wv], rank, lane);
        __syncthreads();
        uint32_t here = 0;
        if (t < kRadix)
            for (int w = 0; w < NW; ++w) here += s_cnt[w][t];
        uint32_t run = scan_256(here, s_wave);
        if (t < kRadix)
            for (int w = 0; w < NW; ++w) {
                const uint32_t c = s_cnt[w][t];
                s_cnt[w][t] = run;
                run += c;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (valid[r]) {
                const uint32_t pos = s_cnt[wv][digit[r]] + rank[r];
                s_key[pos] = key[r];
                s_val[pos] = val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (valid[r]) {
                key[r] = s_key[first + r * 64];
                val[r] = s_val[first + r * 64];
            }
        __syncthreads();
    }
    // offsets: the wave's keys are consecutive, round by round
    uint32_t own[R], before = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t c = valid[r] ? touched_all[val[r]] : 0u;
        uint32_t inc = c;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(inc, o);
            if (lane >= o) inc += u;
        }
        own[r] = before + inc - c;
        before += __shfl(inc, 63);
    }
    if (lane == 0) s_wave[wv] = before;
    __syncthreads();
    uint32_t run = 0, all = 0;
    for (int w = 0; w < NW; ++w) {
        if (w < wv) run += s_wave[w];
        all += s_wave[w];
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (valid[r]) {
            dkeys[first + r * 64] = key[r];
            dvals[first + r * 64] = val[r];
            off[first + r * 64] = run + own[r];
        }
    if (t == 0) *num_pairs = all;
}

template <class K>
__global__ void k_copy_pairs(const K* __restrict__ ks, const uint32_t* __restrict__ vs,
                             K* __restrict__ kd, uint32_t* __restrict__ vd,
                             const uint32_t* __restrict__ num, uint32_t capacity) {
    const uint32_t count = clamp_count(num, capacity);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        kd[i] = ks[i];
        vd[i] = vs[i];
    }
}

__global__ void k_ranges(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ num,
                         uint32_t capacity, uint32_t n_tiles, uint32_t* __restrict__ ranges) {
    const uint32_t count = clamp_count(num, capacity);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        const uint32_t tile = (uint32_t)(keys[i] >> 32);
        if (tile >= n_tiles) continue;
        if (i == 0 || (uint32_t)(keys[i - 1] >> 32) != tile) ranges[tile] = i;
        if (i + 1 == count || (uint32_t)(keys[i + 1] >> 32) != tile) ranges[n_tiles + tile] = i + 1;
    }
}

// Heavy-first tile order: a one-workgroup counting sort of the view's tiles
// by list length in 8-pair buckets, longest first, so the longest tiles start
// first and the launch has no long tail.  Order inside a bucket is arbitrary;
// it only changes scheduling, never a result.
constexpr int kOrderThreads = 1024;
constexpr int kOrderBuckets = 256;

__device__ __forceinline__ uint32_t order_bucket(const uint32_t* ranges, uint32_t n_tiles_total, uint32_t gt) {
    const uint32_t len = ranges[n_tiles_total + gt] - ranges[gt];
    const uint32_t b = len >> 3;
    return (kOrderBuckets - 1) - (b < (uint32_t)(kOrderBuckets - 1) ? b : (uint32_t)(kOrderBuckets - 1));
}

__global__ __launch_bounds__(kOrderThreads) void k_tile_order(const uint32_t* __restrict__ ranges,
                                                              uint32_t n_view, uint32_t offset,
                                                              uint32_t n_tiles_total,
                                                              uint32_t* __restrict__ order) {
    __shared__ uint32_t hist[kOrderBuckets], s_wave[4];
    static_assert(kOrderBuckets == kRadix, "one bucket per scanned thread");
    for (int b = threadIdx.x; b < kOrderBuckets; b += kOrderThreads) hist[b] = 0;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_view; i += kOrderThreads)
        atomicAdd(&hist[order_bucket(ranges, n_tiles_total, offset + i)], 1u);
    __syncthreads();
    const uint32_t place = scan_256(threadIdx.x < kOrderBuckets ? hist[threadIdx.x] : 0u, s_wave);
    if (threadIdx.x < kOrderBuckets) hist[threadIdx.x] = place;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_view; i += kOrderThreads) {
        const uint32_t pos = atomicAdd(&hist[order_bucket(ranges, n_tiles_total, offset + i)], 1u);
        order[pos] = i;
    }
}

struct SortWs {
    uint64_t* keys_alt;
    uint32_t* vals_alt;
    uint32_t* hist;
    uint32_t* partial;
    uint32_t nb;
    bool small;
    size_t bytes;
};

SortWs sort_layout(void* base, uint32_t capacity) {
    SortWs w{};
    w.small = capacity <= kSmallSort;
    w.nb = div_up(capacity, SmallSort::kKeys);
    size_t off = 0;
    char* p = static_cast<char*>(base);
    w.keys_alt = reinterpret_cast<uint64_t*>(p + off); off += align_up((size_t)capacity * 8);
    w.vals_alt = reinterpret_cast<uint32_t*>(p + off); off += align_up((size_t)capacity * 4);
    w.hist = reinterpret_cast<uint32_t*>(p + off); off += align_up((size_t)w.nb * kRadix * 4);
    w.partial = reinterpret_cast<uint32_t*>(p + off); off += scan_workspace(w.nb * kRadix);
    w.bytes = off;
    return w;
}

int sort_passes(int key_bits) { return (key_bits + 7) / 8; }

template <class G, class K>
pgs_status radix_passes(K* kin, uint32_t* vin, K* kout, uint32_t* vout, const uint32_t* num, uint32_t capacity,
                        int passes, const SortWs& w, hipStream_t s, int start_bit, bool first_hist,
                        const uint32_t* gsrc, uint32_t* gdst) {
    for (int p = 0; p < passes; ++p) {
        const int shift = start_bit + 8 * p;
        const bool last = p + 1 == passes;
        if (p > 0 || !first_hist)
            k_radix_hist<G, K><<<w.nb, G::kThreads, 0, s>>>(kin, num, capacity, shift, w.nb, w.hist);
        if (!G::kDirect) {
            pgs_status st = scan_u32(w.hist, w.hist, w.nb * kRadix, nullptr, w.partial, s);
            if (st != PGS_OK) return st;
        }
        k_radix_scatter<G, K><<<w.nb, G::kThreads, 0, s>>>(kin, vin, kout, vout, num, capacity, shift, w.nb, w.hist,
                                                           last ? gsrc : nullptr, last ? gdst : nullptr);
        PGS_CHECK_LAUNCH("radix pass");
        K* tk = kin; kin = kout; kout = tk;
        uint32_t* tv = vin; vin = vout; vout = tv;
    }
    return PGS_OK;
}

// Sorts key bits [start_bit, start_bit + key_bits) (stable) into (keys, vals),
// the workspace holding the ping-pong copy.  The unsorted input is in
// (keys, vals), or with input_in_ws and an odd number of passes in the
// ping-pong copy, which saves the copy back.  first_hist: the caller already
// wrote the first pass's digit histogram into w.hist.  With gdst, the last
// pass also writes gdst[i] = gsrc[value at i].  Keys of type K (uint64_t, or
// uint32_t for the depth sort, whose keys are 32 bits: a third less traffic
// per pass); the ping-pong key buffer is sized for 64-bit keys and holds
// either.
template <class K>
pgs_status radix_sort(K* keys, uint32_t* vals, const uint32_t* num, uint32_t capacity,
                      int key_bits, const SortWs& w, hipStream_t s, int start_bit = 0, bool first_hist = false,
                      const uint32_t* gsrc = nullptr, uint32_t* gdst = nullptr, bool input_in_ws = false) {
    if (capacity == 0) return PGS_OK;
    const int passes = sort_passes(key_bits);
    K* alt = reinterpret_cast<K*>(w.keys_alt);
    const bool swap = input_in_ws && (passes & 1);
    K *kin = swap ? alt : keys, *kout = swap ? keys : alt;
    uint32_t *vin = swap ? w.vals_alt : vals, *vout = swap ? vals : w.vals_alt;
    const pgs_status st =
        w.small ? radix_passes<SmallSort, K>(kin, vin, kout, vout, num, capacity, passes, w, s, start_bit, first_hist, gsrc, gdst)
                : radix_passes<LargeSort, K>(kin, vin, kout, vout, num, capacity, passes, w, s, start_bit, first_hist, gsrc, gdst);
    if (st != PGS_OK) return st;
    if (!swap && (passes & 1)) {
        k_copy_pairs<K><<<1024, 256, 0, s>>>(alt, w.vals_alt, keys, vals, num, capacity);
        PGS_CHECK_LAUNCH("radix copy");
    }
    return PGS_OK;
}

int bits_for(uint32_t v) {  // number of bits needed for values < v
    int b = 0;
    while (b < 32 && ((uint64_t)1 << b) < v) ++b;
    return b;
}

}  // namespace

extern "C" size_t pgs_sort_workspace(uint32_t capacity) { return sort_layout(nullptr, capacity).bytes; }

extern "C" pgs_status pgs_tile_order(const uint32_t* ranges_dev, int32_t tiles_in_view,
                                     int32_t view_tile_offset, int32_t n_tiles, uint32_t* order_dev,
                                     void* stream) {
    PGS_REQUIRE(tiles_in_view > 0 && view_tile_offset >= 0 && view_tile_offset + tiles_in_view <= n_tiles,
                "pgs_tile_order: bad tile counts");
    PGS_REQUIRE(ranges_dev && order_dev, "pgs_tile_order: null pointer");
    k_tile_order<<<1, kOrderThreads, 0, pgs::as_stream(stream)>>>(ranges_dev, (uint32_t)tiles_in_view,
                                                                 (uint32_t)view_tile_offset, (uint32_t)n_tiles,
                                                                 order_dev);
    PGS_CHECK_LAUNCH("pgs_tile_order");
    return PGS_OK;
}

extern "C" pgs_status pgs_sort_pairs(uint64_t* keys_dev, uint32_t* values_dev, const uint32_t* count_dev,
                                     uint32_t capacity, int32_t key_bits, void* workspace_dev,
                                     size_t workspace_bytes, void* stream) {
    PGS_REQUIRE(key_bits >= 1 && key_bits <= 64, "pgs_sort_pairs: key_bits %d", key_bits);
    if (capacity == 0) return PGS_OK;
    PGS_REQUIRE(keys_dev && values_dev && count_dev && workspace_dev, "pgs_sort_pairs: null pointer");
    SortWs w = sort_layout(workspace_dev, capacity);
    PGS_REQUIRE(workspace_bytes >= w.bytes, "pgs_sort_pairs: workspace %zu < %zu", workspace_bytes, w.bytes);
    return radix_sort(keys_dev, values_dev, count_dev, capacity, key_bits, w, pgs::as_stream(stream));
}

// Workspace of pgs_sort_pairs_noalloc: one array per GPU, in the code
// object, alive until the process ends.  Host code must not pass the name
// `scratch` to a kernel (on the host it is a stand-in, not a device
// address); it uses the address hipGetSymbolAddress gave for the device.
static __device__ __align__(256) unsigned char scratch[PGS_SORT_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
pgs_status scratch_address(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        pgs::set_error("pgs_sort_pairs_noalloc: hipGetDevice: %s", hipGetErrorString(e));
        return PGS_ERR_HIP;
    }
    PGS_REQUIRE(dev >= 0 && dev < kMaxDevices, "pgs_sort_pairs_noalloc: device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || ptr == nullptr) {
            pgs::set_error("pgs_sort_pairs_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
            return PGS_ERR_HIP;
        }
        g_scratch_dev[dev] = ptr;
    }
    *out = g_scratch_dev[dev];
    return PGS_OK;
}

}  // namespace

extern "C" pgs_status pgs_sort_pairs_noalloc(uint64_t* keys_dev, uint32_t* values_dev, const uint32_t* count_dev,
                                             uint32_t capacity, int32_t key_bits, void* stream) {
    PGS_REQUIRE(key_bits >= 1 && key_bits <= 64, "pgs_sort_pairs_noalloc: key_bits %d", key_bits);
    PGS_REQUIRE(capacity <= PGS_SORT_NOALLOC_MAX_PAIRS,
                "pgs_sort_pairs_noalloc: capacity %u exceeds the %u pairs its fixed scratch holds "
                "(use pgs_sort_pairs with a workspace)", capacity, (unsigned)PGS_SORT_NOALLOC_MAX_PAIRS);
    if (capacity == 0) return PGS_OK;
    PGS_REQUIRE(keys_dev && values_dev && count_dev, "pgs_sort_pairs_noalloc: null pointer");
    const size_t need = sort_layout(nullptr, capacity).bytes;
    PGS_REQUIRE(need <= sizeof(scratch), "pgs_sort_pairs_noalloc: workspace %zu exceeds the scratch (%zu)", need,
                sizeof(scratch));
    void* ws = nullptr;
    const pgs_status st = scratch_address(&ws);
    if (st != PGS_OK) return st;
    return radix_sort(keys_dev, values_dev, count_dev, capacity, key_bits, sort_layout(ws, capacity),
                      pgs::as_stream(stream));
}

namespace {

// Workspace of a bin/sort over `items` Gaussians (all views) and `capacity`
// pairs: depth keys and item ids, pair offsets, scan partials, the item
// count word, and the two sorts' ping-pong buffers.
struct BinWs {
    uint32_t* dkeys;
    uint32_t* dvals;
    uint32_t* off;
    uint32_t* partial;
    uint32_t* count;
    SortWs items_ws;
    SortWs pairs_ws;
    size_t bytes;
};

BinWs bin_layout(void* base, uint32_t items, uint32_t capacity) {
    BinWs w{};
    char* p = static_cast<char*>(base);
    size_t off = 0;
    w.dkeys = reinterpret_cast<uint32_t*>(p + off); off += align_up((size_t)items * 4);
    w.dvals = reinterpret_cast<uint32_t*>(p + off); off += align_up((size_t)items * 4);
    w.off = reinterpret_cast<uint32_t*>(p + off); off += align_up((size_t)items * 4);
    w.partial = reinterpret_cast<uint32_t*>(p + off); off += scan_workspace(items);
    w.count = reinterpret_cast<uint32_t*>(p + off); off += align_up(4);
    w.items_ws = sort_layout(p ? p + off : nullptr, items); off += w.items_ws.bytes;
    w.pairs_ws = sort_layout(p ? p + off : nullptr, capacity); off += w.pairs_ws.bytes;
    w.bytes = off;
    return w;
}

pgs_status bin_sort_items(uint32_t items, int n, const EmitViews& ev, int n_tiles, const float* proj_all,
                          const uint32_t* rect_all, const uint32_t* touched_all, uint32_t capacity,
                          uint64_t* keys, uint32_t* values, uint32_t* ranges, uint32_t* num_pairs,
                          uint32_t* flags, const BinWs& w, hipStream_t s, const char* who) {
    if (items == 0) {
        k_clear_u32<<<256, 256, 0, s>>>(ranges, 2u * (uint32_t)n_tiles);
        k_clear_u32<<<1, 64, 0, s>>>(num_pairs, 1u);
        PGS_CHECK_LAUNCH(who);
        return PGS_OK;
    }
    // few items: their whole depth order and offsets in one launch; else depth
    // keys with the first depth pass's histogram (and the clears of ranges and
    // pair count), the depth sort, whose last pass gathers tiles_touched into
    // depth order, and the scan.  The emit writes the pair sort's first
    // histogram, and its pairs where an odd number of passes will end in
    // (keys, values).
    const SortWs& iw = w.items_ws;
    const uint32_t n_ranges = 2u * (uint32_t)n_tiles;
    if (items <= kBlockSort) {
        k_depth_order<<<1, 1024, 0, s>>>(items, proj_all, touched_all, w.dkeys, w.dvals, w.off, ranges, n_ranges,
                                         num_pairs);
        PGS_CHECK_LAUNCH(who);
    } else {
        if (iw.small)
            k_depth_keys<SmallSort><<<iw.nb, SmallSort::kThreads, 0, s>>>(items, proj_all, touched_all, w.dkeys,
                                                                          w.dvals, w.count, iw.nb, iw.hist, ranges,
                                                                          n_ranges, num_pairs);
        else
            k_depth_keys<LargeSort><<<iw.nb, LargeSort::kThreads, 0, s>>>(items, proj_all, touched_all, w.dkeys,
                                                                          w.dvals, w.count, iw.nb, iw.hist, ranges,
                                                                          n_ranges, num_pairs);
        PGS_CHECK_LAUNCH(who);
        pgs_status st = radix_sort(w.dkeys, w.dvals, w.count, items, 32, iw, s, 0, true, touched_all, w.off);
        if (st != PGS_OK) return st;
        st = scan_u32(w.off, w.off, items, num_pairs, w.partial, s);
        if (st != PGS_OK) return st;
    }
    const SortWs& pw = w.pairs_ws;
    const int tile_bits = bits_for((uint32_t)n_tiles);
    const bool odd = (sort_passes(tile_bits) & 1) != 0;
    uint64_t* ekeys = odd ? pw.keys_alt : keys;
    uint32_t* evals = odd ? pw.vals_alt : values;
    const uint32_t ge = pw.nb > 0 ? pw.nb : 1u;
    if (pw.small)
        k_emit_sorted<SmallSort><<<ge, SmallSort::kThreads, 0, s>>>(items, n, ev, w.dkeys, rect_all, w.dvals, w.off,
                                                                    num_pairs, capacity, ekeys, evals, flags, pw.nb,
                                                                    pw.hist);
    else
        k_emit_sorted<LargeSort><<<ge, LargeSort::kThreads, 0, s>>>(items, n, ev, w.dkeys, rect_all, w.dvals, w.off,
                                                                    num_pairs, capacity, ekeys, evals, flags, pw.nb,
                                                                    pw.hist);
    PGS_CHECK_LAUNCH(who);
    if (capacity == 0) return PGS_OK;
    pgs_status st = radix_sort(keys, values, num_pairs, capacity, tile_bits, pw, s, 32, true, nullptr, nullptr, true);
    if (st != PGS_OK) return st;
    const uint32_t grid = div_up(capacity, 256) < 4096 ? div_up(capacity, 256) : 4096;
    k_ranges<<<grid, 256, 0, s>>>(keys, num_pairs, capacity, (uint32_t)n_tiles, ranges);
    PGS_CHECK_LAUNCH(who);
    return PGS_OK;
}

}  // namespace

extern "C" size_t pgs_bin_sort_workspace(int32_t n, uint32_t capacity) {
    return bin_layout(nullptr, n > 0 ? (uint32_t)n : 0u, capacity).bytes;
}

extern "C" pgs_status pgs_bin_sort(int32_t n, const float* proj_dev, const uint32_t* rect_dev,
                                   const uint32_t* touched_dev, int32_t tiles_x, int32_t n_tiles,
                                   int32_t view_tile_offset, uint32_t capacity, uint64_t* keys_dev,
                                   uint32_t* values_dev, uint32_t* ranges_dev, uint32_t* num_pairs_dev,
                                   uint32_t* flags_dev, void* workspace_dev, size_t workspace_bytes,
                                   void* stream) {
    PGS_REQUIRE(n >= 0 && tiles_x > 0 && n_tiles > 0 && view_tile_offset >= 0 &&
                    view_tile_offset < n_tiles, "pgs_bin_sort: bad sizes");
    PGS_REQUIRE(ranges_dev && num_pairs_dev && flags_dev, "pgs_bin_sort: null pointer");
    PGS_REQUIRE(n == 0 || (proj_dev && rect_dev && touched_dev), "pgs_bin_sort: null pointer");
    PGS_REQUIRE(capacity == 0 || (keys_dev && values_dev), "pgs_bin_sort: null pointer");
    const size_t need = pgs_bin_sort_workspace(n, capacity);
    PGS_REQUIRE(workspace_dev && workspace_bytes >= need, "pgs_bin_sort: workspace %zu < %zu",
                workspace_bytes, need);
    EmitViews ev{};
    ev.n_views = 1;
    ev.TX[0] = tiles_x;
    ev.tile_off[0] = view_tile_offset;
    const BinWs w = bin_layout(workspace_dev, (uint32_t)n, capacity);
    return bin_sort_items((uint32_t)n, n > 0 ? n : 1, ev, n_tiles, proj_dev, rect_dev, touched_dev, capacity,
                          keys_dev, values_dev, ranges_dev, num_pairs_dev, flags_dev, w, pgs::as_stream(stream),
                          "pgs_bin_sort");
}

extern "C" pgs_status pgs_bin_sort_views(const pgs_view_batch* views, int32_t n, const float* proj_all_dev,
                                         const uint32_t* rect_all_dev, const uint32_t* touched_all_dev,
                                         uint32_t capacity, uint64_t* keys_dev, uint32_t* values_dev,
                                         uint32_t* ranges_dev, uint32_t* num_pairs_dev, uint32_t* flags_dev,
                                         void* workspace_dev, size_t workspace_bytes, void* stream) {
    pgs_status st = pgs::check_views(views, "pgs_bin_sort_views");
    if (st != PGS_OK) return st;
    PGS_REQUIRE(n >= 0 && (int64_t)n * views->n_views < (1ll << 31), "pgs_bin_sort_views: bad n");
    PGS_REQUIRE(ranges_dev && num_pairs_dev && flags_dev, "pgs_bin_sort_views: null pointer");
    PGS_REQUIRE(n == 0 || (proj_all_dev && rect_all_dev && touched_all_dev), "pgs_bin_sort_views: null pointer");
    PGS_REQUIRE(capacity == 0 || (keys_dev && values_dev), "pgs_bin_sort_views: null pointer");
    const int32_t items = n * views->n_views;
    const size_t need = pgs_bin_sort_workspace(items, capacity);
    PGS_REQUIRE(workspace_dev && workspace_bytes >= need, "pgs_bin_sort_views: workspace %zu < %zu",
                workspace_bytes, need);
    const pgs::ViewsLayout lay = pgs::views_layout(*views);
    EmitViews ev{};
    ev.n_views = views->n_views;
    for (int v = 0; v < views->n_views; ++v) {
        ev.TX[v] = lay.TX[v];
        ev.tile_off[v] = lay.tile_off[v];
    }
    const BinWs w = bin_layout(workspace_dev, (uint32_t)items, capacity);
    return bin_sort_items((uint32_t)items, n > 0 ? n : 1, ev, lay.tile_off[views->n_views], proj_all_dev,
                          rect_all_dev, touched_all_dev, capacity, keys_dev, values_dev, ranges_dev, num_pairs_dev,
                          flags_dev, w, pgs::as_stream(stream), "pgs_bin_sort_views");
}
