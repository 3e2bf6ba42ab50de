// Device-side gradient index (Sec. 4.2 "Efficient Tensor Indexing"): the
// contributions to an embedding table -- anchors, positives, negatives -- are
// grouped by row id with a stable least-significant-digit radix sort, so that
// the scatter-add of the backward pass becomes one atomic-free segmented sum per
// touched row, in a fixed order.  A pass counts the digits of every tile and
// scatters the tiles, whose places a scan of these counts gives; no kernel
// contains a data-dependent wait.
//
// The build runs beside the forward pass and is bound by its launches, not by its bytes, until there are
// millions of keys.  Up to SMALL_KEYS keys one workgroup sorts everything in LDS (700 keys of the
// smallest workload: 14 launches and 32 us became one of 9 us; in small models a launch of the forward pass takes it along); up to OWN_TILES tiles every workgroup of the
// scatter adds up the counts for itself, and up to OWN_KEYS keys the segment heads before it too (five launches
// for two passes); beyond, a launch scans the tiles of every digit.
// A tile is put in order in LDS and leaves as runs of equal digits: written from where the keys lie, four bytes at a time all over
// the output, a pass over 4.2 million keys took 80 to 90 us, in this way 30 to 40, beside the forward pass (the whole build 460 -> 210 us).
#include <algorithm>
#include <type_traits>
#include "small_index.h"

namespace ngdb {
namespace {

constexpr int SORT_THREADS = 512, SORT_WAVES = SORT_THREADS / 64;
// Keys of a thread; a tile is SORT_THREADS x ITEMS keys, SORT_WAVES pieces of ITEMS rounds of 64 in their order.
constexpr int FEW_ITEMS = 4, MID_ITEMS = 8, MANY_ITEMS = 16;
constexpr int OWN_TILES = 64;            // most tiles whose counts a workgroup adds up for itself
constexpr int64_t FEW_KEYS = 80000, MID_KEYS = (int64_t)OWN_TILES * SORT_THREADS * MID_ITEMS;
static_assert((FEW_KEYS + SORT_THREADS * FEW_ITEMS - 1) / (SORT_THREADS * FEW_ITEMS) <= OWN_TILES, "short arrays have few tiles");
constexpr int64_t OWN_KEYS = FEW_KEYS;   // most keys whose heads a workgroup counts for itself
inline int items_of(int64_t n) { return n <= FEW_KEYS ? FEW_ITEMS : n <= MID_KEYS ? MID_ITEMS : MANY_ITEMS; }
inline int tiles_of(int64_t n) {
    const int64_t tile = (int64_t)SORT_THREADS * items_of(n);
    return (int)((n + tile - 1) / tile);
}

// The keys of a pass: the sorted ones of the pass before, or (FIRST) head and tail one after the other, the
// value then being the position.
template <bool FIRST>
struct KeySource {
    const int32_t *keys, *vals;       // FIRST: head, tail
    int n_head;
    __device__ __forceinline__ int32_t key(int64_t i) const {
        if (FIRST) return i < n_head ? keys[i] : vals[i - n_head];
        return keys[i];
    }
    __device__ __forceinline__ int32_t val(int64_t i) const { return FIRST ? (int32_t)i : vals[i]; }
};

// hist[digit * n_tiles + tile] = number of keys of the tile with that digit
template <bool FIRST, int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void hist_kernel(const KeySource<FIRST> src, int64_t n, int shift, int n_tiles,
                                                            int32_t* __restrict__ hist) {
    __shared__ int32_t h[RADIX];
    const int64_t base = (int64_t)blockIdx.x * (SORT_THREADS * ITEMS) + threadIdx.x;
    int32_t key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = src.key(min(base + r * SORT_THREADS, n - 1));
    if (threadIdx.x < RADIX) h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (base + r * SORT_THREADS < n) atomicAdd(&h[(key[r] >> shift) & (RADIX - 1)], 1);
    __syncthreads();
    if (threadIdx.x < RADIX) hist[(size_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// exclusive scan over the threads of a workgroup of WAVES wavefronts, *total the sum
template <int WAVES>
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* total) {
    __shared__ int32_t wsum[WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t t = __shfl_up(inc, off, 64);
        if (lane >= off) inc += t;
    }
    __syncthreads();                      // wsum may still be read from a previous call
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t woff = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) woff += wsum[w];
        tot += wsum[w];
    }
    *total = tot;
    return woff + inc - v;
}

// Exclusive scan of every digit's row of hist, in place, its sum to totals: a workgroup a digit.
__global__ __launch_bounds__(256) void scan_rows_kernel(int32_t* __restrict__ hist, int n_tiles, int32_t* __restrict__ totals) {
    int32_t* row = hist + (size_t)blockIdx.x * n_tiles;
    int32_t carry = 0;
    for (int base = 0; base < n_tiles; base += 1024) {
        int32_t x[4], sum = 0, all;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = base + (int)threadIdx.x * 4 + j;
            x[j] = i < n_tiles ? row[i] : 0;
            sum += x[j];
        }
        int32_t run = carry + block_exclusive_scan<4>(sum, &all);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = base + (int)threadIdx.x * 4 + j;
            if (i < n_tiles) row[i] = run;
            run += x[j];
        }
        carry += all;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// The heads of a tile's segments: bit l of heads[r] = key r * 64 + l of this wavefront's piece starts one.
template <int ITEMS>
__device__ __forceinline__ int32_t tile_heads(const int32_t* __restrict__ keys, int64_t n, int64_t piece, int32_t (&key)[ITEMS],
                                              unsigned long long (&heads)[ITEMS]) {
    const int lane = threadIdx.x & 63;
    int32_t last = keys[max((int64_t)0, min(piece, n) - 1)], count = 0;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) key[r] = keys[min(piece + r * 64 + lane, n - 1)];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t i = piece + r * 64 + lane;
        int32_t before = __shfl_up(key[r], 1, 64);
        if (lane == 0) before = last;
        last = lane_value(key[r], 63);
        heads[r] = __ballot(i < n && (i == 0 || key[r] != before));
        count += __popcll(heads[r]);
    }
    return count;
}

// sums[tile] = number of its heads
template <int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void head_sums_kernel(const int32_t* __restrict__ keys, int64_t n, int32_t* __restrict__ sums) {
    __shared__ int32_t wsum[SORT_WAVES];
    const int wave = threadIdx.x >> 6;
    int32_t key[ITEMS];
    unsigned long long heads[ITEMS];
    const int32_t count = tile_heads<ITEMS>(keys, n, ((int64_t)blockIdx.x * SORT_WAVES + wave) * (64 * ITEMS), key, heads);
    if ((threadIdx.x & 63) == 0) wsum[wave] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t all = 0;
        for (int w = 0; w < SORT_WAVES; ++w) all += wsum[w];
        sums[blockIdx.x] = all;
    }
}

// For every head i with rank u: uniq[u] = keys[i], seg_off[u] = i; the last workgroup closes seg_off.  A workgroup adds up the
// sums of the tiles before its own.  OWN: without sums, each counting the heads before it (at most OWN_KEYS keys).
template <bool OWN, int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void heads_kernel(const int32_t* __restrict__ keys, int64_t n,
                                                             const int32_t* __restrict__ sums, int32_t* __restrict__ uniq,
                                                             int32_t* __restrict__ seg_off, int32_t* __restrict__ n_uniq) {
    __shared__ int32_t wsum[SORT_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t piece = ((int64_t)blockIdx.x * SORT_WAVES + wave) * (64 * ITEMS);
    int32_t key[ITEMS], mine = 0, base;
    unsigned long long heads[ITEMS];
    const int32_t count = tile_heads<ITEMS>(keys, n, piece, key, heads);
    if (OWN) {
        // (16 bytes a lane, eight requests on the way; the key before a group of four by a request of its own)
        const int n4 = (int)blockIdx.x * (SORT_THREADS * ITEMS / 4);
        for (int i0 = threadIdx.x; i0 < n4; i0 += 8 * SORT_THREADS) {
            int4 k[8];
            int32_t last[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = min(i0 + j * SORT_THREADS, n4 - 1);
                k[j] = reinterpret_cast<const int4*>(keys)[i];
                last[j] = keys[max(4 * i - 1, 0)];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = i0 + j * SORT_THREADS;
                if (i < n4)
                    mine += (i == 0 || k[j].x != last[j] ? 1 : 0) + (k[j].y != k[j].x ? 1 : 0) + (k[j].z != k[j].y ? 1 : 0) + (k[j].w != k[j].z ? 1 : 0);
            }
        }
    } else {
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += SORT_THREADS) mine += sums[i];
    }
    block_exclusive_scan<SORT_WAVES>(mine, &base);
    if (lane == 0) wsum[wave] = count;
    __syncthreads();
    int32_t run = base, all = base;
#pragma unroll
    for (int w = 0; w < SORT_WAVES; ++w) {
        run += w < wave ? wsum[w] : 0;
        all += wsum[w];
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if ((heads[r] >> lane) & 1) {
            const int32_t u = run + __popcll(heads[r] & ((1ull << lane) - 1ull));
            uniq[u] = key[r];
            seg_off[u] = (int32_t)(piece + r * 64 + lane);
        }
        run += __popcll(heads[r]);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        seg_off[all] = (int32_t)n;
        n_uniq[0] = all;
        n_uniq[1] = 0;
    }
}

__global__ void no_segments_kernel(int32_t* __restrict__ seg_off, int32_t* __restrict__ n_uniq) { seg_off[0] = n_uniq[0] = n_uniq[1] = 0; }

// Stable scatter of one radix pass.  Every wavefront walks its piece of the tile in rounds of 64 keys and counts the digits of its own
// as it goes: a key's place among equal digits is the count so far + the lower lanes of the round.  With the counts of the
// wavefronts before it and of the smaller digits that is its place in the tile, where it is put in LDS; the tile is then written from
// there, neighbours next to one another.
// OWN: offs is the histogram itself (at most OWN_TILES tiles), scanned by every workgroup; else the scan of its rows and totals.
template <bool FIRST, bool OWN, int ITEMS>
__global__ __launch_bounds__(SORT_THREADS) void scatter_kernel(const KeySource<FIRST> src, int64_t n, int shift, int n_tiles,
                                                               const int32_t* __restrict__ offs, const int32_t* __restrict__ totals,
                                                               int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out) {
    constexpr int TILE = SORT_THREADS * ITEMS;
    __shared__ int32_t sk[TILE], sv[TILE];
    __shared__ int32_t cnt[SORT_WAVES][RADIX];            // of a wavefront; then the place of its first key of the digit in the tile
    __shared__ int32_t to[RADIX];                         // what is added to a place in the tile
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * TILE, piece = base + wave * (64 * ITEMS);
    int32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t i = min(piece + r * 64 + lane, n - 1);
        key[r] = src.key(i);
        val[r] = src.val(i);
    }
    // of digit t: keys of all tiles and of those before this one
    int32_t before = 0, total = 0, all;
    if (OWN) {
        if (t < RADIX)
#pragma unroll
            for (int i0 = 0; i0 < OWN_TILES; i0 += 8) {
                if (i0 >= n_tiles) break;
                int32_t x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = offs[t * n_tiles + min(i0 + i, n_tiles - 1)];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    before += i0 + i < (int)blockIdx.x ? x[i] : 0;
                    total += i0 + i < n_tiles ? x[i] : 0;
                }
            }
    } else if (t < RADIX) {
        before = offs[(size_t)t * n_tiles + blockIdx.x];
        total = totals[t];
    }
    for (int i = t; i < SORT_WAVES * RADIX; i += SORT_THREADS) (&cnt[0][0])[i] = 0;
    const int32_t global = block_exclusive_scan<SORT_WAVES>(total, &all) + before;     // (behind its barriers the counts are zero)
    volatile int32_t* mine = cnt[wave];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = piece + r * 64 + lane < n;
        const int digit = (key[r] >> shift) & (RADIX - 1);
        const unsigned long long peers = digit_peers(valid, digit), lower = peers & ((1ull << lane) - 1ull);
        const int32_t so_far = mine[digit];               // (the LDS operations of a wavefront stay in order)
        rank[r] = so_far + __popcll(lower);
        if (valid && lower == 0ull) mine[digit] = so_far + __popcll(peers);      // one writer per digit
    }
    __syncthreads();
    int32_t here = 0;
    if (t < RADIX) {
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) {
            const int32_t c = cnt[w][t];
            cnt[w][t] = here;
            here += c;
        }
    }
    const int32_t first = block_exclusive_scan<SORT_WAVES>(here, &all);
    if (t < RADIX) {
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) cnt[w][t] += first;
        to[t] = global - first;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (piece + r * 64 + lane < n) {
            const int32_t at = cnt[wave][(key[r] >> shift) & (RADIX - 1)] + rank[r];
            sk[at] = key[r];
            sv[at] = val[r];
        }
    __syncthreads();
    const int count = (int)min((int64_t)TILE, n - base);
    for (int i = t; i < count; i += SORT_THREADS) {
        const int32_t k = sk[i], pos = to[(k >> shift) & (RADIX - 1)] + i;
        keys_out[pos] = k;
        vals_out[pos] = sv[i];
    }
}

__global__ __launch_bounds__(SMALL_THREADS) void small_index_kernel(const SmallIndex job) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[SMALL_INDEX_LDS];
    small_index(job, lds);
}

// launches of ITEMS keys a thread
template <int ITEMS>
hipError_t build_tiled(const int32_t* head, int n_head, const int32_t* tail, int64_t n, int bits, const IndexBuffers& buf, int32_t** src_out,
                       hipStream_t s) {
    const int n_tiles = tiles_of(n);
    const bool own = n_tiles <= OWN_TILES;
    int32_t* totals = buf.hist + (size_t)RADIX * n_tiles;
    int32_t *kin = buf.keys_a, *kout = buf.keys_b, *vin = buf.vals_a, *vout = buf.vals_b;
    const dim3 grid(n_tiles), block(SORT_THREADS);
    auto pass = [&](auto src, int shift) {
        constexpr bool FIRST = std::is_same<decltype(src), KeySource<true>>::value;
        hipLaunchKernelGGL((hist_kernel<FIRST, ITEMS>), grid, block, 0, s, src, n, shift, n_tiles, buf.hist);
        if (own) {
            hipLaunchKernelGGL((scatter_kernel<FIRST, true, ITEMS>), grid, block, 0, s, src, n, shift, n_tiles, (const int32_t*)buf.hist,
                               (const int32_t*)nullptr, kout, vout);
        } else {
            hipLaunchKernelGGL(scan_rows_kernel, dim3(RADIX), dim3(256), 0, s, buf.hist, n_tiles, totals);
            hipLaunchKernelGGL((scatter_kernel<FIRST, false, ITEMS>), grid, block, 0, s, src, n, shift, n_tiles, (const int32_t*)buf.hist,
                               (const int32_t*)totals, kout, vout);
        }
        std::swap(kin, kout);
        std::swap(vin, vout);
    };
    pass(KeySource<true>{head, tail, n_head}, 0);
    for (int shift = RADIX_BITS; shift < bits; shift += RADIX_BITS) pass(KeySource<false>{kin, vin, 0}, shift);
    *src_out = vin;
    // segment heads over the sorted keys
    if (n <= OWN_KEYS) {
        hipLaunchKernelGGL((heads_kernel<true, ITEMS>), grid, block, 0, s, (const int32_t*)kin, n, (const int32_t*)nullptr, buf.uniq, buf.seg_off,
                           buf.n_uniq);
    } else {
        hipLaunchKernelGGL((head_sums_kernel<ITEMS>), grid, block, 0, s, (const int32_t*)kin, n, buf.scan_tmp);
        hipLaunchKernelGGL((heads_kernel<false, ITEMS>), grid, block, 0, s, (const int32_t*)kin, n, (const int32_t*)buf.scan_tmp, buf.uniq,
                           buf.seg_off, buf.n_uniq);
    }
    return hipGetLastError();
}

}  // namespace

// (shorter arrays may have more tiles, but at most OWN_TILES)
size_t index_scan_tmp_elems(int64_t n_keys) { return (size_t)std::max(OWN_TILES, tiles_of(std::max<int64_t>(n_keys, 1))); }
size_t index_hist_elems(int64_t n_keys) { return RADIX * (index_scan_tmp_elems(n_keys) + 1); }

inline int bits_below(int32_t bound) {
    int bits = 1;
    while (bits < 31 && (1ll << bits) < (long long)bound) ++bits;
    return bits;
}
bool small_index_job(const int32_t* head, int n_head, const int32_t* tail, int64_t n_tail, int32_t key_bound, const IndexBuffers& buf, SmallIndex* job) {
    const int64_t n = (int64_t)n_head + n_tail;
    if (n <= 0 || n > SMALL_KEYS) return false;
    *job = SmallIndex{head, tail, n_head, (int)n, bits_below(key_bound), buf.vals_a, buf.uniq, buf.seg_off, buf.n_uniq};
    return true;
}

hipError_t build_segment_index(const int32_t* head, int n_head, const int32_t* tail, int64_t n_tail,
                               int32_t key_bound, const IndexBuffers& buf, int32_t** src_out, hipStream_t s) {
    const int64_t n = (int64_t)n_head + n_tail;
    if (n <= 0) {
        hipLaunchKernelGGL(no_segments_kernel, dim3(1), dim3(1), 0, s, buf.seg_off, buf.n_uniq);
        *src_out = buf.vals_a;
        return hipGetLastError();
    }
    SmallIndex job;
    if (small_index_job(head, n_head, tail, n_tail, key_bound, buf, &job)) {
        hipLaunchKernelGGL(small_index_kernel, dim3(1), dim3(SMALL_THREADS), 0, s, job);
        *src_out = buf.vals_a;
        return hipGetLastError();
    }
    const int bits = bits_below(key_bound);
    switch (items_of(n)) {
        case FEW_ITEMS: return build_tiled<FEW_ITEMS>(head, n_head, tail, n, bits, buf, src_out, s);
        case MID_ITEMS: return build_tiled<MID_ITEMS>(head, n_head, tail, n, bits, buf, src_out, s);
        default: return build_tiled<MANY_ITEMS>(head, n_head, tail, n, bits, buf, src_out, s);
    }
}

}  // namespace ngdb
