// Device-side gradient index (Sec. 4.2 "Efficient Tensor Indexing"): the
// contributions to an embedding table -- anchors, positives, negatives -- are
// grouped by row id with a stable least-significant-digit radix sort, so that
// the scatter-add of the backward pass becomes one atomic-free segmented sum per
// touched row, in a fixed order.  Every pass is three kernels (per-tile digit
// histogram, exclusive scan of the digit-major histogram, stable scatter); no
// kernel contains a data-dependent wait.
//
// The build runs beside the forward pass and is bound by its launches, not by its bytes, until there are
// millions of keys.  Up to SMALL_KEYS keys one workgroup sorts everything in LDS (700 keys of the
// smallest workload: 14 launches and 32 us became one of 9 us); up to OWN_TILES tiles every workgroup of the
// scatter adds up the histogram for itself, and up to OWN_KEYS keys the segment heads before it too (five launches
// for two passes); up to MID_TILES tiles the histogram is
// scanned by one launch instead of three, each workgroup adding up what lies before its digit (at
// 66 000 keys 8 launches instead of 14); beyond that this would read the histogram too often.
#include "common.h"

namespace ngdb {
namespace {

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int SORT_THREADS = 256;
constexpr int SORT_ITEMS = 4;                        // keys per thread
constexpr int SORT_TILE = SORT_THREADS * SORT_ITEMS; // keys per workgroup
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

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
template <bool FIRST>
__global__ __launch_bounds__(SORT_THREADS) void hist_kernel(const KeySource<FIRST> src, int64_t n, int shift, int n_tiles,
                                                            int32_t* __restrict__ hist) {
    __shared__ int32_t h[RADIX];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SORT_TILE;
    for (int r = 0; r < SORT_ITEMS; ++r) {
        const int64_t i = base + (int64_t)r * SORT_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[(src.key(i) >> shift) & (RADIX - 1)], 1);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// ---- exclusive scan of int32 in three steps: tile sums, scan of the sums, tile scan
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* total) {
    __shared__ int32_t wsum[SCAN_THREADS / 64];
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
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
        if (w < wave) woff += wsum[w];
        tot += wsum[w];
    }
    *total = tot;
    return woff + inc - v;
}

template <bool HEADS>
__device__ __forceinline__ int32_t scan_input(const int32_t* __restrict__ in, int64_t i) {
    if (!HEADS) return in[i];
    return (i == 0 || in[i] != in[i - 1]) ? 1 : 0;   // segment head flag over sorted keys
}

template <bool HEADS>
__global__ __launch_bounds__(SCAN_THREADS) void scan_sums_kernel(const int32_t* __restrict__ in, int64_t n,
                                                                 int32_t* __restrict__ sums) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t s = 0;
    for (int k = 0; k < SCAN_ITEMS; ++k)
        if (base + k < n) s += scan_input<HEADS>(in, base + k);
    int32_t tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// one workgroup: exclusive scan of sums[0..m) in place, grand total to *total
__global__ __launch_bounds__(SCAN_THREADS) void scan_top_kernel(int32_t* __restrict__ sums, int m,
                                                                int32_t* __restrict__ total) {
    int32_t carry = 0;
    for (int base = 0; base < m; base += SCAN_THREADS) {
        const int i = base + threadIdx.x;
        const int32_t v = i < m ? sums[i] : 0;
        int32_t tot;
        const int32_t ex = block_exclusive_scan(v, &tot);
        if (i < m) sums[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total) total[0] = carry, total[1] = 0;
}

// HEADS=false: out[i] = exclusive prefix.  HEADS=true: for every head position i
// with rank u: uniq[u] = keys[i], seg_off[u] = i; the last workgroup closes seg_off.
template <bool HEADS>
__global__ __launch_bounds__(SCAN_THREADS) void scan_apply_kernel(const int32_t* __restrict__ in, int64_t n,
                                                                  const int32_t* __restrict__ sums,
                                                                  int32_t* __restrict__ out,
                                                                  int32_t* __restrict__ seg_off,
                                                                  const int32_t* __restrict__ total) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS];
    int32_t s = 0;
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        v[k] = base + k < n ? scan_input<HEADS>(in, base + k) : 0;
        s += v[k];
    }
    int32_t tot;
    int32_t run = sums[blockIdx.x] + block_exclusive_scan(s, &tot);
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        if (base + k < n) {
            if (!HEADS) {
                out[base + k] = run;
            } else if (v[k]) {
                out[run] = in[base + k];
                seg_off[run] = (int32_t)(base + k);
            }
        }
        run += v[k];
    }
    if (HEADS && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) seg_off[*total] = (int32_t)n;
}

// Exclusive scan of a short digit-major histogram in one launch: workgroup `digit` adds up the rows before its own
// and scans its own (n_tiles <= MID_TILES <= SCAN_THREADS), out of place.
constexpr int MID_TILES = 256;
__global__ __launch_bounds__(SCAN_THREADS) void scan_rows_kernel(const int32_t* __restrict__ hist, int n_tiles,
                                                                 int32_t* __restrict__ offs) {
    const int digit = blockIdx.x, t = threadIdx.x;
    // 16 bytes a lane, eight loads on the way (one 4-byte load after the other: 18 us at 66 tiles, 33 at 128)
    int32_t before = 0;
    const int n_before = digit * n_tiles, n4 = n_before >> 2;
    const int4* h4 = reinterpret_cast<const int4*>(hist);
    for (int i = t; i < n4; i += 8 * SCAN_THREADS) {
        int4 x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = h4[min(i + j * SCAN_THREADS, n4 - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j) before += i + j * SCAN_THREADS < n4 ? (x[j].x + x[j].y) + (x[j].z + x[j].w) : 0;
    }
    if (t < (n_before & 3)) before += hist[n4 * 4 + t];
    int32_t base, row;
    block_exclusive_scan(before, &base);
    const int32_t v = t < n_tiles ? hist[(size_t)digit * n_tiles + t] : 0;
    const int32_t ex = block_exclusive_scan(v, &row);
    if (t < n_tiles) offs[(size_t)digit * n_tiles + t] = base + ex;
}

// Segment heads of a short sorted array in one launch after the tile sums: like scan_apply_kernel<true>, each workgroup
// adding up the sums of the tiles before it (at most MID_TILES of them).
// OWN: without sums, each counting the heads before it (at most OWN_KEYS keys).
constexpr int OWN_KEYS = 16384;
template <bool OWN>
__global__ __launch_bounds__(SCAN_THREADS) void heads_kernel(const int32_t* __restrict__ keys, int64_t n,
                                                             const int32_t* __restrict__ sums, int32_t* __restrict__ uniq,
                                                             int32_t* __restrict__ seg_off, int32_t* __restrict__ n_uniq) {
    int32_t base, all, tot;
    int32_t mine = 0;
    if (OWN) {
        const int n4 = (int)blockIdx.x * (SCAN_TILE / 4);
        for (int i0 = threadIdx.x; i0 < n4; i0 += 4 * SCAN_THREADS) {
            int4 k[4];
            int32_t last[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = min(i0 + j * SCAN_THREADS, n4 - 1);
                k[j] = reinterpret_cast<const int4*>(keys)[i];
                last[j] = keys[max(4 * i - 1, 0)];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + j * SCAN_THREADS;
                if (i >= n4) break;
                mine += (i == 0 || k[j].x != last[j] ? 1 : 0) + (k[j].y != k[j].x ? 1 : 0) + (k[j].z != k[j].y ? 1 : 0) + (k[j].w != k[j].z ? 1 : 0);
            }
        }
    } else {
        mine = (int)threadIdx.x < (int)blockIdx.x ? sums[threadIdx.x] : 0;
    }
    block_exclusive_scan(mine, &base);
    const int64_t first = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS], s = 0;
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        v[k] = first + k < n ? scan_input<true>(keys, first + k) : 0;
        s += v[k];
    }
    int32_t run = base + block_exclusive_scan(s, &tot);
    for (int k = 0; k < SCAN_ITEMS; ++k)
        if (v[k]) {
            uniq[run] = keys[first + k];
            seg_off[run++] = (int32_t)(first + k);
        }
    all = base + tot;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        seg_off[all] = (int32_t)n;
        n_uniq[0] = all;
        n_uniq[1] = 0;
    }
}

// Lanes of the wavefront that hold a valid key with the lane's digit
__device__ __forceinline__ unsigned long long digit_peers(bool valid, int digit) {
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < RADIX_BITS; ++b) {
        const unsigned long long bal = __ballot((digit >> b) & 1);
        peers &= ((digit >> b) & 1) ? bal : ~bal;
    }
    return peers;
}

// Stable scatter of one radix pass.  The tile is walked in rounds of 256
// consecutive keys (thread t takes key round*256 + t), so the order inside the
// tile is (round, wavefront, lane); the rank of a key among equal digits is
// running count of earlier rounds + counts of lower wavefronts + lower lanes.
// OWN: offs is the histogram itself (at most OWN_TILES tiles), scanned by every workgroup.
constexpr int OWN_TILES = 32;
template <bool FIRST, bool OWN>
__global__ __launch_bounds__(SORT_THREADS) void scatter_kernel(const KeySource<FIRST> src, int64_t n, int shift, int n_tiles,
                                                               const int32_t* __restrict__ offs,
                                                               int32_t* __restrict__ keys_out,
                                                               int32_t* __restrict__ vals_out) {
    __shared__ int32_t running[RADIX];                    // global position of the next key per digit
    __shared__ int32_t wcnt[SORT_THREADS / 64][RADIX];    // per wavefront counts of the current round
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (OWN) {
        int32_t before = 0, total = 0, all;
#pragma unroll
        for (int i0 = 0; i0 < OWN_TILES; i0 += 8) {
            if (i0 >= n_tiles) break;
            int32_t x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = offs[threadIdx.x * n_tiles + min(i0 + i, n_tiles - 1)];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                before += i0 + i < (int)blockIdx.x ? x[i] : 0;
                total += i0 + i < n_tiles ? x[i] : 0;
            }
        }
        running[threadIdx.x] = block_exclusive_scan(total, &all) + before;
    } else {
        running[threadIdx.x] = offs[(size_t)threadIdx.x * n_tiles + blockIdx.x];
    }
    for (int w = 0; w < SORT_THREADS / 64; ++w) wcnt[w][threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SORT_TILE;
    int32_t key[SORT_ITEMS], val[SORT_ITEMS];
#pragma unroll
    for (int r = 0; r < SORT_ITEMS; ++r) {
        const int64_t i = base + (int64_t)r * SORT_THREADS + threadIdx.x;
        key[r] = i < n ? src.key(i) : 0;
        val[r] = i < n ? src.val(i) : 0;
    }
#pragma unroll
    for (int r = 0; r < SORT_ITEMS; ++r) {
        const int64_t i = base + (int64_t)r * SORT_THREADS + threadIdx.x;
        const bool valid = i < n;
        const int digit = (key[r] >> shift) & (RADIX - 1);
        const unsigned long long peers = digit_peers(valid, digit);
        const unsigned long long lower = peers & ((1ull << lane) - 1ull);
        const int rank_in_wave = __popcll(lower);
        if (valid && lower == 0ull) wcnt[wave][digit] = __popcll(peers);   // one writer per digit
        __syncthreads();
        int32_t pos = 0;
        if (valid) {
            pos = running[digit] + rank_in_wave;
            for (int w = 0; w < wave; ++w) pos += wcnt[w][digit];
        }
        __syncthreads();
        {   // thread t owns digit t: advance the running position, clear the round's counts
            int32_t add = 0;
            for (int w = 0; w < SORT_THREADS / 64; ++w) {
                add += wcnt[w][threadIdx.x];
                wcnt[w][threadIdx.x] = 0;
            }
            running[threadIdx.x] += add;
        }
        if (valid) {
            keys_out[pos] = key[r];
            vals_out[pos] = val[r];
        }
        __syncthreads();
    }
}

// The whole index of at most SMALL_KEYS keys by one workgroup, keys and values in LDS: the same stable
// radix passes (rounds of 1024 keys), then the segment heads.
constexpr int SMALL_KEYS = 4096, SMALL_THREADS = 1024, SMALL_WAVES = SMALL_THREADS / 64;
__global__ __launch_bounds__(SMALL_THREADS) void small_index_kernel(const int32_t* __restrict__ head, int n_head,
                                                                    const int32_t* __restrict__ tail, int n, int bits,
                                                                    int32_t* __restrict__ vals_out, int32_t* __restrict__ uniq,
                                                                    int32_t* __restrict__ seg_off, int32_t* __restrict__ n_uniq) {
    __shared__ int32_t ks[2][SMALL_KEYS], vs[2][SMALL_KEYS];
    __shared__ int32_t running[RADIX], wcnt[SMALL_WAVES][RADIX], wsum[SMALL_WAVES];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int i = t; i < n; i += SMALL_THREADS) {
        ks[0][i] = i < n_head ? head[i] : tail[i - n_head];
        vs[0][i] = i;
    }
    int cur = 0;
    for (int shift = 0; shift < bits; shift += RADIX_BITS) {
        if (t < RADIX) running[t] = 0;
        for (int i = t; i < SMALL_WAVES * RADIX; i += SMALL_THREADS) (&wcnt[0][0])[i] = 0;
        __syncthreads();
        for (int i = t; i < n; i += SMALL_THREADS) atomicAdd(&running[(ks[cur][i] >> shift) & (RADIX - 1)], 1);
        __syncthreads();
        if (wave == 0) {          // exclusive scan of the 256 counts, four per lane
            int32_t c[4], sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                c[j] = running[lane * 4 + j];
                sum += c[j];
            }
            int32_t inc = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int32_t v = __shfl_up(inc, off, 64);
                if (lane >= off) inc += v;
            }
            int32_t run = inc - sum;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                running[lane * 4 + j] = run;
                run += c[j];
            }
        }
        __syncthreads();
        for (int base = 0; base < n; base += SMALL_THREADS) {
            const int i = base + t;
            const bool valid = i < n;
            const int32_t key = valid ? ks[cur][i] : 0, val = valid ? vs[cur][i] : 0;
            const int digit = (key >> shift) & (RADIX - 1);
            const unsigned long long peers = digit_peers(valid, digit);
            const unsigned long long lower = peers & ((1ull << lane) - 1ull);
            if (valid && lower == 0ull) wcnt[wave][digit] = __popcll(peers);
            __syncthreads();
            if (t < RADIX) {      // counts of a digit -> its position in every wavefront
                int32_t run = running[t];
                for (int w = 0; w < SMALL_WAVES; ++w) {
                    const int32_t c = wcnt[w][t];
                    wcnt[w][t] = run;
                    run += c;
                }
                running[t] = run;
            }
            __syncthreads();
            if (valid) {
                const int pos = wcnt[wave][digit] + __popcll(lower);
                ks[cur ^ 1][pos] = key;
                vs[cur ^ 1][pos] = val;
            }
            __syncthreads();
            for (int x = t; x < SMALL_WAVES * RADIX; x += SMALL_THREADS) (&wcnt[0][0])[x] = 0;
            __syncthreads();
        }
        cur ^= 1;
    }
    int32_t done = 0;             // heads before the round (the same in all threads)
    for (int base = 0; base < n; base += SMALL_THREADS) {
        const int i = base + t;
        const bool valid = i < n;
        const bool is_head = valid && (i == 0 || ks[cur][i] != ks[cur][i - 1]);
        const unsigned long long m = __ballot(is_head);
        __syncthreads();
        if (lane == 0) wsum[wave] = __popcll(m);
        __syncthreads();
        int32_t at = done + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int w = 0; w < SMALL_WAVES; ++w) {
            at += w < wave ? wsum[w] : 0;
            done += wsum[w];
        }
        if (is_head) {
            uniq[at] = ks[cur][i];
            seg_off[at] = i;
        }
        if (valid) vals_out[i] = vs[cur][i];
    }
    if (t == 0) {
        seg_off[done] = n;
        n_uniq[0] = done;
        n_uniq[1] = 0;
    }
}

inline int tiles_of(int64_t n, int tile) { return (int)((n + tile - 1) / tile); }

// exclusive scan of in[0..n) into out (may alias), scratch `sums` of ceil(n/SCAN_TILE) ints
hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* sums, hipStream_t s) {
    const int nt = tiles_of(n, SCAN_TILE);
    hipLaunchKernelGGL((scan_sums_kernel<false>), dim3(nt), dim3(SCAN_THREADS), 0, s, in, n, sums);
    hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, sums, nt, (int32_t*)nullptr);
    hipLaunchKernelGGL((scan_apply_kernel<false>), dim3(nt), dim3(SCAN_THREADS), 0, s, in, n,
                       (const int32_t*)sums, out, (int32_t*)nullptr, (const int32_t*)nullptr);
    return hipGetLastError();
}

}  // namespace

size_t index_hist_elems(int64_t n_keys) {
    const size_t tiles = tiles_of(std::max<int64_t>(n_keys, 1), SORT_TILE);
    return (size_t)RADIX * std::max(tiles, 2 * std::min<size_t>(tiles, MID_TILES));     // (the short scan is out of place)
}

size_t index_scan_tmp_elems(int64_t n_keys) {
    const int64_t a = tiles_of((int64_t)index_hist_elems(n_keys), SCAN_TILE);
    const int64_t b = tiles_of(std::max<int64_t>(n_keys, 1), SCAN_TILE);
    return (size_t)std::max(a, b) + 1;
}

hipError_t build_segment_index(const int32_t* head, int n_head, const int32_t* tail, int64_t n_tail,
                               int32_t key_bound, const IndexBuffers& buf, int32_t** src_out, hipStream_t s) {
    const int64_t n = (int64_t)n_head + n_tail;
    if (n <= 0) {
        // empty index: n_uniq = 0, seg_off[0] = 0
        hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, buf.seg_off, 0, buf.n_uniq);
        hipLaunchKernelGGL((scan_apply_kernel<true>), dim3(1), dim3(SCAN_THREADS), 0, s,
                           (const int32_t*)buf.keys_a, (int64_t)0, (const int32_t*)buf.scan_tmp, buf.uniq,
                           buf.seg_off, (const int32_t*)buf.n_uniq);
        *src_out = buf.vals_a;
        return hipGetLastError();
    }
    int bits = 1;
    while (bits < 31 && (1ll << bits) < (long long)key_bound) ++bits;
    if (n <= SMALL_KEYS) {
        hipLaunchKernelGGL(small_index_kernel, dim3(1), dim3(SMALL_THREADS), 0, s, head, n_head, tail, (int)n, bits, buf.vals_a,
                           buf.uniq, buf.seg_off, buf.n_uniq);
        *src_out = buf.vals_a;
        return hipGetLastError();
    }
    const int n_tiles = tiles_of(n, SORT_TILE);
    const bool own = n_tiles <= OWN_TILES, mid = !own && n_tiles <= MID_TILES;
    int32_t* offs = mid ? buf.hist + (size_t)RADIX * n_tiles : buf.hist;
    int32_t *kin = buf.keys_a, *kout = buf.keys_b, *vin = buf.vals_a, *vout = buf.vals_b;
    for (int shift = 0; shift < bits; shift += RADIX_BITS) {
        const KeySource<true> first{head, tail, n_head};
        const KeySource<false> sorted{kin, vin, 0};
        if (shift == 0)
            hipLaunchKernelGGL((hist_kernel<true>), dim3(n_tiles), dim3(SORT_THREADS), 0, s, first, n, shift, n_tiles, buf.hist);
        else
            hipLaunchKernelGGL((hist_kernel<false>), dim3(n_tiles), dim3(SORT_THREADS), 0, s, sorted, n, shift, n_tiles, buf.hist);
        if (own) {
        } else if (mid) {
            hipLaunchKernelGGL(scan_rows_kernel, dim3(RADIX), dim3(SCAN_THREADS), 0, s, (const int32_t*)buf.hist, n_tiles, offs);
        } else {
            hipError_t e = scan_exclusive(buf.hist, buf.hist, (int64_t)RADIX * n_tiles, buf.scan_tmp, s);
            if (e != hipSuccess) return e;
        }
#define NGDB_SCATTER(FIRST, OWN, SRC)                                                                                                  \
    hipLaunchKernelGGL((scatter_kernel<FIRST, OWN>), dim3(n_tiles), dim3(SORT_THREADS), 0, s, SRC, n, shift, n_tiles, (const int32_t*)offs, kout, vout)
        if (shift == 0 && own) NGDB_SCATTER(true, true, first);
        else if (shift == 0) NGDB_SCATTER(true, false, first);
        else if (own) NGDB_SCATTER(false, true, sorted);
        else NGDB_SCATTER(false, false, sorted);
#undef NGDB_SCATTER
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    // segment heads over the sorted keys
    const int nt = tiles_of(n, SCAN_TILE);
    if (n <= OWN_KEYS) {
        hipLaunchKernelGGL((heads_kernel<true>), dim3(nt), dim3(SCAN_THREADS), 0, s, (const int32_t*)kin, n, (const int32_t*)nullptr, buf.uniq,
                           buf.seg_off, buf.n_uniq);
        *src_out = vin;
        return hipGetLastError();
    }
    hipLaunchKernelGGL((scan_sums_kernel<true>), dim3(nt), dim3(SCAN_THREADS), 0, s, (const int32_t*)kin, n,
                       buf.scan_tmp);
    if (nt <= MID_TILES) {
        hipLaunchKernelGGL((heads_kernel<false>), dim3(nt), dim3(SCAN_THREADS), 0, s, (const int32_t*)kin, n, (const int32_t*)buf.scan_tmp,
                           buf.uniq, buf.seg_off, buf.n_uniq);
    } else {
        hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, buf.scan_tmp, nt, buf.n_uniq);
        hipLaunchKernelGGL((scan_apply_kernel<true>), dim3(nt), dim3(SCAN_THREADS), 0, s, (const int32_t*)kin, n,
                           (const int32_t*)buf.scan_tmp, buf.uniq, buf.seg_off, (const int32_t*)buf.n_uniq);
    }
    *src_out = vin;
    return hipGetLastError();
}

}  // namespace ngdb
