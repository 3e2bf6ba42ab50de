// The gradient index of few keys by one workgroup (index.hip), here also as part of another launch (level.hip).
#pragma once
#include "common.h"

namespace ngdb {
namespace {

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;

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

// The whole index of at most SMALL_KEYS keys by one workgroup, keys and values in LDS: the same stable
// radix passes (rounds of 1024 keys), then the segment heads.
constexpr int SMALL_THREADS = 1024, SMALL_WAVES = SMALL_THREADS / 64;
struct SmallIndexLds {
    int32_t ks[2][SMALL_KEYS], vs[2][SMALL_KEYS];
    int32_t running[RADIX], wcnt[SMALL_WAVES][RADIX], wsum[SMALL_WAVES];
};
constexpr size_t SMALL_INDEX_LDS = sizeof(SmallIndexLds);
__device__ __forceinline__ void small_index(const SmallIndex& job, void* lds) {
    SmallIndexLds& L = *reinterpret_cast<SmallIndexLds*>(lds);
    auto& ks = L.ks; auto& vs = L.vs; auto& running = L.running; auto& wcnt = L.wcnt; auto& wsum = L.wsum;
    const int32_t *head = job.head, *tail = job.tail;
    const int n_head = job.n_head, n = job.n, bits = job.bits;
    int32_t *vals_out = job.vals_out, *uniq = job.uniq, *seg_off = job.seg_off, *n_uniq = job.n_uniq;
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

}  // namespace
}  // namespace ngdb
