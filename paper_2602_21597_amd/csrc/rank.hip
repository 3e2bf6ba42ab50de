// All-entity ranking (Sec. 3.2: answer a query by ranking every entity by
// f(q,e) = gamma - min_b ||y_b - E[e]||_1): L1 distances of every branch
// embedding to a chunk of entity rows, then a running top-k per query.
//
// The distance pass is bound by plain vector arithmetic (two VALU operations per
// coordinate: subtract, add-absolute; an L1 distance is not a contraction, so the
// matrix cores cannot help): a workgroup owns a tile of (branch rows x entities),
// 128 x 128 where both sides fill it, stages both operands k-major in LDS 16
// coordinates at a time, and every lane accumulates an 8 x 8 block of distances in
// registers, so that one 16-byte LDS read feeds 32 accumulations.  Vector
// families with enough to do go through these kernels for a first sample at most, and
// for what the filter of rank_filter.hip cannot take.
//
// The selection pass looks for a bound, lists what is within it and places that with the running result of
// earlier chunks.  Order is (distance, entity id), so equal distances rank the lower id first.
#include <climits>

#include "common.h"

namespace ngdb {
namespace {

constexpr int DC = 16;

// Tile of 16*RPL rows x 16*EPL entities, RPL x EPL pairs per lane (entities in groups of four, 64
// apart, so that neighbouring lanes read adjacent 16-byte units of LDS).  The distance of a (row,
// entity) pair is summed by one lane over the coordinates in ascending order, so its value does
// not depend on where in a tile, or in which launch, the pair falls.
// BOX (box family): the row side is a box, centre from act and offset from off, and a coordinate
// contributes relu(a - o) + alpha * min(a, o) = max(alpha * a, a - (1 - alpha) * o), a = |e - c|;
// the offsets are staged already multiplied by (1 - alpha): five VALU operations per coordinate.
// Emat16 (if set): the entity rows are read from this bf16 copy of Emat.
// count (if set): tiles without a row whose query has count > room for the tile's piece of the table are left out.
// Three wavefronts per SIMD and two coordinates unrolled: left to itself the compiler unrolled all sixteen, fetched them
// ahead into 512 registers and ran one wavefront per SIMD, waiting for LDS and copying between register files.  At 603 boxes
// (737 rows) x 300 000 entities x 316 coordinates 14.4 -> 6.4 ms, at 512 vectors x 200 000 x 256 2.56 -> 1.52 ms.
__device__ __forceinline__ bool marked_piece(const int32_t* __restrict__ any, int pieces) {
    int32_t some = 0;
    for (int p = 0; p < pieces; ++p) some |= any[p];
    return some != 0;
}
template <bool BOX, int RPL, int EPL>
__global__ __launch_bounds__(256, 3) void l1_tile_kernel(const float* __restrict__ act, const float* __restrict__ off,
                                                      float alpha, const int32_t* __restrict__ row_ids,
                                                      int n_rows, const float* __restrict__ Emat,
                                                      const uint16_t* __restrict__ Emat16, int n_ent, int d,
                                                      float* __restrict__ dist, int ld, const int32_t* __restrict__ row_q,
                                                      const int32_t* __restrict__ count, int room,
                                                      const int32_t* __restrict__ any, int n_queries) {
    const int pieces = (n_ent + RANK_PIECE - 1) / RANK_PIECE;
    if (any && !marked_piece(any, pieces)) return;         // uniform
    constexpr int TQ = 16 * RPL, TE = 16 * EPL, LDQ = TQ + 4, LDE = TE + 4;
    constexpr int LQ = (TQ * 4 + 255) / 256, LE = (TE * 4 + 255) / 256;     // float4 per thread and stage
    __shared__ __attribute__((aligned(16))) float Ys[2][DC][LDQ];
    __shared__ __attribute__((aligned(16))) float Es[2][DC][LDE];
    __shared__ __attribute__((aligned(16))) float Os[BOX ? 2 : 1][BOX ? DC : 1][LDQ];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int r0 = blockIdx.y * TQ;
    uint32_t marked = 0u;                                  // pieces for which the rows of this tile are needed
    if (count) {
        const int r = r0 + tid;
        for (int p = 0; p < pieces; ++p)
            if (__syncthreads_or(tid < TQ && r < n_rows && count[(size_t)p * n_queries + row_q[r]] > room)) marked |= 1u << p;
        if (marked == 0u) return;                          // uniform
    }
    // (a launch that only completes a filtered pass has few workgroups, each with several entity tiles)
    for (int e0 = blockIdx.x * TE; e0 < n_ent; e0 += gridDim.x * TE) {
        if (count && !(marked >> (e0 / RANK_PIECE) & 1u)) continue;          // uniform; a piece is a multiple of every tile

        const float* yrow[LQ];
        const float* orow[LQ];
        const float* erow[LE];
        const uint16_t* erow16[LE];
        const int lkq = tid & 3, lrow = tid >> 2;             // row lrow + 64 * i of either side
        const bool has_y = lrow < TQ, has_e = lrow < TE;      // (a side of 32 rows has work for half the threads)
#pragma unroll
        for (int i = 0; i < LQ; ++i) {
            const int r = min(r0 + lrow + 64 * i, n_rows - 1);          // clamped rows are computed and never stored
            yrow[i] = act + (size_t)row_ids[r] * d;
            orow[i] = BOX ? off + (size_t)row_ids[r] * d : nullptr;
        }
#pragma unroll
        for (int i = 0; i < LE; ++i) {
            const int ec = min(e0 + lrow + 64 * i, n_ent - 1);
            erow[i] = Emat + (Emat16 ? 0 : (size_t)ec * d);
            erow16[i] = Emat16 ? Emat16 + (size_t)ec * d : nullptr;
        }
        float4 ry[LQ], re[LE], ro[LQ];
        const float shrink = 1.f - alpha;
        auto issue = [&](int k0) {
            const int kc = min(k0 + lkq * 4, d - 4);
#pragma unroll
            for (int i = 0; i < LQ; ++i) {
                ry[i] = *reinterpret_cast<const float4*>(yrow[i] + kc);
                if (BOX) ro[i] = *reinterpret_cast<const float4*>(orow[i] + kc);
            }
#pragma unroll
            for (int i = 0; i < LE; ++i)
                re[i] = Emat16 ? bf16x4_to_f32(*reinterpret_cast<const uint2*>(erow16[i] + kc))
                               : *reinterpret_cast<const float4*>(erow[i] + kc);
        };
        auto stage = [&](int buf, int k0) {
            const bool ok = k0 + lkq * 4 < d;                  // coordinates past d contribute |0 - 0|
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < LQ; ++i) {
                if (!has_y) break;
                const int row = lrow + 64 * i;
                const float4 y = ok ? ry[i] : zero;
                Ys[buf][lkq * 4 + 0][row] = y.x; Ys[buf][lkq * 4 + 1][row] = y.y;
                Ys[buf][lkq * 4 + 2][row] = y.z; Ys[buf][lkq * 4 + 3][row] = y.w;
                if (BOX) {
                    const float4 o = ok ? ro[i] : zero;
                    Os[buf][lkq * 4 + 0][row] = shrink * o.x; Os[buf][lkq * 4 + 1][row] = shrink * o.y;
                    Os[buf][lkq * 4 + 2][row] = shrink * o.z; Os[buf][lkq * 4 + 3][row] = shrink * o.w;
                }
            }
#pragma unroll
            for (int i = 0; i < LE; ++i) {
                if (!has_e) break;
                const int row = lrow + 64 * i;
                const float4 e = ok ? re[i] : zero;
                Es[buf][lkq * 4 + 0][row] = e.x; Es[buf][lkq * 4 + 1][row] = e.y;
                Es[buf][lkq * 4 + 2][row] = e.z; Es[buf][lkq * 4 + 3][row] = e.w;
            }
        };

        float acc[RPL][EPL];
#pragma unroll
        for (int i = 0; i < RPL; ++i)
#pragma unroll
            for (int j = 0; j < EPL; ++j) acc[i][j] = 0.f;

        const int nk = (d + DC - 1) / DC;
        issue(0);
        stage(0, 0);
        __syncthreads();
        for (int kt = 0; kt < nk; ++kt) {
            const int buf = kt & 1;
            if (kt + 1 < nk) issue((kt + 1) * DC);
#pragma unroll 2
            for (int k = 0; k < DC; ++k) {
                float yv[RPL], ov[RPL], ev[EPL];
#pragma unroll
                for (int i = 0; i < RPL; ++i) {
                    yv[i] = Ys[buf][k][ty * RPL + i];
                    ov[i] = BOX ? Os[BOX ? buf : 0][BOX ? k : 0][ty * RPL + i] : 0.f;
                }
#pragma unroll
                for (int j = 0; j < EPL; j += 4) {
                    const float4 x = *reinterpret_cast<const float4*>(&Es[buf][k][(j >> 2) * 64 + tx * 4]);
                    ev[j] = x.x; ev[j + 1] = x.y; ev[j + 2] = x.z; ev[j + 3] = x.w;
                }
#pragma unroll
                for (int i = 0; i < RPL; ++i)
#pragma unroll
                    for (int j = 0; j < EPL; ++j) {
                        const float a = fabsf(yv[i] - ev[j]);
                        acc[i][j] += BOX ? fmaxf(alpha * a, a - ov[i]) : a;
                    }
            }
            if (kt + 1 < nk) stage(buf ^ 1, (kt + 1) * DC);
            __syncthreads();
        }

#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int r = r0 + ty * RPL + i;
            if (r >= n_rows) continue;
#pragma unroll
            for (int j = 0; j < EPL; j += 4) {
                const int e = e0 + (j >> 2) * 64 + tx * 4;
                float* out = dist + (size_t)r * ld + e;
                if (e + 3 < n_ent) {
                    *reinterpret_cast<float4*>(out) = make_float4(acc[i][j], acc[i][j + 1], acc[i][j + 2], acc[i][j + 3]);
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (e + t < n_ent) out[t] = acc[i][j + t];
                }
            }
        }
    }
}

constexpr int KMAX = NGDB_MAX_TOPK;

__device__ __forceinline__ bool before(float d, int i, float d2, int i2) { return d < d2 || (d == d2 && i < i2); }

// One workgroup per query: merges the chunk's distances into the query's running top-k.  Two looks at the distances (a
// union query takes the minimum over its branch rows): the first finds every lane's smallest, and the k-th smallest of
// these in a wavefront is a bound that k entities keep; the second lists what is within the least of these bounds,
// some ten times k entities, whose places are counted directly.  (Sorted lists of KMAX per lane, merged: 78 us more at
// 15 000 entities, 290 at 50 000.)  Should the list be too short for ties, the k best are found one after the other.
// REST: completes a filtered pass, for the queries that have a mark in count (cleared here), several to a workgroup.
constexpr int TOPK_T = 1024, TOPK_LIST = 2048, TOPK_FEW = 512;
template <bool REST>
__global__ __launch_bounds__(TOPK_T) void topk_kernel(const float* __restrict__ dist, int ld, const int32_t* __restrict__ root_off,
                                                      int n_queries, int ent_base, int n_ent, int k, bool first_chunk,
                                                      float* __restrict__ out_dist, int32_t* __restrict__ out_ids,
                                                      const int32_t* __restrict__ gave_up, int32_t* __restrict__ count, int room,
                                                      const int32_t* __restrict__ any) {
    const int pieces = REST ? (n_ent + RANK_PIECE - 1) / RANK_PIECE : 1;
    if (*gave_up) n_ent = 0;             // (uniform)
    if (REST && !marked_piece(any, pieces)) return;        // uniform
    __shared__ float s_d[TOPK_LIST], s_bound[TOPK_T / 64], s_run[KMAX];
    __shared__ int s_i[TOPK_LIST], s_run_i[KMAX], s_n;
    const int t = threadIdx.x, T = blockDim.x, lane = t & 63, wave = t >> 6;
    for (int q = blockIdx.x; q < n_queries; q += gridDim.x) {
        uint32_t marked = 0u;
        for (int p = 0; REST && p < pieces; ++p)
            if (count[(size_t)p * n_queries + q] > room) marked |= 1u << p;
        if (REST && marked == 0u) continue;              // uniform: the filter has dealt with this query's pieces
        const int r0 = root_off[q], nb = root_off[q + 1] - r0;
        const float* row = dist + (size_t)r0 * ld;
        auto four = [&](int e) {                         // entities e .. e + 3, those past the end or dealt with not a number
            if (REST && !(marked >> (e / RANK_PIECE) & 1u)) return make_float4(NAN, NAN, NAN, NAN);
            float4 v = *reinterpret_cast<const float4*>(row + e);
            for (int b = 1; b < nb; ++b) {
                const float4 w = *reinterpret_cast<const float4*>(row + (size_t)b * ld + e);
                v.x = fminf(v.x, w.x); v.y = fminf(v.y, w.y); v.z = fminf(v.z, w.z); v.w = fminf(v.w, w.w);
            }
            if (e + 1 >= n_ent) v.y = NAN;
            if (e + 2 >= n_ent) v.z = NAN;
            if (e + 3 >= n_ent) v.w = NAN;
            return v;
        };
        if (t == 0) s_n = 0;
        if (t < KMAX) {
            const bool have = !first_chunk && t < k;
            s_run[t] = have ? out_dist[(size_t)q * k + t] : INFINITY;
            s_run_i[t] = have ? out_ids[(size_t)q * k + t] : -1;
        }
        float least = INFINITY;
#pragma unroll 4
        for (int e = 4 * t; e < n_ent; e += 4 * T) {
            const float4 v = four(e);
            least = fminf(least, fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
        }
        int smaller = 0;                                 // lanes before this one
#pragma unroll
        for (int j = 0; j < 64; ++j) {
            const float o = lane_value(least, j);
            smaller += (o < least || (o == least && j < lane)) ? 1 : 0;
        }
        const float bound_w = lane_value(least, __ffsll(__ballot(smaller == k - 1)) - 1);
        if (lane == 0) s_bound[wave] = bound_w;
        __syncthreads();
        float bound = INFINITY;
        for (int w = 0; w < T / 64; ++w) bound = fminf(bound, s_bound[w]);
        if (s_run_i[k - 1] >= 0) bound = fminf(bound, s_run[k - 1]);
        auto list = [&](float d, int id) {
            const int at = atomicAdd(&s_n, 1);
            if (at < TOPK_LIST) {
                s_d[at] = d;
                s_i[at] = id;
            }
        };
        if (t < k && s_run_i[t] >= 0) list(s_run[t], s_run_i[t]);
#pragma unroll 4
        for (int e = 4 * t; e < n_ent; e += 4 * T) {
            const float4 v = four(e);
            if (v.x <= bound) list(v.x, ent_base + e);
            if (v.y <= bound) list(v.y, ent_base + e + 1);
            if (v.z <= bound) list(v.z, ent_base + e + 2);
            if (v.w <= bound) list(v.w, ent_base + e + 3);
        }
        __syncthreads();
        const int n = s_n;
        if (n <= TOPK_LIST) {
            for (int x = t; x < n; x += T) {
                const float d = s_d[x];
                const int id = s_i[x];
                int place = 0;
                for (int j = 0; j < n; ++j) place += before(s_d[j], s_i[j], d, id) ? 1 : 0;
                if (place < k) {
                    out_dist[(size_t)q * k + place] = d;
                    out_ids[(size_t)q * k + place] = id;
                }
            }
            if (t >= n && t < k) {
                out_dist[(size_t)q * k + t] = INFINITY;
                out_ids[(size_t)q * k + t] = -1;
            }
        } else {
            float pd = -INFINITY;
            int pi = -1;
            for (int r = 0; r < k; ++r) {                // the first one after (pd, pi)
                float md = INFINITY;
                int mi = INT_MAX;
                auto look = [&](float d, int id) {
                    if (before(pd, pi, d, id) && before(d, id, md, mi)) {
                        md = d;
                        mi = id;
                    }
                };
                if (t < k && s_run_i[t] >= 0) look(s_run[t], s_run_i[t]);
                for (int e = 4 * t; e < n_ent; e += 4 * T) {
                    const float4 v = four(e);
                    look(v.x, ent_base + e); look(v.y, ent_base + e + 1); look(v.z, ent_base + e + 2); look(v.w, ent_base + e + 3);
                }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const float od = __shfl_xor(md, off, 64);
                    const int oi = __shfl_xor(mi, off, 64);
                    if (before(od, oi, md, mi)) {
                        md = od;
                        mi = oi;
                    }
                }
                __syncthreads();                         // s_d / s_i of the round before have been read
                if (lane == 0) {
                    s_d[wave] = md;
                    s_i[wave] = mi;
                }
                __syncthreads();
                for (int w = 0; w < T / 64; ++w)
                    if (before(s_d[w], s_i[w], md, mi)) {
                        md = s_d[w];
                        mi = s_i[w];
                    }
                pd = md;
                pi = mi;
                if (t == 0) {
                    out_dist[(size_t)q * k + r] = md;
                    out_ids[(size_t)q * k + r] = mi == INT_MAX ? -1 : mi;
                }
            }
        }
        if (!REST) return;
        if (t < pieces) count[(size_t)t * n_queries + q] = 0;
        __syncthreads();
    }
}

// ---------------------------------------------------------------- filtered ranks of listed answers
// query of answer a: largest q with ans_off[q] <= a
__device__ __forceinline__ int query_of_answer(const int32_t* __restrict__ ans_off, int n_queries, int a) {
    int lo = 0, hi = n_queries;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ans_off[mid] <= a) lo = mid; else hi = mid;
    }
    return lo;
}

constexpr int CNT_SLAB = 8192;    // entities per workgroup of the counting pass
constexpr int CNT_AT_ONCE = 8;    // answers a lane counts for in one look at its distances

// count[a] += number of entities of the slab strictly closer to a's query than thr[a].
// Grid (slabs, queries).  Counters in registers, summed over the workgroup at the end; one integer atomic per answer and
// workgroup reaches global memory (integer sums do not depend on the order).  (A ballot and an LDS counter per answer
// and 64 entities took 44 us more for 100 queries of six answers over 50 000 entities.)
__global__ __launch_bounds__(256) void count_less_kernel(const float* __restrict__ dist, int ld,
                                                         const int32_t* __restrict__ root_off,
                                                         const int32_t* __restrict__ ans_off,
                                                         const float* __restrict__ thr, int n_ent,
                                                         int32_t* __restrict__ count, const int32_t* __restrict__ listed,
                                                         int room) {
    __shared__ int32_t s_cnt[4][CNT_AT_ONCE];
    const int q = blockIdx.y;
    const int a_lo = ans_off[q], a_hi = ans_off[q + 1];
    if (a_lo >= a_hi || (listed && listed[q] <= room)) return;        // uniform
    const int r_lo = root_off[q], nb = root_off[q + 1] - r_lo;
    const float* row = dist + (size_t)r_lo * ld;
    const int e_lo = blockIdx.x * CNT_SLAB, e_hi = min(n_ent, e_lo + CNT_SLAB);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int t0 = a_lo; t0 < a_hi; t0 += CNT_AT_ONCE) {
        float th[CNT_AT_ONCE];
        int cnt[CNT_AT_ONCE];
#pragma unroll
        for (int j = 0; j < CNT_AT_ONCE; ++j) {
            th[j] = t0 + j < a_hi ? thr[t0 + j] : -INFINITY;          // (nothing is closer)
            cnt[j] = 0;
        }
#pragma unroll 2
        for (int e = e_lo + 4 * t; e < e_hi; e += 4 * 256) {
            float4 v = *reinterpret_cast<const float4*>(row + e);
            for (int b = 1; b < nb; ++b) {
                const float4 w = *reinterpret_cast<const float4*>(row + (size_t)b * ld + e);
                v.x = fminf(v.x, w.x); v.y = fminf(v.y, w.y); v.z = fminf(v.z, w.z); v.w = fminf(v.w, w.w);
            }
            if (e + 1 >= e_hi) v.y = INFINITY;                        // entities past the end are closer to nothing
            if (e + 2 >= e_hi) v.z = INFINITY;
            if (e + 3 >= e_hi) v.w = INFINITY;
#pragma unroll
            for (int j = 0; j < CNT_AT_ONCE; ++j)
                cnt[j] += (v.x < th[j] ? 1 : 0) + (v.y < th[j] ? 1 : 0) + (v.z < th[j] ? 1 : 0) + (v.w < th[j] ? 1 : 0);
        }
#pragma unroll
        for (int j = 0; j < CNT_AT_ONCE; ++j) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) cnt[j] += __shfl_xor(cnt[j], off, 64);
        }
        __syncthreads();                                              // the counters of the round before have been read
        if (lane == 0)
#pragma unroll
            for (int j = 0; j < CNT_AT_ONCE; ++j) s_cnt[wave][j] = cnt[j];
        __syncthreads();
        if (t < CNT_AT_ONCE && t0 + t < a_hi) {
            const int c = (s_cnt[0][t] + s_cnt[1][t]) + (s_cnt[2][t] + s_cnt[3][t]);
            if (c) atomicAdd(&count[t0 + t], c);
        }
    }
}

// rank[a] = 1 + count[a] - #{other listed answers b of the same query with thr[b] < thr[a]}
__global__ __launch_bounds__(256) void finish_rank_kernel(const int32_t* __restrict__ count,
                                                          const float* __restrict__ thr,
                                                          const int32_t* __restrict__ ans_off, int n_queries,
                                                          int n_ans, const int32_t* __restrict__ gave_up, int32_t* __restrict__ rank) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n_ans) return;
    if (*gave_up) {                      // (uniform: no entity is closer than an answer at no distance, which would be rank 1)
        rank[a] = 0;
        return;
    }
    const int q = query_of_answer(ans_off, n_queries, a);
    const float t = thr[a];
    int closer = 0;
    for (int b = ans_off[q]; b < ans_off[q + 1]; ++b) closer += thr[b] < t ? 1 : 0;
    rank[a] = 1 + count[a] - closer;
}

// out[0] = mean reciprocal rank, out[1..3] = Hit@1, @3, @10: per query the mean over its first
// n_take[q] listed answers (all if n_take is null), then the mean over the queries that have one.
// One workgroup, fixed summation order: the queries of 1024 threads at a time, then 256 sums of every 256th query, then these
// (a thread per sum for all of its queries: 1024 queries of 8 answers 12 us, 5.6 so).  A query's sums and the inverse of its count are
// handed over apart: its mean is rounded once, with the sum that it is added to.
constexpr int METRIC_T = 1024;
__global__ __launch_bounds__(METRIC_T) void rank_metrics_kernel(const int32_t* __restrict__ rank,
                                                                const int32_t* __restrict__ ans_off,
                                                                const int32_t* __restrict__ n_take, int n_queries,
                                                                float* __restrict__ out) {
    __shared__ float per[METRIC_T][5], part[256][5];
    float acc[5] = {0.f, 0.f, 0.f, 0.f, 0.f};      // MRR, H@1, H@3, H@10, queries counted
    for (int q0 = 0; q0 < n_queries; q0 += METRIC_T) {
        const int q = q0 + threadIdx.x;
        float v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};    // the four sums, the inverse of their count (0: no answer)
        if (q < n_queries) {
            const int lo = ans_off[q];
            const int n = n_take ? min(n_take[q], ans_off[q + 1] - lo) : ans_off[q + 1] - lo;
#pragma unroll 4
            for (int j = 0; j < n; ++j) {
                const int r = rank[lo + j];
                v[0] += 1.f / (float)r;
                v[1] += r <= 1 ? 1.f : 0.f;
                v[2] += r <= 3 ? 1.f : 0.f;
                v[3] += r <= 10 ? 1.f : 0.f;
            }
            if (n > 0) v[4] = 1.f / (float)n;
        }
        __syncthreads();                               // the round before has been read
        for (int k = 0; k < 5; ++k) per[threadIdx.x][k] = v[k];
        __syncthreads();
        if (threadIdx.x < 256)
            for (int i = threadIdx.x; i < METRIC_T; i += 256) {
                const float inv = per[i][4];
                for (int k = 0; k < 4; ++k) acc[k] = fmaf(per[i][k], inv, acc[k]);
                acc[4] += inv > 0.f ? 1.f : 0.f;
            }
    }
    if (threadIdx.x < 256)
        for (int k = 0; k < 5; ++k) part[threadIdx.x][k] = acc[k];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            for (int k = 0; k < 5; ++k) part[threadIdx.x][k] += part[threadIdx.x + off][k];
        __syncthreads();
    }
    if (threadIdx.x < 4) out[threadIdx.x] = part[0][4] > 0.f ? part[0][threadIdx.x] / part[0][4] : 0.f;
}

__global__ __launch_bounds__(256) void fill_zero_i32_kernel(int32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

hipError_t launch_l1_tile(const float* act, const float* off, float alpha, const int32_t* row_ids, int n_rows,
                          const float* Emat, int n_ent, int d, float* dist, int ld, hipStream_t s, const uint16_t* Emat16,
                          const Overflowed* only) {
    if (n_rows <= 0 || n_ent <= 0) return hipSuccess;
    if ((d & 3) || (ld & 3) || (off && !(alpha >= 0.f && alpha <= 1.f))) return hipErrorInvalidValue;
    // 128 x 128 tiles where they fill the chip's 256 compute units; smaller ones for few rows (a tile's time does
    // not depend on how many of its rows exist) and for small tables; 32 rows where 64 x 64 tiles would leave compute units idle
    // (590 rows x 1280 entities x 400 coordinates, 200 tiles: 41 us, as 380 tiles 34.6)
    const int rpl = n_rows <= 32 || (long)((n_rows + 63) / 64) * ((n_ent + 63) / 64) < 256 ? 2 : (n_rows <= 64 || (long)((n_rows + 127) / 128) * ((n_ent + 127) / 128) < 512 ? 4 : 8);
    const int epl = (long)((n_rows + 16 * rpl - 1) / (16 * rpl)) * ((n_ent + 127) / 128) < 512 ? 4 : 8;
    int tiles_e = (n_ent + 16 * epl - 1) / (16 * epl);
    if (only) tiles_e = std::min(tiles_e, 64);
    if (only && n_ent > RANK_PIECES * RANK_PIECE) return hipErrorInvalidValue;
    const dim3 grid(tiles_e, (n_rows + 16 * rpl - 1) / (16 * rpl)), block(256);
#define NGDB_L1(BOX, R, C)                                                                                             \
    hipLaunchKernelGGL((l1_tile_kernel<BOX, R, C>), grid, block, 0, s, act, off, alpha, row_ids, n_rows, Emat, Emat16,   \
                       n_ent, d, dist, ld, only ? only->row_q : nullptr, only ? (const int32_t*)only->count : nullptr,   \
                       only ? only->room : 0, only ? only->any : nullptr, only ? only->n_queries : 0)
#define NGDB_L1_SIZES(BOX)                                                                  \
    if (rpl == 8) { if (epl == 8) NGDB_L1(BOX, 8, 8); else NGDB_L1(BOX, 8, 4); }             \
    else if (rpl == 4) { if (epl == 8) NGDB_L1(BOX, 4, 8); else NGDB_L1(BOX, 4, 4); }        \
    else { if (epl == 8) NGDB_L1(BOX, 2, 8); else NGDB_L1(BOX, 2, 4); }
    if (off) { NGDB_L1_SIZES(true) } else { NGDB_L1_SIZES(false) }
#undef NGDB_L1_SIZES
#undef NGDB_L1
    return hipGetLastError();
}

hipError_t launch_count_less(const float* dist, int ld, const int32_t* root_off, const int32_t* ans_off,
                             const float* thr, int n_queries, int n_ent, int32_t* count, hipStream_t s,
                             const Overflowed* only) {
    if (n_queries <= 0 || n_ent <= 0) return hipSuccess;
    if (n_queries > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(count_less_kernel, dim3((n_ent + CNT_SLAB - 1) / CNT_SLAB, n_queries), dim3(256), 0, s, dist, ld,
                       root_off, ans_off, thr, n_ent, count, only ? (const int32_t*)only->count : nullptr, only ? only->room : 0);
    return hipGetLastError();
}

hipError_t launch_finish_rank(const int32_t* count, const float* thr, const int32_t* ans_off, int n_queries, int n_ans,
                              const int32_t* gave_up, int32_t* rank, hipStream_t s) {
    if (n_ans <= 0) return hipSuccess;
    hipLaunchKernelGGL(finish_rank_kernel, dim3((n_ans + 255) / 256), dim3(256), 0, s, count, thr, ans_off, n_queries,
                       n_ans, gave_up, rank);
    return hipGetLastError();
}

hipError_t launch_rank_metrics(const int32_t* rank, const int32_t* ans_off, const int32_t* n_take, int n_queries,
                               float* out, hipStream_t s) {
    hipLaunchKernelGGL(rank_metrics_kernel, dim3(1), dim3(METRIC_T), 0, s, rank, ans_off, n_take, n_queries, out);
    return hipGetLastError();
}

hipError_t launch_fill_zero_i32(int32_t* p, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_topk_merge(const float* dist, int ld, const int32_t* root_off, int n_queries, int ent_base, int n_ent,
                             int k, bool first_chunk, float* out_dist, int32_t* out_ids, const int32_t* gave_up, hipStream_t s,
                             const Overflowed* only) {
    if (n_queries <= 0) return hipSuccess;
    if (!gave_up) return hipErrorInvalidValue;
    if (k < 1 || k > KMAX) return hipErrorInvalidValue;
    if (ld & 3) return hipErrorInvalidValue;
    const dim3 block(n_ent > 4096 ? TOPK_T : 256);
    if (only)
        hipLaunchKernelGGL(topk_kernel<true>, dim3(std::min(n_queries, TOPK_FEW)), block, 0, s, dist, ld, root_off, n_queries, ent_base, n_ent, k,
                           first_chunk, out_dist, out_ids, gave_up, only->count, only->room, only->any);
    else
        hipLaunchKernelGGL(topk_kernel<false>, dim3(n_queries), block, 0, s, dist, ld, root_off, n_queries, ent_base, n_ent, k, first_chunk, out_dist,
                           out_ids, gave_up, (int32_t*)nullptr, 0, (const int32_t*)nullptr);
    return hipGetLastError();
}

}  // namespace ngdb
