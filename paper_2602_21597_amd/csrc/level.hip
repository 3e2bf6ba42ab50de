// The operators of one depth in one launch, for models whose MLPs are small: assembly of the input rows, both layers
// and the intersection's pooling, or the reverse of it in the backward pass.
//
// At small widths a step is bound by its launches, not by their work: three a depth in either direction, 3 to 5 us each
// for contractions of a few MFLOP.  A workgroup takes 16 rows (of an intersection: all inputs of 16 / k members, so
// that the pooling needs nobody else), keeps their inputs and hidden rows in LDS and reads the weights of both
// layers from the L2, 16 output columns at a time per wavefront, eight k-steps ahead (sixteen wavefronts: with eight and
// six steps ahead 112 against 101 us for a forward pass at d = h = 256).  What it costs over the
// separate launches is that every 16 rows read all weights again and that a row block's matrix work stays on one
// compute unit.  Measured, device time of a forward pass with scoring of 256 queries (two launches a depth less, 41 -> 25 us of
// host time) and of a training step with 32 negatives, separate -> here: d = 64, h = 128: 59 -> 45 and 149 -> 128 us;
// 128, 128: 62 -> 56, 157 -> 148; 100, 200: 65 -> 59, 163 -> 165; 32, 512: 66 -> 67, 165 -> 182; 128, 256: 62 -> 72, 160 -> 184.
// Boxes (more launches apart): 128, 128: 46 -> 39, 112 -> 106; 128, 256: 48 -> 46, 116 -> 123; 64, 512: 49 -> 49, 117 -> 132,
// and with 16 queries 56 -> 47 and 100 -> 104.
#include <algorithm>
#include "small_index.h"

namespace ngdb {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int LV_ROWS = 16, LV_WAVES = 16, LV_T = LV_WAVES * 64;
constexpr int LV_AHEAD = 8;      // k-steps of 16 on the way per wavefront

__host__ __device__ constexpr int lv_pitch(int n) { return (n + 15) / 16 * 16 + 4; }

// One layer, out = A * W^T (BT: A * W) for the 16 rows of A in LDS; wavefront w computes the column blocks w, w + 16, ...  start()
// requests the first weights (long before A is there), run() hands a lane's four values (rows 4 (lane / 16) .. +3 of
// column n) to done.  Within a k-step lane group g holds k = 4g .. 4g+3 of both operands, one of them per matrix instruction.
// These add product after product to an fp32 sum, so k goes through sums of at most 16 products, four at a time, which are
// then added: the error against fp64 stays at that of the separate launches, which split k over eight wavefronts.  (Two sums
// over all of k: outputs at d = 128, h = 256 off by 2.2e-7 instead of 1.3e-7, at 256, 128 2.4e-7 instead of 1.3e-7; a step
// 167.9 -> 174.5 us at 100, 200, 186.5 -> 193.4 at 128, 256, 134.4 -> 136.7 at 64, 128.  Eight sums folded half as often
// spill, and k split over wavefronts waits longer at the barrier than it saves.)
template <bool BT>
struct Layer {
    const float* W;
    int ldw, K, N, steps, col, kg, lb, ls;
    float4 w[LV_AHEAD];
    __device__ __forceinline__ float4 fetch() {       // (past the last block: clamped, never used)
        const int n = min(lb * 16 + col, N - 1), k = ls * 16 + kg, kc = min(k, K - 4);
        float4 v;
        if (!BT) {
            v = *reinterpret_cast<const float4*>(W + (size_t)n * ldw + kc);
        } else {
            const float* p = W + (size_t)kc * ldw + n;
            v = make_float4(p[0], p[ldw], p[2 * ldw], p[3 * ldw]);
        }
        if (k >= K) v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (++ls == steps) {
            ls = 0;
            lb += LV_WAVES;
        }
        return v;
    }
    __device__ __forceinline__ void start(const float* W_, int ldw_, int K_, int N_) {
        W = W_; ldw = ldw_; K = K_; N = N_;
        steps = (K + 15) / 16;
        col = threadIdx.x & 15;
        kg = ((threadIdx.x & 63) >> 4) * 4;
        lb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        ls = 0;
#pragma unroll
        for (int q = 0; q < LV_AHEAD; ++q) w[q] = fetch();
    }
    template <class Done>
    __device__ __forceinline__ void run(const float* As, int ap, Done done) {
        int b = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), s = 0;
        const int blocks = (N + 15) / 16;
        const int total = b < blocks ? ((blocks - b + LV_WAVES - 1) / LV_WAVES) * steps : 0;
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        floatx4 sum[4] = {zero, zero, zero, zero}, all = zero;
        const float* arow = As + col * ap + kg;
        for (int t0 = 0; t0 < total; t0 += LV_AHEAD) {
#pragma unroll
            for (int q = 0; q < LV_AHEAD; ++q) {
                if (t0 + q >= total) return;
                const float4 x = *reinterpret_cast<const float4*>(arow + s * 16);
                sum[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, w[q].x, sum[0], 0, 0, 0);
                sum[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, w[q].y, sum[1], 0, 0, 0);
                sum[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, w[q].z, sum[2], 0, 0, 0);
                sum[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, w[q].w, sum[3], 0, 0, 0);
                if (t0 + q + LV_AHEAD < total) w[q] = fetch();
                const bool last = ++s == steps;      // uniform
                if (q % 4 == 3 || last) {
                    all += (sum[0] + sum[1]) + (sum[2] + sum[3]);
                    sum[0] = sum[1] = sum[2] = sum[3] = zero;
                }
                if (last) {
                    done(b * 16 + col, all);
                    all = zero;
                    s = 0;
                    b += LV_WAVES;
                }
            }
        }
    }
};

// Several depths in one launch (CHAIN): a workgroup takes the next number, and with it the next tile of the depths in their
// order, requests its weights, waits until all tiles of the depth before are through, and counts itself when its rows are stored.  Numbers are
// handed out in the order of dependence, so whoever is waited for has its number and runs, whatever part of the launch is resident and whoever
// else is on the card.  What one depth hands to the next (rows of act, or of dact) is stored and loaded at the scope of the card, past
// the L2s of the dies: a store is where everybody finds it when its wavefront's wait is over, and no cache has to be written
// back or dropped.  The launch between two depths that this replaces costs 4 us of host time and 2 to 3 of the card's beyond
// the wait: steps of 64 queries x 8 negatives at d = 32, h = 64 73.0 -> 68.0 us, 256 x 32 at 64, 128 135 -> 123, 64 x 16 at 100, 200 142 -> 130,
// boxes of 200 x 32 at 128, 128 116 -> 105.
template <bool CHAIN>
__device__ __forceinline__ float4 row_get(const float* p) {
    if (!CHAIN) return *reinterpret_cast<const float4*>(p);
    const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float4(__uint_as_float((uint32_t)lo), __uint_as_float((uint32_t)(lo >> 32)), __uint_as_float((uint32_t)hi),
                       __uint_as_float((uint32_t)(hi >> 32)));
}
template <bool CHAIN>
__device__ __forceinline__ float row_get1(const float* p) {
    return CHAIN ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool CHAIN>
__device__ __forceinline__ void row_put1(float* p, float v) {
    if (CHAIN) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}
template <bool CHAIN>
__device__ __forceinline__ void row_put(float* p, float4 v) {
    if (!CHAIN) { *reinterpret_cast<float4*>(p) = v; return; }
    row_put1<true>(p, v.x); row_put1<true>(p + 1, v.y); row_put1<true>(p + 2, v.z); row_put1<true>(p + 3, v.w);
}
// counts[0]: numbers handed out, counts[1]: tiles through, counts[2 + l]: tiles of depth l through (but the last).  A wait that no
// working card comes near ends all the same, after so many looks that they take seconds: the rows of its tile are not valid then, and its
// depth's count goes past all tiles there are by GAVE_UP, so that whoever waits for that depth gives up at once too.
static_assert(LEVEL_CHAIN_TILES < GAVE_UP && (long)LEVEL_CHAIN_TILES * (GAVE_UP + 1) < INT32_MAX, "counts of tiles and of those that gave up in one word");
// whether all tiles of that depth have their rows stored (known to the first thread, which looks)
__device__ __forceinline__ bool wait_for_depth(const int32_t* through, int tiles, int polls) {
    int32_t n = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < polls && (n = __hip_atomic_load(through, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < tiles; ++i) __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
    __syncthreads();
    return n == tiles;
}

// Box family: projections have no MLP (16 members a workgroup: centre plus, offset plus relu of the relation's rows); the
// offset side of an intersection pools by the least input times the gate of the mean logit.
template <bool BWD, bool CHAIN>
__device__ __forceinline__ void box_projection(const LevelArgs& a, const LevelProblem& p, int i0) {
    const int d4 = a.d >> 2;
    const int n = min(LV_ROWS, p.n - i0) * d4;
    for (int idx = threadIdx.x; idx < n; idx += LV_T) {
        const int i = i0 + idx / d4, c = (idx % d4) * 4;
        const size_t out = (size_t)(p.out0 + i) * a.d + c;
        if (BWD) {
            const size_t in = (size_t)a.dst_row[p.ref_off + i] * a.d + c;
            row_put<CHAIN>(a.dact + in, row_get<CHAIN>(a.dact + out));
            row_put<CHAIN>(a.doff + in, row_get<CHAIN>(a.doff + out));
            continue;
        }
        const int32_t ref = a.refs[p.ref_off + i];
        const size_t r = (size_t)a.rel[p.rel_off + i] * a.d + c;
        float4 x, o = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ref >= 0) {
            x = row_get<CHAIN>(a.act + (size_t)ref * a.d + c);
            o = row_get<CHAIN>(a.off + (size_t)ref * a.d + c);
        } else {
            x = *reinterpret_cast<const float4*>(a.E + (size_t)(-1 - ref) * a.d + c);
        }
        const float4 rc = *reinterpret_cast<const float4*>(a.R + r), ro = *reinterpret_cast<const float4*>(a.Ro + r);
        x.x += rc.x; x.y += rc.y; x.z += rc.z; x.w += rc.w;
        o.x += fmaxf(ro.x, 0.f); o.y += fmaxf(ro.y, 0.f); o.z += fmaxf(ro.z, 0.f); o.w += fmaxf(ro.w, 0.f);
        row_put<CHAIN>(a.act + out, x);
        row_put<CHAIN>(a.off + out, o);
    }
}

// tile `block` of problem p; before(): what it reads of other depths is there
template <bool BWD, bool BOX, bool CHAIN, class Before>
__device__ __forceinline__ void level_tile(const LevelArgs& a, const LevelProblem& p, int block, float* lds, Before before) {
    __shared__ int row_of[LV_ROWS], out_of[LV_ROWS], in_of[LV_ROWS], rel_of[LV_ROWS];     // MLP row / output row / input reference / relation of a tile row
    const LevelMlp w = a.mlp[p.type];
    const int d = a.d, h = a.h, xp = lv_pitch(d), hp = lv_pitch(h);
    float *Xs = lds, *Ls = Xs + LV_ROWS * xp, *Hs = Ls + LV_ROWS * xp, *bias = Hs + LV_ROWS * hp;
    const int tid = threadIdx.x, lane = tid & 63;
    const int m = LV_ROWS / p.k, i0 = block * m;
    const bool inter = p.pool != 0;
    if (BOX && p.pool == LEVEL_PROJECTION) {
        before();
        box_projection<BWD, CHAIN>(a, p, i0);
        return;
    }
    const bool gate = BOX && p.pool == LEVEL_GATE;
    float* const act = gate ? a.off : a.act;
    float* const dact = gate ? a.doff : a.dact;
    float* const Att = gate ? a.Gate : a.Att;
    float* const dAtt = gate ? a.dGate : a.dAtt;
    Layer<BWD> first, second;
    if (BWD) first.start(w.Wb, h, d, h);
    else first.start(w.Wa, d, d, h);
    if (BWD) second.start(w.Wa, d, h, d);
    else second.start(w.Wb, h, h, d);
    if (tid < LV_ROWS) {
        const int j = tid / m, i = i0 + tid - j * m;
        const bool ok = j < p.k && i < p.n;
        const int r = j * p.n + i;
        row_of[tid] = ok ? p.row0 + r : -1;
        if (BWD) {
            in_of[tid] = ok ? a.dst_row[p.ref_off + r] : 0;
            out_of[tid] = p.out0 + min(i, p.n - 1);
        } else {
            const int o = p.out0 + min(i, p.n - 1);
            out_of[tid] = a.out_row ? a.out_row[o] : o;
            in_of[tid] = ok ? a.refs[p.ref_off + r] : 0;
            rel_of[tid] = ok && p.rel_off >= 0 ? a.rel[p.rel_off + r] : 0;
        }
    }
    if (!BWD)
        for (int i = tid; i < h + d; i += LV_T) bias[i] = i < h ? w.ba[i] : w.bb[i - h];
    before();
    // rows of the tile that are no rows, and the columns that fill up the last k-step, count as zeros
    if (!BWD) {
        __syncthreads();
        const int c4 = (xp - 4) >> 2;
        for (int idx = tid; idx < LV_ROWS * c4; idx += LV_T) {
            const int lr = idx / c4, c = (idx - lr * c4) * 4;
            const int j = lr / m, i = i0 + lr - j * m;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < p.k && i < p.n && c < d) {
                const int r = j * p.n + i;
                const int32_t ref = in_of[lr];
                if (ref >= 0) v = row_get<CHAIN>(act + (size_t)ref * d + c);
                else v = *reinterpret_cast<const float4*>(a.E + (size_t)(-1 - ref) * d + c);
                if (p.rel_off >= 0) {
                    const float4 t = *reinterpret_cast<const float4*>(a.R + (size_t)rel_of[lr] * d + c);
                    v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
                }
                if (a.keep) *reinterpret_cast<float4*>(w.Z + (size_t)(p.row0 + r) * d + c) = v;
            }
            *reinterpret_cast<float4*>(Xs + lr * xp + c) = v;
        }
        __syncthreads();
        first.run(Xs, xp, [&](int n, floatx4 v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int lr = (lane >> 4) * 4 + e;
                const float y = n < h ? fmaxf(v[e] + bias[min(n, h - 1)], 0.f) : 0.f;
                Hs[lr * hp + n] = y;
                const int r = row_of[lr];
                if (a.keep && r >= 0 && n < h) w.H[(size_t)r * h + n] = y;
            }
        });
        __syncthreads();
        second.run(Hs, hp, [&](int n, floatx4 v) {
            if (n >= d) return;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int lr = (lane >> 4) * 4 + e, r = row_of[lr];
                const float y = v[e] + bias[h + n];
                if (inter) {
                    Ls[lr * xp + n] = y;
                    if (a.keep && r >= 0) Att[(size_t)r * d + n] = y;
                } else if (r >= 0) {
                    row_put1<CHAIN>(act + (size_t)out_of[lr] * d + n, y);
                }
            }
        });
        if (!inter) return;
        __syncthreads();
        for (int idx = tid; idx < m * d; idx += LV_T) {
            const int ii = idx / d, c = idx - ii * d;
            if (i0 + ii >= p.n) break;
            if (gate) {
                float mean = 0.f, mn = INFINITY;
                for (int j = 0; j < p.k; ++j) {
                    mean += Ls[(j * m + ii) * xp + c];
                    mn = fminf(mn, Xs[(j * m + ii) * xp + c]);
                }
                row_put1<CHAIN>(act + (size_t)out_of[ii] * d + c, mn * sigmoid_f(mean / (float)p.k));
                continue;
            }
            float e[NGDB_MAX_CARD], mx = -INFINITY, den = 0.f, y = 0.f;
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                e[j] = Ls[(min(j, p.k - 1) * m + ii) * xp + c];
                if (j < p.k) mx = fmaxf(mx, e[j]);
            }
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                e[j] = j < p.k ? expf(e[j] - mx) : 0.f;
                den += e[j];
            }
            const float inv = 1.f / den;
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) y += e[j] * inv * Xs[(min(j, p.k - 1) * m + ii) * xp + c];
            row_put1<CHAIN>(act + (size_t)out_of[ii] * d + c, y);
        }
        return;
    }
    // ---- backward: gradients of the second layer's outputs in Xs, the hidden rows (for the sign) in Hs, the direct
    // gradient of an intersection's inputs in Ls
    {
        const int c4 = (xp - 4) >> 2, e4 = (hp - 4) >> 2;
        for (int idx = tid; idx < LV_ROWS * c4; idx += LV_T) {
            const int lr = idx / c4, c = (idx - lr * c4) * 4;
            const int j = lr / m, i = i0 + lr - j * m;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!inter && j < p.k && i < p.n && c < d) v = row_get<CHAIN>(dact + (size_t)(p.out0 + i) * d + c);
            *reinterpret_cast<float4*>(Xs + lr * xp + c) = v;
        }
        for (int idx = tid; idx < LV_ROWS * e4; idx += LV_T) {
            const int lr = idx / e4, c = (idx - lr * e4) * 4;
            const int j = lr / m, i = i0 + lr - j * m;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < p.k && i < p.n && c < h) v = *reinterpret_cast<const float4*>(w.H + (size_t)(p.row0 + j * p.n + i) * h + c);
            *reinterpret_cast<float4*>(Hs + lr * hp + c) = v;
        }
        __syncthreads();
        if (inter) {
            for (int idx = tid; idx < m * d; idx += LV_T) {
                const int ii = idx / d, c = idx - ii * d;
                if (i0 + ii >= p.n) break;
                float e[NGDB_MAX_CARD], x[NGDB_MAX_CARD], mx = -INFINITY, den = 0.f, tall = 0.f;
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                    const size_t at = (size_t)(p.row0 + min(j, p.k - 1) * p.n + i0 + ii) * d + c;
                    e[j] = Att[at];
                    x[j] = w.Z[at];
                    if (j < p.k) mx = fmaxf(mx, e[j]);
                }
                const float dy = row_get1<CHAIN>(dact + (size_t)(p.out0 + i0 + ii) * d + c);
                if (gate) {
                    float mean = 0.f, mn = INFINITY;
                    int arg = 0;
#pragma unroll
                    for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                        if (j < p.k) {
                            mean += e[j];
                            if (x[j] < mn) {       // strict: equal offsets keep the lower input
                                mn = x[j];
                                arg = j;
                            }
                        }
                    }
                    const float g = sigmoid_f(mean / (float)p.k), dpre = dy * mn * g * (1.f - g) / (float)p.k;
                    for (int j = 0; j < p.k; ++j) {
                        Xs[(j * m + ii) * xp + c] = dpre;
                        Ls[(j * m + ii) * xp + c] = j == arg ? dy * g : 0.f;
                        dAtt[(size_t)(p.row0 + j * p.n + i0 + ii) * d + c] = dpre;
                    }
                    continue;
                }
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                    e[j] = j < p.k ? expf(e[j] - mx) : 0.f;
                    den += e[j];
                }
                const float inv = 1.f / den;
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j) tall += e[j] * inv * x[j] * dy;
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                    if (j < p.k) {
                        const float wj = e[j] * inv, g = wj * (dy * x[j] - tall);
                        Xs[(j * m + ii) * xp + c] = g;
                        Ls[(j * m + ii) * xp + c] = wj * dy;
                        dAtt[(size_t)(p.row0 + j * p.n + i0 + ii) * d + c] = g;
                    }
                }
            }
            __syncthreads();
        }
        first.run(Xs, xp, [&](int n, floatx4 v) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int lr = (lane >> 4) * 4 + e, r = row_of[lr];
                const float y = Hs[lr * hp + n] > 0.f ? v[e] : 0.f;       // (zero beyond h)
                Hs[lr * hp + n] = y;
                if (r >= 0 && n < h) w.dH[(size_t)r * h + n] = y;
            }
        });
        __syncthreads();
        second.run(Hs, hp, [&](int n, floatx4 v) {
            if (n >= d) return;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int lr = (lane >> 4) * 4 + e;
                if (row_of[lr] >= 0) row_put1<CHAIN>(dact + (size_t)in_of[lr] * d + n, v[e] + (inter ? Ls[lr * xp + n] : 0.f));
            }
        });
    }
}

__device__ __forceinline__ int problem_of(const LevelTiles& t, int tile) {
    int q = 0;
    for (int i = 1; i < t.count; ++i)
        if (tile >= t.tile_start[i]) q = i;
    return q;
}

template <bool BWD, bool BOX>
__global__ __launch_bounds__(LV_T) void level_kernel(const LevelArgs a) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int q = problem_of(a.t, (int)blockIdx.x);
    level_tile<BWD, BOX, false>(a, a.t.p[q], (int)blockIdx.x - a.t.tile_start[q], lds, [] {});
}

struct LevelRun {                   // the first depth's tiles stand in a
    LevelArgs a;
    LevelTiles more[LEVEL_CHAIN - 1];
    int n, first[LEVEL_CHAIN + 1];      // depths, the first tile of each
    LevelSync sync;
    SmallIndex index;               // (n: 0 without one)
    PlanCopy copy;                  // (n: 0 without one)
};
static_assert(LV_T == SMALL_THREADS, "the index of few keys is a workgroup's job here too");
// INDEX: the first workgroup builds the gradient index meanwhile, which nothing here reads.  A launch of its own for it was 5 to 10 us
// of a small step (64 x 8 at 32, 64 68.0 -> 62.6 us, 64 x 16 at 100, 200 130 -> 120, 16 x 4 boxes at 64, 64 66 -> 56).
template <bool BWD, bool BOX, bool INDEX>
__global__ __launch_bounds__(LV_T) void levels_kernel(const LevelRun r) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ int number;
    if (INDEX && blockIdx.x == 0) {
        small_index(r.index, lds);
        return;
    }
    if (!BWD && r.copy.n > 0 && blockIdx.x == gridDim.x - 1) {
        for (int i = threadIdx.x; i < r.copy.n; i += LV_T) r.copy.dst[i] = r.copy.src[i];
        return;
    }
    // (requested here: where it is needed it would cost a round trip to the argument segment)
    int32_t* const counts = r.sync.counts;
    const int polls = r.sync.polls;
    asm volatile("" ::"s"(counts), "s"(polls));
    if (threadIdx.x == 0) number = __hip_atomic_fetch_add(counts, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int at = __builtin_amdgcn_readfirstlane(number);
    int l = 0;
    for (int i = 1; i < r.n; ++i)
        if (at >= r.first[i]) l = i;
    const LevelTiles& t = l == 0 ? r.a.t : r.more[l - 1];
    const int tile = at - r.first[l], q = problem_of(t, tile);
    bool there = true;              // (of the first thread; of the others nobody asks.  A tile that gave up goes on like any other: what it reads
                                    // are numbers, and a branch here would hold back the requests for what comes after the wait)
    level_tile<BWD, BOX, true>(r.a, t.p[q], tile - t.tile_start[q], lds, [&] {
        if (l > 0) there = wait_for_depth(counts + 1 + l, r.first[l] - r.first[l - 1], polls);
    });
    wait_vm<0>();                   // this wavefront's rows are where the next depth finds them,
    __syncthreads();                // ... and everybody's
    if (threadIdx.x != 0) return;
    if (!there) {
        __hip_atomic_store(r.sync.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(r.sync.host_gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // (nobody waits for the last depth; the counts of the others were seen in full by whoever gets there, so none of them can
    // still be on its way when they are cleared.  In a pass that gave up one can: nothing is launched on these counts any more)
    if (l + 1 < r.n) __hip_atomic_fetch_add(counts + 2 + l, there ? 1 : GAVE_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the last one through leaves the counts as they were found
    if (__hip_atomic_fetch_add(counts + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != r.first[r.n] - 1) return;
    for (int i = 0; i < LEVEL_SYNC; ++i) __hip_atomic_store(counts + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The forward pass of a handful of queries (every layer has a few rows only: gemm.hip's rows_kernel, whose sums these are): all layers of
// all depths in one launch.  As a launch a layer such a pass is bound by the host, 4 us each, and the first of them, which copies the plan,
// is spared too: the references travel as arguments and one more workgroup copies the plan for whoever follows.  A tile requests its weights,
// all of them, before it waits for the layer before; what an intersection pools are its tile's own columns.  Rows and values of one layer
// reach the next as in levels_kernel, and a wait ends like there; a tile that gave up leaves NaN, and so does then every tile of the layers behind it.
// Tiles are dealt by workgroup number (TileHelp), and a tile that is through says so by a bit of a word that few others share: tickets and counts, each in one word taken by a few
// hundred workgroups one after the other, were 14 us a layer; a tile that is taken before it is worked on costs the launch 3 us, a word a tile 1.
// Scoring against 1000 candidates, a launch a layer and like this, us a call with its plan, on average over six batches of all structures (those with an inner
// depth of too many words keep their launches): one query at d = 400, h = 800 41.3 and 26.7 (35 to 55 and 21 to 35), four 50.3 and 37.3, eight 60 and 52; one at 512, 1024 41.3
// and 27.0, eight at 132, 260 58 and 43.  Of a call of one query with three depths 23.4 are this launch.
constexpr int CHAIN_ROWS = 4, CHAIN_COLS = 4, CHAIN_T = 256;
constexpr int CHAIN_TILES = 2048;
static_assert(CHAIN_CARD <= CHAIN_ROWS && CHAIN_ROWS * CHAIN_COLS <= 64, "an intersection is a tile, its sums a lane each");
__host__ __device__ inline int chain_row_groups(const RowsProblem& p, bool second) {
    return second && p.k > 1 ? p.n : (p.n * p.k + CHAIN_ROWS - 1) / CHAIN_ROWS;
}
__host__ __device__ inline int chain_col_groups(int n) { return (n + 4 * CHAIN_COLS - 1) / (4 * CHAIN_COLS); }
// The bits of a lane's word once all `tiles` of a layer are through
__device__ __forceinline__ unsigned long long rows_all(int tiles, int lane) {
    return lane < CHAIN_LINES && lane < tiles ? (CHAIN_GAVE_UP - 1ull) >> (CHAIN_BITS - (tiles - lane + CHAIN_LINES - 1) / CHAIN_LINES) : 0ull;
}
__device__ __forceinline__ unsigned long long rows_word(const unsigned long long* layer, int line) {
    return __hip_atomic_load(layer + min(line, CHAIN_LINES - 1) * CHAIN_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until all tiles of the layer before l are through (helps: or there is one to compute meanwhile): TILE_GO, TILE_GAVE_UP or whose tile that is.  By one
// wavefront.
__device__ __forceinline__ int rows_wait(const RowsChain& r, const unsigned long long* through, int l, int polls, bool helps) {
    const int lane = threadIdx.x & 63;
    const unsigned long long want = rows_all(r.first[l] - r.first[l - 1], lane);
    int again = max(r.help.patience, 0);
    for (int i = 0; i < polls; ++i) {
        const unsigned long long now = rows_word(through + (l - 1) * CHAIN_LAYER, lane);
        if (__ballot(lane < CHAIN_LINES && now != want) == 0ull) return TILE_GO;
        if (__ballot(now >= CHAIN_GAVE_UP) != 0ull) break;
        if (__builtin_expect(helps && i >= again, 0)) {
            for (int m = 0; m < l; ++m) {        // (the first layer that is not through: it waits for nothing)
                const unsigned long long open = rows_all(r.first[m + 1] - r.first[m], lane) & ~rows_word(through + m * CHAIN_LAYER, lane);
                unsigned long long lines = __ballot(open != 0ull);
                if (lines == 0ull) continue;
                for (int skip = (int)blockIdx.x % __popcll(lines); skip > 0; --skip) lines &= lines - 1ull;       // (not all the same one)
                const int line = __ffsll(lines) - 1, bit = __builtin_amdgcn_readlane(__ffsll(open) - 1, line);
                if (lane == 0) __hip_atomic_fetch_add(r.help.helped, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return r.first[m] + bit * CHAIN_LINES + line;
            }
            again = i + TILE_AGAIN;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return TILE_GAVE_UP;
}
// The tile of workgroup `at`.  first: the workgroup that runs it begins with it; helps: may leave it for another one while it waits.  Returns whose tile to
// compute first (>= 0), or TILE_GO: done.
__device__ __forceinline__ int rows_tile(const RowsChain& r, int at, bool helps, bool first, float* lds, int* state) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));        // (where tiles are computed in a loop nothing that follows from it is kept from one to the next)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int layers = 2 * r.depths;
    const int polls = r.sync.polls;
    unsigned long long* const through = r.through;
    asm volatile("" ::"s"(polls), "s"(through));
    int l = 0;                       // layer: 2 * depth, and one more for the second of the depth
    for (int i = 1; i < layers; ++i)
        if (at >= r.first[i]) l = i;
    const bool second = l & 1;
    const int K = second ? r.h : r.d, N = second ? r.d : r.h, cols = chain_col_groups(N), in_layer = at - r.first[l];
    if (first && l + 1 < layers)
        tile_late(r.help, at, [&] { return (rows_word(through + l * CHAIN_LAYER, in_layer % CHAIN_LINES) >> (in_layer / CHAIN_LINES) & 1ull) != 0ull; });
    int tile = in_layer, q = 0;
    for (; q + 1 < r.count[l >> 1]; ++q) {
        const int n = chain_row_groups(r.p[l >> 1][q], second) * cols;
        if (tile < n) break;
        tile -= n;
    }
    const RowsProblem p = r.p[l >> 1][q];
    const int rg = tile / cols, nb = tile - rg * cols;
    const bool pooled = second && p.k > 1;
    const int M = pooled ? p.k : min(CHAIN_ROWS, p.n * p.k - rg * CHAIN_ROWS), row_lo = pooled ? rg : rg * CHAIN_ROWS, row_step = pooled ? p.n : 1;
    const int n0 = (nb * 4 + wave) * CHAIN_COLS, k4 = K >> 2;
    const float* W = second ? r.Wb[p.type] : r.Wa[p.type];
    const float* bias_of = second ? r.bb[p.type] : r.ba[p.type];
    float4 w[CHAIN_COLS][CHAIN_WIDTH / 256];
#pragma unroll
    for (int c = 0; c < CHAIN_WIDTH / 256; ++c)
#pragma unroll
        for (int j = 0; j < CHAIN_COLS; ++j)
            if (c * 64 < k4) w[j][c] = *reinterpret_cast<const float4*>(W + (size_t)min(n0 + j, N - 1) * K + min(c * 64 + lane, k4 - 1) * 4);
    float bias[CHAIN_COLS];
#pragma unroll
    for (int j = 0; j < CHAIN_COLS; ++j) bias[j] = bias_of[min(n0 + j, N - 1)];
    // a wavefront takes an input row (the last one again where there are fewer)
    const int mine = row_lo + min(wave, M - 1) * row_step;
    const int32_t ref = second ? 0 : r.words[p.at + mine];
    const bool related = !second && p.type == 0;
    const float* rel = r.R + (related ? (size_t)r.words[p.at + p.n + mine] * K : 0);
    // (lane CHAIN_COLS m + j stores column n0 + j of row m, and has that of input m of an intersection)
    const int m_out = pooled ? 0 : min(lane / CHAIN_COLS, M - 1), col = n0 + lane % CHAIN_COLS;
    const int out_row = second ? r.words[p.at + p.n * p.k + (p.type == 0 ? p.n : 0) + row_lo + m_out] : p.row0 + row_lo + m_out;
    float* const to = (second ? r.act : r.H[p.type]) + (size_t)out_row * N + col;
    float4 x[CHAIN_WIDTH / 256], y[CHAIN_WIDTH / 256];
#pragma unroll
    for (int c = 0; c < CHAIN_WIDTH / 256; ++c) {
        const int k = min(c * 64 + lane, k4 - 1) * 4;
        if (related && c * 64 < k4) y[c] = *reinterpret_cast<const float4*>(rel + k);
        if (ref < 0 && c * 64 < k4) x[c] = *reinterpret_cast<const float4*>(r.E + (size_t)(-1 - ref) * K + k);
    }
    int got = TILE_GO;
    if (l > 0) {
        if (wave == 0) {
            got = rows_wait(r, through, l, polls, helps);
            if (lane == 0) *state = got;
        }
        asm volatile("" ::: "memory");
        __syncthreads();
    }
    if (ref >= 0) {
        const float* row = second ? r.H[p.type] + (size_t)(p.row0 + mine) * K : r.act + (size_t)ref * K;
#pragma unroll
        for (int c = 0; c < CHAIN_WIDTH / 256; ++c)
            if (c * 64 < k4) x[c] = row_get<true>(row + min(c * 64 + lane, k4 - 1) * 4);
    }
    float input = 0.f;
    if (pooled) input = row_get1<true>(r.Z + (size_t)(p.row0 + row_lo + min(lane / CHAIN_COLS, p.k - 1) * row_step) * r.d + min(col, N - 1));
    if (l > 0) {                     // (looked at when the rows are requested)
        got = __builtin_amdgcn_readfirstlane(*state);
        if (got >= 0) return got;
    }
    const bool there = got == TILE_GO;
    if (wave < M) {
#pragma unroll
        for (int c = 0; c < CHAIN_WIDTH / 256; ++c) {
            if (c * 64 + lane >= k4) break;
            float4 v = x[c];
            if (related) { v.x += y[c].x; v.y += y[c].y; v.z += y[c].z; v.w += y[c].w; }
            *reinterpret_cast<float4*>(lds + wave * K + (c * 64 + lane) * 4) = v;
            if (nb == 0 && !second && p.k > 1) row_put<true>(r.Z + (size_t)(p.row0 + mine) * K + (c * 64 + lane) * 4, v);
        }
    }
    __syncthreads();
    float out = 0.f, sum[CHAIN_ROWS][CHAIN_COLS];
#pragma unroll
    for (int m = 0; m < CHAIN_ROWS; ++m) {
        if (m >= M) continue;        // uniform
        float acc[CHAIN_COLS];
#pragma unroll
        for (int j = 0; j < CHAIN_COLS; ++j) acc[j] = 0.f;
#pragma unroll
        for (int c = 0; c < CHAIN_WIDTH / 256; ++c) {
            if (c * 64 + lane >= k4) break;
            const float4 v = *reinterpret_cast<const float4*>(lds + m * K + (c * 64 + lane) * 4);
#pragma unroll
            for (int j = 0; j < CHAIN_COLS; ++j) acc[j] += (v.x * w[j][c].x + v.y * w[j][c].y) + (v.z * w[j][c].z + v.w * w[j][c].w);
        }
#pragma unroll
        for (int j = 0; j < CHAIN_COLS; ++j) {
            float v = wave_sum_dpp(acc[j]) + bias[j];
            if (!second) v = fmaxf(v, 0.f);
            sum[m][j] = v;
            if (lane == m * CHAIN_COLS + j) out = v;
        }
    }
    if (pooled) {
#pragma unroll
        for (int j = 0; j < CHAIN_COLS; ++j) {
            float mx = -INFINITY, den = 0.f, v = 0.f;
#pragma unroll
            for (int m = 0; m < CHAIN_ROWS; ++m)
                if (m < M) mx = fmaxf(mx, sum[m][j]);
#pragma unroll
            for (int m = 0; m < CHAIN_ROWS; ++m) {
                sum[m][j] = m < M ? expf(sum[m][j] - mx) : 0.f;
                den += sum[m][j];
            }
            const float inv = 1.f / den;
#pragma unroll
            for (int m = 0; m < CHAIN_ROWS; ++m)
                if (m < M) v += sum[m][j] * inv * lane_value(input, m * CHAIN_COLS + j);
            if (lane == j) out = v;
        }
    }
    if (!there) out = NAN;
    if (lane < (pooled ? 1 : M) * CHAIN_COLS && col < N) row_put1<true>(to, out);
    wait_vm<0>();                    // this wavefront's values are where the next layer finds them,
    __syncthreads();                 // ... and everybody's
    if (tid == 0) {
        if (!there) {
            __hip_atomic_store(r.sync.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(r.sync.host_gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (l + 1 < layers)
            __hip_atomic_fetch_or(through + l * CHAIN_LAYER + in_layer % CHAIN_LINES * CHAIN_STRIDE, there ? 1ull << (in_layer / CHAIN_LINES) : CHAIN_GAVE_UP, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    return TILE_GO;
}
__global__ __launch_bounds__(CHAIN_T) void rows_chain_kernel(const RowsChain r) {
    extern __shared__ __attribute__((aligned(16))) float lds[];      // [CHAIN_ROWS][K]
    __shared__ int state;
    const int own = (int)blockIdx.x;
    if (own == r.first[2 * r.depths]) {           // (only where there is something to copy)
        for (int i = threadIdx.x; i < r.copy.n; i += CHAIN_T) r.copy.dst[i] = r.copy.src[i];
        return;
    }
    if (own + 1 == r.first[2 * r.depths])         // (a tile that has time)
        for (int i = threadIdx.x; i < 2 * LEVEL_CHAIN * CHAIN_LINES; i += CHAIN_T) r.clear[i * CHAIN_STRIDE] = 0ull;
    int other = rows_tile(r, own, true, true, lds, &state);
    if (__builtin_expect(other < 0, 1)) return;
    // (code of its own: around the tile above this loop would cost it registers)
#pragma clang loop unroll(disable)
    for (;;) {
        __syncthreads();
        int again = 0;               // (and no argument is kept from tile to tile)
        asm volatile("" : "+s"(again));
        const bool home = other < 0;
        other = rows_tile((&r)[again], home ? own : other, home, false, lds, &state);
        if (home && other < 0) return;
    }
}

size_t lv_lds(int d, int h) { return ((size_t)LV_ROWS * (2 * lv_pitch(d) + lv_pitch(h)) + d + h) * sizeof(float); }

}  // namespace

bool level_add(LevelArgs& a, int type, int pool, int n, int k, int ref_off, int rel_off, int row0, int out0) {
    if (n <= 0) return true;
    LevelTiles& t = a.t;
    if (t.count == LEVEL_MAX || k < 1 || k > NGDB_MAX_CARD) return false;
    t.p[t.count] = LevelProblem{type, pool, n, k, ref_off, rel_off, row0, out0};
    const int m = LV_ROWS / k;
    t.tile_start[t.count + 1] = t.tile_start[t.count] + (n + m - 1) / m;
    return (long)t.tile_start[++t.count] * a.d * a.h <= LEVEL_WORK;
}

bool level_fits(int d, int h, bool box) { return d <= 256 && h <= 512 && d * h <= (box ? LEVEL_WEIGHTS_BOX : LEVEL_WEIGHTS); }

hipError_t launch_level(const LevelArgs& a, bool backward, hipStream_t s) {
    if (a.t.count == 0) return hipSuccess;
    if (!level_fits(a.d, a.h, true) || (a.d & 3) || (a.h & 3)) return hipErrorInvalidValue;
    const dim3 grid(a.t.tile_start[a.t.count]);
    const size_t lds = lv_lds(a.d, a.h);
    if (a.off && backward) hipLaunchKernelGGL((level_kernel<true, true>), grid, dim3(LV_T), lds, s, a);
    else if (a.off) hipLaunchKernelGGL((level_kernel<false, true>), grid, dim3(LV_T), lds, s, a);
    else if (backward) hipLaunchKernelGGL((level_kernel<true, false>), grid, dim3(LV_T), lds, s, a);
    else hipLaunchKernelGGL((level_kernel<false, false>), grid, dim3(LV_T), lds, s, a);
    return hipGetLastError();
}

bool rows_chain_lay_out(RowsChain& r) {
    if (r.depths < 1 || r.depths > LEVEL_CHAIN || r.d < 4 || r.h < 4 || (r.d & 3) || (r.h & 3) || std::max(r.d, r.h) > CHAIN_WIDTH || r.n_words > CHAIN_WORDS) return false;
    int tiles = 0;
    for (int l = 0; l < 2 * r.depths; ++l) {
        if (l > 0 && tiles - r.first[l - 1] > CHAIN_LINES * CHAIN_BITS) return false;
        r.first[l] = tiles;
        if (r.count[l >> 1] < 1 || r.count[l >> 1] > CHAIN_PROBLEMS) return false;
        for (int q = 0; q < r.count[l >> 1]; ++q) {
            const RowsProblem& p = r.p[l >> 1][q];
            if (p.n < 1 || p.k < 1 || p.k > CHAIN_CARD || p.type < 0 || p.type > 2 || p.at < 0 || p.at + p.n * (p.k + 1 + (p.type == 0 ? 1 : 0)) > r.n_words) return false;
            tiles += chain_row_groups(p, l & 1) * chain_col_groups(l & 1 ? r.d : r.h);
        }
    }
    for (int l = 2 * r.depths; l <= 2 * LEVEL_CHAIN; ++l) r.first[l] = tiles;
    return tiles <= CHAIN_TILES;
}

hipError_t launch_rows_chain(const RowsChain& r, hipStream_t s) {
    const int tiles = r.first[2 * LEVEL_CHAIN];
    if (tiles < 1 || tiles > CHAIN_TILES || !r.through || !r.clear || !r.help.helped || !r.sync.gave_up || !r.sync.host_gave_up || r.copy.n < 0 ||
        (r.copy.n > 0 && (!r.copy.src || !r.copy.dst)))
        return hipErrorInvalidValue;
    const size_t bytes = (size_t)CHAIN_ROWS * std::max(r.d, r.h) * sizeof(float);
    hipLaunchKernelGGL(rows_chain_kernel, dim3(tiles + (r.copy.n > 0 ? 1 : 0)), dim3(CHAIN_T), bytes, s, r);
    return hipGetLastError();
}

bool levels_chain(const LevelArgs* a, int n) {
    int tiles = 0;
    for (int l = 0; l < n; ++l) {
        if (a[l].t.count == 0) return false;
        tiles += a[l].t.tile_start[a[l].t.count];
    }
    return n > 1 && n <= LEVEL_CHAIN && tiles <= LEVEL_CHAIN_TILES;
}

hipError_t launch_levels(const LevelArgs* a, int n, bool backward, const LevelSync& sync, const SmallIndex* index, const PlanCopy& copy, hipStream_t s) {
    if (!levels_chain(a, n) || !sync.counts || !sync.gave_up || !sync.host_gave_up || !level_fits(a[0].d, a[0].h, true) || (a[0].d & 3) || (a[0].h & 3)) return hipErrorInvalidValue;
    LevelRun r{};
    r.a = a[0];
    r.n = n;
    r.sync = sync;
    for (int l = 0; l < n; ++l) {
        if (l > 0) r.more[l - 1] = a[l].t;
        r.first[l + 1] = r.first[l] + a[l].t.tile_start[a[l].t.count];
    }
    const bool with_index = index && index->n > 0;
    if (with_index && backward) return hipErrorInvalidValue;
    if (with_index) r.index = *index;
    if (copy.n < 0 || (copy.n > 0 && (backward || !copy.src || !copy.dst))) return hipErrorInvalidValue;
    r.copy = copy;
    const dim3 grid(r.first[n] + (with_index ? 1 : 0) + (copy.n > 0 ? 1 : 0));
    const size_t lds = std::max(lv_lds(r.a.d, r.a.h), with_index ? SMALL_INDEX_LDS : 0);
#define NGDB_LEVELS(...)                                                                                                                    \
    do {                                                                                                                                    \
        if (lds > 64 * 1024)                                                                                                                \
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(levels_kernel<__VA_ARGS__>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
        hipLaunchKernelGGL((levels_kernel<__VA_ARGS__>), grid, dim3(LV_T), lds, s, r);                                                      \
    } while (0)
    if (r.a.off && backward) NGDB_LEVELS(true, true, false);
    else if (r.a.off && with_index) NGDB_LEVELS(false, true, true);
    else if (r.a.off) NGDB_LEVELS(false, true, false);
    else if (backward) NGDB_LEVELS(true, false, false);
    else if (with_index) NGDB_LEVELS(false, false, true);
    else NGDB_LEVELS(false, false, false);
#undef NGDB_LEVELS
    return hipGetLastError();
}

}  // namespace ngdb
