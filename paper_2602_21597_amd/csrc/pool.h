// Pooling of intersections, both families: a thread takes four coordinates of a member.  The cardinality is
// that of the whole job: classes of two and three inputs, nearly all there are, read what they need and no more
// (walking every class to the largest cardinality under a predicate, a coordinate a thread, read 16 words where a class of two needs
// four).  Backward, d = 400, us a launch: 512 queries 4.7 -> 4.1, 1024 7.6 -> 5.3, 4096 15.5 -> 11.2, 509 boxes 5.4 -> 4.4.
#pragma once
#include "common.h"

namespace ngdb {
namespace pool {

struct Four { float v[4]; };
__device__ __forceinline__ Four load4(const float* p) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    return {{x.x, x.y, x.z, x.w}};
}
__device__ __forceinline__ void store4(float* p, const Four& f) { *reinterpret_cast<float4*>(p) = make_float4(f.v[0], f.v[1], f.v[2], f.v[3]); }

// y_i = sum_j softmax_j(att_j)_c * x_j,c over k <= K inputs of member i, coordinates c .. c + 3 (k == K unless K is the largest cardinality)
template <bool BWD, int K>
__device__ __forceinline__ void attention(const InterJob& jb, int d, int i, int c) {
    const int n = jb.n, k = K == NGDB_MAX_CARD ? jb.k : K;
    Four a[K], x[K], dy{}, y{};
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const size_t at = ((size_t)min(j, k - 1) * n + i) * d + c;
        a[j] = load4(jb.Att + at);
        x[j] = load4(jb.X + at);
    }
    if (BWD) dy = load4(jb.dY + (size_t)i * d + c);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float mx = -INFINITY, den = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (j < k) mx = fmaxf(mx, a[j].v[q]);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            a[j].v[q] = j < k ? expf(a[j].v[q] - mx) : 0.f;
            den += a[j].v[q];
        }
        const float inv = 1.f / den;
        if (!BWD) {
#pragma unroll
            for (int j = 0; j < K; ++j) y.v[q] += a[j].v[q] * inv * x[j].v[q];
        } else {
            const float g = dy.v[q];
            float tall = 0.f;
#pragma unroll
            for (int j = 0; j < K; ++j) tall += a[j].v[q] * inv * x[j].v[q] * g;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const float w = a[j].v[q] * inv;
                a[j].v[q] = w * (g * x[j].v[q] - tall);
                x[j].v[q] = w * g;
            }
        }
    }
    if (!BWD) {
        store4(jb.out + (size_t)(jb.out_row ? jb.out_row[i] : i) * d + c, y);
        return;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j >= k) break;
        const size_t at = ((size_t)j * n + i) * d + c;
        store4(jb.dAtt + at, a[j]);
        store4(jb.Dx + at, x[j]);
    }
}

// Offsets of boxes: the smallest input offset times sigmoid of the mean gate; the first of equal offsets takes the gradient
template <bool BWD, int K>
__device__ __forceinline__ void smallest(const InterJob& jb, int d, int i, int c) {
    const int n = jb.n, k = K == NGDB_MAX_CARD ? jb.k : K;
    Four g[K], x[K], dy{}, y{}, dpre{};
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const size_t at = ((size_t)min(j, k - 1) * n + i) * d + c;
        g[j] = load4(jb.Att + at);
        x[j] = load4(jb.X + at);
    }
    if (BWD) dy = load4(jb.dY + (size_t)i * d + c);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float mean = 0.f, mn = INFINITY;
        int arg = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (j >= k) break;
            mean += g[j].v[q];
            if (x[j].v[q] < mn) {       // strict: equal offsets keep the lower input
                mn = x[j].v[q];
                arg = j;
            }
        }
        const float gate = sigmoid_f(mean / (float)k);
        if (!BWD) {
            y.v[q] = mn * gate;
        } else {
            const float up = dy.v[q];
            dpre.v[q] = up * mn * gate * (1.f - gate) / (float)k;
#pragma unroll
            for (int j = 0; j < K; ++j) x[j].v[q] = j == arg ? up * gate : 0.f;
        }
    }
    if (!BWD) {
        store4(jb.out + (size_t)i * d + c, y);
        return;
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j >= k) break;
        const size_t at = ((size_t)j * n + i) * d + c;
        store4(jb.dAtt + at, dpre);
        store4(jb.Dx + at, x[j]);
    }
}

// thread t of a job (k is uniform)
template <bool BWD, bool OFFSETS>
__device__ __forceinline__ void member(const InterJob& jb, int d, size_t t) {
    const int d4 = d >> 2;
    if (t >= (size_t)jb.n * d4) return;
    const int i = (int)(t / d4), c = (int)(t % d4) * 4;
    if (jb.k == 2) OFFSETS ? smallest<BWD, 2>(jb, d, i, c) : attention<BWD, 2>(jb, d, i, c);
    else if (jb.k == 3) OFFSETS ? smallest<BWD, 3>(jb, d, i, c) : attention<BWD, 3>(jb, d, i, c);
    else OFFSETS ? smallest<BWD, NGDB_MAX_CARD>(jb, d, i, c) : attention<BWD, NGDB_MAX_CARD>(jb, d, i, c);
}
constexpr int THREADS = 128;      // (few members a depth: more workgroups)

}  // namespace pool
}  // namespace ngdb
