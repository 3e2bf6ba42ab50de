// Shared declarations of the library's translation units (host side) and the
// small device helpers every kernel file uses.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <utility>

#include "ngdb.h"

namespace ngdb {

constexpr int WAVE = 64;

// ---------------------------------------------------------------- device helpers
#if defined(__HIPCC__)
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}
__device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }
__device__ __forceinline__ float sgn(float x) { return (float)((x > 0.f) - (x < 0.f)); }
// bf16 bit patterns <-> fp32 (round to nearest, ties to even)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float x) {
    const uint32_t b = __float_as_uint(x);
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_round_f32(float x) { return __uint_as_float(f32_to_bf16_bits(x) << 16); }
// 4 consecutive bf16 values (8 bytes) -> float4
__device__ __forceinline__ float4 bf16x4_to_f32(uint2 v) {
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xFFFF0000u));
}
// Sum over the 64 lanes of a wavefront on the vector ALU alone (data-parallel primitives: adds inside
// quads, inside rows of 16 lanes, then across the four rows through row broadcasts), returned in
// every lane.  No LDS round trips: a chain of six ds_bpermute exchanges costs several hundred
// cycles of latency per sum.  Fixed summation order.
__device__ __forceinline__ float wave_sum_dpp(float v) {
#define NGDB_DPP_ADD(ctrl, rows)                                                                        \
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xf, false))
    NGDB_DPP_ADD(0xB1, 0xf);    // quad_perm [1,0,3,2]: lane ^ 1
    NGDB_DPP_ADD(0x4E, 0xf);    // quad_perm [2,3,0,1]: lane ^ 2
    NGDB_DPP_ADD(0x141, 0xf);   // row_half_mirror: the other quad of the half row
    NGDB_DPP_ADD(0x140, 0xf);   // row_mirror: the other half row -> every lane holds its row's sum
    NGDB_DPP_ADD(0x142, 0xa);   // row_bcast15 into rows 1 and 3: sums of rows 0+1 and 2+3
    NGDB_DPP_ADD(0x143, 0xc);   // row_bcast31 into rows 2 and 3: row 3 holds the total
#undef NGDB_DPP_ADD
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
// The value lane `l` holds, for an l that is the same in all lanes: a register read, where a
// shuffle with a per-lane index would go through LDS hardware.
__device__ __forceinline__ int32_t lane_value(int32_t v, int l) {
    return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(l));
}
__device__ __forceinline__ float lane_value(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), __builtin_amdgcn_readfirstlane(l)));
}
// A direct load from global memory into LDS (gfx950): lane l's 16 (4) bytes land at lds_base + l * 16 (4), whatever
// global address the lane gives; lds_base is wave-uniform (it travels in M0).  The loads are
// issued from inline assembly and waited for by hand (s_waitcnt vmcnt): left to the compiler,
// every LDS read after such a load would wait for all of them, also those of the stages ahead.
__device__ __forceinline__ void lds_load16(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory");
}
// the same from a wave-uniform address and a lane's byte offset
__device__ __forceinline__ void lds_load16_at(const void* base, uint32_t offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(offset), "s"(base) : "memory");
}
__device__ __forceinline__ void lds_load4(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory");
}
// What workgroups of one launch hand to each other across the dies: loads and stores past the L2s, at the scope of the card.
__device__ __forceinline__ void lds_load16_card(const void* gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off sc1" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(gptr) : "memory");
}
__device__ __forceinline__ float2 card_get2(const float* p) {          // (8-byte aligned, like the next)
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}
__device__ __forceinline__ void card_put2(float* p, float x, float y) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__float_as_uint(y) << 32 | __float_as_uint(x), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
// at most n vector-memory operations of this wavefront still in flight (they complete in order)
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt has 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// all LDS operations of this wavefront done
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4)); }
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// Hardware transcendental approximations (about 1 ulp each; the results they feed are held to 1e-4).
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
// exp(-a) for a >= 0
__device__ __forceinline__ float fast_exp_neg(float a) { return __builtin_amdgcn_exp2f(a * -1.44269504088896341f); }
// log(1 + e) for 0 <= e <= 1: the series where 1 + e would lose e's bits, else the hardware logarithm
__device__ __forceinline__ float fast_log1p_unit(float e) {
    const float series = e * (1.f - e * (0.5f - e * (1.f / 3.f)));
    const float direct = __builtin_amdgcn_logf(1.f + e) * 0.693147180559945309f;
    return e < 0.01f ? series : direct;
}
// sign(x) as -1, 0 or +1 in two instructions and without the condition register: x scaled by 2^252
// is 0 for 0, at least 2^103 in size for every other finite x (denormals included), or infinite;
// clamped to [-1, 1].  c * sign(x) then fuses into the accumulating multiply-add.
__device__ __forceinline__ float sign_unit(float x) {
    return __builtin_amdgcn_fmed3f(__builtin_ldexpf(x, 252), -1.f, 1.f);
}
__device__ __forceinline__ float signed_by(float c, float x) { return c * sign_unit(x); }
// ---- the integer grid of a filtered ranking (rank_filter.hip): a coordinate becomes q = round((x - lo) * inv) within [0, top], the
// grid point lo + step * q; what the row errs by is summed exactly.
// SLACK: of a row's own sums.  A lane adds up to 16 terms (quantise_kernel) or 52 (sem_fuse_kernel) one after the other, then a tree of at
// most six levels follows; a rounding of half a unit each, and some more for the terms themselves: 1.5e-6 and 4e-6.
constexpr float SLACK = 1e-5f;
constexpr int SLACK_TERMS = 64;      // a lane may add as many
static_assert((SLACK_TERMS + 6 + 8) * 6e-8f < SLACK, "the slack covers the sums' rounding");
constexpr int32_t SLACK_CAP = 100000000;      // an error of this or more bounds nothing (a row's parts are added, each capped)
__device__ __forceinline__ float to_grid(float x, float lo, float step, float inv, float top, float* err) {
    const float qf = fminf(fmaxf(rintf((x - lo) * inv), 0.f), top);           // (a NaN becomes 0; its error stays NaN)
    const float on = fmaf(qf, step, lo);                                       // the grid point, itself rounded
    *err += fabsf(x - on) + fabsf(on) * 6e-8f;
    return qf;
}
__device__ __forceinline__ int32_t slack_steps(float err, float inv) {         // in steps, rounded up
    const float s = err * (1.f + SLACK) * inv + 2.f;
    return s < (float)SLACK_CAP ? (int32_t)s : SLACK_CAP;
}
// log(1+exp(x)) and 1/(1+exp(-x)) without overflow
__device__ __forceinline__ float softplus_f(float x) { return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x))); }
__device__ __forceinline__ float sigmoid_f(float x) {
    const float e = expf(-fabsf(x));
    return x >= 0.f ? 1.f / (1.f + e) : e / (1.f + e);
}
#endif

// ---------------------------------------------------------------- GEMM (gemm.hip)
// C[M,N] = A[M,K] * B[K,N] with fp32 MFMA.  Element (m,k) of A is at
// A[m*lda+k] if a_kcontig else A[k*lda+m]; element (k,n) of B is at B[n*ldb+k]
// if b_kcontig else B[k*ldb+n].  Epilogue, in this order: + bias[n]; relu;
// * (mask[m*ldmask+n] > 0); + addend[m*ldadd+n]; row m goes to C row
// dst_row[m] if dst_row else m.
// Fused gather (k-contiguous A only): if a_ref is set, row m of A is
// a_base0 + a_ref[m]*lda for a_ref[m] >= 0, else a_base1 + (-1-a_ref[m])*lda, plus
// row a_add_idx[m] of a_add if a_add_idx is set; the assembled rows are also
// written to a_copy (same leading dimension) if it is set.
struct GemmArgs {
    const int32_t* a_ref = nullptr;
    const float* a_base0 = nullptr;
    const float* a_base1 = nullptr;
    const int32_t* a_add_idx = nullptr;
    const float* a_add = nullptr;
    float* a_copy = nullptr;
    const float* A = nullptr;
    const float* B = nullptr;
    float* C = nullptr;
    const float* bias = nullptr;
    const float* mask = nullptr;
    const float* addend = nullptr;
    const int32_t* dst_row = nullptr;
    const uint16_t* b_pieces = nullptr;
    // The same for A (rows of A in blocks of 32: tile (m / 32, k / 16), a_kt tiles per block row), and
    // for the output, written once more in that form where c_pieces is given (c_kt tiles per block
    // row, at least 2 * ceil(N / 32); no dst_row) for the launch that reads it as its A operand.
    const uint16_t* a_pieces = nullptr;
    uint16_t* c_pieces = nullptr;
    // The output rows are the logits of intersections of pool_k inputs (row j * n + i: input j of member i, M = n * pool_k):
    // row i of pool_out, or row pool_row[i], receives sum_j softmax_j(C[j * n + i]) * pool_X[j * n + i] (leading dimension ldc).
    // C may be null then.  Only launches of split weights do this; others return hipErrorNotSupported.
    const float* pool_X = nullptr;
    float* pool_out = nullptr;
    const int32_t* pool_row = nullptr;
    int pool_k = 0;
    int M = 0, N = 0, K = 0;
    int lda = 0, ldb = 0, ldc = 0;
    int ldmask = 0, ldadd = 0;
    int b_kt = 0, a_kt = 0, c_kt = 0;
    int a_row0 = 0;                // row 0 of A is row a_row0 of a_pieces (with pool_k only)
    int arith = 0;                 // GEMM_AUTO / GEMM_FP32 / GEMM_SPLIT: how the products are formed
    bool a_kcontig = true, b_kcontig = true;
    bool relu = false;
};
// GEMM_FP32: fp32 MFMA.  GEMM_SPLIT: every fp32 operand value as the exact sum of three bf16
// values, the six largest of the nine partial products on the bf16 MFMA with fp32 accumulation
// (what is left out is below 2^-23 of a product, about 2^-27 on average).  GEMM_AUTO: GEMM_SPLIT
// where it is faster, else GEMM_FP32.
constexpr int GEMM_AUTO = 0, GEMM_FP32 = 1, GEMM_SPLIT = 2;
hipError_t launch_gemm(const GemmArgs& a, hipStream_t s);
// Up to GEMM_MAX_GROUP independent contractions with the same operand layout in one
// launch (the operator groups of one depth, or the weight gradients of all types).
constexpr int GEMM_MAX_GROUP = 6;
template <int MOST_>
struct GemmGroupOf {
    static constexpr int MOST = MOST_;
    int count;
    int tile_start[MOST + 1];             // first workgroup of every problem
    GemmArgs p[MOST];
};
using GemmGroup = GemmGroupOf<GEMM_MAX_GROUP>;
// *route (if given) receives the arithmetic the launch used: GEMM_FP32 or GEMM_SPLIT; *emitted (if
// given) whether the launch wrote c_pieces (only gemm_kernel does where it reads its B operand as pieces,
// in launches of few tiles, and only if every problem of the group asks for it).
// *kernel (if given) receives which kernel the launch went to.
enum GemmKernel { GEMM_K_TILES, GEMM_K_PRODUCT_ONE, GEMM_K_PRODUCT_PAIR, GEMM_K_ROWS };
hipError_t launch_gemm_group(const GemmArgs* problems, int count, hipStream_t s, int* route = nullptr, bool* emitted = nullptr, int* kernel = nullptr);
// Weight gradients: C[M,N] = A^T B over the K rows of A [K][lda] and B [K][ldb] (the rows of an operator type),
// and colsum[m] = sum of column m of A (the gradient of the layer's bias).  M, N and the leading
// dimensions multiples of 4; K >= 0.  Up to GEMM_MAX_GROUP of them in one launch.
struct WgradArgs {
    const float *A, *B;
    float *C, *colsum;
    int M, N, K, lda, ldb, ldc;
};
hipError_t launch_wgrad_group(const WgradArgs* problems, int count, hipStream_t s, bool aside = false);

// Whether a forward layer of M rows is computed row by row (and has no use for split weights).
bool gemm_takes_rows(int M, int K);

// A row-major matrix W [R][C] as B operand of the bf16 MFMA block in both forms, each value split
// into three bf16 pieces, stored tile by tile (32 n x 16 k) in lane order and zero beyond the
// matrix: out_rk holds B[n = row][k = column] (ceil(R/32) x ceil(C/16) tiles), out_ck holds
// B[n = column][k = row] (ceil(C/32) x ceil(R/16) tiles).  C a multiple of 4.
constexpr int PIECE_MAX_JOBS = 6;
struct PieceJob {
    const float* W;
    uint16_t *out_rk, *out_ck;     // (out_ck may be null)
    int R, C;
};
struct PieceJobs {
    int count;
    PieceJob job[PIECE_MAX_JOBS];
    int block0[PIECE_MAX_JOBS + 1];
    // and copy_n x 16 bytes from copy_src to copy_dst (a plan, from host memory) by the first copy_blocks workgroups
    float4* copy_dst;
    const float4* copy_src;
    int copy_n, copy_blocks;
    // and clear_n words from clear on are zero afterwards (those that launches of several layers count in)
    int32_t* clear;
    int clear_n;
};
inline size_t pieces_elems(int N, int K) { return (size_t)((N + 31) / 32) * ((K + 15) / 16) * 1536; }
hipError_t launch_weight_pieces(PieceJobs& jobs, hipStream_t s);

// ---------------------------------------------------------------- elementwise ops (ops.hip)
// Intersections of one level, one job per cardinality class: n members with k inputs each,
// rows j*n+i of X (inputs) and Att (logits).  Forward: out[i] = sum_j w_j x_j, w = softmax over
// the inputs per coordinate.  Backward: dAtt[j*n+i] = w_j*(dy*x_j - sum_l w_l dy x_l),
// Dx[j*n+i] = w_j*dy.
constexpr int INTER_MAX_JOBS = 8;
struct InterJob {
    const float *X, *Att, *dY;
    float *out, *dAtt, *Dx;
    int n, k;
    const int32_t* out_row;   // forward: member i is written to row out_row[i] of out (null: row i)
};
struct InterJobs {
    int count;
    int d;
    InterJob job[INTER_MAX_JOBS];
};
hipError_t launch_inter(const InterJobs& jobs, bool backward, hipStream_t s);
// Box family, offset part of the intersections (same job layout: X = the inputs' offsets, Att =
// the per-input outputs of the offset MLP).  Forward: out[i] = min_j x_j * sigmoid(mean_j att_j).
// Backward: dAtt[j*n+i] = dy * min * g(1-g) / k;  Dx[j*n+i] = dy * g for the first j attaining
// the minimum, 0 for the others.
hipError_t launch_box_offset(const InterJobs& jobs, bool backward, hipStream_t s);

// Box family, projections of one group: member i reads its input box through ref[i] (slot, or
// -1-entity: centre E[e], offset 0) and writes (c + Rc[rel[i]], o + relu(Ro[rel[i]])) to slot
// out_base + i.  Backward copies the gradient rows of slot out_base + i (centre and offset) to
// the input's gradient rows gslot[i].
struct BoxProjArgs {
    const int32_t *ref, *gslot, *rel;
    const float *E, *Rc, *Ro;
    float *act_c, *act_o, *dact_c, *dact_o;
    int n, d, out_base;
};
hipError_t launch_box_proj(const BoxProjArgs& a, bool backward, hipStream_t s);
// Both poolings of the box family's intersections in one launch: jobs flagged in gate_mask are
// offset jobs (launch_box_offset), the others centre jobs (launch_inter).  With has_proj the
// projections of a group of the same level (independent of the intersections) ride along as
// one more job.
struct BoxPoolJobs {
    InterJobs jobs;
    uint32_t gate_mask;
    int has_proj;
    BoxProjArgs proj;
};
hipError_t launch_box_pool(const BoxPoolJobs& jobs, bool backward, hipStream_t s);
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
// calibration access patterns (ngdb_debug_stream)
hipError_t launch_stream_pattern(int mode, void* dst, const void* src, size_t bytes, const int32_t* rows, int64_t n_rows,
                                 int row_floats, hipStream_t s);

struct AdamHyper {
    float lr, beta1, beta2, eps;
    float bc1, bc2;   // 1 - beta^t for the step being applied
    const int32_t* gave_up = nullptr;      // nothing is updated if this word is set (null: none): gradients of a pass that gave up
};
struct DenseAdamJob {
    float* p[13];
    float* m[13];
    float* v[13];
    const float* g[13];
    int64_t n[13];
    int count;
};
#ifdef __HIPCC__
// one tensor by the threads start, start + stride, ...
__device__ __forceinline__ void dense_adam(const DenseAdamJob& job, int t, const AdamHyper& hp, int64_t start, int64_t stride) {
    float* __restrict__ p = job.p[t];
    float* __restrict__ m = job.m[t];
    float* __restrict__ v = job.v[t];
    const float* __restrict__ g = job.g[t];
    const int64_t n = hp.gave_up && *hp.gave_up != 0 ? 0 : job.n[t];
    for (int64_t i = start; i < n; i += stride) {
        const float gi = g[i];
        const float mi = hp.beta1 * m[i] + (1.f - hp.beta1) * gi;
        const float vi = hp.beta2 * v[i] + (1.f - hp.beta2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= hp.lr * (mi / hp.bc1) / (sqrtf(vi / hp.bc2) + hp.eps);
    }
}
#endif
hipError_t launch_dense_adam(const DenseAdamJob& job, const AdamHyper& hp, hipStream_t s);
// loss[0] = scale * sum_i terms[i]
hipError_t launch_loss_reduce(const float* terms, int n, float scale, float* loss, hipStream_t s);

// ---------------------------------------------------------------- small models (level.hip)
// The operators of one depth in one launch.  A problem is a projection or negation group (k = 1, pool = 0) or one class of
// intersections (k inputs each, pool = 1): MLP rows row0 + j * n + i of type's buffers, references ref_off + j * n + i
// (and relations rel_off + ..., -1: none), outputs out0 + i.
// Taken up to LEVEL_WEIGHTS weights a layer (a step of 64, 256 and 1024 queries at 100 x 200, separate launches against this one,
// planning included: 157 and 147, 172 and 169, 211 and 212 us; at 128 x 256 152 and 163, 168 and 188, 210 and 230; beyond, the
// weights read by every row block cost more than the launches).  Up to LEVEL_WEIGHTS_BOX by boxes, whose separate launches
// are more (at 128 x 256 122 and 111, 129 and 131, 157 and 158), and by depths of at most LEVEL_FEW row blocks (at 128 x 256,
// separate, all depths here and these depths here: 16 queries 159, 149 and 149, 32 queries 162, 155 and 149, 64 queries 152,
// 163 and 139, 512 queries 182, 200 and 170).  Never above LEVEL_WORK = row blocks x weights of a depth (from 4096 queries
// on the separate launches are as fast, 386 against 395 us).
constexpr int LEVEL_MAX = 10, LEVEL_WEIGHTS = 20480, LEVEL_WEIGHTS_BOX = 32768, LEVEL_FEW = 4;
constexpr long LEVEL_WORK = 512l * LEVEL_WEIGHTS_BOX;
constexpr int LEVEL_GATE = 2, LEVEL_PROJECTION = 3;      // box family (off set): pooling of offsets, projection without MLP
struct LevelProblem { int type, pool, n, k, ref_off, rel_off, row0, out0; };
struct LevelMlp { const float *Wa, *ba, *Wb, *bb; float *Z, *H, *dH; };
struct LevelTiles {                 // the problems of a depth and the first of their workgroups
    int count;
    int tile_start[LEVEL_MAX + 1];
    LevelProblem p[LEVEL_MAX];
};
struct LevelArgs {
    int d, h;
    bool keep;                      // forward: inputs, hidden rows and logits are kept for a backward pass
    LevelTiles t;
    LevelMlp mlp[3];
    const int32_t *refs, *rel, *out_row, *dst_row;   // out_row: row of act per output (null: itself); dst_row: of dact per reference
    const float *E, *R;
    float *act, *Att, *dact, *dAtt;
    const float* Ro;
    float *off, *Gate, *doff, *dGate;
};
bool level_fits(int d, int h, bool box);
// adds a problem; false if the launch has no room for it
bool level_add(LevelArgs& a, int type, int pool, int n, int k, int ref_off, int rel_off, int row0, int out0);
hipError_t launch_level(const LevelArgs& a, bool backward, hipStream_t s);
// All depths of a pass in one launch, in the order of their dependence; alike but for their tiles.  Taken for at most LEVEL_CHAIN
// depths of at most LEVEL_CHAIN_TILES workgroups together.  index: a small gradient index built beside them, by one more
// workgroup (null: none).
struct SmallIndex;
constexpr int LEVEL_CHAIN = 4, LEVEL_CHAIN_TILES = 256, LEVEL_SYNC = 2 + LEVEL_CHAIN;
// What such launches share: counts, zero, and zero again behind each of them, and what is set for good once one of them has given up
// waiting for a depth: rows are not valid then, whatever is computed from them, and launches that hand out results look at the mark instead.
struct LevelSync {
    int32_t* counts = nullptr;      // LEVEL_SYNC words
    int32_t* gave_up = nullptr;     // a word on the device, for the launches that follow
    int32_t* host_gave_up = nullptr;        // the same in pinned host memory, for the next call
    int32_t polls = 0;              // looks at a count before a wait gives up (0: it does at once)
};
constexpr int32_t GAVE_UP = 1 << 16;      // what a tile that gave up adds to a count of tiles
// A launch whose tiles, dealt by workgroup number, wait for one another has to come to its end whatever else holds places on the card, other
// launches of its kind among them, on other streams or of other processes: nobody may wait for good for a workgroup that has not started.  So a
// workgroup that has looked `patience` times for the layer before computes another one's tile, and then begins its own again.  Of the layers that are not through
// the first is always worked on, then: its tiles wait for nothing.
// rows_chain_kernel: a bit is set when its tile is through, and whoever helps computes one of the first layer that is not, which its own workgroup or others may do as
// well: they write the same values, to rows that nothing else of the launch is written to, and set the same bit.
// tile_chain_kernel, whose rows may be used again by a later depth: a workgroup takes its tile before it works on it, by setting the tile's word, and whoever helps takes
// the first tile that nobody has (what it works on lies before everything that is not taken, so that it never waits for such a tile itself, and
// whoever has a tile of the first layer that is not through works on that one).  Tiles of the last layer, which nobody waits for, are not taken.
// patience < 0, for tests: waiting workgroups help at once, and every eighth one looks -patience times whether its tile is done or taken before it begins itself.
struct TileHelp {
    int32_t* helped = nullptr;              // counts the tiles that another workgroup computed
    int32_t patience = 0;
};
constexpr int TILE_PATIENCE = 1024, TILE_AGAIN = 64;       // (looks of 0.3 us and more; a launch takes up to 60 us)
// What a workgroup learns before it needs the layer before: goes on; goes on, but its rows are not valid; has no tile any more.  Else: whose tile to compute first.
constexpr int TILE_GO = -1, TILE_GAVE_UP = -2, TILE_TAKEN = -3;
template <class Over>
__device__ __forceinline__ void tile_late(const TileHelp& c, int at, Over over) {
    if (__builtin_expect(c.patience < 0 && (at & 7) == 7, 0))
        for (int i = 0; i < -c.patience && !over(); ++i) __builtin_amdgcn_s_sleep(64);
}
// The plan, copied from pinned memory for the launches that follow, by one more workgroup (n: 16-byte units, 0: nothing to copy).
struct PlanCopy {
    const float4* src = nullptr;
    float4* dst = nullptr;
    int n = 0;
};
// A forward pass of a handful of queries, all layers of all depths in one launch (level.hip: rows_chain_kernel).  A problem is a projection or
// negation group (k = 1) or one class of intersections (k inputs each): rows row0 + j * n + i of its type's buffers, which no other depth uses; words[at ..] holds
// its n k references, the relations of a projection and its n output rows, so that nothing waits for the plan to reach the device.
// Limits: words of all problems, inputs of an intersection, values of a row.
constexpr int CHAIN_PROBLEMS = 5, CHAIN_WORDS = 160, CHAIN_CARD = 4, CHAIN_WIDTH = 1024;
// Tiles of a layer by bits of CHAIN_LINES words on lines of their own, the highest bit of each for a tile that gave up.  A launch clears the words of the next one.
constexpr int CHAIN_LINES = 16, CHAIN_STRIDE = 16, CHAIN_LAYER = CHAIN_LINES * CHAIN_STRIDE, CHAIN_BITS = 63, CHAIN_SYNC = 2 * LEVEL_CHAIN * CHAIN_LAYER;
constexpr unsigned long long CHAIN_GAVE_UP = 1ull << CHAIN_BITS;
struct RowsProblem { int type, k, n, at, row0; };
struct RowsChain {                                  // (what every tile needs first stands together)
    int d, h, depths = 0, n_words = 0;
    unsigned long long *through, *clear;            // CHAIN_SYNC words each: zero at first; zero at last
    TileHelp help;
    LevelSync sync;                                 // (its counts are not used)
    int count[LEVEL_CHAIN] = {}, first[2 * LEVEL_CHAIN + 1] = {};    // problems of a depth; tiles before each layer (rows_chain_lay_out)
    RowsProblem p[LEVEL_CHAIN][CHAIN_PROBLEMS];
    const float *Wa[3], *ba[3], *Wb[3], *bb[3];     // by type: projection, intersection, negation
    const float *E, *R;
    float *act, *Z, *H[3];                          // outputs; inputs of intersections; hidden rows by type
    PlanCopy copy;
    int32_t words[CHAIN_WORDS];
};
// Counts its tiles.  False: too many for one launch, or not such a pass.
bool rows_chain_lay_out(RowsChain& r);
hipError_t launch_rows_chain(const RowsChain& r, hipStream_t s);
// All layers of a pass over up to some hundred rows a depth in one launch (gemm.hip: tile_chain_kernel).  A problem is a projection or negation
// group (k = 1) or one class of intersections (k inputs each): rows row0 + j * n + i of its type's buffers, references ref0 + ... (and
// relations rel0 + ..., -1: none), outputs out0 + i.  Limits: inputs of an intersection, input values and hidden values of a row, problems of a depth.
constexpr int TILE_CARD = 4, TILE_D = 512, TILE_H = 1024, TILE_PROBLEMS = 8, TILE_PARTS = 32, TILE_WORDS = 8192;
// words of counts, zero before the launch: of the layers of a forward pass (two a depth), then of a backward one (up to three a depth)
constexpr int TILE_LINES = 16, TILE_STRIDE = 32, TILE_LAYER = TILE_LINES * TILE_STRIDE;
constexpr int TILE_LAYERS = 2 * LEVEL_CHAIN, TILE_LAYERS_BWD = 3 * LEVEL_CHAIN, TILE_SYNC = (TILE_LAYERS + TILE_LAYERS_BWD) * TILE_LAYER;
struct TileProblem { int type, k, n, row0, ref0, rel0, out0; };
// What the tiles of a part do.  Backward: the gradient of the hidden rows (from that of the outputs), of the inputs (from that of the
// hidden rows), and before both the pooling of a class.  Boxes: intersections once for the centres (type 1) and once for the offsets (type 2: pooled by the
// least input times the gate), projections (type 0) coordinate by coordinate, in the first layer of their depth.
enum TileKind { TILE_FIRST = 0, TILE_SECOND = 1, TILE_POOLED = 3, TILE_PLAIN = 2 };
// The tiles of a problem in one layer: mt = quotient of a tile's number by `by` (the row tile) or its remainder, mem members each; number: of its first tile
// in the layer.  inv_*: what a product's upper half divides by.
struct TilePart { int M, row0, ref0, rel0, out0, number, tiles, by; uint32_t inv_by; int m_major, mem, inv_mem, n_mem, cls, pools; };
struct TileChain {
    int d, h, layers = 0, parts = 0;
    int keep = 0;                                   // forward: inputs, hidden rows and logits are kept for a backward pass
    int tiles[TILE_LAYERS_BWD] = {};                // of a layer
    uint32_t start[TILE_PARTS];                     // of a part: its first workgroup << 8 | layer << 4 | type << 2 | kind
    TilePart part[TILE_PARTS];
    const uint16_t* W[2][3];                        // by layer of the MLP (backward: in the order they are taken) and type: pieces of the weights, biases,
    const float* bias[2][3];                        // ... inputs of the second layer and outputs of the first
    float *Z[3], *H[3];
    const float *E, *R;
    const int32_t *refs, *rel, *out_row;            // out_row: row of act per output (null: itself); backward: refs = row of dact per reference
    float *act, *Att;
    float *dact, *dAtt, *Dx, *dH[3];                // backward
    const float* Ro;                                // boxes: relations and the same buffers for the offsets
    float *off, *Gate, *doff, *dGate, *DxO;
    LevelSync sync;                                 // (its counts are not used)
    int32_t* chain;                                 // a word of TILE_LINES on lines of their own per layer
    unsigned long long* taken;                      // TILE_WORDS, by workgroup number: the number of the last launch that took it, ...
    unsigned long long launch = 0;                  // ... which no other launch of the context has, so that nothing is cleared between them
    TileHelp help;
    int blocks = 0;
};
// Tiles of a layer of n columns over members of k rows each that belong together, and of what is done coordinate by coordinate; the most that
// a layer may have for such a launch to be the better way (0: widths it does not take).
int tile_chain_tiles(int members, int k, int n);
int tile_chain_plain(int members, int d);
int tile_chain_most(int d, int h, bool box, bool trains);
// Lays out the tiles of n depths in the order given (count[l] problems each).  False: more parts than one launch has room for.
bool tile_chain_lay_out(TileChain& r, const TileProblem (*p)[TILE_PROBLEMS], const int* count, int n, bool backward, bool box);
hipError_t launch_tile_chain(const TileChain& r, bool backward, bool box, hipStream_t s);
bool levels_chain(const LevelArgs* a, int n);
hipError_t launch_levels(const LevelArgs* a, int n, bool backward, const LevelSync& sync, const SmallIndex* index, const PlanCopy& copy, hipStream_t s);

// ---------------------------------------------------------------- scoring (score.hip)
struct ScoreArgs {
    const float* act;          // [n_slots, d]
    const float* E;            // [N, d]
    const int32_t* root_off;   // [B+1]
    const int32_t* root_slot;  // [n_roots]
    const int32_t* pos;        // [B] or null (then candidates only)
    const int32_t* cand;       // [B, C]
    int B, C, d, max_branch;
    float gamma;
    // outputs
    float* score;              // [B, C + (pos?1:0)]
    float* coef;               // same shape, dL/ds (training only)
    int32_t* win;              // same shape, root slot of the winning branch (training, if set)
    void* mask;                // if set (training with text features): [pairs, 64] sign codes of (winning branch - entity row), 2 bits per
                               // coordinate; lane l of a wavefront owns coordinates 4l..4l+3 of every
                               // 256-coordinate chunk: 1, 2 or 4 bytes per lane for d <= 256, 512, 1024
                               // (one of win / mask is set in training)
    float* dact;               // gradient arena (training only)
    float* loss_terms;         // [B] (training only)
    // box family (off set): act holds the centres, off the offsets [n_slots, d]; the distance is
    // sum relu(|e-c| - o) + alpha * sum min(|e-c|, o); doff receives dL/d(offset) of the roots
    const float* off = nullptr;
    float* doff = nullptr;
    float alpha = 0.f;
    // candidate rows from a bf16 copy of the table [N, d] (bit patterns) instead of E
    const uint16_t* E16 = nullptr;
    bool streaming = false;    // E is a table beyond the caches
    const int32_t* gave_up = nullptr;      // as LevelSync: scores are minus infinity if it is set (not in training)
    size_t table_bytes = 0;    // of the candidates' rows
};
hipError_t launch_score(const ScoreArgs& a, bool train, hipStream_t s);

// ---------------------------------------------------------------- ranking (rank.hip)
// Entities of a piece of the table: an unfiltered ranking takes one at a time, the filter chunks of several (RANK_PIECES at most).
constexpr int RANK_PIECE = 1 << 16, RANK_PIECES = 4;
// dist[r*ld + e] = ||act[row_ids[r]] - Emat[e]||_1 for r < n_rows, e < n_ent.
// With off (box family, 0 <= alpha <= 1): the box distance of (act row, off row) to the entity row.
// With Emat16 (bf16 bit patterns, same shape as Emat) the entity rows are read from it.
// With `only` (this call completes a filtered pass): row tiles without a query whose list overflowed
// are left out, and so are, in the two launches below, the queries whose list did not.  launch_l1_tile and launch_topk_merge
// take several pieces of RANK_PIECE entities at a time, each with its own lists.
struct Overflowed {
    const int32_t* row_q;      // query of every branch row
    int32_t* count;            // [pieces, queries] listed entities; more than room: overflowed
    int room;
    const int32_t* any;        // [pieces] whether there is such a query
    int n_queries;
};
hipError_t launch_l1_tile(const float* act, const float* off, float alpha, const int32_t* row_ids, int n_rows,
                          const float* Emat, int n_ent, int d, float* dist, int ld, hipStream_t s,
                          const uint16_t* Emat16 = nullptr, const Overflowed* only = nullptr);
// count[a] += #{entities e < n_ent of this chunk: min over rows dist[row, e] < thr[a]}
hipError_t launch_count_less(const float* dist, int ld, const int32_t* root_off, const int32_t* ans_off,
                             const float* thr, int n_queries, int n_ent, int32_t* count, hipStream_t s,
                             const Overflowed* only = nullptr);
// rank[a] = 1 + count[a] - #{listed answers b of a's query: thr[b] < thr[a]}; 0 if *gave_up is set
hipError_t launch_finish_rank(const int32_t* count, const float* thr, const int32_t* ans_off, int n_queries, int n_ans,
                              const int32_t* gave_up, int32_t* rank, hipStream_t s);
// out[0..3] = MRR, Hit@1, Hit@3, Hit@10 over the first n_take[q] (null: all) answers of every query
hipError_t launch_rank_metrics(const int32_t* rank, const int32_t* ans_off, const int32_t* n_take, int n_queries,
                               float* out, hipStream_t s);
hipError_t launch_fill_zero_i32(int32_t* p, int n, hipStream_t s);
// per query q: entity value = min over rows root_off[q]..root_off[q+1]-1 of dist; merges the
// k best (value, ent_base + e) of this chunk into out_dist/out_ids [n_queries, k]
hipError_t launch_topk_merge(const float* dist, int ld, const int32_t* root_off, int n_queries, int ent_base, int n_ent,
                             int k, bool first_chunk, float* out_dist, int32_t* out_ids, const int32_t* gave_up, hipStream_t s,
                             const Overflowed* only = nullptr);

// Ranking with a filter on integer sums (rank_filter.hip): buffers of one pass.  Rows as words of 4
// (bits = 8) or 2 (bits = 16) coordinates, word-major; leading dimensions are multiples of 128.
struct RankFilter {
    int d, bits, words;              // words: rank_filter_words(d, bits)
    float *part, *lo, *grid;         // [32 * d] scratch, [d] grid origin, [2] step and its inverse
    uint32_t* Yq; int ldy;           // branch rows [words, ldy]
    float* base;                     // [2 * ldy] constant of every branch row in a bound from below, from above
    int32_t* row_q;                  // [ldy] its query
    uint32_t* Eq; int lde;           // entity rows of a chunk [words, lde]
    int32_t* slack; int parts;       // [parts, lde] error of an entity row, in steps: the sum over the parts
    // top-k: what the tiles of a chunk found, [ldy, tiles] words (zero between chunks) and rank_found_bytes(ldy, lde)
    uint32_t *found, *found_pair;
    // filtered ranks: per query the entities to be computed in fp32 [queries, room], their number (chunks of one piece).  Both: a
    // number above room marks a query for the fp32 pass of a piece, count [pieces of a chunk, queries]
    int32_t *list, *count; int room;
    int32_t* overflowed;             // per piece of the pass: a list had no room (behind count: n_counters in all, cleared with the grid)
    int n_counters;
    const int32_t* gave_up;          // nobody is near if this word is set
};
int rank_filter_words(int d, int bits);
size_t rank_found_bytes(int ldy, int lde);
// the grid of a pass from n_rows rows of a table, row_step apart; clears found and the counters
hipError_t launch_rank_grid(const RankFilter& f, const float* E, const uint16_t* E16, int64_t row_step, int n_rows, hipStream_t s);
// the branch rows of a pass, and the entity rows of a chunk, on the grid: both in one launch (8 us of one's own for the few branch rows), or
// either (rows null; n_ent 0)
struct RankRows { const float* act; const int32_t* ids; int n; const int32_t* root_off; int n_queries; };
hipError_t launch_quantise(const RankFilter& f, const RankRows* rows, const float* E, const uint16_t* E16, int n_ent, hipStream_t s);
// lists the chunk's entities that may be among the k nearest (best: running [queries, k] distances), and merges them
hipError_t launch_near_tile(const RankFilter& f, int n_rows, int n_ent, const float* best, int k, hipStream_t s);
hipError_t launch_near_merge(const RankFilter& f, int piece, const float* act, const int32_t* row_ids, const int32_t* root_off,
                             int n_queries, const float* E, const uint16_t* E16, int ent_base, int n_ent, int k, float* out_dist,
                             int32_t* out_ids, hipStream_t s);
// the k nearest of a table (RANK_PIECES pieces at most) from its sums (ld >= n_ent rounded up to 4); queries whose list has no room get no result and a mark
hipError_t launch_pick(const RankFilter& f, const uint32_t* sums, int ld, const float* act, const int32_t* row_ids, const int32_t* root_off,
                       int n_queries, const float* E, const uint16_t* E16, int n_ent, int k, float* out_dist, int32_t* out_ids, hipStream_t s);
// sums[r * ld + e] of the chunk; chunk_count[a] = entities certainly closer than answer a, the undecided
// ones listed; these computed, total[a] += both
hipError_t launch_sum_tile(const RankFilter& f, int n_rows, int n_ent, uint32_t* sums, int ld, hipStream_t s);
hipError_t launch_count_sure(const RankFilter& f, const uint32_t* sums, int ld, const int32_t* root_off, const int32_t* ans_off,
                             const float* thr, int n_queries, int n_ent, int32_t* chunk_count, hipStream_t s);
hipError_t launch_count_open(const RankFilter& f, int chunk, const uint32_t* sums, int ld, const float* act, const int32_t* row_ids, const int32_t* root_off,
                             const int32_t* ans_off, const float* thr, int n_queries, const float* E, const uint16_t* E16,
                             int32_t* chunk_count, int32_t* total, hipStream_t s);
// thr[a] = fp32 distance of answer a to its query, a0 <= a < a0 + cnt (row ans[a] of E, or row a - a0 where ans is null);
// counters[a] = counters[n_ans + a] = 0 for them
hipError_t launch_answer_distance(const float* act, const float* off, float alpha, const int32_t* row_ids, const int32_t* root_off,
                                  const int32_t* ans_off, int n_queries, const int32_t* ans, int a0, int cnt, const float* E,
                                  const uint16_t* E16, int d, const int32_t* gave_up, float* thr, int32_t* counters, int n_ans, hipStream_t s);

// ---------------------------------------------------------------- index (index.hip)
struct IndexBuffers {   // device scratch owned by the context, sized for n_keys
    int32_t *keys_a, *keys_b, *vals_a, *vals_b;   // [n_keys]
    int32_t* hist;                                // [256 * n_tiles] + totals of the digits
    int32_t* scan_tmp;                            // heads of a tile
    int32_t *uniq, *seg_off;                      // [n_keys], [n_keys+1]
    int32_t* n_uniq;                              // device scalar
};
size_t index_hist_elems(int64_t n_keys);
size_t index_scan_tmp_elems(int64_t n_keys);
// Up to SMALL_KEYS keys: the build as a job for one workgroup of 1024 threads (false: not so few, or none).  The order lands in vals_a.
constexpr int SMALL_KEYS = 4096;
struct SmallIndex {
    const int32_t *head, *tail;
    int n_head, n, bits;
    int32_t *vals_out, *uniq, *seg_off, *n_uniq;
};
bool small_index_job(const int32_t* head, int n_head, const int32_t* tail, int64_t n_tail, int32_t key_bound, const IndexBuffers& buf, SmallIndex* job);
// keys = [head[0..n_head) | tail[0..n_tail)], values < key_bound.  On return
// (stream order) uniq/seg_off/n_uniq are filled and the contribution order is in
// *src_out (one of vals_a / vals_b).
hipError_t build_segment_index(const int32_t* head, int n_head, const int32_t* tail, int64_t n_tail,
                               int32_t key_bound, const IndexBuffers& buf, int32_t** src_out,
                               hipStream_t s);

// ---------------------------------------------------------------- tables (table.hip)
struct TableArgs {
    float *P, *Mo, *Vo;            // table and moments [rows, d]
    const int32_t* uniq;           // [n_uniq] row ids
    const int32_t* seg_off;        // [n_uniq+1]
    const int32_t* n_uniq_dev;     // device scalar
    int d;
    // contribution records in segment order, gradient rows before pairs inside a segment:
    // rec_row[t] < 0 is row -1-rec_row[t] of dact, added as it is; rec_row[t] >= 0 is a
    // (query, candidate) pair and the contribution is rec_coef[t] * sign: without mask,
    // rec_row[t] is a row of act and sign = sign(act row - table row); with mask (text
    // features) it is the pair number and the signs are the pair's entry of mask (layout:
    // ScoreArgs::mask).  rec_coef may be null if all records are gradient rows.
    const float* rec_coef;
    const int32_t* rec_row;
    // the records unresolved (at the end of a step only): contribution numbers in segment order and what
    // launch_resolve makes records of; rec_coef and rec_row are not read then
    const int32_t* src = nullptr;
    const float* pair_coef = nullptr;
    const int32_t* pair_win = nullptr;
    int n_rowsrc = 0, row_base = 0, B = 0, K = 1;
    const float* dact;
    const float* act;
    const void* mask;              // set together with g_bf16
    float* g_out;                  // if set: write gradients [n_uniq, d] instead of updating
    // text-feature fusion: the row gradient is also left in g_bf16 [n_uniq, d] (bf16 bit
    // patterns) for the gradient of the projection
    uint16_t* g_bf16 = nullptr;
    // box family: pair records carry rows of act (centres) and off (offsets); the contribution is
    // rec_coef * w * sign(centre - table row), w = 1 where |centre - row| > offset, else alpha
    const float* off = nullptr;
    float alpha = 0.f;
    // the row's gradient is multiplied by [table row > 0] (a table that is used through relu)
    bool relu_gate = false;
    // A pass over the rows that do not wait for the backward pass (`later` set): rows whose first record is a gradient
    // row are left out, their positions in uniq appended to later (*n_later of them, zero before).  The pass over
    // those (`pick` set): the positions pick[0..*n_uniq_dev).
    int32_t* later = nullptr;
    int32_t* n_later = nullptr;
    const int32_t* pick = nullptr;
    // bf16 copy of the table [rows, d] that the scoring pass reads: pair signs are taken against
    // the rounded row, and the updated row is rounded into the copy
    uint16_t* shadow = nullptr;
    // the table and its moments are far larger than the caches: their rows move with non-temporal
    // loads and stores (single-table launches only)
    bool streaming = false;
};
// sorted contribution numbers -> records: c < n_rowsrc is gradient row row_base + c,
// otherwise a (query, candidate) pair in the order [B positives | B*K negatives]
// (win: winning rows per pair -> records carry act rows; null -> records carry pair numbers).
// With loss_terms [B] the same launch also writes loss[0] = loss_scale * sum of the terms (infinite if *gave_up is set).
hipError_t launch_resolve(const int32_t* src, int64_t n, int n_rowsrc, int row_base, int B, int K, const float* coef,
                          const int32_t* win, float* rec_coef, int32_t* rec_row, const float* loss_terms,
                          float loss_scale, float* loss, const int32_t* gave_up, hipStream_t s);
// few: by one workgroup per compute unit (a pass that has time and should leave the chip to others); max_rows: at most so many
// touched rows.  table_takes_once: by a wavefront a row, which may resolve the records of its row (a.src)
bool table_takes_once(const TableArgs& a, bool few, int64_t max_rows);
hipError_t launch_table_update(const TableArgs& a, const AdamHyper& hp, bool few, int64_t max_rows, hipStream_t s);
// The end of a step in one launch: the main table (at most max_rows touched rows; 0: not part of it), up to two small
// plain tables of the same width (no text features, box weights or bf16 copy: the relation tables, each of at most
// small_rows touched rows), and the dense tensors.
struct TableTail {
    int main_blocks, dense_blocks;     // dense_blocks: of every tensor
    int blocks[2];
    TableArgs job[2];
    DenseAdamJob dense;
    // one more workgroup: loss[0] = loss_scale * sum of the loss terms (null: not here)
    const float* loss_terms;
    int n_loss;
    float loss_scale;
    float* loss;
    const int32_t* gave_up;
};
struct LossSum { const float* terms; int n; float scale; float* loss; const int32_t* gave_up; };       // gave_up: the loss is infinite if it is set
hipError_t launch_step_tail(const TableArgs& a, int64_t max_rows, const TableArgs* small, int n_small, int small_rows,
                            const DenseAdamJob& dense, const LossSum& loss, const AdamHyper& hp, hipStream_t s);

// ---------------------------------------------------------------- text-feature fusion (sem.hip)
hipError_t launch_cast_bf16(const float* x, uint16_t* y, int64_t n, hipStream_t s);
// inv[src[t]] = u for seg_off[u] <= t < seg_off[u+1]
hipError_t launch_inverse_index(const int32_t* src, const int32_t* seg_off, const int32_t* n_uniq_dev, int64_t n,
                                int32_t* inv, hipStream_t s);
// out[i] = in_ref[i] if it is a slot, else -1 - inv[in_gslot[i] - n_slots] (anchor -> its touched-row position)
hipError_t launch_translate_refs(const int32_t* in_ref, const int32_t* in_gslot, int n, int n_slots,
                                 const int32_t* inv, int32_t* out, hipStream_t s);
// out[u, :] = E[id(u), :] + Wb * H[id(u), :] for u < n_rows; id(u) = ids[u], or id_base + u for u < n_seq and
// (u - n_seq) * spread from there on
struct SemFuseArgs {
    const uint16_t* H;          // [N, ds] bf16
    const uint16_t* Wb;         // [d, ds] bf16
    const float* E;             // [N, d]
    const int32_t* ids;         // [n_rows] or null
    int64_t id_base;
    int n_seq = INT32_MAX, spread = 0;
    const int32_t* n_rows_dev;  // device scalar (then n_rows is an upper bound) or null
    int n_rows;
    int d, ds;                  // ds a multiple of 64
    float* out;                 // [n_rows, d]
    // the rows on the integer grid of a ranking as well (bits: 8, 16, or 0 for not): words of row u at Q[w * ldq + u], the error that
    // column part c of the row adds at err[c * ldq + u] (sem_fuse_parts(d) parts)
    int bits = 0, ldq = 0, words = 0;
    const float *lo = nullptr, *grid = nullptr;
    uint32_t* Q = nullptr;
    int32_t* err = nullptr;
};
int sem_fuse_parts(int d);
hipError_t launch_sem_fuse(const SemFuseArgs& a, hipStream_t s);
// out[m, n] = sum_u G[u, m] * H[ids[u], n] over u < *n_rows_dev
struct SemWgradArgs {
    const uint16_t* H;
    const int32_t* ids;
    const uint16_t* G;          // [n_rows, d] bf16, d a multiple of 8
    const int32_t* n_rows_dev;
    int n_rows;                 // upper bound
    int d, ds;
    int n_splits;               // from sem_wgrad_splits
    float* partial;             // [n_splits, d, ds]
};
int sem_wgrad_splits(int64_t n_rows_bound, int d, int ds);
hipError_t launch_sem_wgrad(const SemWgradArgs& a, float* out, hipStream_t s);

}  // namespace ngdb
