// Contractions of the grouped operator MLPs (Sec. 4.1's batched kernels): gemm_kernel forward and
// for data gradients, product_kernel the same over many rows, rows_kernel forward over few rows, wgrad_kernel for
// weight gradients.
//
// The groups of one batch are small next to the chip (a few hundred to a few
// thousand rows against 256 compute units), so a contraction is latency bound,
// not throughput bound: what matters is the length of the dependent chain
// "global load -> LDS -> MFMA" of one workgroup.  Therefore the k extent is
// split over the wavefronts of a workgroup: every wavefront walks its own
// k-tiles (tile w, w+NW, ...) through a private LDS staging area and
// accumulates the whole BM x BN output tile with 32x32x2 MFMA blocks; the NW
// partial tiles are then summed through LDS in a fixed order (deterministic) and
// the epilogue is applied to the sum.  The A operand can be assembled on the fly
// from row references (gather of operator inputs fused into the first layer).
//
// Results are fp32 either way, but the products are formed on one of two routes: fp32
// MFMA blocks, or (SPLIT) bf16 MFMA blocks on operands that are split, while a tile is
// staged, into three bf16 pieces whose sum is the fp32 value exactly; six of the nine
// partial products are kept.  The matrix unit then needs 2.7 times less time per tile.
// On the split route the small tile can take operands that were split beforehand (BP: the
// weights, once per pass, by weight_pieces_kernel; AP: the hidden rows, by the epilogue of
// the launch that produced them): such pieces lie in global memory tile by tile in the lane
// order of the MFMA and go from there straight into its operand registers.
#include <type_traits>
#include "common.h"

namespace ngdb {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BK = 16;    // k extent of one staged tile
constexpr int PAD = 4;    // keeps LDS rows 16-byte aligned and spreads banks

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int NW, bool SPLIT = false, bool BP = false, bool AP = false>
struct Smem {
    // SPLIT: per wavefront and operand three bf16 pieces of a [32][BK] tile (BP, AP: that operand
    // comes ready-made from global memory and is not staged)
    static constexpr int STAGE = SPLIT ? NW * ((AP ? 0 : BM / 32) + (BP ? 0 : BN / 32)) * 960 : NW * BK * (BM + PAD + BN + PAD);   // floats
    // partial tiles held in LDS at once: all of them in the small tile (one barrier less than folding
    // the upper half of the wavefronts into the lower half first, 34 KB for eight)
    static constexpr int NR = (NW > 4 && BM * BN > 32 * 32) ? NW / 2 : NW;
    static constexpr int REDUCE = NR * BM * (BN + 1);
    static constexpr int FLOATS = STAGE > REDUCE ? STAGE : REDUCE;
};

// Operand staging is written as force-inlined functions over register arrays of
// compile-time size (no lambdas, no run-time indices) so that the tiles in
// flight stay in VGPRs.  Issuing a tile is nothing but address arithmetic and
// loads: addresses are clamped into the operand, never branched on, and nothing
// touches the loaded values before the tile is staged, so the loads of the next
// tile stay in flight while the current one is multiplied.
// A 16-byte load from global memory.  Row pointers picked at run time among several bases lose their
// address space, and the loads through them would be FLAT ones: those count as LDS operations as
// well, so every LDS read of the current tile would wait for the tile requested ahead.
// (through a built-in vector type: float4 is a class, and copying one goes through a generic reference)
__device__ __forceinline__ float4 load_global4(const float* p) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    typedef const floatx4 __attribute__((address_space(1))) * global_floatx4;
    const floatx4 v = *(global_floatx4)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

template <int BM, int LA, bool AK>
__device__ __forceinline__ void issue_a(const GemmArgs& a, int lane, int m0, int k0, bool has_add,
                                        const float* const (&arow)[LA], const float* const (&aadd)[LA],
                                        float4 (&ra)[LA], float4 (&rd)[LA]) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int idx = lane + i * 64;
        if (AK) {
            const int gkc = min(k0 + (idx % (BK / 4)) * 4, a.K - 4);
            ra[i] = load_global4(arow[i] + gkc);
            if (has_add) rd[i] = load_global4(aadd[i] + gkc);
        } else {
            const int gk = k0 + idx / (BM / 4), gm = m0 + (idx % (BM / 4)) * 4;
            ra[i] = load_global4(a.A + (size_t)min(gk, a.K - 1) * a.lda + min(gm, a.M - 4));
        }
    }
}

template <int BN, int LB, bool BKC>
__device__ __forceinline__ void issue_b(const GemmArgs& a, int lane, int n0, int k0, float4 (&rb)[LB]) {
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int idx = lane + i * 64;
        const float* p;
        if (BKC) {
            const int gn = n0 + idx / (BK / 4), gk = k0 + (idx % (BK / 4)) * 4;
            p = a.B + (size_t)min(gn, a.N - 1) * a.ldb + min(gk, a.K - 4);
        } else {
            const int gk = k0 + idx / (BN / 4), gn = n0 + (idx % (BN / 4)) * 4;
            p = a.B + (size_t)min(gk, a.K - 1) * a.ldb + min(gn, a.N - 4);
        }
        rb[i] = load_global4(p);
    }
}

// registers -> this wavefront's LDS tile [BK][LD].  Here the values are completed:
// relation row added, entries outside the operand zeroed, assembled A rows copied out.
template <int BM, int LA, int LD, bool AK>
__device__ __forceinline__ void stage_a(const GemmArgs& a, float* __restrict__ dst, int lane, int m0, int k0,
                                        bool has_add, bool copy_out, const bool (&avalid)[LA],
                                        const float4 (&ra)[LA], const float4 (&rd)[LA]) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int idx = lane + i * 64;
        float4 v = ra[i];
        if (AK) {
            const int m = idx / (BK / 4), kq = idx % (BK / 4);
            const int gk = k0 + kq * 4;
            if (has_add) { v.x += rd[i].x; v.y += rd[i].y; v.z += rd[i].z; v.w += rd[i].w; }
            const bool ok = avalid[i] && gk < a.K;
            v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
            if (copy_out && ok) *reinterpret_cast<float4*>(a.a_copy + (size_t)(m0 + m) * a.lda + gk) = v;
            dst[(kq * 4 + 0) * LD + m] = v.x;
            dst[(kq * 4 + 1) * LD + m] = v.y;
            dst[(kq * 4 + 2) * LD + m] = v.z;
            dst[(kq * 4 + 3) * LD + m] = v.w;
        } else {
            const int k = idx / (BM / 4), mq = idx % (BM / 4);
            const bool ok = k0 + k < a.K && m0 + mq * 4 < a.M;
            v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
            *reinterpret_cast<float4*>(&dst[k * LD + mq * 4]) = v;
        }
    }
}

template <int BN, int LB, int LD, bool BKC>
__device__ __forceinline__ void stage_b(const GemmArgs& a, float* __restrict__ dst, int lane, int n0, int k0,
                                        const float4 (&rb)[LB]) {
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int idx = lane + i * 64;
        float4 v = rb[i];
        if (BKC) {
            const int n = idx / (BK / 4), kq = idx % (BK / 4);
            const bool ok = n0 + n < a.N && k0 + kq * 4 < a.K;
            v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
            dst[(kq * 4 + 0) * LD + n] = v.x;
            dst[(kq * 4 + 1) * LD + n] = v.y;
            dst[(kq * 4 + 2) * LD + n] = v.z;
            dst[(kq * 4 + 3) * LD + n] = v.w;
        } else {
            const int k = idx / (BN / 4), nq = idx % (BN / 4);
            const bool ok = k0 + k < a.K && n0 + nq * 4 < a.N;
            v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
            *reinterpret_cast<float4*>(&dst[k * LD + nq * 4]) = v;
        }
    }
}

// An fp32 value is the exact sum of three bf16 values: x rounded to bf16, the remainder rounded
// to bf16, and what is then left (at most 6 bits).  Rounding is to nearest (the hardware
// conversion), so the pieces carry signs of their own and nothing is biased: with pieces cut off
// instead, every product would come out a little short, and the scores, whose loss weights
// depend on them exponentially, would shift in one direction.  A product of two fp32 values is a
// sum of nine bf16 products, of which the six largest are kept; the three left out are below
// 2^-23 of the product (second piece at most 2^-8, third at most 2^-16 of the value), with
// either sign.  bf16 products are exact in the fp32 accumulator of the matrix unit,
// which multiplies bf16 sixteen times as fast as fp32.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk(float first, float second) {   // first in the lower half
    const floatx2 v = {first, second};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// pieces of two values, packed pairwise: h, m, l words
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = cvt_pk(a, b);
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = cvt_pk(ra, rb);
    l = cvt_pk(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
}
struct Pieces {
    uint2 h, m, l;     // 4 consecutive k each, bf16 bit patterns
};
__device__ __forceinline__ Pieces split3(float4 v) {
    Pieces p;
    split2(v.x, v.y, p.h.x, p.m.x, p.l.x);
    split2(v.z, v.w, p.h.y, p.m.y, p.l.y);
    return p;
}
// Pieces of a [32][BK] tile in LDS: 16-byte units (8 consecutive k of a row); unit index
// = k-half * 32 + row, piece after piece -- the operand layout of the 32x32x16 bf16 MFMA
// (lane = k-half * 32 + row reads unit `lane`).  In the tiles of an operand that is staged from
// its k-strided layout (GAPS) one unit is left empty after every four: the 32-bit stores of that
// staging then spread over all banks (8-way conflicts without the gaps; the 64-bit stores of the
// k-contiguous staging need none and are slower with them).  Room per piece: 80 units = 640
// bf16 either way; the three pieces of 32 rows take 1920.
template <bool GAPS>
__device__ __forceinline__ int unit_at(int u) { return (GAPS ? u + (u >> 2) : u) * 8; }
constexpr int PIECE = 640, SUBTILE = 3 * PIECE;
__device__ __forceinline__ void store_pieces(uint16_t* tile, int row, int kq, const Pieces& p) {
    uint16_t* at = tile + unit_at<false>((kq >> 1) * 32 + row) + (kq & 1) * 4;
    *reinterpret_cast<uint2*>(at) = p.h;
    *reinterpret_cast<uint2*>(at + PIECE) = p.m;
    *reinterpret_cast<uint2*>(at + 2 * PIECE) = p.l;
}

// Operand stored with k as the slow index ([K][X], X = rows or columns of the output): a lane
// takes two consecutive k of four consecutive x (8 lanes cover 128 contiguous bytes), so that
// the pieces of a (k, k+1) pair fill one 32-bit word of the tile.
__device__ __forceinline__ void issue_strided(const float* base, int ld, int K, int X, int k0, int x0, int lane,
                                              float4 (&r)[2]) {
    const int gk = k0 + 2 * (lane >> 3), gx = min(x0 + (lane & 7) * 4, X - 4);
    r[0] = load_global4(base + (size_t)min(gk, K - 1) * ld + gx);
    r[1] = load_global4(base + (size_t)min(gk + 1, K - 1) * ld + gx);
}
__device__ __forceinline__ void stage_strided(uint16_t* tile, int K, int X, int k0, int x0, int lane,
                                              const float4 (&r)[2]) {
    const int kp = lane >> 3, q = lane & 7;
    const bool okx = x0 + q * 4 < X;
    const bool ok0 = okx && k0 + 2 * kp < K, ok1 = okx && k0 + 2 * kp + 1 < K;
    const float e[4] = {r[0].x, r[0].y, r[0].z, r[0].w}, o[4] = {r[1].x, r[1].y, r[1].z, r[1].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t h, m, l;
        split2(ok0 ? e[j] : 0.f, ok1 ? o[j] : 0.f, h, m, l);
        uint32_t* at = reinterpret_cast<uint32_t*>(tile + unit_at<true>((kp >> 2) * 32 + q * 4 + j) + (kp & 3) * 2);
        at[0] = h;
        at[PIECE / 2] = m;
        at[PIECE] = l;
    }
}

// Weight matrices as ready-made B operands of the bf16 MFMA block: the three bf16 pieces of every
// value (see split3), laid out tile by tile in the order the lanes of a wavefront consume them.
// Tile (nb, kt) covers rows n = nb*32 .. +31 and k = kt*16 .. +15 of the operand B[n][k]; it holds
// per piece 64 x 16 bytes: lane l's eight values B[nb*32 + (l & 31)][kt*16 + (l >> 5)*8 + 0..7].
// A wavefront fetches a piece of a tile with one fully coalesced 1 KiB load straight into the
// registers of the MFMA: no staging through LDS, no arithmetic.  Tiles beyond the matrix (the
// launcher pads the tile grid to what its kernels walk) hold zeros, so the consumers need no bounds.
constexpr int WTILE = 3 * 512;            // bf16 values of one tile
// One workgroup reads a block of 32 rows x 64 columns of a row-major matrix W [R][C] (coalesced),
// and writes the tiles that block contributes to both operand forms: B[n = row][k = column]
// (four tiles along k) and B[n = column][k = row] (two tile rows x two k-tiles).
__global__ __launch_bounds__(256) void weight_pieces_kernel(const PieceJobs J) {
    __shared__ float blk[32][65];
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < J.clear_n; i += gridDim.x * 256) J.clear[i] = 0;
    if ((int)blockIdx.x < J.copy_blocks) {
        for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < J.copy_n; i += J.copy_blocks * 256) J.copy_dst[i] = J.copy_src[i];
        return;
    }
    const int block = (int)blockIdx.x - J.copy_blocks;
    int j = 0;
#pragma unroll
    for (int i = 1; i < PIECE_MAX_JOBS; ++i)
        if (i < J.count && block >= J.block0[i]) j = i;
    PieceJob jb = J.job[0];
#pragma unroll
    for (int i = 1; i < PIECE_MAX_JOBS; ++i)
        if (i == j) jb = J.job[i];
    const int b = block - J.block0[j];
    const int cblocks = (jb.C + 63) / 64;
    const int r0 = (b / cblocks) * 32, c0 = (b % cblocks) * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int q = 0; q < 2; ++q) {         // 512 float4 of the block, 16 per row
        const int idx = tid + q * 256, r = idx >> 4, c4 = (idx & 15) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r0 + r < jb.R && c0 + c4 < jb.C) v = *reinterpret_cast<const float4*>(jb.W + (size_t)(r0 + r) * jb.C + c0 + c4);
        blk[r][c4 + 0] = v.x; blk[r][c4 + 1] = v.y; blk[r][c4 + 2] = v.z; blk[r][c4 + 3] = v.w;
    }
    __syncthreads();
    float v[8];
    // B[n = row][k = column]: wavefront w writes k-tile w of the block
    {
        const int kt = c0 / 16 + wave, KT = (jb.C + 15) / 16;
        if (kt < KT) {
            const int n = lane & 31, kk = wave * 16 + (lane >> 5) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = blk[n][kk + e];
            const Pieces p0 = split3(make_float4(v[0], v[1], v[2], v[3])), p1 = split3(make_float4(v[4], v[5], v[6], v[7]));
            uint16_t* out = jb.out_rk + ((size_t)(r0 / 32) * KT + kt) * WTILE + lane * 8;
            *reinterpret_cast<uint4*>(out) = make_uint4(p0.h.x, p0.h.y, p1.h.x, p1.h.y);
            *reinterpret_cast<uint4*>(out + 512) = make_uint4(p0.m.x, p0.m.y, p1.m.x, p1.m.y);
            *reinterpret_cast<uint4*>(out + 1024) = make_uint4(p0.l.x, p0.l.y, p1.l.x, p1.l.y);
        }
    }
    // B[n = column][k = row]: wavefront w writes tile row w / 2, k-tile w % 2 of the block
    if (!jb.out_ck) return;
    {
        const int nb = c0 / 32 + (wave >> 1), kt = r0 / 16 + (wave & 1), KT = (jb.R + 15) / 16;
        if (nb < (jb.C + 31) / 32 && kt < KT) {
            const int n = (wave >> 1) * 32 + (lane & 31), kk = (wave & 1) * 16 + (lane >> 5) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = blk[kk + e][n];
            const Pieces p0 = split3(make_float4(v[0], v[1], v[2], v[3])), p1 = split3(make_float4(v[4], v[5], v[6], v[7]));
            uint16_t* out = jb.out_ck + ((size_t)nb * KT + kt) * WTILE + lane * 8;
            *reinterpret_cast<uint4*>(out) = make_uint4(p0.h.x, p0.h.y, p1.h.x, p1.h.y);
            *reinterpret_cast<uint4*>(out + 512) = make_uint4(p0.m.x, p0.m.y, p1.m.x, p1.m.y);
            *reinterpret_cast<uint4*>(out + 1024) = make_uint4(p0.l.x, p0.l.y, p1.l.x, p1.l.y);
        }
    }
}

// (at: the lane's place in the first piece of a tile)
__device__ __forceinline__ bf16x8 piece_at(const uint16_t* at, int q) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(at + q * 512));
}

// POOL: problems with pool_k set take whole intersections: a tile is all inputs of 32 / pool_k members, and the pooling
// is the end of the epilogue (a launch of its own cost 3 to 5 us at each depth).
template <int BM, int BN, int NW, bool AK, bool BKC, bool SPLIT = false, int PF = 1, bool BP = false, bool AP = false, bool POOL = false, class Group = GemmGroup>
__global__ __launch_bounds__(NW * 64) void gemm_kernel(const Group g) {
    static_assert(!BP || (SPLIT && AK), "B operand from split pieces: split route with k-contiguous A only");
    static_assert(!AP || (BP && BM == 32), "A operand from split pieces: with B from pieces, one block of rows");
    static_assert(!SPLIT || BK == 16, "split path: one 32x32x16 MFMA step per staged tile");
    __shared__ __attribute__((aligned(16))) float smem[Smem<BM, BN, NW, SPLIT, BP, AP>::FLOATS];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    // which problem of the group this workgroup works on (uniform, stays in scalar registers)
    int p = 0, first = g.tile_start[0], last = g.tile_start[1];
#pragma unroll
    for (int i = 1; i < Group::MOST; ++i)
        if (i < g.count && (int)blockIdx.x >= g.tile_start[i]) {
            p = i;
            first = g.tile_start[i];
            last = g.tile_start[i + 1];
        }
    const GemmArgs& a = g.p[p];        // (the group lies in the kernel argument segment: a scalar load at a uniform offset)
    // Workgroups are dealt round-robin to the 8 dies, each with its own L2.  Every problem
    // owns a multiple of 8 workgroups, and die x takes the x-th eighth of the problem's
    // tiles, ordered so that this eighth is a slab along the longer output side: a die then
    // reads one slab of one operand and the whole of the other, not both whole.
    const int local = (int)blockIdx.x - first;
    const int per_die = (last - first) >> 3;
    const int tile = (local & 7) * per_die + (local >> 3);
    const int cls = POOL && a.pool_k ? a.pool_k : 1, mem = BM / cls, n_mem = a.M / cls;     // POOL: inputs, members per tile and in all
    const int tiles_m = POOL ? (n_mem + mem - 1) / mem : (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    if (tile >= tiles_m * tiles_n) return;
    const bool m_major = a.M >= a.N;
    const int mt = m_major ? tile / tiles_n : tile % tiles_m;
    const int m0 = mt * BM;
    auto pool_row_of = [&](int lr, bool* ok) {          // POOL: row of A and C that row lr of the tile is
        const int j = lr / mem, i = mt * mem + lr - j * mem;
        *ok = j < cls && i < n_mem;
        return *ok ? j * n_mem + i : a.M - 1;
    };
    const int n0 = (m_major ? tile % tiles_n : tile / tiles_m) * BN;
    const bool first_n_tile = n0 == 0;
    constexpr int TM = BM / 32, TN = BN / 32;
    constexpr int LDA = BM + PAD, LDB = BN + PAD;
    // (SPLIT: per 32 rows of an operand three pieces, SUBTILE bf16 = 960 floats)
    float* As = smem + (SPLIT ? wave * ((AP ? 0 : TM) + (BP ? 0 : TN)) * 960 : wave * BK * (LDA + LDB));     // [BK][LDA] of this wavefront
    float* Bs = As + (SPLIT ? (AP ? 0 : TM) * 960 : BK * LDA);                                      // [BK][LDB]

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    constexpr int LA = BM * BK / 4 / 64;   // float4 per lane per tile
    constexpr int LB = BN * BK / 4 / 64;
    float4 ra[PF][LA], rd[PF][LA], rb[PF][LB];
    bf16x8 bq[PF][BP ? BN / 32 : 1][3];       // BP: the B operand blocks of a tile, ready for the MFMA
    bf16x8 aq[PF][3];                         // AP: the A operand block likewise
    const bool has_add = AK && a.a_ref != nullptr && a.a_add_idx != nullptr;   // uniform
    const bool copy_out = AK && a.a_copy != nullptr && first_n_tile;           // uniform

    // rows of A (k-contiguous layout), possibly assembled from references: resolved once
    // per lane; rows past M point at row M-1 and are zeroed after the load
    const float* arow[LA];
    const float* aadd[LA];
    bool avalid[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        arow[i] = a.A;
        aadd[i] = a.A;
        avalid[i] = false;
        if (AK && !AP) {
            const int gm = m0 + (lane + i * 64) / (BK / 4);
            avalid[i] = gm < a.M;
            int gmc = min(gm, a.M - 1);
            if (POOL) gmc = pool_row_of((lane + i * 64) / (BK / 4), &avalid[i]);
            if (a.a_ref) {
                const int32_t r = a.a_ref[gmc];
                arow[i] = r >= 0 ? a.a_base0 + (size_t)r * a.lda : a.a_base1 + (size_t)(-1 - r) * a.lda;
                if (a.a_add_idx) aadd[i] = a.a_add + (size_t)a.a_add_idx[gmc] * a.lda;
            } else {
                arow[i] = a.A + (size_t)gmc * a.lda;
            }
        }
    }

    // AP: this lane's place in the first k-tile of the A pieces
    size_t a_lane = 0;
    if (AP) {
        if (POOL) {
            bool ok;
            const int r = pool_row_of(lane & 31, &ok) + a.a_row0;
            a_lane = (size_t)(r >> 5) * a.a_kt * WTILE + ((lane >> 5) * 32 + (r & 31)) * 8;
        } else {
            a_lane = (size_t)(m0 / 32) * a.a_kt * WTILE + lane * 8;
        }
    }

    // Epilogue operands of this thread's output elements (clamped addresses, uniform flags).
    // Small tiles (launches that are latency bound) request them here, ahead of the k loop, so
    // that nothing is waited for after the last MFMA; large tiles request them after the loop:
    // held across it they would cost the registers of a second resident wavefront per SIMD (the
    // 4-wavefront small tile with split arithmetic likewise: 5 instead of 4 wavefronts per SIMD).
    constexpr int EPT = BM * BN / (NW * 64);
    constexpr bool EARLY_EPILOGUE = BM * BN <= 32 * 32 && !(SPLIT && NW == 4) && PF == 1;
    float e_bias[EPT], e_mask[EPT], e_add[EPT];
    int e_orow[EPT];
    const bool has_bias = a.bias != nullptr, has_mask = a.mask != nullptr, has_addend = a.addend != nullptr,
               has_dst = a.dst_row != nullptr;
#define NGDB_LOAD_EPILOGUE()                                                                \
    _Pragma("unroll") for (int q = 0; q < EPT; ++q) {                                      \
        const int e = tid + q * NW * 64;                                                    \
        const int lr = e / BN, lc = e % BN;                                                 \
        bool row_ok;                                                                        \
        const int row = POOL ? pool_row_of(lr, &row_ok) : min(m0 + lr, a.M - 1), col = min(n0 + lc, a.N - 1); \
        e_bias[q] = has_bias ? a.bias[col] : 0.f;                                           \
        e_mask[q] = has_mask ? a.mask[(size_t)row * a.ldmask + col] : 1.f;                  \
        e_add[q] = has_addend ? a.addend[(size_t)row * a.ldadd + col] : 0.f;                \
        e_orow[q] = has_dst ? a.dst_row[row] : row;                                         \
    }
    if (EARLY_EPILOGUE) { NGDB_LOAD_EPILOGUE() }

    // A wavefront stages its tiles in its own LDS area and LDS executes a wavefront's
    // instructions in order, so the k loop needs no workgroup barrier: wavefronts run
    // independently (their memory waits do not line up) and only over the tiles they own.
    const int nk = (a.K + BK - 1) / BK;
    const int rounds = nk > wave ? (nk - wave + NW - 1) / NW : 0;
    // (operands that come as fp32 values, to be staged, and operands that come as pieces)
#define NGDB_ISSUE_VALUES(u, kc)                                                             \
    if (AP) {                                                                                \
    } else if (SPLIT && !AK) {                                                               \
        _Pragma("unroll") for (int t = 0; t < TM; ++t)                                      \
            issue_strided(a.A, a.lda, a.K, a.M, kc, m0 + 32 * t, lane, reinterpret_cast<float4(&)[2]>(ra[u][2 * t])); \
    } else {                                                                                 \
        issue_a<BM, LA, AK>(a, lane, m0, kc, has_add, arow, aadd, ra[u], rd[u]);            \
    }                                                                                        \
    if (BP) {                                                                                \
    } else if (SPLIT && !BKC) {                                                              \
        _Pragma("unroll") for (int t = 0; t < TN; ++t)                                      \
            issue_strided(a.B, a.ldb, a.K, a.N, kc, n0 + 32 * t, lane, reinterpret_cast<float4(&)[2]>(rb[u][2 * t])); \
    } else {                                                                                 \
        issue_b<BN, LB, BKC>(a, lane, n0, kc, rb[u]);                                       \
    }
#define NGDB_ISSUE_PIECES(u, kc, live)                                                       \
    if (AP) {                                                                                \
        const uint16_t* at = (live) ? a.a_pieces + (size_t)((kc) / BK) * WTILE + a_lane : a.a_pieces; \
        _Pragma("unroll") for (int q = 0; q < 3; ++q) aq[u][q] = piece_at(at, q);           \
    }                                                                                        \
    if (BP) {                                                                                \
        _Pragma("unroll") for (int j = 0; j < BN / 32; ++j) {                               \
            const uint16_t* at = (live) ? a.b_pieces + ((size_t)(n0 / 32 + j) * a.b_kt + (kc) / BK) * WTILE + lane * 8 : a.b_pieces; \
            _Pragma("unroll") for (int q = 0; q < 3; ++q) bq[u][BP ? j : 0][q] = piece_at(at, q); \
        }                                                                                    \
    }
    // PF tiles are in flight per wavefront.  With more than one, every stage of the loop requests
    // its next tile whether or not there is one (beyond the end: the first k-tile once more for the
    // staged values, one 16-byte word for all lanes for the pieces, neither used): with the same
    // loads on every path the compiler can wait for a stage's own loads alone (vmcnt = what was
    // requested after them), where a request under a condition makes it wait for everything outstanding.
#pragma unroll
    for (int u = 0; u < PF; ++u) {
        const bool live = u < rounds;
        const int kc = live ? (u * NW + wave) * BK : 0;
        if (SPLIT && PF > 1) {
            NGDB_ISSUE_VALUES(u, kc)
            NGDB_ISSUE_PIECES(u, kc, live)
        } else if (live) {
            NGDB_ISSUE_VALUES(u, kc)
            NGDB_ISSUE_PIECES(u, kc, true)
        }
    }
    for (int it0 = 0; SPLIT && it0 < rounds; it0 += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int it = it0 + u;
        const bool live_next = it + PF < rounds;
        const int knext = live_next ? ((it + PF) * NW + wave) * BK : 0;
        if (it < rounds) {
            const int kcur = (it * NW + wave) * BK;
            uint16_t* Ap = reinterpret_cast<uint16_t*>(As);
            uint16_t* Bp = reinterpret_cast<uint16_t*>(Bs);
            if (!AK) {
#pragma unroll
                for (int t = 0; t < TM; ++t)
                    stage_strided(Ap + t * SUBTILE, a.K, a.M, kcur, m0 + 32 * t, lane,
                                  reinterpret_cast<const float4(&)[2]>(ra[u][2 * t]));
            }
#pragma unroll
            for (int i = 0; AK && !AP && i < LA; ++i) {
                const int idx = lane + i * 64;
                const int m = idx / (BK / 4), kq = idx % (BK / 4);
                const int gk = kcur + kq * 4;
                float4 v = ra[u][i];
                if (has_add) { v.x += rd[u][i].x; v.y += rd[u][i].y; v.z += rd[u][i].z; v.w += rd[u][i].w; }
                const bool ok = avalid[i] && gk < a.K;
                v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
                if (copy_out && ok) *reinterpret_cast<float4*>(a.a_copy + (size_t)(m0 + m) * a.lda + gk) = v;
                store_pieces(Ap + (m >> 5) * SUBTILE, m & 31, kq, split3(v));
            }
            if (!BKC && !BP) {
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    stage_strided(Bp + t * SUBTILE, a.K, a.N, kcur, n0 + 32 * t, lane,
                                  reinterpret_cast<const float4(&)[2]>(rb[u][2 * t]));
            }
#pragma unroll
            for (int i = 0; BKC && !BP && i < LB; ++i) {
                const int idx = lane + i * 64;
                const int n = idx / (BK / 4), kq = idx % (BK / 4);
                float4 v = rb[u][i];
                const bool ok = n0 + n < a.N && kcur + kq * 4 < a.K;
                v.x = ok ? v.x : 0.f; v.y = ok ? v.y : 0.f; v.z = ok ? v.z : 0.f; v.w = ok ? v.w : 0.f;
                store_pieces(Bp + (n >> 5) * SUBTILE, n & 31, kq, split3(v));
            }
            if (!AP) __builtin_amdgcn_wave_barrier();
            // Operands that came as pieces are multiplied from the registers they were loaded into, and
            // those registers are requested again only after the MFMAs: copied aside first, the compiler
            // would load into temporaries and wait for them in the middle of the MFMAs.
            bf16x8 ap[TM][3], bp[TN][3];
            if (AP) {
#pragma unroll
                for (int q = 0; q < 3; ++q) ap[0][q] = aq[u][q];
            }
            if (BP) {
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 3; ++q) bp[j][q] = bq[u][BP ? j : 0][q];
            }
            // the staged values' registers are free again: their next tile is under way during the MFMAs
            // (one tile in flight: nothing for the compiler to count, and no request beyond the end)
            if (PF == 1 && live_next) { NGDB_ISSUE_VALUES(u, knext) }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
#pragma unroll
                for (int i = 0; !AP && i < TM; ++i)
                    ap[i][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Ap + i * SUBTILE + q * PIECE + unit_at<!AK>(lane)));
#pragma unroll
                for (int j = 0; !BP && j < TN; ++j)
                    bp[j][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Bp + j * SUBTILE + q * PIECE + unit_at<!BKC>(lane)));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {   // smallest products first
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][2], bp[j][0], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][0], bp[j][2], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][1], bp[j][1], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][1], bp[j][0], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][0], bp[j][1], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[i][0], bp[j][0], acc[i][j], 0, 0, 0);
                }
            if (!AP) __builtin_amdgcn_wave_barrier();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (PF > 1) { NGDB_ISSUE_VALUES(u, knext) }
        if (PF > 1 || live_next) {
            NGDB_ISSUE_PIECES(u, knext, live_next)
        }
      }
    }
    for (int it0 = 0; !SPLIT && it0 < rounds; it0 += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int it = it0 + u;
        if (it >= rounds) break;
        const int kcur = (it * NW + wave) * BK;
        stage_a<BM, LA, LDA, AK>(a, As, lane, m0, kcur, has_add, copy_out, avalid, ra[u], rd[u]);
        stage_b<BN, LB, LDB, BKC>(a, Bs, lane, n0, kcur, rb[u]);
        __builtin_amdgcn_wave_barrier();        // staged tile before its reads (compiler ordering only)
        if (it + PF < rounds) {
            const int kc = ((it + PF) * NW + wave) * BK;
            NGDB_ISSUE_VALUES(u, kc)
        }
        // all LDS operand reads of the tile are issued before the first MFMA, so that the
        // matrix pipe never waits for an LDS round trip between k steps
        float av[BK / 2][TM], bv[BK / 2][TN];
#pragma unroll
        for (int kk = 0; kk < BK / 2; ++kk) {
            const int krow = kk * 2 + (lane >> 5);
#pragma unroll
            for (int i = 0; i < TM; ++i) av[kk][i] = As[krow * LDA + i * 32 + (lane & 31)];
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[kk][j] = Bs[krow * LDB + j * 32 + (lane & 31)];
        }
        __builtin_amdgcn_sched_barrier(0);      // keep the reads ahead of the MFMAs
#pragma unroll
        for (int kk = 0; kk < BK / 2; ++kk)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk][i], bv[kk][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_wave_barrier();        // reads of this tile before the next one is staged
      }
    }
    if (!EARLY_EPILOGUE) { NGDB_LOAD_EPILOGUE() }   // in flight during the reduction
    constexpr int PQ = POOL ? std::max(1, BM / 2 * BN / (NW * 64)) : 1;      // pooled values of a thread (at most 16 members a tile)
    float px[PQ][NGDB_MAX_CARD];
    if (POOL && a.pool_k) {
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int e = tid + q * NW * 64, i = min(mt * mem + e / BN, n_mem - 1), col = min(n0 + e % BN, a.N - 1);
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) px[q][j] = a.pool_X[(size_t)(min(j, cls - 1) * n_mem + i) * a.ldc + col];
        }
    }
#undef NGDB_LOAD_EPILOGUE
#undef NGDB_ISSUE_VALUES
#undef NGDB_ISSUE_PIECES
    __syncthreads();                            // the staging areas are reused for the reduction

    // partial tiles -> LDS.  Accumulator layout of a 32x32 block: lane owns column
    // (lane & 31) and rows 8*(r/4) + 4*(lane/32) + r%4, r = 0..15.
    constexpr int NR = Smem<BM, BN, NW, SPLIT, BP, AP>::NR;
    float* red = smem + (wave % NR) * BM * (BN + 1);
#define NGDB_ACC_TO_LDS()                                                                   \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                         \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                         \
    _Pragma("unroll") for (int r = 0; r < 16; ++r) {                                       \
        const int row = i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);                  \
        red[row * (BN + 1) + j * 32 + (lane & 31)] = acc[i][j][r];                          \
    }
    if (NW > NR) {   // fold the upper half of the wavefronts into the lower half first
        if (wave >= NR) { NGDB_ACC_TO_LDS() }
        __syncthreads();
        if (wave < NR) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                        acc[i][j][r] += red[row * (BN + 1) + j * 32 + (lane & 31)];
                    }
        }
        __syncthreads();
    }
    if (wave < NR) { NGDB_ACC_TO_LDS() }
#undef NGDB_ACC_TO_LDS
    __syncthreads();

    // epilogue: the partial tiles are summed, the operands requested before the k loop applied
    const bool emit = a.c_pieces != nullptr;    // uniform
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
        const int e = tid + q * NW * 64;
        const int lr = e / BN, lc = e % BN;
        float v = smem[lr * (BN + 1) + lc];
#pragma unroll
        for (int w = 1; w < NR; ++w) v += smem[w * BM * (BN + 1) + lr * (BN + 1) + lc];
        v += e_bias[q];
        if (a.relu) v = fmaxf(v, 0.f);
        v = e_mask[q] > 0.f ? v : 0.f;
        v += e_add[q];
        bool inside = m0 + lr < a.M && n0 + lc < a.N;
        if (POOL) {
            (void)pool_row_of(lr, &inside);
            inside = inside && n0 + lc < a.N;
            if (a.pool_k) smem[lr * (BN + 1) + lc] = v;      // (read by the thread that owns the element only, as below)
        }
        if (inside && (!POOL || a.C)) a.C[(size_t)e_orow[q] * a.ldc + n0 + lc] = v;
        // (a slot of the first partial tile is read by the thread that owns the element only)
        if (BM == 32 && BN == 32 && SPLIT && emit) smem[lr * (BN + 1) + lc] = inside ? v : 0.f;
    }
    if (POOL && a.pool_k) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int e = tid + q * NW * 64, ii = e / BN, lc = e % BN, i = mt * mem + ii;
            if (ii >= mem || i >= n_mem || n0 + lc >= a.N) continue;
            float z[NGDB_MAX_CARD], mx = -INFINITY, den = 0.f, y = 0.f;
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                z[j] = smem[(min(j, cls - 1) * mem + ii) * (BN + 1) + lc];
                if (j < cls) mx = fmaxf(mx, z[j]);
            }
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) {
                z[j] = j < cls ? expf(z[j] - mx) : 0.f;
                den += z[j];
            }
            const float inv = 1.f / den;
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j) y += z[j] * inv * px[q][j];
            a.pool_out[(size_t)(a.pool_row ? a.pool_row[i] : i) * a.ldc + n0 + lc] = y;
        }
    }
    // The output once more as bf16 pieces in tile order (zero beyond the matrix), for the launch that
    // takes it as its A operand: block row m0/32, k-tiles n0/16 and n0/16 + 1; a lane of the first
    // two wavefronts splits eight consecutive values of a row.
    if (BM == 32 && BN == 32 && SPLIT && emit) {
        __syncthreads();
        if (tid < 128) {
            const int lr = tid & 31, u = tid >> 5;
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = smem[lr * (BN + 1) + u * 8 + j];
            const Pieces p0 = split3(make_float4(x[0], x[1], x[2], x[3])), p1 = split3(make_float4(x[4], x[5], x[6], x[7]));
            uint16_t* out = a.c_pieces + ((size_t)(m0 / 32) * a.c_kt + n0 / 16 + (u >> 1)) * WTILE + ((u & 1) * 32 + lr) * 8;
            *reinterpret_cast<uint4*>(out) = make_uint4(p0.h.x, p0.h.y, p1.h.x, p1.h.y);
            *reinterpret_cast<uint4*>(out + 512) = make_uint4(p0.m.x, p0.m.y, p1.m.x, p1.m.y);
            *reinterpret_cast<uint4*>(out + 1024) = make_uint4(p0.l.x, p0.l.y, p1.l.x, p1.l.y);
        }
    }
}

// Weight gradients.  Both operands have k (the rows) as the slow index.  A wavefront owns a 64 x 64 tile of the
// output over every fourth block of 16 rows and needs nobody: the blocks of both operands travel from global memory
// straight into its own LDS (256 bytes of a row by 16 lanes), are read as the 8 rows x 32 columns a lane group of
// the 32x32x16 MFMA wants, split into pieces in registers, and multiplied: 24 MFMAs (768 cycles) beside 176 vector
// operations (704) and 8 KB of operands a block, every split value feeding two MFMA blocks.  A block's
// buffer is requested again as soon as its values are in registers, so that two blocks are on the way during
// the arithmetic at 64 KB of LDS per workgroup, two workgroups per compute unit.  (Staged through registers
// and LDS as pieces, with one block ahead, a block took 4500 cycles: 51 us for the six contractions of 512
// queries at d=400, h=800 (1356, 730 and 182 rows) and 5 us for the bias gradients, against 29 us here; 88 and
// 53 us against 48 for 1024.)  The column sums of A that the bias gradients are fall out of the values read.
// Six bf16 products stand for an fp32 one, whatever the size of the step.  The five small ones have accumulators of their own,
// so that the large sums are rounded once a block: against fp64 the error is 0.4 to 0.9 of that of fp32 matrix instructions on
// eight partial sums (16 to 5000 rows; gradients with rows of one size or many, hidden rows of one sign or both).  All six
// in one accumulator were up to 1.9 times as far off as those, from 130 rows on.  185 -> 249 registers, still two
// wavefronts per SIMD and the same time.
constexpr int WG_T = 64, WG_LD = WG_T + 1;
struct WgradGroup {
    int count;
    int tile_start[GEMM_MAX_GROUP + 1];
    WgradArgs p[GEMM_MAX_GROUP];
};
__global__ __launch_bounds__(256, 2) void wgrad_kernel(const WgradGroup g) {
    constexpr int BUF = 16 * WG_T * 4;                      // bytes of 16 rows of one operand
    constexpr int WAVE_LDS = WG_T * WG_LD * 4;              // >= two buffers of both operands; the partial tile at the end
    static_assert(WAVE_LDS >= 4 * BUF, "staging fits the reduction area");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * WAVE_LDS];
    __shared__ float cs[4][WG_T];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int p = 0;
#pragma unroll
    for (int i = 1; i < GEMM_MAX_GROUP; ++i)
        if (i < g.count && (int)blockIdx.x >= g.tile_start[i]) p = i;
    const WgradArgs& a = g.p[p];
    // (tiles to dies as in gemm_kernel)
    const int local = (int)blockIdx.x - g.tile_start[p], per_die = (g.tile_start[p + 1] - g.tile_start[p]) >> 3;
    const int tile = (local & 7) * per_die + (local >> 3);
    const int tiles_m = (a.M + WG_T - 1) / WG_T, tiles_n = (a.N + WG_T - 1) / WG_T;
    if (tile >= tiles_m * tiles_n) return;
    const bool m_major = a.M >= a.N;
    const int m0 = (m_major ? tile / tiles_n : tile % tiles_m) * WG_T;
    const int n0 = (m_major ? tile % tiles_n : tile / tiles_m) * WG_T;

    const int nk = (a.K + 15) / 16;
    const int rounds = nk > wave ? (nk - wave + 3) / 4 : 0;
    unsigned char* mine = lds + wave * WAVE_LDS;
    const uint32_t at = lds_addr(mine);
    const int row_in = lane >> 4, col_in = (lane & 15) * 4;
    const float* acol = a.A + min(m0 + col_in, a.M - 4);
    const float* bcol = a.B + min(n0 + col_in, a.N - 4);
    // (rounds past the end fetch the last one again; rows past K the last row, zeroed after the read)
    auto issue = [&](int it) {
        const int k0 = (min(it, rounds - 1) * 4 + wave) * 16;
        const uint32_t to = at + (uint32_t)(it & 1) * 2 * BUF;
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_load16(acol + (size_t)min(k0 + q * 4 + row_in, a.K - 1) * a.lda, to + q * 1024);
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_load16(bcol + (size_t)min(k0 + q * 4 + row_in, a.K - 1) * a.ldb, to + BUF + q * 1024);
    };
    floatx16 acc[2][2], low[2][2];      // products of the first pieces; the other five of the six
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = low[i][j][r] = 0.f;
    float csum[2] = {0.f, 0.f};
    float v[4][8];                      // values of a block: A columns 0-31, 32-63, B columns 0-31, 32-63
    bf16x8 pc[2][4][3];                 // pieces of the block being multiplied and of the next
    auto fetch = [&](int it) {
        wait_vm<8>();
        asm volatile("" ::: "memory");
        // lane: column (lane & 31) of a group of 32, rows 8 * (lane >> 5) .. + 7
        const float* src = reinterpret_cast<const float*>(mine + (it & 1) * 2 * BUF) + (lane >> 5) * 8 * WG_T + (lane & 31);
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 8; ++r) v[o * 2 + b][r] = src[o * (BUF / 4) + r * WG_T + b * 32];
        wait_lds();
        issue(it + 2);
        const int k0 = (it * 4 + wave) * 16;
        if (k0 + 16 > a.K) {            // the last block, or beyond it: rows past the end count nothing
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (k0 + (lane >> 5) * 8 + r >= a.K) v[0][r] = v[1][r] = v[2][r] = v[3][r] = 0.f;
        }
    };
    auto split = [&](bf16x8 (&to)[4][3]) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
            csum[b] += ((v[b][0] + v[b][1]) + (v[b][2] + v[b][3])) + ((v[b][4] + v[b][5]) + (v[b][6] + v[b][7]));
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            u32x4 h, m, l;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t wh, wm, wl;
                split2(v[b][2 * q], v[b][2 * q + 1], wh, wm, wl);
                h[q] = wh; m[q] = wm; l[q] = wl;
            }
            to[b][0] = __builtin_bit_cast(bf16x8, h);
            to[b][1] = __builtin_bit_cast(bf16x8, m);
            to[b][2] = __builtin_bit_cast(bf16x8, l);
        }
    };
    // smallest products first; the output is built transposed (a lane holds 4 consecutive columns of a row)
    auto multiply = [&](const bf16x8 (&of)[4][3]) {
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    floatx16& to = t < 5 ? low[i][j] : acc[i][j];
                    to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(of[2 + j][PB[t]], of[i][PA[t]], to, 0, 0, 0);
                }
    };
    if (rounds > 0) {
        issue(0);
        issue(1);
        fetch(0);
        split(pc[0]);
        // the next block is split between the MFMAs of this one: matrix and vector unit work side by side in one
        // wavefront (a block beyond the last is zeros)
        for (int it0 = 0; it0 < rounds; it0 += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (it0 + u < rounds) {     // uniform
                    fetch(it0 + u + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(pc[u]);
                    split(pc[u ^ 1]);
#pragma unroll
                    for (int q = 0; q < 24; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);    // one MFMA,
                        __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);    // then vector operations
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    wait_vm<0>();                       // (the requests past the end land before their place is used again)
    float* part = reinterpret_cast<float*>(mine);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[(i * 32 + (lane & 31)) * WG_LD + j * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3)] = acc[i][j][r] + low[i][j][r];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const float both = csum[b] + __shfl_xor(csum[b], 32, 64);
        if (lane < 32) cs[wave][b * 32 + lane] = both;
    }
    __syncthreads();
    const float* all = reinterpret_cast<const float*>(lds);
#pragma unroll
    for (int q = 0; q < WG_T * WG_T / 4 / 256; ++q) {
        const int idx = tid + q * 256, lr = idx / (WG_T / 4), lc = (idx % (WG_T / 4)) * 4;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] += all[w * (WAVE_LDS / 4) + lr * WG_LD + lc + j];
        if (m0 + lr < a.M && n0 + lc < a.N)
            *reinterpret_cast<float4*>(a.C + (size_t)(m0 + lr) * a.ldc + n0 + lc) = make_float4(o[0], o[1], o[2], o[3]);
    }
    if (a.colsum && n0 == 0 && tid < WG_T && m0 + tid < a.M)
        a.colsum[m0 + tid] = (cs[0][tid] + cs[1][tid]) + (cs[2][tid] + cs[3][tid]);
}

// Forward layers and data gradients over many rows, weights from pieces.  A tile of 32 WM rows x 64 columns belongs to
// WM x WK wavefronts: one takes 32 rows x 64 columns over every WK-th block of 16 k.  Rows (fp32) and pieces travel from global
// memory straight into LDS: a wavefront's own rows, and for the WM of a block the pieces together.  A wavefront reads both as
// MFMA operands, splits the rows on the way (44 vector operations a block) and multiplies (12 MFMAs, 384 cycles); a block's
// requests are on their way for one turn.  Every operand reaches a compute unit once a tile instead of once a wavefront, and a
// row is split once per 64 columns: gemm_kernel's 32 x 32 tiles fetch 5 KB a block of 6 MFMAs, which at 2000 rows is 190 MB
// through the L1s.  What is left is bound by LDS (8 KB read and 5 KB written a block and wavefront) and by issue; it takes four
// wavefronts a SIMD to hide that (128 registers), and 64 x 64 accumulators on two, or three stages in LDS, were slower.
// us a launch at d = 400, h = 800 (first layer with relations and copy, second layer, their gradients), against gemm_kernel:
// 480 rows 7.8 7.9 7.8 6.6 (8.8 8.2 8.2 7.9), 1000 rows 11.0 8.3 8.2 8.4 (14.9 10.8 10.8 12.1), 2000 rows 17.3 11.7 11.7 13.7
// (22.5 18.9 19.1 19.7), 7900 rows 57 40 40 44 (76 59 60 64).  The whole forward pass of 1024 queries (launches and their gaps included)
// 136 -> 121 us, of 4096 314 -> 261.
// 64 bytes of a row and block land per row; 16-byte unit c of row r is stored at c ^ tile_swizzle(r), which spreads the reads
// of 16 rows over all banks.
// ADD: problems may add a second gathered row (the relation's) to every row of A; it is staged likewise.
// POOL: as in gemm_kernel, 32 WM / pool_k members to a tile.
// The sums are formed as in gemm_kernel (WK partial sums of blocks, six products each, smallest first).
constexpr int FIRST = 3;      // products ahead of the wait for a block's reads
constexpr int PN = 64, PN_LD = PN + 4;      // columns of a tile
__device__ __forceinline__ int tile_swizzle(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }
template <int WM, int WK, bool ADD, bool POOL, class Group>
__global__ __launch_bounds__(WM * WK * 64, WM > 1 ? 4 : 2) void product_kernel(const Group g) {
    constexpr int NW = WM * WK, BM = 32 * WM;
    constexpr int AB = 2048, BB = 2 * WTILE * 2;             // bytes of 32 rows of a block, of two tiles of pieces
    constexpr int ROWS = (ADD ? 2 : 1) * AB, GROUP = 2 * BB + WM * ROWS;
    // partial sums of a group of wavefronts: where one wavefront alone staged (its own requests are in), else behind a barrier
    constexpr int PART = WM == 1 ? GROUP : BM * PN_LD * 4;
    static_assert(PART >= BM * PN_LD * 4, "a partial tile fits its place");
    constexpr int BL = (6 + WM - 1) / WM;                    // loads of pieces per wavefront and stage
    __shared__ __attribute__((aligned(1024))) unsigned char lds[WK * (GROUP > PART ? GROUP : PART)];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave / WM, wm = wave % WM;      // (in scalar registers)
    int p = 0;
#pragma unroll
    for (int i = 1; i < Group::MOST; ++i)
        if (i < g.count && (int)blockIdx.x >= g.tile_start[i]) p = i;
    const GemmArgs& a = g.p[p];
    // (all of the arguments that are used late are requested here: one by one each costs a round trip to the argument segment)
    const float *bias = a.bias, *mask = a.mask, *addend = a.addend, *X = a.pool_X;
    const int32_t *dst_row = a.dst_row, *pool_row = a.pool_row;
    float *C = a.C, *a_copy = a.a_copy, *pool_out = a.pool_out;
    const int ldc = a.ldc, ldmask = a.ldmask, ldadd = a.ldadd, relu = a.relu;
    asm volatile("" ::"s"(bias), "s"(mask), "s"(addend), "s"(dst_row), "s"(C), "s"(a_copy), "s"(ldc), "s"(ldmask), "s"(ldadd), "s"(relu));
    if (POOL) asm volatile("" ::"s"(X), "s"(pool_row), "s"(pool_out));
    // (tiles to dies as in gemm_kernel)
    const int local = (int)blockIdx.x - g.tile_start[p], per_die = (g.tile_start[p + 1] - g.tile_start[p]) >> 3;
    const int tile = (local & 7) * per_die + (local >> 3);
    const int cls = POOL && a.pool_k ? a.pool_k : 1, mem = BM / cls, n_mem = a.M / cls;
    const int tiles_m = (n_mem + mem - 1) / mem, tiles_n = (a.N + PN - 1) / PN;
    if (tile >= tiles_m * tiles_n) return;
    const bool m_major = a.M >= a.N;
    const int mt = m_major ? tile / tiles_n : tile % tiles_m;
    const int nt = m_major ? tile % tiles_n : tile / tiles_m, n0 = nt * PN;
    auto row_of = [&](int lr, bool* ok) {          // row of A and C that row lr of the tile is (past the end: the last one)
        const int j = POOL ? lr / mem : 0, i = mt * mem + lr - j * mem;
        *ok = j < cls && i < n_mem;
        return *ok ? j * n_mem + i : a.M - 1;
    };

    const int nk = (a.K + 15) / 16, stages = (nk + WK - 1) / WK, k_last = a.K - 4;
    const uint32_t at = lds_addr(lds) + kg * GROUP, at_a = at + 2 * BB + wm * ROWS;
    const bool has_add = ADD && a.a_add_idx != nullptr;      // uniform
    // (the second tile of a last column block that has one only: the first once more, its columns are not stored)
    const uint16_t* btile = a.b_pieces + (size_t)(n0 / 32) * a.b_kt * WTILE;
    const uint32_t b_next = n0 + 32 < a.N ? (uint32_t)a.b_kt * WTILE : 0u;
    uint32_t b_at[BL];                  // this wavefront's pieces of a stage: i % 3 of tile i / 3
#pragma unroll
    for (int q = 0; q < BL; ++q) {
        const int i = min(wm * BL + q, 5);
        b_at[q] = i >= 3 ? b_next + (i - 3) * 512 : i * 512;
    }
    // (stages past the end fetch the last block again; k past the end the last four, which meet zeros in the pieces)
    auto issue_b = [&](int s, int half) {
        const uint16_t* b = btile + (uint32_t)min(s * WK + kg, nk - 1) * WTILE;
#pragma unroll
        for (int q = 0; q < BL; ++q) lds_load16_at(b + b_at[q], lane * 16, at + half * BB + min(wm * BL + q, 5) * 1024);
    };
    issue_b(0, 0);                      // on their way while the rows are looked up
    issue_b(1, 1);
    const int unit = ((lane & 3) ^ tile_swizzle(lane >> 2)) * 4;                // k of the 16 bytes this lane fetches
    const float *arow[2], *radd[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        bool ok;
        const int m = row_of(wm * 32 + q * 16 + (lane >> 2), &ok);
        if (a.a_ref) {
            const int32_t r = a.a_ref[m];
            arow[q] = r >= 0 ? a.a_base0 + (size_t)r * a.lda : a.a_base1 + (size_t)(-1 - r) * a.lda;
        } else {
            arow[q] = a.A + (size_t)m * a.lda;
        }
        if (ADD) radd[q] = has_add ? a.a_add + (size_t)a.a_add_idx[m] * a.lda : arow[q];
    }
    auto issue_a = [&](int s, auto added) {
        const uint32_t k = (uint32_t)min(min(s * WK + kg, nk - 1) * 16 + unit, k_last);
#pragma unroll
        for (int q = 0; q < 2; ++q) lds_load16(arow[q] + k, at_a + q * 1024);
        if (decltype(added)::value) {
#pragma unroll
            for (int q = 0; q < 2; ++q) lds_load16(radd[q] + k, at_a + AB + q * 1024);
        }
    };
    floatx16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    float v[8];                         // values of a block of A
    bf16x8 pa[2][3], pb[2][2][3];       // pieces of the block being multiplied and of the next
    // lane: row (lane & 31) of 32, k = 8 * (lane >> 5) .. + 7 = units 2 * (lane >> 5) and the next
    const int f = tile_swizzle(lane & 15), u0 = (lane >> 5) * 2;
    const unsigned char* rows = lds + kg * GROUP + 2 * BB + wm * ROWS + (lane & 31) * 64;
    const unsigned char* pieces = lds + kg * GROUP + lane * 16;
    auto fetch = [&](int half, bf16x8 (&b)[2][3], auto added) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int off = ((u0 + h) ^ f) * 16;
            float4 x = *reinterpret_cast<const float4*>(rows + off);
            if (decltype(added)::value) {
                const float4 y = *reinterpret_cast<const float4*>(rows + AB + off);
                x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
            }
            v[h * 4] = x.x; v[h * 4 + 1] = x.y; v[h * 4 + 2] = x.z; v[h * 4 + 3] = x.w;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q) b[j][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(pieces + half * BB + (j * 3 + q) * 1024));
    };
    auto split = [&](bf16x8 (&to)[3]) {
        u32x4 h, m, l;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t wh, wm_, wl;
            split2(v[2 * q], v[2 * q + 1], wh, wm_, wl);
            h[q] = wh; m[q] = wm_; l[q] = wl;
        }
        to[0] = __builtin_bit_cast(bf16x8, h);
        to[1] = __builtin_bit_cast(bf16x8, m);
        to[2] = __builtin_bit_cast(bf16x8, l);
    };
    // smallest products first; the output is built transposed (a lane holds 4 consecutive columns of a row)
    auto multiply = [&](const bf16x8 (&fa)[3], const bf16x8 (&fb)[2][3], auto from, auto to) {
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int t = decltype(from)::value; t < decltype(to)::value; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j][PB[t]], fa[PA[t]], acc[j], 0, 0, 0);
    };
    using N0 = std::integral_constant<int, 0>;
    using N1 = std::integral_constant<int, 1>;
    using NF = std::integral_constant<int, FIRST>;
    using N6 = std::integral_constant<int, 6>;
    auto walk = [&](auto added) {
        // what was asked for has landed, everybody's, and everybody has read what it fetched
        auto arrive = [&]() {
            asm volatile("" ::: "memory");
            wait_lds();
            wait_vm<0>();
            if (WM > 1) __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        auto turn = [&](int s, auto half) {
            constexpr int u = decltype(half)::value;
            arrive();
            fetch(u ^ 1, pb[u ^ 1], added);
            issue_b(s + 2, u);
            multiply(pa[u], pb[u], N0(), NF());         // (while the reads are on their way)
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            wait_lds();
            issue_a(s + 2, added);                      // the rows' place is this wavefront's own
            __builtin_amdgcn_sched_barrier(0);
            multiply(pa[u], pb[u], NF(), N6());
            split(pa[u ^ 1]);
#pragma unroll
            for (int q = 0; q < 12 - 2 * FIRST; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);    // one MFMA,
                __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);    // then vector operations
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        issue_a(0, added);
        arrive();
        fetch(0, pb[0], added);
        wait_lds();
        issue_a(1, added);
        split(pa[0]);
        // (in the last stage not every group of wavefronts has a block)
        const bool last = (stages - 1) * WK + kg < nk;
        int s = 0;
        for (; s + 2 < stages; s += 2) {
            turn(s, N0());
            turn(s + 1, N1());
        }
        if (s + 1 < stages) {
            turn(s, N0());
            if (last) multiply(pa[1], pb[1], N0(), N6());
        } else if (last) {
            multiply(pa[0], pb[0], N0(), N6());
        }
    };
    if (has_add) walk(std::true_type());
    else walk(std::false_type());
    wait_vm<0>();                       // (the requests past the end land before their place is used again)
    if (WM > 1) __syncthreads();
    // The rows as gathered, for who reads them later: every tile copies its share of their columns, a wavefront its rows and its
    // share of these (requested here, stored last).
    const bool copies = !POOL && a_copy != nullptr;
    const int k4 = a.K >> 2, per = (k4 + tiles_n - 1) / tiles_n, c_end = min(k4, (nt + 1) * per);
    int c = nt * per + kg * 4;
    float4 cy[2], cz[2];
    auto copy_load = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int k = min(c + (lane & 3), k4 - 1) * 4;
            cy[q] = load_global4(arow[q] + k);
            if (has_add) cz[q] = load_global4(radd[q] + k);
        }
    };
    auto copy_store = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int m = mt * BM + wm * 32 + q * 16 + (lane >> 2), k = c + (lane & 3);
            if (has_add) { cy[q].x += cz[q].x; cy[q].y += cz[q].y; cy[q].z += cz[q].z; cy[q].w += cz[q].w; }
            if (m < a.M && k < c_end) *reinterpret_cast<float4*>(a_copy + (size_t)m * a.lda + k * 4) = cy[q];
        }
    };
    if (copies) copy_load();
    // operands of the epilogue: four consecutive columns of ER rows per thread, in flight during the reduction
    constexpr int ER = BM * PN / 4 / (NW * 64), RS = NW * 4;      // rows of a thread, RS apart
    const int lc = (tid & 15) * 4, col = min(n0 + lc, a.N - 4);
    float4 e_mask[ER], e_add[ER];
    float e_bias[4];
    int row[ER], orow[ER];
    bool inside[ER];
#pragma unroll
    for (int j = 0; j < 4; ++j) e_bias[j] = bias ? bias[col + j] : 0.f;
#pragma unroll
    for (int q = 0; q < ER; ++q) {
        row[q] = row_of((tid >> 4) + q * RS, &inside[q]);
        e_mask[q] = mask ? load_global4(mask + (size_t)row[q] * ldmask + col) : make_float4(1.f, 1.f, 1.f, 1.f);
        e_add[q] = addend ? load_global4(addend + (size_t)row[q] * ldadd + col) : make_float4(0.f, 0.f, 0.f, 0.f);
        inside[q] = inside[q] && n0 + lc < a.N;
    }
#pragma unroll
    for (int q = 0; q < ER; ++q) orow[q] = dst_row ? dst_row[row[q]] : row[q];
    float* part = reinterpret_cast<float*>(lds + kg * PART) + (wm * 32 + (lane & 31)) * PN_LD;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<float4*>(part + j * 32 + r * 8 + (lane >> 5) * 4) =
                make_float4(acc[j][r * 4], acc[j][r * 4 + 1], acc[j][r * 4 + 2], acc[j][r * 4 + 3]);
    __syncthreads();
    float* all = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int q = 0; q < ER; ++q) {
        float* mine4 = all + ((tid >> 4) + q * RS) * PN_LD + lc;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WK; ++w) {
            const float4 x = *reinterpret_cast<const float4*>(mine4 + w * (PART / 4));
            o[0] += x.x; o[1] += x.y; o[2] += x.z; o[3] += x.w;
        }
        const float mk[4] = {e_mask[q].x, e_mask[q].y, e_mask[q].z, e_mask[q].w}, ad[4] = {e_add[q].x, e_add[q].y, e_add[q].z, e_add[q].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] += e_bias[j];
            if (relu) o[j] = fmaxf(o[j], 0.f);
            o[j] = mk[j] > 0.f ? o[j] : 0.f;
            o[j] += ad[j];
        }
        const float4 out = make_float4(o[0], o[1], o[2], o[3]);
        if (inside[q] && (!POOL || C)) *reinterpret_cast<float4*>(C + (size_t)orow[q] * ldc + n0 + lc) = out;
        if (POOL && a.pool_k) *reinterpret_cast<float4*>(mine4) = out;      // (read before by this thread only)
    }
    if (copies) {
        copy_store();
        for (c += 4 * WK; c < c_end; c += 4 * WK) {
            copy_load();
            copy_store();
        }
    }
    if (POOL && a.pool_k) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < (ER + 1) / 2; ++q) {                 // (at most BM / 2 members a tile)
            const int ii = (tid >> 4) + q * RS, i = mt * mem + ii;
            if (ii >= mem || i >= n_mem || n0 + lc >= a.N) continue;
            float4 z[NGDB_MAX_CARD], x[NGDB_MAX_CARD];
#pragma unroll
            for (int j = 0; j < NGDB_MAX_CARD; ++j)
                if (j < cls) {
                    x[j] = load_global4(X + (size_t)(j * n_mem + i) * ldc + n0 + lc);
                    z[j] = *reinterpret_cast<const float4*>(all + (j * mem + ii) * PN_LD + lc);
                }
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                auto of = [&](const float4& f4) { return e == 0 ? f4.x : (e == 1 ? f4.y : (e == 2 ? f4.z : f4.w)); };
                float mx = -INFINITY, den = 0.f, w[NGDB_MAX_CARD];
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j)
                    if (j < cls) mx = fmaxf(mx, of(z[j]));
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j)
                    if (j < cls) { w[j] = expf(of(z[j]) - mx); den += w[j]; }
                const float inv = 1.f / den;
                y[e] = 0.f;
#pragma unroll
                for (int j = 0; j < NGDB_MAX_CARD; ++j)
                    if (j < cls) y[e] += w[j] * inv * of(x[j]);
            }
            *reinterpret_cast<float4*>(pool_out + (size_t)(pool_row ? pool_row[i] : i) * ldc + n0 + lc) = make_float4(y[0], y[1], y[2], y[3]);
        }
    }
}

// A pass over up to some hundred rows a depth, all layers of all depths in one launch a direction (or of the deep ones, where the first have more rows).
// As launches such layers take 6 to 10 us and a gap of 2 before each; what bounds them is the chain from the arguments over references, rows and weights to the
// sums, not the 1 to 2 us of the matrix unit.  Here a workgroup has one tile of 32 rows x 32 columns, requests its first weights and
// relations and looks its rows up before it waits for the layer before, and then brings its rows into LDS at once; the weights go from
// global memory into the registers they are multiplied from.  k is dealt to the eight wavefronts in blocks of 16, four of them on the way; 64 KB
// of LDS and 128 registers leave room for two workgroups a compute unit.  Rows handed from layer to layer are stored and loaded at
// the scope of the card (level.hip: levels_kernel).  Tiles are dealt by workgroup number (TileHelp), waits and
// giving up are those of rows_chain_kernel; the counts are cleared by the launch that splits the weights.  Sums are formed as in product_kernel with eight partial sums.
// What a workgroup has to know first comes in two round trips to the argument segment, its part of the layer, then that part's values
// and pointers (looked up one by one, with divisions, the start of a tile took 2 to 6 us instead of 1.0 to 2.5).  A layer takes 4.3 us at k = 400 and 5.3 at
// 800: 0.9 until a count is seen, 0.7 for the rows, 1.3 and 2.3 for the products, 0.5 to 1 for sums and pooling, 0.5 for the stores.
// Scoring and training with 8 negatives, by launches and like this, us: 40 queries at d = 400, h = 800 75 and 162 against 64 and 137, 160
// queries 84 and 186 against 76 and 175, 320 95 and 222 against 91 and 216; 40 at 208, 416 63 and 141 against 50 and 108, 160 70 and 155 against 52 and 123, 512 76
// and 181 against 66 and 171; 40 at 512, 1024 77 and 177 against 69 and 157.
// Boxes, whose projections are parts of their own: 40 queries at d = 300, h = 500 49 and 108 against 40 and 90, 160 56 and 118 against 43 and 102, 80 at 400, 800 58 and
// 120 against 44 and 101, 160 at 160, 320 56 and 109 against 34 and 87.
constexpr int TC_WAVES = 8, TC_T = TC_WAVES * 64, TC_AHEAD = 4, TC_LD = 36;
static_assert(TC_AHEAD * TC_WAVES * 16 >= TILE_D && 2 * TC_AHEAD * TC_WAVES * 16 >= TILE_H, "relations in registers; two chunks at most");
// (the number of the launch that had taken it before)
__device__ __forceinline__ unsigned long long tc_take(const TileChain& r, int at) {
    return __hip_atomic_exchange(r.taken + at, r.launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tc_taken(const TileChain& r, int at) {
    return __hip_atomic_load(r.taken + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == r.launch;
}
// The first tile of the workgroups before `end` that nobody has, taken; TILE_GO: there is none.  By one wavefront.
__device__ __forceinline__ int tc_take_first(const TileChain& r, int end) {
    const int lane = threadIdx.x & 63;
    for (int base = 0; base < end; base += 64) {
        unsigned long long open = __ballot(base + lane < end && !tc_taken(r, min(base + lane, end - 1)));
        for (; open != 0ull; open &= open - 1ull) {
            const int at = base + __ffsll(open) - 1;
            if (__ballot(lane == 0 && tc_take(r, at) != r.launch) == 0ull) continue;
            if (lane == 0) __hip_atomic_fetch_add(r.help.helped, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return at;
        }
    }
    return TILE_GO;
}
// Waits until all tiles of the layer before are through, each counted in one of its words; *state: what to do (TILE_*), for all threads.  taken: (of the first
// thread) what tc_take said of its tile, looked at only here, as the answer is slow; helps: may take another tile meanwhile.
__device__ __forceinline__ void tc_wait(const TileChain& r, int l, const int32_t* before_counts, int before_tiles, int polls, unsigned long long taken, bool helps, int* state) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x, want = (before_tiles - lane + TILE_LINES - 1) / TILE_LINES;       // of this lane's word
        const int32_t* word = before_counts + min(lane, TILE_LINES - 1) * TILE_STRIDE;
        asm volatile("" : "+v"(taken));
        int got = __builtin_amdgcn_readfirstlane((int)(taken != r.launch)) ? TILE_GO : TILE_TAKEN, again = max(r.help.patience, 0);
        if (got == TILE_GO && l > 0) {
            got = TILE_GAVE_UP;
            for (int i = 0; i < polls; ++i) {
                const int n = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__ballot(lane < TILE_LINES && n != want) == 0ull) {
                    got = TILE_GO;
                    break;
                }
                if (__ballot(lane < TILE_LINES && n > want) != 0ull) break;
                if (__builtin_expect(helps && i >= again, 0)) {
                    int part = 0;                          // (the first of this layer)
                    while (part + 1 < r.parts && (int)(r.start[part] >> 4 & 15) < l) ++part;
                    const int at = tc_take_first(r, (int)(r.start[part] >> 8));
                    if (at >= 0) {
                        got = at;
                        break;
                    }
                    again = i + TILE_AGAIN;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        if (lane == 0) *state = got;
    }
    asm volatile("" ::: "memory");
    __syncthreads();
}
// The end of a tile that others wait for (number: in its layer; counts: null where nobody does)
__device__ __forceinline__ void tc_through(const TileChain& r, int32_t* counts, int number, bool there) {
    if (!counts && there) return;
    wait_vm<0>();                    // this wavefront's values are where the next layer finds them,
    __syncthreads();                 // ... and everybody's
    if (threadIdx.x != 0) return;
    if (!there) {
        __hip_atomic_store(r.sync.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(r.sync.host_gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (counts) __hip_atomic_fetch_add(counts + number % TILE_LINES * TILE_STRIDE, there ? 1 : GAVE_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A tile of a class's pooling, backward (pool.h: attention<true>, and smallest<true> for the offsets of boxes): a thread takes four coordinates of a member.
template <bool OFFSETS>
__device__ __forceinline__ int tc_pool_backward(const TileChain& r, const TilePart& p, int tile, int l, const int32_t* before_counts, int before_tiles, int polls,
                                                int32_t* counts, unsigned long long taken, bool helps, int* state) {
    const int d = r.d, d4 = d >> 2, k = p.cls, t = tile * TC_T + (int)threadIdx.x;
    const bool inside = t < p.n_mem * d4;
    const int i = min((int)__umulhi((uint32_t)t, p.inv_by), p.n_mem - 1), c = min(t - i * d4, d4 - 1) * 4;      // (inv_by: by d4)
    float4 a[TILE_CARD], x[TILE_CARD];
#pragma unroll
    for (int j = 0; j < TILE_CARD; ++j) {
        const size_t at = (size_t)(p.row0 + min(j, k - 1) * p.n_mem + i) * d + c;
        a[j] = load_global4((OFFSETS ? r.Gate : r.Att) + at);
        x[j] = load_global4(r.Z[OFFSETS ? 2 : 1] + at);
    }
    tc_wait(r, l, before_counts, before_tiles, polls, taken, helps, state);
    const float* from = (OFFSETS ? r.doff : r.dact) + (size_t)(p.out0 + i) * d + c;
    const float2 g0 = card_get2(from), g1 = card_get2(from + 2);
    const int got = __builtin_amdgcn_readfirstlane(*state);      // (looked at when the values are requested)
    if (got >= 0 || got == TILE_TAKEN) return got;
    const bool there = got == TILE_GO;
    auto one = [&](float g, auto of) {
        if (OFFSETS) {
            float mean = 0.f, mn = INFINITY;
            int arg = 0;
#pragma unroll
            for (int j = 0; j < TILE_CARD; ++j) {
                if (j >= k) break;
                mean += of(a[j]);
                if (of(x[j]) < mn) {                         // strict: equal offsets keep the lower input
                    mn = of(x[j]);
                    arg = j;
                }
            }
            const float gate = sigmoid_f(mean / (float)k), dpre = g * mn * gate * (1.f - gate) / (float)k;
#pragma unroll
            for (int j = 0; j < TILE_CARD; ++j) {
                of(a[j]) = there ? dpre : NAN;
                of(x[j]) = j == arg ? g * gate : 0.f;
            }
            return;
        }
        float mx = -INFINITY, den = 0.f, tall = 0.f;
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j)
            if (j < k) mx = fmaxf(mx, of(a[j]));
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j) {
            of(a[j]) = j < k ? expf(of(a[j]) - mx) : 0.f;
            den += of(a[j]);
        }
        const float inv = 1.f / den;
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j) tall += of(a[j]) * inv * of(x[j]) * g;
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j) {
            const float w = of(a[j]) * inv;
            of(a[j]) = there ? w * (g * of(x[j]) - tall) : NAN;
            of(x[j]) = w * g;
        }
    };
    one(g0.x, [](float4& f) -> float& { return f.x; });
    one(g0.y, [](float4& f) -> float& { return f.y; });
    one(g1.x, [](float4& f) -> float& { return f.z; });
    one(g1.y, [](float4& f) -> float& { return f.w; });
#pragma unroll
    for (int j = 0; j < TILE_CARD; ++j) {
        if (j >= k || !inside) break;
        const size_t at = (size_t)(p.row0 + j * p.n_mem + i) * d + c;
        float *const da = (OFFSETS ? r.dGate : r.dAtt) + at, *const dx = (OFFSETS ? r.DxO : r.Dx) + at;
        card_put2(da, a[j].x, a[j].y);
        card_put2(da + 2, a[j].z, a[j].w);
        card_put2(dx, x[j].x, x[j].y);
        card_put2(dx + 2, x[j].z, x[j].w);
    }
    tc_through(r, counts, p.number + tile, there);
    return TILE_GO;
}
// A tile of the projections of boxes (box.hip: proj_body), likewise.
template <bool BWD>
__device__ __forceinline__ int tc_box_projection(const TileChain& r, const TilePart& p, int tile, int l, const int32_t* before_counts, int before_tiles, int polls,
                                                 int32_t* counts, unsigned long long taken, bool helps, int* state) {
    const int d = r.d, d4 = d >> 2, t = tile * TC_T + (int)threadIdx.x;
    const bool inside = t < p.n_mem * d4;
    const int i = min((int)__umulhi((uint32_t)t, p.inv_by), p.n_mem - 1), c = min(t - i * d4, d4 - 1) * 4;
    const int32_t ref = r.refs[p.ref0 + i];                  // (backward: the row of the input's gradient)
    const size_t out = (size_t)(p.out0 + i) * d + c;
    auto get = [](const float* from) {
        const float2 a = card_get2(from), b = card_get2(from + 2);
        return make_float4(a.x, a.y, b.x, b.y);
    };
    float4 x, o = make_float4(0.f, 0.f, 0.f, 0.f), rc = o, ro = o;
    if (!BWD) {
        const size_t rel = (size_t)r.rel[p.rel0 + i] * d + c;
        rc = load_global4(r.R + rel);
        ro = load_global4(r.Ro + rel);
    }
    tc_wait(r, l, before_counts, before_tiles, polls, taken, helps, state);
    float *to_x, *to_o;
    if (BWD) {
        x = get(r.dact + out);
        o = get(r.doff + out);
        to_x = r.dact + (size_t)ref * d + c;
        to_o = r.doff + (size_t)ref * d + c;
    } else {
        if (ref >= 0) {
            x = get(r.act + (size_t)ref * d + c);
            o = get(r.off + (size_t)ref * d + c);
        } else {
            x = load_global4(r.E + (size_t)(-1 - ref) * d + c);
        }
        x.x += rc.x; x.y += rc.y; x.z += rc.z; x.w += rc.w;
        o.x += fmaxf(ro.x, 0.f); o.y += fmaxf(ro.y, 0.f); o.z += fmaxf(ro.z, 0.f); o.w += fmaxf(ro.w, 0.f);
        to_x = r.act + out;
        to_o = r.off + out;
    }
    const int got = __builtin_amdgcn_readfirstlane(*state);
    if (got >= 0 || got == TILE_TAKEN) return got;
    const bool there = got == TILE_GO;
    if (!there) x = o = make_float4(NAN, NAN, NAN, NAN);
    if (inside) {
        card_put2(to_x, x.x, x.y);
        card_put2(to_x + 2, x.z, x.w);
        card_put2(to_o, o.x, o.y);
        card_put2(to_o + 2, o.z, o.w);
    }
    tc_through(r, counts, p.number + tile, there);
    return TILE_GO;
}
// BWD: the reverse.  An intersection's pooling is a layer of its own, four coordinates of a member a thread, ahead of its depth's other two.
// The tile of workgroup `at`.  takes: the workgroup that runs it still has to take it; helps: may take another one while it waits.  Returns whose tile to
// compute first (>= 0), or that this one is done with (TILE_GO) or somebody else's (TILE_TAKEN).
template <bool BWD, bool BOX>
__device__ __forceinline__ int tc_tile(const TileChain& r, uint32_t at, bool helps, bool takes, unsigned char* lds, int* state) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));        // (where tiles are computed in a loop nothing that follows from it is kept from one to the next)
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int layers = r.layers;
    int32_t* const counts = r.chain;
    const int polls = r.sync.polls, d = r.d, h = r.h;
    float *const act1 = BWD ? r.dact : r.act, *const Dx1 = r.Dx, *const act2 = BWD ? r.doff : r.off, *const Dx2 = r.DxO;
    const float *const E = r.E, *const R = r.R;
    const int32_t *const refs = r.refs, *const rels = r.rel, *const out_row = r.out_row;
    const int keep = r.keep;
    unsigned long long* const words = r.taken;
    const unsigned long long launch = r.launch;
    const int patience = r.help.patience;
    asm volatile("" ::"s"(counts), "s"(polls), "s"(d), "s"(h), "s"(act1), "s"(refs), "s"(layers), "s"(words), "s"(launch), "s"(patience));
    if (BOX) asm volatile("" ::"s"(act2), "s"(Dx2));
    if (BWD) asm volatile("" ::"s"(Dx1));
    else asm volatile("" ::"s"(E), "s"(R), "s"(rels), "s"(out_row), "s"(keep));
    int e = 0;
    uint32_t start = r.start[0];
#pragma unroll
    for (int i = 1; i < TILE_PARTS; ++i)
        if (at >= r.start[i] >> 8) { e = i; start = r.start[i]; }
    const int l = start >> 4 & 15, type = start >> 2 & 3, kind = start & 3;
    const bool second = kind & 1, pooled = !BWD && kind == TILE_POOLED;
    const TilePart p = r.part[e];
    const uint16_t* W = r.W[kind & 1][type];
    const float* bias_of = r.bias[kind & 1][type];
    float *const H = r.H[type], *const Z = r.Z[type], *const dH = r.dH[type];
    const int before_tiles = r.tiles[l > 0 ? l - 1 : 0];
    asm volatile("" ::"s"(p.M), "s"(p.row0), "s"(p.out0), "s"(p.inv_mem), "s"(W), "s"(H), "s"(before_tiles));
    if (BWD) asm volatile("" ::"s"(dH));
    else asm volatile("" ::"s"(bias_of), "s"(Z));
    int32_t* const my_counts = l + 1 < layers ? counts + l * TILE_LAYER : nullptr;
    const int32_t* const before_counts = counts + (l - 1) * TILE_LAYER;
    const int local = (int)(at - (start >> 8)), tile = (BWD || BOX) && kind == TILE_PLAIN ? local : (local & 7) * ((p.tiles + 7) >> 3) + (local >> 3);
    unsigned long long taken = 0;
    if (takes && my_counts && tid == 0) {
        tile_late(r.help, (int)at, [&] { return tc_taken(r, (int)at); });
        taken = tc_take(r, (int)at);
    }
    if (tile >= p.tiles) return TILE_GO;
    if ((BWD || BOX) && kind == TILE_PLAIN) {
        if (BOX && type == 0) return tc_box_projection<BWD>(r, p, tile, l, before_counts, before_tiles, polls, my_counts, taken, helps, state);
        if (BOX && type == 2) return tc_pool_backward<true>(r, p, tile, l, before_counts, before_tiles, polls, my_counts, taken, helps, state);
        if (BWD) return tc_pool_backward<false>(r, p, tile, l, before_counts, before_tiles, polls, my_counts, taken, helps, state);
    }
    const bool offsets = BOX && type == 2;
    float *const act = offsets ? act2 : act1, *const Dx = offsets ? Dx2 : Dx1;
    const int K = second ? h : d, N = second ? d : h, tiles_n = (N + 31) >> 5;
    const int M = p.M, number = p.number + tile;
    const int quo = p.by == 1 ? tile : (int)__umulhi((uint32_t)tile, p.inv_by), rem = tile - quo * p.by;
    const int mt = p.m_major ? quo : rem, nt = p.m_major ? rem : quo, n0 = nt * 32;
    // (a tile is mem members of a class that pools, with all their inputs, else 32 rows)
    const int mem = p.mem, n_mem = p.n_mem, cls = p.cls;
    auto row_of = [&](int lr, bool* ok) {          // row of the problem that row lr of the tile is (past the end: the last one)
        const int j = lr * p.inv_mem >> 16, i = mt * mem + lr - j * mem;
        *ok = j < cls && i < n_mem;
        return *ok ? j * n_mem + i : M - 1;
    };
    const int nk = (K + 15) >> 4;
    const bool two = nk > TC_AHEAD * TC_WAVES;      // chunks of k
    auto block_of = [&](int c, int j) { return (c * TC_AHEAD + j) * TC_WAVES + wave; };
    W += (size_t)nt * nk * WTILE + lane * 8;
    bf16x8 b[TC_AHEAD][3];
    auto issue_b = [&](int blk, int j) {
        const uint16_t* from = W + (size_t)blk * WTILE;
#pragma unroll
        for (int i = 0; i < 3; ++i) b[j][i] = piece_at(from, i);
    };
    // a lane fetches 16 bytes of rows lane / 4 and 16 + lane / 4 of a block, and multiplies 8 values of row lane % 32; a thread ends with two
    // columns of a row
    const bool related = !BWD && !second && p.rel0 >= 0, mapped = !BWD && second && out_row != nullptr;        // uniform
    bool ok, mine_ok, inside;
    const int m0 = row_of(lane >> 2, &ok), m1 = row_of(16 + (lane >> 2), &ok), mine = row_of(lane & 31, &mine_ok), k_in = (lane >> 5) * 8;
    const int erow = tid >> 4, lc = (tid & 15) * 2, col = min(n0 + lc, N - 2);
    const int em = row_of(erow, &inside), out_i = pooled ? min(mt * mem + erow, n_mem - 1) : em;
    inside = inside && n0 + lc < N;
    // (numbers of rows are read whether or not this layer has a use for them: all at once, from where there are some)
    const int32_t *ref_of = refs + p.ref0, *rel_of = related ? rels + p.rel0 : ref_of, *out_of = mapped ? out_row + p.out0 : ref_of;
    const int32_t ref0 = BWD ? 0 : ref_of[m0], ref1 = BWD ? 0 : ref_of[m1], my_rel = BWD ? 0 : rel_of[mine], my_out = out_of[mapped ? out_i : em];
    // (added in the end; backward: a hidden value that the relu cut off has no gradient)
    float2 bias = make_float2(0.f, 0.f), mask = make_float2(1.f, 1.f);
    if (!BWD) bias = make_float2(bias_of[col], bias_of[col + 1]);
    else if (!second) mask = *reinterpret_cast<const float2*>(H + (size_t)(p.row0 + em) * h + col);
    // (blocks past the end: the last one again, not multiplied)
#pragma unroll
    for (int j = 0; j < TC_AHEAD; ++j) issue_b(min(block_of(0, j), nk - 1), j);
    const float* arow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int32_t ref = i ? ref1 : ref0, m = i ? m1 : m0;
        if (BWD) {
            arow[i] = second ? dH + (size_t)(p.row0 + m) * h : (p.pools ? (offsets ? r.dGate : r.dAtt) + (size_t)(p.row0 + m) * d : act + (size_t)(p.out0 + m) * d);
        } else {
            const float* of_depths = ref >= 0 ? act + (size_t)ref * d : E + (size_t)(-1 - ref) * d;
            arow[i] = second ? H + (size_t)(p.row0 + m) * h : of_depths;
        }
    }
    const int orow = !second ? p.row0 + em : (BWD || mapped ? my_out : p.out0 + out_i);
    // first layer: the relations' values; second: the inputs that a thread pools, once they are there
    float4 rel[TC_AHEAD][2];
    if (related) {
        const float* row = R + (size_t)my_rel * d;
#pragma unroll
        for (int j = 0; j < TC_AHEAD; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) rel[j][i] = load_global4(row + min(min(block_of(0, j), nk - 1) * 16 + k_in + i * 4, K - 4));
    }

    const uint32_t at_a = lds_addr(lds) + wave * (TC_AHEAD * 2048);
    const int unit = ((lane & 3) ^ tile_swizzle(lane >> 2)) * 4;
    auto issue_a = [&](int blk, int j) {
        const int k = min(blk * 16 + unit, K - 4);
#pragma unroll
        for (int i = 0; i < 2; ++i) lds_load16_card(arow[i] + k, at_a + j * 2048 + i * 1024);
    };
    auto first_rows = [&] {
#pragma unroll
        for (int j = 0; j < TC_AHEAD; ++j)
            if (block_of(0, j) < nk) issue_a(block_of(0, j), j);
    };
    if (l == 0) first_rows();        // (wait for no layer)
    tc_wait(r, l, before_counts, before_tiles, polls, taken, helps, state);
    if (l > 0) first_rows();
    const int got = __builtin_amdgcn_readfirstlane(*state);      // (looked at when the rows are requested)
    if (got >= 0 || got == TILE_TAKEN) {
        wait_vm<0>();
        return got;
    }
    const bool there = got == TILE_GO;
    if (pooled) {
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j) {
            const float2 x = card_get2(Z + (size_t)(p.row0 + min(j, cls - 1) * n_mem + out_i) * d + col);
            rel[j][0].x = x.x; rel[j][0].y = x.y;
        }
    }
    if (BWD && second && p.pools) bias = card_get2(Dx + (size_t)(p.row0 + em) * d + col);       // what the pooling passes on directly
    const bool copies = !BWD && !second && (keep || p.pools);        // uniform
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    const int f = tile_swizzle(lane & 15), u0 = (lane >> 5) * 2;
    const unsigned char* rows = lds + wave * (TC_AHEAD * 2048) + (lane & 31) * 64;
    auto chunk = [&](auto which, bool more) {
        constexpr int c = decltype(which)::value;
        asm volatile("" ::: "memory");
        wait_vm<0>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < TC_AHEAD; ++j) {
            const int blk = block_of(c, j);
            if (blk >= nk) break;                            // uniform
            float4 v[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                v[i] = *reinterpret_cast<const float4*>(rows + j * 2048 + ((u0 + i) ^ f) * 16);
                if (c == 0 && related) { v[i].x += rel[j][i].x; v[i].y += rel[j][i].y; v[i].z += rel[j][i].z; v[i].w += rel[j][i].w; }
            }
            // the rows as gathered, for who reads them later: a block of k by the tile whose turn it is
            if (c == 0 && copies && (unsigned)blk % (unsigned)tiles_n == (unsigned)nt) {
                float* to = Z + (size_t)(p.row0 + mine) * d + blk * 16 + k_in;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (mine_ok && blk * 16 + k_in + i * 4 < K) {
                        if (p.pools) {
                            card_put2(to + i * 4, v[i].x, v[i].y);
                            card_put2(to + i * 4 + 2, v[i].z, v[i].w);
                        } else {
                            *reinterpret_cast<float4*>(to + i * 4) = v[i];
                        }
                    }
            }
            u32x4 hi, mi, lo;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t w0, w1, w2;
                split2(v[i].x, v[i].y, w0, w1, w2);
                hi[2 * i] = w0; mi[2 * i] = w1; lo[2 * i] = w2;
                split2(v[i].z, v[i].w, w0, w1, w2);
                hi[2 * i + 1] = w0; mi[2 * i + 1] = w1; lo[2 * i + 1] = w2;
            }
            if (c == 0 && more && block_of(1, j) < nk) {     // (the values are read: their place is this wavefront's own)
                asm volatile("" ::: "memory");
                wait_lds();
                issue_a(block_of(1, j), j);
            }
            const bf16x8 a[3] = {__builtin_bit_cast(bf16x8, hi), __builtin_bit_cast(bf16x8, mi), __builtin_bit_cast(bf16x8, lo)};
            constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};      // smallest products first
#pragma unroll
            for (int t = 0; t < 6; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j][PB[t]], a[PA[t]], acc, 0, 0, 0);
            if (c == 0 && more && block_of(1, j) < nk) issue_b(block_of(1, j), j);
        }
    };
    chunk(std::integral_constant<int, 0>(), two);
    if (two) chunk(std::integral_constant<int, 1>(), false);
    __syncthreads();
    float* all = reinterpret_cast<float*>(lds);
    float* part = all + (wave * 32 + (lane & 31)) * TC_LD;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        *reinterpret_cast<float4*>(part + i * 8 + (lane >> 5) * 4) = make_float4(acc[i * 4], acc[i * 4 + 1], acc[i * 4 + 2], acc[i * 4 + 3]);
    __syncthreads();
    float* own = all + erow * TC_LD + lc;
    float o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < TC_WAVES; ++w) {
        const float2 v = *reinterpret_cast<const float2*>(own + w * 32 * TC_LD);
        o0 += v.x; o1 += v.y;
    }
    o0 += bias.x; o1 += bias.y;
    if (BWD) {
        o0 = mask.x > 0.f ? o0 : 0.f; o1 = mask.y > 0.f ? o1 : 0.f;
    } else if (!second) {
        o0 = fmaxf(o0, 0.f); o1 = fmaxf(o1, 0.f);
    }
    if (pooled) {
        if (inside && keep) *reinterpret_cast<float2*>((offsets ? r.Gate : r.Att) + (size_t)(p.row0 + em) * d + n0 + lc) = make_float2(o0, o1);
        *reinterpret_cast<float2*>(own) = make_float2(o0, o1);           // (read before by this thread only)
        __syncthreads();
        inside = erow < mem && mt * mem + erow < n_mem && n0 + lc < N;
        float2 z[TILE_CARD];
#pragma unroll
        for (int j = 0; j < TILE_CARD; ++j) z[j] = *reinterpret_cast<const float2*>(all + (min(j, cls - 1) * mem + min(erow, mem - 1)) * TC_LD + lc);
        auto pool = [&](auto logit, auto input) {
            if (offsets) {
                float mean = 0.f, mn = INFINITY;
#pragma unroll
                for (int j = 0; j < TILE_CARD; ++j)
                    if (j < cls) {
                        mean += logit(j);
                        if (input(j) < mn) mn = input(j);
                    }
                return mn * sigmoid_f(mean / (float)cls);
            }
            float mx = -INFINITY, den = 0.f, w[TILE_CARD], y = 0.f;
#pragma unroll
            for (int j = 0; j < TILE_CARD; ++j)
                if (j < cls) mx = fmaxf(mx, logit(j));
#pragma unroll
            for (int j = 0; j < TILE_CARD; ++j)
                if (j < cls) { w[j] = expf(logit(j) - mx); den += w[j]; }
            const float inv = 1.f / den;
#pragma unroll
            for (int j = 0; j < TILE_CARD; ++j)
                if (j < cls) y += w[j] * inv * input(j);
            return y;
        };
        o0 = pool([&](int j) { return z[j].x; }, [&](int j) { return rel[j][0].x; });
        o1 = pool([&](int j) { return z[j].y; }, [&](int j) { return rel[j][0].y; });
    }
    if (!there) o0 = o1 = NAN;
    float* const rows_out = BWD ? dH : H;
    if (inside) card_put2((second ? act + (size_t)orow * d : rows_out + (size_t)orow * h) + n0 + lc, o0, o1);
    tc_through(r, my_counts, number, there);
    return TILE_GO;
}
template <bool BWD, bool BOX>
__global__ __launch_bounds__(TC_T, 4) void tile_chain_kernel(const TileChain r) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[TC_WAVES * TC_AHEAD * 2048];
    __shared__ int state;
    static_assert(sizeof(lds) >= TC_WAVES * 32 * TC_LD * sizeof(float), "partial sums lie over the rows");
    int other = tc_tile<BWD, BOX>(r, blockIdx.x, true, true, lds, &state);
    if (__builtin_expect(other < 0, 1)) return;
    // (code of its own: around the tile above this loop would cost it 20 vector registers more than there are)
#pragma clang loop unroll(disable)
    for (;;) {
        __syncthreads();
        int again = 0;               // (and no argument is kept from tile to tile)
        asm volatile("" : "+s"(again));
        const bool own = other < 0;
        other = tc_tile<BWD, BOX>((&r)[again], own ? blockIdx.x : (uint32_t)other, own, false, lds, &state);
        if (own && other < 0) return;
    }
}

// Forward layers of very few rows (a handful of queries): a matrix-vector product per row.  The time is reading
// the weights once, 1.3 MB at d=400, h=800, spread over the chip: a wavefront takes ROWS_N output columns, reads
// their weight rows (k-contiguous, a float4 per lane) and multiplies them with up to MR assembled rows held in
// LDS; fp32 FMAs throughout.  One row: 3.4 us a layer against 6.5 to 7.1 for the tile kernel, and no split weights
// are needed (9 us a pass).
// Rows go to workgroups of four, two where there are no more.  (A workgroup that took all rows assembled, multiplied and reduced them one
// after the other on a card that was nearly empty.  1, 2, 3, 4 and 16 rows of 400 into 800 columns 2.7, 3.2, 4.5, 4.9 and 11.0 us, now 2.7,
// 2.9, 3.4, 3.5 and 4.2; of 800 into 400 3.1, 3.7, 5.8, 6.4 and 14.9, now 3.1, 3.3, 4.1, 4.2 and 4.3.)  From 17 rows on the tiles pool
// intersections in their epilogues, which costs a launch here: up to 32 rows here 40 queries of all structures score in 89 against 81 us at
// d = 512, h = 1024, 12 without intersections in 53 against 57 at 400, 800.
constexpr int ROWS_N = 2, ROWS_M = 4, ROWS_MAX = 16, ROWS_LDS = 16384;
template <int MR, class Group>
__global__ __launch_bounds__(256) void rows_kernel(const Group g) {
    extern __shared__ __attribute__((aligned(16))) float xs[];      // [MR][K]
    int p = 0;
#pragma unroll
    for (int i = 1; i < Group::MOST; ++i)
        if (i < g.count && (int)blockIdx.x >= g.tile_start[i]) p = i;
    const GemmArgs& a = g.p[p];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (the arguments in one request and what they point to in another: one by one each costs a round trip, which is most of what a
    // launch of one row takes)
    const int32_t *a_ref = a.a_ref, *a_add_idx = a.a_add_idx, *dst_row = a.dst_row;
    const float *A = a.A, *base0 = a.a_base0, *base1 = a.a_base1, *a_add = a.a_add, *B = a.B, *a_bias = a.bias;
    float *C = a.C, *a_copy = a.a_copy;
    const int rows = a.M, N = a.N, K = a.K, lda = a.lda, ldb = a.ldb, ldc = a.ldc, relu = a.relu;
    asm volatile("" ::"s"(a_ref), "s"(a_add_idx), "s"(dst_row), "s"(A), "s"(base0), "s"(base1), "s"(a_add), "s"(B), "s"(a_bias), "s"(C), "s"(a_copy));
    asm volatile("" ::"s"(rows), "s"(N), "s"(K), "s"(lda), "s"(ldb), "s"(ldc), "s"(relu));
    const int groups_n = (N + 4 * ROWS_N - 1) / (4 * ROWS_N), block = (int)blockIdx.x - g.tile_start[p];
    const int m0 = MR == 2 ? 0 : block / groups_n * MR, nb = MR == 2 ? block : block % groups_n, M = min(MR, rows - m0);      // (two rows: all there are)
    const int k4 = K >> 2;
    const int n0 = (nb * 4 + wave) * ROWS_N;
    // the first piece of the weight rows is on its way while the inputs are assembled
    const float* wrow[ROWS_N];
#pragma unroll
    for (int j = 0; j < ROWS_N; ++j) wrow[j] = B + (size_t)min(n0 + j, N - 1) * ldb;
    float4 w[ROWS_N];
#pragma unroll
    for (int j = 0; j < ROWS_N; ++j) w[j] = load_global4(wrow[j] + min(lane, k4 - 1) * 4);
    // a wavefront takes an input row (the last one again where there are fewer); a bias a column, a place a row.  (What is not
    // given is read from the weights, and not used.)
    const int mine = m0 + min(wave, M - 1);
    const int32_t* none = reinterpret_cast<const int32_t*>(B);
    const int32_t ref = (a_ref ? a_ref : none)[a_ref ? mine : 0], add_at = (a_add_idx ? a_add_idx : none)[a_add_idx ? mine : 0];
    float bias[ROWS_N];
    int to[MR];
#pragma unroll
    for (int j = 0; j < ROWS_N; ++j) bias[j] = (a_bias ? a_bias : B)[a_bias ? min(n0 + j, N - 1) : 0];
#pragma unroll
    for (int m = 0; m < MR; ++m) to[m] = (dst_row ? dst_row : none)[dst_row ? m0 + min(m, M - 1) : 0];
    asm volatile("" ::"s"(ref), "s"(add_at), "s"(bias[0]), "s"(bias[1]), "s"(to[0]), "s"(to[MR - 1]));
    static_assert(ROWS_N == 2, "biases named above");
#pragma unroll
    for (int j = 0; j < ROWS_N; ++j) bias[j] = a_bias ? bias[j] : 0.f;
#pragma unroll
    for (int m = 0; m < MR; ++m) to[m] = dst_row ? to[m] : m0 + m;
    const float* row = !a_ref ? A + (size_t)mine * lda : ref >= 0 ? base0 + (size_t)ref * lda : base1 + (size_t)(-1 - ref) * lda;
    const bool has_add = a_ref && a_add_idx;
    const float* add = has_add ? a_add + (size_t)add_at * lda : row;
    for (int c0 = lane * 4; wave < M && c0 < K; c0 += 1024) {
        float4 x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = min(c0 + u * 256, K - 4);
            x[u] = load_global4(row + c);
            if (has_add) y[u] = load_global4(add + c);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * 256;
            if (c >= K) break;
            float4 v = x[u];
            if (has_add) { v.x += y[u].x; v.y += y[u].y; v.z += y[u].z; v.w += y[u].w; }
            *reinterpret_cast<float4*>(xs + wave * K + c) = v;
            if (nb == 0 && a_copy) *reinterpret_cast<float4*>(a_copy + (size_t)mine * lda + c) = v;
        }
    }
    __syncthreads();
    float acc[MR][ROWS_N];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int j = 0; j < ROWS_N; ++j) acc[m][j] = 0.f;
    for (int q0 = 0; q0 < k4; q0 += 64) {
        float4 nx[ROWS_N];
#pragma unroll
        for (int j = 0; j < ROWS_N; ++j) nx[j] = load_global4(wrow[j] + min(q0 + 64 + lane, k4 - 1) * 4);
        const int q = q0 + lane;
        if (q < k4) {
#pragma unroll
            for (int m = 0; m < MR; ++m) {
                const float4 x = *reinterpret_cast<const float4*>(xs + min(m, M - 1) * K + q * 4);
#pragma unroll
                for (int j = 0; j < ROWS_N; ++j)
                    acc[m][j] += (x.x * w[j].x + x.y * w[j].y) + (x.z * w[j].z + x.w * w[j].w);
            }
        }
#pragma unroll
        for (int j = 0; j < ROWS_N; ++j) w[j] = nx[j];
    }
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        if (MR == 2 && m >= M) break;        // uniform
#pragma unroll
        for (int j = 0; j < ROWS_N; ++j) {
            float v = wave_sum_dpp(acc[m][j]) + bias[j];
            if (relu) v = fmaxf(v, 0.f);
            if (lane == 0 && m < M && n0 + j < N) C[(size_t)to[m] * ldc + n0 + j] = v;
        }
    }
}

// Launches of more than this many tiles of 32 x 64 take product_kernel; below, half of them would leave compute units idle, and
// gemm_kernel's smaller tiles are through first.  At d = 400, h = 800, first layer, gemm_kernel against this one: 130 tiles 6.9 and 7.4 us,
// 169 tiles 9.0 and 7.7; second layer 112 tiles 7.9 and 7.8, 154 tiles 10.7 and 8.1; at d = 256, h = 512 104 tiles 5.7 and 6.7, 176
// tiles 7.6 and 6.9.  Short k needs more tiles: k = 128 with 188 tiles 5.8 and 6.1, with 376 tiles 8.5 and 7.6; k = 184 with 188 tiles 6.7
// and 7.0; k = 152 with 282 tiles 9.3 and 8.0.  Up to 256 tiles, one to a compute unit, k is split over all eight wavefronts of one; beyond,
// pairs of them share the pieces (1000 rows at d = 400, h = 800: second layer 224 tiles 8.3 against 10.6 us, first layer 416 tiles
// 13.5 against 11.0).
constexpr long PRODUCT_ONE_EACH = 256;
long product_from(int max_k) { return max_k < 256 ? PRODUCT_ONE_EACH : 140; }

bool takes_rows_kernel(const GemmArgs& a) {
    return a.arith == GEMM_AUTO && a.a_kcontig && a.b_kcontig && a.M <= ROWS_MAX && (long)a.M * a.K <= ROWS_LDS && !a.mask &&
           !a.addend && !a.a_pieces;
}

// Launches of few problems are given the room of a smaller group: a launch costs the host 1 us for every KB of its arguments (a group
// of six takes 1.3 KB, of three 0.7; launch_with(f) calls f with the smallest that holds g).
template <int MOST>
GemmGroupOf<MOST> smaller(const GemmGroup& g) {
    GemmGroupOf<MOST> s;
    s.count = g.count;
    for (int i = 0; i <= MOST; ++i) s.tile_start[i] = g.tile_start[i];
    for (int i = 0; i < MOST; ++i) s.p[i] = g.p[i];
    return s;
}
template <class Launch>
hipError_t launch_with(const GemmGroup& g, Launch launch) {
    if (g.count == 1) launch(smaller<1>(g));
    else if (g.count <= 3) launch(smaller<3>(g));
    else launch(g);
    return hipGetLastError();
}

hipError_t dispatch_rows(GemmGroup& g, hipStream_t s) {
    int blocks = 0, most = 1, words = 4;
    for (int i = 0; i < g.count; ++i) most = std::max(most, g.p[i].M);
    const int mr = most <= 2 ? 2 : ROWS_M;
    for (int i = 0; i < g.count; ++i) {
        words = std::max(words, std::min(mr, g.p[i].M) * g.p[i].K);      // (at most ROWS_LDS: every problem is laid out by its own K)
        g.tile_start[i] = blocks;
        blocks += (g.p[i].M + mr - 1) / mr * ((g.p[i].N + 4 * ROWS_N - 1) / (4 * ROWS_N));
    }
    for (int i = g.count; i <= GEMM_MAX_GROUP; ++i) g.tile_start[i] = blocks;
    const size_t lds = (size_t)words * sizeof(float);
    return launch_with(g, [&](const auto& f) {
        using Group = std::decay_t<decltype(f)>;
        if (mr == 2) hipLaunchKernelGGL((rows_kernel<2, Group>), dim3(blocks), dim3(256), lds, s, f);
        else hipLaunchKernelGGL((rows_kernel<ROWS_M, Group>), dim3(blocks), dim3(256), lds, s, f);
    });
}

template <int BM, int BN, int NW, bool SPLIT = false>
hipError_t dispatch_layout(GemmGroup& g, hipStream_t s) {
    int tiles = 0;
    for (int i = 0; i < g.count; ++i) {
        g.tile_start[i] = tiles;
        tiles += (((g.p[i].M + BM - 1) / BM) * ((g.p[i].N + BN - 1) / BN) + 7) / 8 * 8;
    }
    for (int i = g.count; i <= GEMM_MAX_GROUP; ++i) g.tile_start[i] = tiles;
    dim3 grid(tiles), block(NW * 64);
    const GemmArgs& a = g.p[0];
    if (!a.a_kcontig && (a.b_kcontig || (SPLIT && BM != 32))) return hipErrorInvalidValue;     // (both row-contiguous: the large tile in fp32 only)
    return launch_with(g, [&](const auto& f) {
        using Group = std::decay_t<decltype(f)>;
        if (a.a_kcontig && a.b_kcontig)
            hipLaunchKernelGGL((gemm_kernel<BM, BN, NW, true, true, SPLIT, 1, false, false, false, Group>), grid, block, 0, s, f);
        else if (a.a_kcontig)
            hipLaunchKernelGGL((gemm_kernel<BM, BN, NW, true, false, SPLIT, 1, false, false, false, Group>), grid, block, 0, s, f);
        else
            hipLaunchKernelGGL((gemm_kernel<BM, BN, NW, false, false, SPLIT && BM == 32, 1, false, false, false, Group>), grid, block, 0, s, f);
    });
}

template <int WM, int WK>
hipError_t dispatch_product(GemmGroup& g, bool pool, hipStream_t s) {
    int tiles = 0;
    bool add = false;
    for (int i = 0; i < g.count; ++i) {
        g.tile_start[i] = tiles;
        const int k = g.p[i].pool_k ? g.p[i].pool_k : 1, rows = WM * 32 / k, n = g.p[i].M / k;
        tiles += (((n + rows - 1) / rows) * ((g.p[i].N + PN - 1) / PN) + 7) / 8 * 8;
        add = add || g.p[i].a_add_idx != nullptr;
    }
    for (int i = g.count; i <= GEMM_MAX_GROUP; ++i) g.tile_start[i] = tiles;
    const dim3 grid(tiles), block(WM * WK * 64);
    if (pool && add) return hipErrorInvalidValue;
    return launch_with(g, [&](const auto& f) {
        using Group = std::decay_t<decltype(f)>;
        if (pool) hipLaunchKernelGGL((product_kernel<WM, WK, false, true, Group>), grid, block, 0, s, f);
        else if (add) hipLaunchKernelGGL((product_kernel<WM, WK, true, false, Group>), grid, block, 0, s, f);
        else hipLaunchKernelGGL((product_kernel<WM, WK, false, false, Group>), grid, block, 0, s, f);
    });
}

template <bool AP, int PF>
hipError_t dispatch_pieces(GemmGroup& g, bool pool, hipStream_t s) {
    constexpr int BM = 32, BN = 32, NW = 8;
    int tiles = 0;
    for (int i = 0; i < g.count; ++i) {
        g.tile_start[i] = tiles;
        const int k = g.p[i].pool_k ? g.p[i].pool_k : 1, rows = BM / k, n = g.p[i].M / k;
        tiles += (((n + rows - 1) / rows) * ((g.p[i].N + BN - 1) / BN) + 7) / 8 * 8;
    }
    for (int i = g.count; i <= GEMM_MAX_GROUP; ++i) g.tile_start[i] = tiles;
    return launch_with(g, [&](const auto& f) {
        using Group = std::decay_t<decltype(f)>;
        if (pool) hipLaunchKernelGGL((gemm_kernel<BM, BN, NW, true, true, true, PF, true, AP, true, Group>), dim3(tiles), dim3(NW * 64), 0, s, f);
        else hipLaunchKernelGGL((gemm_kernel<BM, BN, NW, true, true, true, PF, true, AP, false, Group>), dim3(tiles), dim3(NW * 64), 0, s, f);
    });
}

}  // namespace

hipError_t launch_gemm_group(const GemmArgs* problems, int count, hipStream_t s, int* route, bool* emitted, int* kernel) {
    if (kernel) *kernel = GEMM_K_TILES;
    if (route) *route = GEMM_FP32;
    if (emitted) *emitted = false;
    GemmGroup g{};
    uint16_t* c_pieces[GEMM_MAX_GROUP] = {};
    long blocks_small = 0;
    int max_k = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs& a = problems[i];
        if (a.M <= 0 || a.N <= 0) continue;
        if (g.count == GEMM_MAX_GROUP) return hipErrorInvalidValue;
        // float4 operand loads: leading dimensions and the contiguous extents must be multiples of 4
        if ((a.lda & 3) || (a.ldb & 3)) return hipErrorInvalidValue;
        if ((a.a_kcontig ? a.K : a.M) & 3) return hipErrorInvalidValue;
        if ((a.b_kcontig ? a.K : a.N) & 3) return hipErrorInvalidValue;
        if (a.a_ref && !a.a_kcontig) return hipErrorInvalidValue;
        if (g.count && (a.a_kcontig != g.p[0].a_kcontig || a.b_kcontig != g.p[0].b_kcontig))
            return hipErrorInvalidValue;   // one operand layout per launch
        if (g.count && a.arith != g.p[0].arith) return hipErrorInvalidValue;
        c_pieces[g.count] = a.c_pieces;
        g.p[g.count] = a;
        g.p[g.count++].c_pieces = nullptr;    // (only the kernels chosen below for ready-made B operands write them)
        blocks_small += (long)((a.M + 31) / 32) * ((a.N + 63) / 64);
        max_k = std::max(max_k, a.K);
    }
    if (g.count == 0) return hipSuccess;
    bool pool = false;
    for (int i = 0; i < g.count; ++i) pool = pool || g.p[i].pool_k > 0;
    bool few_rows = true;
    for (int i = 0; i < g.count; ++i) few_rows = few_rows && takes_rows_kernel(g.p[i]);
    if (few_rows && kernel) *kernel = GEMM_K_ROWS;
    if (few_rows) return pool ? hipErrorNotSupported : dispatch_rows(g, s);
    const int arith = g.p[0].arith;
    const bool auto_split = arith == GEMM_AUTO && g.p[0].a_kcontig && max_k >= 128;
    // every B operand comes ready-made (weights split once per pass), and rows of four columns can be stored at once
    bool b_ready = g.p[0].a_kcontig;
    for (int i = 0; i < g.count; ++i) {
        const GemmArgs& a = g.p[i];
        b_ready = b_ready && a.b_pieces != nullptr && a.b_kt >= (a.K + 15) / 16 && ((a.N | a.ldc) & 3) == 0 && (!a.mask || (a.ldmask & 3) == 0) &&
                  (!a.addend || (a.ldadd & 3) == 0) &&
                  (((uintptr_t)a.C | (uintptr_t)a.mask | (uintptr_t)a.addend | (uintptr_t)a.pool_X | (uintptr_t)a.pool_out | (uintptr_t)a.a_copy) & 15) == 0;
    }
    if (pool && (!b_ready || !auto_split)) return hipErrorNotSupported;
    for (int i = 0; pool && i < g.count; ++i)
        if (g.p[i].pool_k == 1 || g.p[i].pool_k > NGDB_MAX_CARD || (g.p[i].pool_k > 0 && g.p[i].M % g.p[i].pool_k)) return hipErrorInvalidValue;
    if (b_ready && (auto_split || arith == GEMM_SPLIT) && blocks_small > product_from(max_k)) {
        if (route) *route = GEMM_SPLIT;
        if (kernel) *kernel = blocks_small <= PRODUCT_ONE_EACH ? GEMM_K_PRODUCT_ONE : GEMM_K_PRODUCT_PAIR;
        return blocks_small <= PRODUCT_ONE_EACH ? dispatch_product<1, 8>(g, pool, s) : dispatch_product<2, 4>(g, pool, s);
    }
    if (blocks_small >= 2048 && arith != GEMM_SPLIT) {
        if (route && auto_split) *route = GEMM_SPLIT;
        return auto_split ? dispatch_layout<64, 64, 4, true>(g, s) : dispatch_layout<64, 64, 4>(g, s);
    }
    // below that the launches of a step do not fill the chip: the smallest tile the MFMA block
    // allows spreads a launch over the most compute units (a tile's MFMA work runs on one)
    // (more than two such tiles per compute unit: 4 wavefronts per tile keep them all resident)
    // fp32 operands as three bf16 pieces each (six bf16 MFMAs per k-tile instead of eight fp32
    // ones that take twice as long each): launches whose A operand is k-contiguous, i.e. the
    // forward and data-gradient contractions.  (With k as the slow index of both operands, which a step leaves to
    // wgrad_kernel, these kernels serve ngdb_debug_gemm: products of fp32 matrix instructions to measure that one against.)
    // (with a k extent below 128 the matrix unit is idle either way and the splitting only adds work)
    if (arith == GEMM_SPLIT || auto_split) {
        if (route) *route = GEMM_SPLIT;
        if (b_ready) {      // no staging of B at all
            // ... and the A operand too where the launch before left its output as pieces
            bool a_too = true;
            for (int i = 0; i < g.count; ++i)
                a_too = a_too && g.p[i].a_pieces != nullptr && !g.p[i].a_ref && !g.p[i].a_copy && g.p[i].a_kt >= (g.p[i].K + 15) / 16;
            if (emitted) {
                *emitted = true;
                for (int i = 0; i < g.count; ++i)
                    *emitted = *emitted && c_pieces[i] != nullptr && !g.p[i].dst_row && g.p[i].c_kt >= 2 * ((g.p[i].N + 31) / 32);
                for (int i = 0; i < g.count; ++i)
                    if (*emitted) g.p[i].c_pieces = c_pieces[i];
            }
            return a_too ? dispatch_pieces<true, 2>(g, pool, s) : dispatch_pieces<false, 1>(g, pool, s);
        }
        if (blocks_small * 2 > 512) return dispatch_layout<32, 32, 4, true>(g, s);
        return dispatch_layout<32, 32, 8, true>(g, s);
    }
    if (blocks_small * 2 > 512) return dispatch_layout<32, 32, 4>(g, s);
    return dispatch_layout<32, 32, 8>(g, s);
}

hipError_t launch_wgrad_group(const WgradArgs* problems, int count, hipStream_t s, bool aside) {
    WgradGroup g{};
    for (int i = 0; i < count; ++i) {
        const WgradArgs& a = problems[i];
        if (a.M <= 0 || a.N <= 0) continue;
        if (g.count == GEMM_MAX_GROUP || (a.M & 3) || (a.N & 3) || (a.lda & 3) || (a.ldb & 3) || (a.ldc & 3) || a.K < 0)
            return hipErrorInvalidValue;
        // the contractions over the most rows first: their tiles take longest
        int at = g.count++;
        for (; at > 0 && g.p[at - 1].K < a.K; --at) g.p[at] = g.p[at - 1];
        g.p[at] = a;
    }
    if (g.count == 0) return hipSuccess;
    int tiles = 0;
    for (int i = 0; i < g.count; ++i) {
        g.tile_start[i] = tiles;
        tiles += (((g.p[i].M + WG_T - 1) / WG_T) * ((g.p[i].N + WG_T - 1) / WG_T) + 7) / 8 * 8;
    }
    for (int i = g.count; i <= GEMM_MAX_GROUP; ++i) g.tile_start[i] = tiles;
    // Beside a long memory-bound pass on another stream the LDS asked for leaves room for one workgroup per
    // compute unit: two of them hold the wavefront slots that the other pass needs to keep memory busy
    // (6.84 against 6.76 ms for the step over a 2.5 M-entity table, which that pass bounds).
    hipLaunchKernelGGL(wgrad_kernel, dim3(tiles), dim3(256), aside ? 40 * 1024 : 0, s, g);
    return hipGetLastError();
}

// The card holds 512 such tiles at a time, and what exceeds them starts a layer late; a launch a layer has larger tiles then, which the longer k is the sooner
// pays.  Scoring and training, us, by launches and with at most 400, 512 and 800 tiles a layer here: 512 queries at d = 208, h = 416 76 and 181
// against 66 and 171, 72 and 181, 73 and 182; at 400, 800 100 and 245 against 97 and 243, 102 and 246, 108 and 255.  With 400 and 260 (by
// TILE_CHAIN_WORK): 320 at 512, 1024 99 and 245 against 103 and 252, 99 and 242; 160 at 512, 1024 90 and 204 against 87 and 206, 85 and 196.
// Boxes (scoring and training at 300, 500): 512 of them with at most 300 to 400 tiles 64 and 149 against 61 and 145, with 500 151; 1024, whose layer of 306
// tiles 400 lets in, 79 and 170.5 against 74 and 174.
// Forward-only passes, whose tiles are all that the card has: with 400, 300 and 220 tiles 40 drawn calls of 250 to 1000 queries 0.92 to 1.08 of the speed of launches (8 of
// them below 0.97), 0.98 to 1.08 and 0.94 to 1.08 (4).
constexpr int TILE_CHAIN_MOST = 400, TILE_CHAIN_MOST_FORWARD = 300, TILE_CHAIN_MOST_BOX = 300, TILE_CHAIN_WORK = 400000;
static_assert(TILE_CHAIN_MOST < GAVE_UP, "counts of tiles and of those that gave up in one word");
int tile_chain_tiles(int members, int k, int n) { return (members + 32 / k - 1) / (32 / k) * ((n + 31) / 32); }
int tile_chain_plain(int members, int d) { return (int)(((long)members * (d / 4) + TC_T - 1) / TC_T); }
int tile_chain_most(int d, int h, bool box, bool trains) {
    if ((d & 3) || (h & 3) || d < 128 || h < 128 || d > TILE_D || h > TILE_H) return 0;
    return std::min(box ? TILE_CHAIN_MOST_BOX : (trains ? TILE_CHAIN_MOST : TILE_CHAIN_MOST_FORWARD), TILE_CHAIN_WORK / (d + h));
}
bool tile_chain_lay_out(TileChain& r, const TileProblem (*problems)[TILE_PROBLEMS], const int* count, int n, bool backward, bool box) {
    if (n < 1 || n > LEVEL_CHAIN || tile_chain_most(r.d, r.h, box, true) == 0) return false;
    const auto up = [](int by) { return by == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + by - 1) / by); };
    int blocks = 0;
    r.parts = r.layers = 0;
    for (int l = 0; l < n; ++l) {
        if (count[l] < 1) return false;
        // layers of a depth: forward first and second, backward pooling, gradient of the hidden rows, of the inputs
        for (int layer_of = backward ? 0 : 1; layer_of < 3; ++layer_of) {
            const bool second = layer_of == 2, plain_turn = layer_of == (backward ? 0 : 1);
            const int N = second ? r.d : r.h, tiles_n = (N + 31) / 32, layer = r.layers;
            int tiles = 0;
            for (int q = 0; q < count[l]; ++q) {
                const TileProblem& p = problems[l][q];
                if (p.n < 1 || p.k < 1 || p.k > TILE_CARD || p.type < 0 || p.type > 2 || (long)p.n * p.k > 1 << 16) return false;
                const bool projection = box && p.type == 0, plain = projection || layer_of == 0;
                if (projection ? !plain_turn : layer_of == 0 && p.k == 1) continue;
                if (r.parts == TILE_PARTS) return false;
                const bool pooled = second && !backward && p.k > 1;
                TilePart& t = r.part[r.parts];
                t.M = p.n * p.k; t.row0 = p.row0; t.ref0 = p.ref0; t.rel0 = p.rel0; t.out0 = p.out0; t.pools = p.k > 1;
                t.cls = pooled || plain ? p.k : 1; t.mem = 32 / t.cls; t.n_mem = t.M / t.cls; t.inv_mem = (65535 + t.mem) / t.mem;
                const int tiles_m = (t.n_mem + t.mem - 1) / t.mem;
                t.m_major = t.M >= N;
                t.by = plain ? r.d / 4 : (t.m_major ? tiles_n : tiles_m);
                t.inv_by = up(t.by);
                t.tiles = plain ? tile_chain_plain(t.n_mem, r.d) : tiles_m * tiles_n;
                t.number = tiles;
                const int kind = plain ? TILE_PLAIN : (pooled ? TILE_POOLED : (second ? TILE_SECOND : TILE_FIRST));
                r.start[r.parts++] = (uint32_t)blocks << 8 | layer << 4 | p.type << 2 | kind;
                tiles += t.tiles;
                blocks += (t.tiles + 7) / 8 * 8;
                if (blocks > TILE_WORDS) return false;
            }
            if (tiles == 0) continue;                // (a depth without intersections)
            r.tiles[r.layers++] = tiles;
        }
    }
    for (int i = r.parts; i < TILE_PARTS; ++i) r.start[i] = 0xFFFFFFFFu;
    r.blocks = blocks;
    return true;
}

hipError_t launch_tile_chain(const TileChain& r, bool backward, bool box, hipStream_t s) {
    if (!r.chain || !r.taken || !r.help.helped || !r.sync.gave_up || !r.sync.host_gave_up || r.blocks < 1 || r.blocks > TILE_WORDS || r.parts < 1) return hipErrorInvalidValue;
    const dim3 grid(r.blocks), block(TC_T);
    if (box && backward) hipLaunchKernelGGL((tile_chain_kernel<true, true>), grid, block, 0, s, r);
    else if (box) hipLaunchKernelGGL((tile_chain_kernel<false, true>), grid, block, 0, s, r);
    else if (backward) hipLaunchKernelGGL((tile_chain_kernel<true, false>), grid, block, 0, s, r);
    else hipLaunchKernelGGL((tile_chain_kernel<false, false>), grid, block, 0, s, r);
    return hipGetLastError();
}

bool gemm_takes_rows(int M, int K) {
    GemmArgs a;
    a.M = M; a.K = K;
    return takes_rows_kernel(a);
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s) { return launch_gemm_group(&a, 1, s, nullptr); }

hipError_t launch_weight_pieces(PieceJobs& J, hipStream_t s) {
    if (J.count <= 0 && J.copy_n <= 0) return hipSuccess;
    if (J.count > PIECE_MAX_JOBS || J.copy_n < 0 || J.clear_n < 0 || (J.clear_n > 0 && !J.clear)) return hipErrorInvalidValue;
    int blocks = 0;
    for (int i = 0; i < J.count; ++i) {
        if ((J.job[i].C & 3) || J.job[i].R <= 0 || J.job[i].C <= 0) return hipErrorInvalidValue;
        J.block0[i] = blocks;
        blocks += ((J.job[i].R + 31) / 32) * ((J.job[i].C + 63) / 64);
    }
    J.block0[J.count] = blocks;
    J.copy_blocks = std::min((J.copy_n + 255) / 256, 256);
    hipLaunchKernelGGL(weight_pieces_kernel, dim3(blocks + J.copy_blocks), dim3(256), 0, s, J);
    return hipGetLastError();
}

}  // namespace ngdb
