// Text-feature fusion of entity rows (Sec. 4.4: the frozen encoder's outputs are
// cached in HBM as H_sem, a batch gathers its rows and a learned linear map
// brings them to the embedding width):
//     Ef[e] = E[e] + bf16(Wp) * H_sem[e]
// computed once per step for the entity rows the batch touches (the rows of the
// gradient index, so every repeated negative is projected once), with
// bf16 16x16x32 MFMA blocks and fp32 accumulation; and the gradient of the
// projection, dWp = sum over touched rows of g_row (x) H_sem[row], as a
// contraction over the touched rows split over workgroups and summed in a
// fixed order.
//
// Both kernels bring their operand rows from global memory straight into LDS
// (direct loads, a few stages ahead, counted and waited for by hand) and keep one
// workgroup of large tiles per compute unit: what limits them is how many cache
// lines a compute unit has in flight, so every row piece is brought in as few
// times as the accumulator registers allow.  The gradient's operands both have
// the contraction index (rows) as the slow one: they are fetched from LDS with
// the transposing read of gfx950 instead of being transposed on the way in.
#include "common.h"

namespace ngdb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int KS = 64;          // the feature width is a multiple of this
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t to_bf16_bits(float x) {   // round to nearest, ties to even
    const uint32_t b = __float_as_uint(x);
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

__global__ __launch_bounds__(256) void cast_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = (uint16_t)to_bf16_bits(x[i]);
}

// inv[contribution number] = position of its entity in the list of touched rows
__global__ __launch_bounds__(256) void inverse_index_kernel(const int32_t* __restrict__ src,
                                                            const int32_t* __restrict__ seg_off,
                                                            const int32_t* __restrict__ n_uniq_dev, int64_t n,
                                                            int32_t* __restrict__ inv) {
    const int n_uniq = *n_uniq_dev;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        int lo = 0, hi = n_uniq;                    // largest u with seg_off[u] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)seg_off[mid] <= t) lo = mid; else hi = mid;
        }
        inv[src[t]] = lo;
    }
}

// operator input references with anchors redirected to their fused row: inv[anchor], or the anchor's number
__global__ __launch_bounds__(256) void translate_refs_kernel(const int32_t* __restrict__ in_ref,
                                                             const int32_t* __restrict__ in_gslot, int n, int n_slots,
                                                             const int32_t* __restrict__ inv, int32_t* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t r = in_ref[i];
    if (r >= 0) {
        out[i] = r;
        return;
    }
    const int32_t anchor = in_gslot[i] - n_slots;
    out[i] = -1 - (inv ? inv[anchor] : anchor);
}

// ---- building blocks of the projection kernels (gfx950)
// Transposing LDS read of 16-bit values: within 16 lanes, lane 4r + c gives the address of 4
// consecutive values of row r (c-th group of 4 columns); lane i receives column i of the
// 4 x 16 block: rows 0..3.  Two of them make the 8 consecutive k of a 16x16x32 MFMA operand
// from a tile that is stored with k as the slow index.
typedef short short4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ short4v read_tr(const uint16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)p);
}
__device__ __forceinline__ bf16x8 join8(short4v a, short4v b) {
    typedef short short8v __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, short8v{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
}

// ------------------------------------------------------------------ forward
// out[u, :] = E[id(u), :] + Wb * H[id(u), :].  Workgroup tile: 256 rows x 208 coordinates (two
// tiles cover d = 400, so a feature row is brought into LDS twice), k stages of 64 = 128 bytes of
// every row = one cache line per row and stage.  What bounds the kernel is how much a compute unit has in flight between its
// barriers (35 GB/s per unit; an L2 hit path that is kept full delivers 122), so every request is a whole line and the tile is as wide
// as the accumulators allow.
// A stage is 64 direct loads of 1 KiB, 8 per wavefront: load l of an area covers rows 8l .. 8l+7,
// 128 bytes each; a lane's 16 bytes land at its lane number, so the lane picks the column that
// belongs there: column c of row r is stored at c ^ (r / 2 % 8), which spreads the 16 rows x 16
// bytes one MFMA operand fetch touches over all banks.
constexpr int SF_BU = 256, SF_N = 208, SF_NBLK = SF_N / 16, SF_KS = 64;
constexpr int SF_NW = 8;                                      // wavefronts: 32 rows x 208 coordinates each (104 accumulator registers)
constexpr int SF_HL = SF_BU / 8, SF_WL = 32;                  // loads per stage: feature rows, weight rows (26 used)
static_assert(SF_NBLK * 4 <= SLACK_TERMS, "a lane's part of a row's error");
constexpr int SF_STAGE = (SF_HL + SF_WL) * 1024, SF_NB = 2, SF_PER_WAVE = (SF_HL + SF_WL) / SF_NW;
// BITS: the rows also go onto the integer grid of a ranking, from the accumulators.  For 65 536 rows of 400 coordinates and 1024 feature
// values 86 -> 99 us; the pass that read the rows again took 27.
template <int BITS>
__global__ __launch_bounds__(SF_NW * 64) void sem_fuse_kernel(const SemFuseArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char tiles[SF_NB * SF_STAGE];
    const int n_rows = a.n_rows_dev ? min(*a.n_rows_dev, a.n_rows) : a.n_rows;
    const int n_tiles = (a.d + SF_N - 1) / SF_N;
    // workgroups are dealt round-robin to the 8 dies: the coordinate tiles of one
    // row tile go to the same die one after the other and share its L2
    const int die = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int u0 = ((j / n_tiles) * 8 + die) * SF_BU;
    const int n0 = (j % n_tiles) * SF_N;
    if (u0 >= n_rows) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // entity of a row of the tile (rows past the end: the last row's); the row numbers are read
    // unconditionally (from a valid address when the rows are no list)
    const bool listed = a.ids != nullptr;
    const int32_t* id_src = listed ? a.ids : reinterpret_cast<const int32_t*>(a.E);
    constexpr int HQ = SF_HL / SF_NW, WQ = SF_WL / SF_NW;     // loads per wavefront: 4 + 4
    int urow[HQ + 2];
#pragma unroll
    for (int q = 0; q < HQ; ++q) urow[q] = min(u0 + (wave + SF_NW * q) * 8 + (lane >> 3), n_rows - 1);   // feature rows this lane fetches
#pragma unroll
    for (int q = 0; q < 2; ++q) urow[HQ + q] = min(u0 + wave * 32 + q * 16 + (lane & 15), n_rows - 1);   // rows of its accumulator blocks
    int32_t listed_id[HQ + 2];
#pragma unroll
    for (int q = 0; q < HQ + 2; ++q) listed_id[q] = id_src[listed ? urow[q] : 0];
    int64_t ent[HQ + 2];
#pragma unroll
    for (int q = 0; q < HQ + 2; ++q)
        ent[q] = listed ? (int64_t)listed_id[q] : urow[q] < a.n_seq ? a.id_base + urow[q] : (int64_t)(urow[q] - a.n_seq) * a.spread;
    // sources of this lane's loads at k = 0 (row r of the area = 8 * load + lane / 8, stored column lane % 8)
    const uint16_t* src[SF_PER_WAVE];
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
        const int r = (wave + SF_NW * q) * 8 + (lane >> 3);
        src[q] = a.H + ent[q] * a.ds + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    }
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
        const int r = (wave + SF_NW * q) * 8 + (lane >> 3);          // (rows past the tile's 208: padding, the last row again)
        src[HQ + q] = a.Wb + (size_t)min(n0 + min(r, SF_N - 1), a.d - 1) * a.ds + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    }
    // The accumulators start from the structural rows: a lane holds, per block, 4 consecutive
    // coordinates of one row (clamped addresses; rows and coordinates past the end are never stored).
    floatx4 acc[2][SF_NBLK];
#pragma unroll
    for (int bu = 0; bu < 2; ++bu) {
        const float* erow = a.E + ent[HQ + bu] * a.d;
#pragma unroll
        for (int bn = 0; bn < SF_NBLK; ++bn) {
            const float4 e = *reinterpret_cast<const float4*>(erow + min(n0 + bn * 16 + (lane >> 4) * 4, a.d - 4));
            acc[bu][bn] = floatx4{e.x, e.y, e.z, e.w};
        }
    }
    const uint32_t tiles_at = lds_addr(tiles);
    const int stages = a.ds / SF_KS;
    auto issue = [&](int s) {                // (stages past the end fetch the last one again; nobody reads them)
        const int k0 = min(s, stages - 1) * SF_KS;
        const uint32_t base = tiles_at + (uint32_t)(s % SF_NB) * SF_STAGE;
#pragma unroll
        for (int q = 0; q < HQ; ++q) lds_load16(src[q] + k0, base + (uint32_t)(wave + SF_NW * q) * 1024u);
#pragma unroll
        for (int q = 0; q < WQ; ++q) lds_load16(src[HQ + q] + k0, base + (uint32_t)(SF_HL + wave + SF_NW * q) * 1024u);
    };
    issue(0);
    issue(1);
    // The structural rows have to be in their registers before the loop: the compiler's own count of
    // loads in flight does not know the direct loads, and its waits inside the loop would throttle them.
    wait_vm<0>();
    // operand fetch: row R = 16 b + lane % 16 of an area, columns 4 h + lane / 16 (h = which half of the stage's k)
    const int ri = lane & 15;
    int frag_at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        frag_at[h] = (ri >> 3) * 1024 + (ri & 7) * 128 + (((4 * h + (lane >> 4)) ^ ((ri >> 1) & 7))) * 16;
    for (int s = 0; s < stages; ++s) {
        wait_vm<SF_PER_WAVE>();              // all but the next stage's loads: stage s is in LDS
        __syncthreads();                     // ... every wavefront's part of it
        const unsigned char* buf = tiles + (s % SF_NB) * SF_STAGE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8 fh[2], fw[SF_NBLK];
#pragma unroll
            for (int bu = 0; bu < 2; ++bu)
                fh[bu] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + (wave * 2 + bu) * 2048 + frag_at[h]));
#pragma unroll
            for (int bn = 0; bn < SF_NBLK; ++bn)
                fw[bn] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(buf + SF_HL * 1024 + bn * 2048 + frag_at[h]));
#pragma unroll
            for (int bu = 0; bu < 2; ++bu)
#pragma unroll
                for (int bn = 0; bn < SF_NBLK; ++bn)
                    acc[bu][bn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[bn], fh[bu], acc[bu][bn], 0, 0, 0);
        }
        __syncthreads();                     // everybody is done with this buffer
        issue(s + 2);
    }
    wait_vm<0>();                            // the loads issued past the end land before the workgroup gives up its LDS
    const float step = BITS ? a.grid[0] : 0.f, inv = BITS ? a.grid[1] : 0.f;
    constexpr float TOP = BITS == 8 ? 255.f : 65535.f;
    float er[2] = {0.f, 0.f};
#pragma unroll
    for (int bn = 0; bn < SF_NBLK; ++bn) {
        const int n = n0 + bn * 16 + (lane >> 4) * 4;
        float4 lo = make_float4(0.f, 0.f, 0.f, 0.f);
        if (BITS) lo = *reinterpret_cast<const float4*>(a.lo + min(n, a.d - 4));
#pragma unroll
        for (int bu = 0; bu < 2; ++bu) {
            const int u = u0 + wave * 32 + bu * 16 + (lane & 15);
            if (u >= n_rows) continue;
            const float4 v = make_float4(acc[bu][bn][0], acc[bu][bn][1], acc[bu][bn][2], acc[bu][bn][3]);
            if (n < a.d) *reinterpret_cast<float4*>(a.out + (size_t)u * a.d + n) = v;
            if (!BITS || n * BITS >= a.words * 32) continue;
            // (words past the last coordinate are zero)
            float dropped = 0.f, *e = n < a.d ? &er[bu] : &dropped;
            uint32_t q[4] = {(uint32_t)to_grid(v.x, lo.x, step, inv, TOP, e), (uint32_t)to_grid(v.y, lo.y, step, inv, TOP, e),
                             (uint32_t)to_grid(v.z, lo.z, step, inv, TOP, e), (uint32_t)to_grid(v.w, lo.w, step, inv, TOP, e)};
            if (n >= a.d) q[0] = q[1] = q[2] = q[3] = 0u;
            if (BITS == 8) {
                a.Q[(size_t)(n >> 2) * a.ldq + u] = q[0] | q[1] << 8 | q[2] << 16 | q[3] << 24;
            } else {
                a.Q[(size_t)(n >> 1) * a.ldq + u] = q[0] | q[1] << 16;
                a.Q[(size_t)((n >> 1) + 1) * a.ldq + u] = q[2] | q[3] << 16;
            }
        }
    }
    if (BITS) {
#pragma unroll
        for (int bu = 0; bu < 2; ++bu) {
            const int u = u0 + wave * 32 + bu * 16 + (lane & 15);
            float e = er[bu] + __shfl_xor(er[bu], 16, 64);
            e += __shfl_xor(e, 32, 64);
            if (lane < 16 && u < n_rows) a.err[(size_t)(n0 / SF_N) * a.ldq + u] = slack_steps(e, inv);
        }
    }
}

// The same, for rows that go nowhere else and at least ST_FROM feature values: one workgroup a compute unit takes tile after tile, and
// the memory is asked for something all the time.  Four wavefronts of 64 rows x 208 coordinates: an operand fetched from LDS feeds twice
// the products (17 instead of 30 KB a wavefront and 104 products), and with one wavefront a SIMD all of its registers are there, 208
// for the accumulators and two sets of operands, one being multiplied while the other is fetched.  Feature rows are two stages ahead
// (they come from HBM; a wavefront fetches and reads its own), weight rows one (from L2); the last stages of a tile request the first
// ones of the next, and each block of results leaves just before the next tile's structural rows are requested into its registers.
// 262 144 rows of 400 coordinates and 1024 values 421 -> 366 us (floor at the rate of a copy 281), 20 000 x 128 x 512 25.5 -> 23.5,
// 65 536 x 632 x 256 108 -> 104; but x 424 x 192 62.2 and 63.6, x 48 x 128 13.8 and 15.0.  Rows that are also put on a
// ranking's grid stay with the kernel above: a form of this one for them took 335 instead of 393 us for 262 144, but the integer sums that
// follow then took 1035 instead of 907 us, 28.0 instead of 26.5 ms a pass (the cause was not looked for).
// What the compiler does not know of here (products and accumulator loads) is checked in the listing it makes: tests/test_hand_scheduled_kernels.py.
// It lets no vector write come just before a product that reads it; a wait in every product would do without the check and costs 1 %
// of this kernel's time, and 8 % of sem_wgrad_kernel's (2.50 -> 2.70 ms), whose products are issued the same way.
constexpr int ST_FROM = 256;
constexpr int ST_NW = 4, ST_RB = SF_BU / ST_NW / 16;          // wavefronts; row blocks of each
constexpr int ST_HL = SF_BU / 8 / ST_NW, ST_WL = 7;           // loads a wavefront and stage: its own feature rows, a quarter of the weight rows (26 used)
constexpr int ST_HB = SF_BU * 128, ST_WB = ST_NW * ST_WL * 1024, ST_HS = 3, ST_WS = 2;       // bytes of a stage, stages
constexpr int ST_WG = 256;
static_assert(ST_FROM >= ST_HS * SF_KS, "a tile has all the stages that are requested ahead");
__global__ __launch_bounds__(ST_NW * 64) __attribute__((amdgpu_waves_per_eu(1, 1))) void sem_stream_kernel(const SemFuseArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char tiles[ST_HS * ST_HB + ST_WS * ST_WB];
    const int n_rows = a.n_rows_dev ? min(*a.n_rows_dev, a.n_rows) : a.n_rows;
    const int n_tiles = (a.d + SF_N - 1) / SF_N;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // tile t of a die is coordinate tile t % n_tiles of its row tile t / n_tiles (side by side on one die: one L2)
    const int die = blockIdx.x & 7, t_step = gridDim.x >> 3;
    auto rows_at = [&](int tile) { return (tile / n_tiles * 8 + die) * SF_BU; };
    auto cols_at = [&](int tile) { return tile % n_tiles * SF_N; };
    int t = blockIdx.x >> 3;
    if (rows_at(t) >= n_rows) return;

    // entities of this lane's rows of a tile (rows past the end: the last row's): feature rows it fetches, rows of its accumulator
    // blocks.  The row numbers are read unconditionally (from a valid address when the rows are no list).
    const bool listed = a.ids != nullptr;
    const int32_t* id_src = listed ? a.ids : reinterpret_cast<const int32_t*>(a.E);
    auto row_of = [&](int u0, int q) {
        const int r = q < ST_HL ? q * 8 + (lane >> 3) : (q - ST_HL) * 16 + (lane & 15);
        return min(u0 + wave * 64 + r, n_rows - 1);
    };
    int32_t ent[ST_HL + ST_RB];              // of the tile that is requested next
    auto read_ids = [&](int u0) {
#pragma unroll
        for (int q = 0; q < ST_HL + ST_RB; ++q) ent[q] = id_src[listed ? row_of(u0, q) : 0];
    };
    auto take_ids = [&](int u0) {
#pragma unroll
        for (int q = 0; q < ST_HL + ST_RB; ++q) {
            const int r = row_of(u0, q);
            if (!listed) ent[q] = r < a.n_seq ? (int32_t)a.id_base + r : (r - a.n_seq) * a.spread;
        }
    };
    // sources of this lane's loads at k = 0 (row r of the area = 8 * load + lane / 8, stored column lane % 8)
    const uint16_t* hsrc[ST_HL];
    uint32_t wsrc[ST_WL];
    auto point_h = [&]() {
#pragma unroll
        for (int q = 0; q < ST_HL; ++q) hsrc[q] = a.H + (int64_t)ent[q] * a.ds + ((lane & 7) ^ ((q * 4 + (lane >> 4)) & 7)) * 8;
    };
    auto point_w = [&](int n0) {
#pragma unroll
        for (int q = 0; q < ST_WL; ++q) {
            const int r = (wave * ST_WL + q) * 8 + (lane >> 3);      // (rows past the tile's 208: padding, the last row again)
            wsrc[q] = ((uint32_t)min(n0 + min(r, SF_N - 1), a.d - 1) * (uint32_t)a.ds + (uint32_t)((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2;
        }
    };
    // The accumulators start from the structural rows: a lane holds, per block, 4 consecutive coordinates of one row (clamped addresses;
    // rows and coordinates past the end are never stored).  They are loaded straight into the accumulator registers, behind the
    // compiler's back, and are there after wait_vm<0>.  Nothing may touch them in between: the loads are in and out operands of the
    // same registers, all 208 of them are taken by the accumulators, and no branch over single loads parts them.
    floatx4 acc[ST_RB][SF_NBLK];
    auto structural = [&](int bu, int n0) {
        const float* row = a.E + (int64_t)ent[ST_HL + bu] * a.d;
#pragma unroll
        for (int bn = 0; bn < SF_NBLK; ++bn) {
            const float* from = row + min(n0 + bn * 16 + (lane >> 4) * 4, a.d - 4);
            asm volatile("global_load_dwordx4 %0, %1, off" : "+a"(acc[bu][bn]) : "v"(from) : "memory");
        }
    };
    const uint32_t h_at = lds_addr(tiles) + wave * (ST_HL * 1024), w_at = lds_addr(tiles) + ST_HS * ST_HB + wave * (ST_WL * 1024);
    const int stages = a.ds / SF_KS;
    auto issue_h = [&](int k, int buf) {
#pragma unroll
        for (int q = 0; q < ST_HL; ++q) lds_load16(hsrc[q] + k * SF_KS, h_at + (uint32_t)(buf * ST_HB + q * 1024));
    };
    auto issue_w = [&](int k, int buf) {
#pragma unroll
        for (int q = 0; q < ST_WL; ++q) lds_load16_at(a.Wb + k * SF_KS, wsrc[q], w_at + (uint32_t)(buf * ST_WB + q * 1024));
    };
    // operand fetch: row R = 16 b + lane % 16 of an area, columns 4 h + lane / 16 (h = which half of the stage's k)
    const int ri = lane & 15;
    int frag_at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        frag_at[h] = (ri >> 3) * 1024 + (ri & 7) * 128 + (((4 * h + (lane >> 4)) ^ ((ri >> 1) & 7))) * 16;
    constexpr int FETCHES = ST_RB + SF_NBLK, PRODUCTS = ST_RB * SF_NBLK;
    struct Operands { bf16x8 f[FETCHES]; };
    auto fetch = [&](Operands& o, int hbuf, int wbuf, int h, int i) {
        const unsigned char* at = tiles + frag_at[h] + (i < ST_RB ? hbuf * ST_HB + wave * (ST_HL * 1024) + i * 2048 : ST_HS * ST_HB + wbuf * ST_WB + (i - ST_RB) * 2048);
        o.f[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(at));
    };
    // (the accumulators stay where they are: with the builtin the compiler copies 200 and more of them about in every stage)
    auto product = [&](const Operands& o, int m) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[m % ST_RB][m / ST_RB]) : "v"(o.f[ST_RB + m / ST_RB]), "v"(o.f[m % ST_RB]));
    };

    int u0 = rows_at(t), n0 = cols_at(t), hbuf = 0, wbuf = 0;
#pragma unroll
    for (int bu = 0; bu < ST_RB; ++bu)
#pragma unroll
        for (int bn = 0; bn < SF_NBLK; ++bn) acc[bu][bn] = floatx4{0.f, 0.f, 0.f, 0.f};
    read_ids(u0);
    take_ids(u0);
#pragma unroll
    for (int bu = 0; bu < ST_RB; ++bu) structural(bu, n0);
    point_h();
    point_w(n0);
    issue_h(0, 0);
    issue_w(0, 0);
    issue_h(1, 1);
    issue_w(1, 1);
    issue_h(2, 2);
    for (;;) {
        const int t_next = t + t_step, u_next = rows_at(t_next), n_next = cols_at(t_next);
        const bool more = u_next < n_rows;
        if (more) read_ids(u_next);
        wait_vm<0>();
        if (more) take_ids(u_next);
        __syncthreads();
        Operands o0, o1;
#pragma unroll
        for (int i = 0; i < FETCHES; ++i) fetch(o0, hbuf, wbuf, 0, i);
        int hk = min(ST_HS, stages - 1), wk = ST_WS;          // stages to be requested next
        for (int s = 0; s < stages; ++s) {
            const int hnext = hbuf == ST_HS - 1 ? 0 : hbuf + 1;
#pragma unroll
            for (int m = 0; m < PRODUCTS; ++m) {
                product(o0, m);
                if (m % 2 == 0 && m / 2 < FETCHES) fetch(o1, hbuf, wbuf, 1, m / 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the last stages request the next tile's first ones (without one, the last stage again: nobody reads it)
            if (more && s + ST_HS == stages) { point_h(); hk = 0; }
            if (more && s + ST_WS == stages) { point_w(n_next); wk = 0; }
            wait_vm<ST_HL>();                // all but the rows of the stage after the next: the next one is in LDS
            wait_lds();                      // ... and this one in registers,
            __syncthreads();                 // ... every wavefront's part
            const uint16_t* w_from = a.Wb + wk * SF_KS;
            const uint32_t w_to = w_at + (uint32_t)(wbuf * ST_WB), h_to = h_at + (uint32_t)(hbuf * ST_HB);
#pragma unroll
            for (int m = 0; m < PRODUCTS; ++m) {
                product(o1, m);
                if (m % 2 == 0 && m / 2 < FETCHES) fetch(o0, hnext, wbuf ^ 1, 0, m / 2);
                if (m % 3 == 1 && m / 3 < ST_WL) lds_load16_at(w_from, wsrc[m / 3], w_to + (m / 3) * 1024);
                if (m % 3 == 1 && m / 3 >= ST_WL && m / 3 < ST_WL + ST_HL) lds_load16(hsrc[m / 3 - ST_WL] + hk * SF_KS, h_to + (m / 3 - ST_WL) * 1024);
                __builtin_amdgcn_sched_barrier(0);
            }
            hk = min(hk + 1, stages - 1);
            wk = min(wk + 1, stages - 1);
            hbuf = hnext;
            wbuf ^= 1;
        }
        // block of rows by block: results out, the next tile's structural rows in
#pragma unroll
        for (int bu = 0; bu < ST_RB; ++bu) {
            // (a result is read 18 cycles after its product at the earliest; the compiler does not know the products)
            asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc[bu][0]), "+a"(acc[bu][1]), "+a"(acc[bu][2]), "+a"(acc[bu][3]), "+a"(acc[bu][4]), "+a"(acc[bu][5]),
                         "+a"(acc[bu][6]), "+a"(acc[bu][7]), "+a"(acc[bu][8]), "+a"(acc[bu][9]), "+a"(acc[bu][10]), "+a"(acc[bu][11]), "+a"(acc[bu][12]));
            const int u = u0 + wave * 64 + bu * 16 + (lane & 15);
            if (u < n_rows) {
#pragma unroll
                for (int bn = 0; bn < SF_NBLK; ++bn) {
                    if (n0 + bn * 16 >= a.d) break;          // uniform
                    const int n = n0 + bn * 16 + (lane >> 4) * 4;
                    if (n < a.d) *reinterpret_cast<floatx4*>(a.out + (size_t)u * a.d + n) = acc[bu][bn];
                }
            }
            if (more) structural(bu, n_next);
        }
        if (!more) break;
        t = t_next;
        u0 = u_next;
        n0 = n_next;
    }
    wait_vm<0>();                            // the loads issued past the end land before the workgroup gives up its LDS
}

// ------------------------------------------------------------------ gradient of Wp
constexpr int WG_SEM = 256;     // text-feature coordinates per workgroup tile of the gradient

// LDS of one 32-row stage: H rows [32][256 feature coordinates] at a pitch of 544 bytes (34
// chunks of 16: with 17 * 32 bytes per row the 16 consecutive rows one transposing read touches
// spread over all banks), G rows [32][208 embedding coordinates] at 416 bytes (13 * 32: likewise).
constexpr int WG_KS = 32;                                     // rows per stage = one MFMA step
constexpr int WG_M = 208, WG_MB = WG_M / 16;                  // embedding coordinates per workgroup tile, MFMA blocks
constexpr int WG_HP = 544, WG_GP = 2 * WG_M;                  // row pitches, bytes
constexpr int WG_HL = 17, WG_GL = 13;                         // wave-loads of 1 KiB per stage: H area, G area
constexpr int WG_STAGE = (WG_HL + WG_GL) * 1024;
constexpr int WG_NB = 5;                                      // stages in LDS: one being fetched from, four in flight or landing
constexpr int WG_PER_WAVE = (WG_HL + WG_GL + 3) / 4;          // data loads per wavefront and stage (the last two of 32 carry nothing)

// partial[split, m, n] = sum over the split's rows u of G[u, m] * H[id(u), n]
// Workgroup tile: 208 embedding x 256 feature coordinates (two tiles cover d = 400, so a feature
// row is brought into LDS twice per step and a gradient row four times; the tile is as large as the accumulators allow and LDS is all
// staging).  Rows travel from global memory straight into LDS (no registers, no transposition on the way): every wavefront issues 8 loads
// of 1 KiB per stage, up to five stages ahead of the one being multiplied, and one load of the row numbers three stages further; the
// operands of the MFMA blocks are fetched with transposing reads, those of the next stage between the products of this one.
// One workgroup barrier per stage.  What bounds it is the wait for a stage's last rows (3.1 TB/s from HBM, each stage 1830 cycles of which the
// products take 832): with operands fetched and multiplied in turn and four stages in LDS 2.72 ms for the 2.7 million rows of a step
// over 5 million entities, 2.46 with the fetches between the products, 2.40 with five stages.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void sem_wgrad_kernel(const SemWgradArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char tiles[WG_NB * WG_STAGE + 2048];       // (the end takes the loads that carry nothing)
    __shared__ __attribute__((aligned(256))) int32_t id_ring[4][4][64];     // per wavefront: row numbers of four stages
    const int n_rows = min(*a.n_rows_dev, a.n_rows);
    const int m_tiles = (a.d + WG_M - 1) / WG_M, n_tiles = (a.ds + WG_SEM - 1) / WG_SEM;
    const int tiles_mn = m_tiles * n_tiles;
    const int die = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int split = (j / tiles_mn) * 8 + die;
    if (split >= a.n_splits) return;
    const int tile = j % tiles_mn;
    const int m0 = (tile % m_tiles) * WG_M, n0 = (tile / m_tiles) * WG_SEM;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int stages = (n_rows + WG_KS - 1) / WG_KS;
    const int per_split = (stages + a.n_splits - 1) / a.n_splits;
    const int s_lo = split * per_split, s_hi = min(stages, s_lo + per_split);

    floatx4 acc[4][WG_MB];
#pragma unroll
    for (int bn = 0; bn < 4; ++bn)
#pragma unroll
        for (int bm = 0; bm < WG_MB; ++bm) {
            acc[bn][bm] = floatx4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[bn][bm]));        // (in accumulator registers from here on)
        }

    if (s_lo < s_hi) {
        // What this lane fetches in each of its wavefront's loads of a stage (the same every stage).
        // The H tile is 32 rows x 34 chunks of 16 bytes = 17 loads of 64 chunks (chunk c = row c/34, column
        // c%34; columns 32 and 33 are padding and fetch columns 0 and 1 again), the G tile 32 x 26 = 13 loads.
        // Loads 0..16 of a stage are the H tile, loads 17..29 the G tile.
        constexpr int G_AT = WG_HL;                                       // the G tile starts at this KiB of the stage
        int row[WG_PER_WAVE];
        const uint16_t* from[WG_PER_WAVE];                                // the lane's column of row 0
#pragma unroll
        for (int q = 0; q < WG_PER_WAVE; ++q) {
            const int l = wave + 4 * q;                                   // load number within the stage, 0..31
            if (l < G_AT) {
                const int c = l * 64 + lane;
                row[q] = c / 34;
                from[q] = a.H + min(n0 + ((c % 34) & 31) * 8, a.ds - 8);
            } else {
                const int c = (l - G_AT) * 64 + lane;
                row[q] = min(c / (WG_GP / 16), WG_KS - 1);                // (loads 30, 31: the last row again)
                from[q] = a.G + min(m0 + (c % (WG_GP / 16)) * 8, a.d - 8);
            }
        }
        static_assert(WG_HL * 1024 >= WG_KS * WG_HP && WG_GL * 1024 >= WG_KS * WG_GP && 4 * WG_PER_WAVE - (WG_HL + WG_GL) == 2, "stage layout");
        const uint32_t tiles_at = lds_addr(tiles), ring_at = lds_addr(&id_ring[wave][0][0]);
        auto issue_ids = [&](int s) {        // row numbers of stage s (rows past the end: the last row's)
            lds_load4(a.ids + min(s * WG_KS + (lane & (WG_KS - 1)), n_rows - 1), ring_at + (uint32_t)(s & 3) * 256u);
        };
        // load q of a stage; the row numbers of the stage have to be in the ring
        auto source_row = [&](int s, int q) { return wave + 4 * q < G_AT ? id_ring[wave][s & 3][row[q]] : min(s * WG_KS + row[q], n_rows - 1); };
        auto issue_data = [&](int buf, int q, int r) {
            const int l = wave + 4 * q;
            const uint16_t* src = from[q] + (size_t)(uint32_t)r * (uint32_t)(l < G_AT ? a.ds : a.d);
            lds_load16(src, tiles_at + (uint32_t)(l < WG_HL + WG_GL ? buf * WG_STAGE + l * 1024 : WG_NB * WG_STAGE + (l - WG_HL - WG_GL) * 1024));
        };
        auto issue_stage = [&](int s, int buf) {
#pragma unroll
            for (int q = 0; q < WG_PER_WAVE; ++q) issue_data(buf, q, source_row(s, q));
        };
        // lane group g = lane / 16 reads rows 4g .. 4g+3 (first read) and 16 + 4g .. (second) of the 32 rows:
        // the order of the 32 products within an MFMA step is free as long as both operands agree
        const int row_in = (lane >> 4) * 4 + ((lane & 15) >> 2), col_in = (lane & 3) * 4;
        const int h_in = row_in * WG_HP + (wave * 64 + col_in) * 2, g_in = G_AT * 1024 + row_in * WG_GP + col_in * 2;
        constexpr int FETCHES = 2 * (4 + WG_MB), PRODUCTS = 4 * WG_MB;
        struct Operands { short4v f[FETCHES]; };                          // H blocks, then G blocks, two reads each
        auto fetch = [&](Operands& o, const unsigned char* buf, int i) {
            const int b = i >> 1, half = i & 1;
            o.f[i] = read_tr(reinterpret_cast<const uint16_t*>(b < 4 ? buf + h_in + half * 16 * WG_HP + b * 32 : buf + g_in + half * 16 * WG_GP + (b - 4) * 32));
        };
        auto product = [&](const Operands& o, int m) {
            const int bn = m % 4, bm = m / 4;
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[bn][bm]) : "v"(join8(o.f[2 * bn], o.f[2 * bn + 1])), "v"(join8(o.f[8 + 2 * bm], o.f[9 + 2 * bm])));
        };
        // stage s has landed, its last rows may lie past the end: these hold copies of the last row and count as zeros through G
        auto clear_tail = [&](int s, int buf) {
            if ((s + 1) * WG_KS <= n_rows || s >= s_hi) return;
            uint32_t* g = reinterpret_cast<uint32_t*>(tiles + buf * WG_STAGE + G_AT * 1024);
            for (int i = (n_rows - s * WG_KS) * (WG_GP / 4) + tid; i < WG_KS * (WG_GP / 4); i += 256) g[i] = 0u;
            __syncthreads();
        };
        // Stage s is multiplied from registers while stage s + 1 is fetched from LDS, the stages up to s + 4 are on their way and stage s + 5
        // is requested into the buffer that stage s was fetched from.
        int buf = 0;                         // of stage s
        auto stage = [&](const Operands& now, Operands& next, int s) {
            // stage s + 1 and the row numbers of stage s + 5 are in LDS: all but the data of stage s + 2 and what follows it
            wait_vm<3 * WG_PER_WAVE + 2>();
            wait_lds();                      // (stage s is in this wavefront's registers)
            __syncthreads();                 // ... those of every wavefront
            const int next_buf = buf == WG_NB - 1 ? 0 : buf + 1;
            clear_tail(s + 1, next_buf);
            int r[WG_PER_WAVE];
#pragma unroll
            for (int q = 0; q < WG_PER_WAVE; ++q) r[q] = source_row(s + 5, q);
            issue_ids(s + 8);
#pragma unroll
            for (int m = 0; m < PRODUCTS; ++m) {
                product(now, m);
                if (m < FETCHES) fetch(next, tiles + next_buf * WG_STAGE, m);
                if (m % 5 == 4 && m / 5 < WG_PER_WAVE) issue_data(buf, m / 5, r[m / 5]);        // (stages past the end fetch valid rows that nobody reads)
                __builtin_amdgcn_sched_barrier(0);
            }
            buf = next_buf;
        };
        // prologue: in flight afterwards, oldest first: data of the first stage, of the second, then, as in the loop, the row numbers of
        // stage s + 3 before the data of stage s: ids(5) data(2) | ids(6) data(3) | ids(7) data(4)
#pragma unroll
        for (int i = 0; i < 4; ++i) issue_ids(s_lo + i);
        wait_vm<0>();
        issue_stage(s_lo, 0);
        issue_ids(s_lo + 4);
        issue_stage(s_lo + 1, 1);
        wait_vm<WG_PER_WAVE>();              // the first stage and the row numbers of the fifth
#pragma unroll
        for (int i = 2; i < WG_NB; ++i) {
            issue_ids(s_lo + 3 + i);
            issue_stage(s_lo + i, i);
        }
        __syncthreads();
        clear_tail(s_lo, 0);
        Operands o0, o1;
#pragma unroll
        for (int i = 0; i < FETCHES; ++i) fetch(o0, tiles, i);
        for (int s = s_lo;;) {
            stage(o0, o1, s);
            if (++s == s_hi) break;
            stage(o1, o0, s);
            if (++s == s_hi) break;
        }
        wait_vm<0>();                        // the loads issued past the end land before the workgroup gives up its LDS
    }
#pragma unroll
    for (int bn = 0; bn < 4; ++bn)           // (a result is read 18 cycles after its product at the earliest; the compiler does not know the products)
        asm volatile("s_nop 15\n\ts_nop 7" : "+a"(acc[bn][0]), "+a"(acc[bn][1]), "+a"(acc[bn][2]), "+a"(acc[bn][3]), "+a"(acc[bn][4]), "+a"(acc[bn][5]),
                     "+a"(acc[bn][6]), "+a"(acc[bn][7]), "+a"(acc[bn][8]), "+a"(acc[bn][9]), "+a"(acc[bn][10]), "+a"(acc[bn][11]), "+a"(acc[bn][12]));
    // a lane holds, per block, 4 consecutive feature coordinates n of one embedding coordinate m
#pragma unroll
    for (int bm = 0; bm < WG_MB; ++bm) {
        const int m = m0 + bm * 16 + (lane & 15);
        if (m >= a.d) continue;
        float* prow = a.partial + ((size_t)split * a.d + m) * a.ds;
#pragma unroll
        for (int bn = 0; bn < 4; ++bn) {
            const int n = n0 + wave * 64 + bn * 16 + (lane >> 4) * 4;
            if (n >= a.ds) continue;
            *reinterpret_cast<float4*>(prow + n) =
                make_float4(acc[bn][bm][0], acc[bn][bm][1], acc[bn][bm][2], acc[bn][bm][3]);
        }
    }
}

// A workgroup sums 64 groups of four coefficients, each of its eight wavefronts an eighth of the splits, eight loads
// on the way.  (One thread per group and one load after the other: 25 us for 26 splits at d = 128 and 512 features.)
constexpr int RED_PARTS = 8;
__global__ __launch_bounds__(64 * RED_PARTS) void sem_wgrad_reduce_kernel(const float* __restrict__ partial, int n_splits,
                                                                          int64_t n4, float* __restrict__ out) {
    __shared__ float4 part[RED_PARTS][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const int64_t at = i < n4 ? i : n4 - 1;
    const int per = (n_splits + RED_PARTS - 1) / RED_PARTS, lo = wave * per, hi = min(n_splits, lo + per);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = lo; k0 < hi; k0 += 8) {
        float4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = reinterpret_cast<const float4*>(partial)[(size_t)min(k0 + q, hi - 1) * n4 + at];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (k0 + q >= hi) break;
            s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w;
        }
    }
    part[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || i >= n4) return;
#pragma unroll
    for (int w = 1; w < RED_PARTS; ++w) {
        const float4 v = part[w][lane];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    reinterpret_cast<float4*>(out)[i] = s;
}

}  // namespace

hipError_t launch_cast_bf16(const float* x, uint16_t* y, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 2048);
    hipLaunchKernelGGL(cast_bf16_kernel, dim3(blocks), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

hipError_t launch_inverse_index(const int32_t* src, const int32_t* seg_off, const int32_t* n_uniq_dev, int64_t n,
                                int32_t* inv, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(inverse_index_kernel, dim3(blocks), dim3(256), 0, s, src, seg_off, n_uniq_dev, n, inv);
    return hipGetLastError();
}

hipError_t launch_translate_refs(const int32_t* in_ref, const int32_t* in_gslot, int n, int n_slots,
                                 const int32_t* inv, int32_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(translate_refs_kernel, dim3((n + 255) / 256), dim3(256), 0, s, in_ref, in_gslot, n, n_slots,
                       inv, out);
    return hipGetLastError();
}

int sem_fuse_parts(int d) { return (d + SF_N - 1) / SF_N; }

hipError_t launch_sem_fuse(const SemFuseArgs& a, hipStream_t s) {
    if (a.n_rows <= 0) return hipSuccess;
    if (a.bits && (a.ids || a.n_rows > a.ldq)) return hipErrorInvalidValue;
    if (a.ds <= 0 || a.ds % KS || a.d % 4) return hipErrorInvalidValue;
    const int64_t u_tiles = (a.n_rows + SF_BU - 1) / SF_BU;
    const int64_t n_tiles = (a.d + SF_N - 1) / SF_N;
    const int64_t blocks = ((u_tiles + 7) / 8) * 8 * n_tiles;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (!a.bits && a.ds >= ST_FROM) {
        hipLaunchKernelGGL(sem_stream_kernel, dim3((unsigned)std::min<int64_t>(blocks, ST_WG)), dim3(ST_NW * 64), 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)blocks), block(SF_NW * 64);
    if (a.bits == 8) hipLaunchKernelGGL((sem_fuse_kernel<8>), grid, block, 0, s, a);
    else if (a.bits == 16) hipLaunchKernelGGL((sem_fuse_kernel<16>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sem_fuse_kernel<0>), grid, block, 0, s, a);
    return hipGetLastError();
}

int sem_wgrad_splits(int64_t n_rows_bound, int d, int ds) {
    const int tiles = ((d + WG_M - 1) / WG_M) * ((ds + WG_SEM - 1) / WG_SEM);
    const int64_t stages = (n_rows_bound + WG_KS - 1) / WG_KS;
    // one resident set of workgroups, no second round: the five stages in LDS leave room for one
    // workgroup per compute unit; the splits of a launch are dealt to the 8 dies in turn, 32
    // compute units each
    const int cap = std::max(1, 32 / tiles) * 8;
    return (int)std::max<int64_t>(1, std::min<int64_t>(stages / 4, cap));
}

hipError_t launch_sem_wgrad(const SemWgradArgs& a, float* out, hipStream_t s) {
    if (a.ds <= 0 || a.ds % KS || a.d % 8 || a.n_splits < 1) return hipErrorInvalidValue;
    const int tiles = ((a.d + WG_M - 1) / WG_M) * ((a.ds + WG_SEM - 1) / WG_SEM);
    const int blocks = ((a.n_splits + 7) / 8) * 8 * tiles;
    hipLaunchKernelGGL(sem_wgrad_kernel, dim3(blocks), dim3(256), 0, s, a);
    const int64_t n4 = (int64_t)a.d * a.ds / 4;
    hipLaunchKernelGGL(sem_wgrad_reduce_kernel, dim3((unsigned)((n4 + 63) / 64)), dim3(64 * RED_PARTS), 0, s,
                       (const float*)a.partial, a.n_splits, n4, out);
    return hipGetLastError();
}

}  // namespace ngdb
