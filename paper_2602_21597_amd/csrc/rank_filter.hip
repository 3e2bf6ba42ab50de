// Ranking with a filter (Sec. 3.2: the answers are the entities nearest to a query's embedding).
//
// An L1 distance costs the vector ALU two operations per coordinate, and the all-entity passes are
// bound by nothing else.  The hardware also sums absolute differences of packed unsigned integers --
// four 8-bit or two 16-bit coordinates in one operation -- so the entity rows and the branch
// embeddings are rounded to integers on one common grid, the integer sums are formed for every
// pair, and only the pairs that the integer sum leaves undecided are computed in fp32.  What a
// rounded row is off by is summed exactly per row, so an integer sum bounds the fp32 distance
// from both sides and the results are those of the fp32 pass: the same distances, formed in the
// same order of summation, and the same order of ids.
//
// Grid: coordinate c of a row becomes round((x - lo[c]) / step), clamped to the range of the type;
// `step` is common to all coordinates (the sums need one unit), lo[c] and step come from a sample
// of the table.  A coordinate outside the grid is clamped.  With e' = lo + step * q(e) the entity
// side, |e - e'| summed over the row is the entity's error (clamped outliers included); the branch
// side splits |y - e'| into the part inside the grid and the excess |y - clamp(y)|, which adds up
// to a constant of the row (exact for every e' on the grid), and errs by |clamp(y) - y'|.  So
//     | dist(y, e) - (excess_y + step * SAD) | <= err_y + err_e.
// fp32 rounding is covered by relative slacks (SLACK on a row's sums, rounding_of(d) on a distance) and by
// half a unit in the last place of every grid point.  A row that holds an infinity or a NaN gets an
// error that leaves every one of its pairs undecided.
//
// Top-k: the first rows of the table are ranked in fp32; the k-th distance so far is a bound, and the
// 8-bit sums of the next chunk leave some tens to hundreds of entities per query that can be below it, which
// one workgroup per query computes and merges.  Chunks grow with what has been ranked.  1024 queries
// (1171 branch rows) x 5 M entities x 400: distance tiles 182.6 ms and merges 32.6 became integer sums 17.5 (34 T
// operations of 4 coordinates a second; the instruction alone reaches 36) and merges 1.0.
// Top-k of a table of one piece (65 536 rows) or few: the 8-bit sums of all entities go to memory, and one workgroup per query takes its nearest
// from them (pick_kernel).  512 queries x 15 000 x 400: fp32 rows 43 us, tiles of the rest 56 and merges 29 became sums 42 and 27.
// Filtered ranks: the 16-bit sums decide all but about 0.1 % of the (entity, answer) comparisons: 1024
// queries x 63 000 entities with 8 answers each, tiles 2.78 ms (0.32 of them for the answers' own
// distances, now computed pair by pair) and counting 0.24 became 0.46 and 0.26.
// Lists have a fixed room per query; a query whose list overflows takes the fp32 pass for that piece of
// the table (launched always, its workgroups leave at once where nothing overflowed).
#include <climits>

#include "common.h"

namespace ngdb {
namespace {

constexpr int UNBOUNDED = INT_MAX / 4;
__device__ __forceinline__ int32_t slack_of(int32_t sum) { return sum >= SLACK_CAP ? UNBOUNDED : sum; }
// relative rounding of an fp32 distance: d additions and d subtractions in sequence
inline float rounding_of(int d) { return (float)(d + 16) * 6e-8f; }
constexpr int SAMPLE_SLABS = 16;

// ---------------------------------------------------------------- the grid
// per coordinate the smallest and largest value of a slab of the sampled rows; grid (d/64, slabs).  On the way n_found words of found
// (a multiple of 4) are cleared.
__global__ __launch_bounds__(256) void sample_range_kernel(const float* __restrict__ E, const uint16_t* __restrict__ E16,
                                                           int64_t row_step, int n_rows, int d, float* __restrict__ part,
                                                           uint32_t* __restrict__ found, int n_found) {
    for (int i = ((blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x) * 4; i < n_found; i += gridDim.x * gridDim.y * 1024)
        *reinterpret_cast<uint4*>(found + i) = make_uint4(0u, 0u, 0u, 0u);
    __shared__ float slo[4][64], shi[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = min((int)blockIdx.x * 64 + lane, d - 1);
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll 8
    for (int i = blockIdx.y * 4 + wave; i < n_rows; i += SAMPLE_SLABS * 4) {
        const size_t at = (size_t)i * row_step * d + c;
        const float x = E16 ? __uint_as_float((uint32_t)E16[at] << 16) : E[at];
        lo = fminf(lo, x);
        hi = fmaxf(hi, x);
    }
    slo[wave][lane] = lo;
    shi[wave][lane] = hi;
    __syncthreads();
    if (wave == 0 && (int)blockIdx.x * 64 + lane < d) {
#pragma unroll
        for (int w = 1; w < 4; ++w) { lo = fminf(lo, slo[w][lane]); hi = fmaxf(hi, shi[w][lane]); }
        part[((size_t)blockIdx.y * 2 + 0) * d + c] = lo;
        part[((size_t)blockIdx.y * 2 + 1) * d + c] = hi;
    }
}

// One workgroup, one coordinate per thread: lo[c], and grid[0] = step, grid[1] = 1/step.  The step spans
// the widest coordinate, but at most three times the mean width: a few wide coordinates then clamp (and
// err) rather than coarsen the grid of all others.  The pass's counters are cleared on the way.
__global__ __launch_bounds__(1024) void make_grid_kernel(const float* __restrict__ part, int d, int levels,
                                                         float* __restrict__ lo_out, float* __restrict__ grid,
                                                         int32_t* __restrict__ counters, int n_counters) {
    __shared__ float smax[16], ssum[16];
    const int c = threadIdx.x, lane = c & 63, wave = c >> 6;
    for (int i = c; i < n_counters; i += 1024) counters[i] = 0;
    float lo = INFINITY, hi = -INFINITY;
    if (c < d) {
#pragma unroll
        for (int s = 0; s < SAMPLE_SLABS; ++s) {
            lo = fminf(lo, part[((size_t)s * 2 + 0) * d + c]);
            hi = fmaxf(hi, part[((size_t)s * 2 + 1) * d + c]);
        }
    }
    const float w = c < d ? hi - lo : 0.f;
    float wmax = w;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wmax = fmaxf(wmax, __shfl_xor(wmax, off, 64));
    const float wsum = wave_sum(w);
    if (lane == 0) {
        smax[wave] = wmax;
        ssum[wave] = wsum;
    }
    __syncthreads();
    float all_max = 0.f, all_sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        all_max = fmaxf(all_max, smax[i]);
        all_sum += ssum[i];
    }
    const float width = fminf(all_max, 3.f * all_sum / (float)d);
    // (a table of equal rows has no width: any grid serves)
    const float step = fmaxf(width, 1e-30f) / (float)(levels - 1);
    if (c < d) lo_out[c] = 0.5f * (lo + hi) - 0.5f * step * (float)(levels - 1);   // centred on the sampled range
    if (c == 0) {
        grid[0] = step;
        grid[1] = 1.f / step;
    }
}

// ---------------------------------------------------------------- rows -> grid
// Q[w * ld + i]: word w of row i, 32 / BITS consecutive coordinates each, words beyond the row zero (on
// both sides of a sum: they add nothing).  A wavefront takes 16 rows of the workgroup's 64, one after
// the other, a float4 per lane; the words pass through LDS so that they leave 64 rows at a time.
// ENT: slack[i] = the row's error in steps, rounded up (SLACK_CAP where it is not finite or larger).
// !ENT (branch rows, ids): base[i] = excess - err and base[ld + i] = excess + err (for bounds from
// below and from above), and row_q[i] = the query the row belongs to.
template <int BITS, bool ENT, int RW>
__device__ __forceinline__ void quantise(int block, const float* __restrict__ X, const uint16_t* __restrict__ X16,
                                         const int32_t* __restrict__ ids, int n_rows, int d, int words,
                                         const float* __restrict__ lo, const float* __restrict__ grid,
                                         uint32_t* __restrict__ Q, int ld, int32_t* __restrict__ slack,
                                         float* __restrict__ base, const int32_t* __restrict__ root_off,
                                         int n_queries, int32_t* __restrict__ row_q, uint32_t* lds) {
    constexpr int WPQ = BITS == 8 ? 1 : 2;       // words of four coordinates
    constexpr float TOP = BITS == 8 ? 255.f : 65535.f;
    constexpr int LD = 4 * RW + 1;
    uint32_t (*tile)[LD] = reinterpret_cast<uint32_t (*)[LD]>(lds);      // [64 * WPQ]: 64 float4 columns of 4 * RW rows
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = block * 4 * RW;
    const float step = grid[0], inv = grid[1];
    float err[RW], excess[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) err[r] = excess[r] = 0.f;
    for (int q0 = 0; q0 * WPQ < words; q0 += 64) {
        const int q4 = q0 + lane;
        const bool inside = q4 * 4 < d;
        const float4 l4 = *reinterpret_cast<const float4*>(lo + (inside ? q4 * 4 : 0));
        const float l[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int i = min(i0 + wave * RW + r, n_rows - 1);
            const size_t at = (size_t)(ids ? ids[i] : i) * d + (inside ? q4 * 4 : 0);
            const float4 v4 = X16 ? bf16x4_to_f32(*reinterpret_cast<const uint2*>(X16 + at)) : *reinterpret_cast<const float4*>(X + at);
            const float v[4] = {v4.x, v4.y, v4.z, v4.w};
            uint32_t w[2] = {0u, 0u};
            float er = 0.f, ex = 0.f, dropped = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float qf;
                if (ENT) {
                    qf = to_grid(v[j], l[j], step, inv, TOP, &er);
                } else {
                    const float cl = fminf(fmaxf(v[j], l[j]), fmaf(TOP, step, l[j]));
                    ex += fabsf(v[j] - cl);
                    qf = to_grid(v[j], l[j], step, inv, TOP, &dropped);
                    const float on = fmaf(qf, step, l[j]);
                    er += fabsf(cl - on) + fabsf(on) * 6e-8f + 0.f * v[j];     // (not a number where v is infinite or none)
                }
                const uint32_t qi = (uint32_t)qf;
                if (BITS == 8) w[0] |= qi << (8 * j);
                else w[j >> 1] |= qi << (16 * (j & 1));
            }
            if (inside) { err[r] += er; excess[r] += ex; }
#pragma unroll
            for (int p = 0; p < WPQ; ++p) tile[lane * WPQ + p][wave * RW + r] = inside ? w[p] : 0u;
        }
        __syncthreads();
        const int n_w = min(64 * WPQ, words - q0 * WPQ);
        for (int x = threadIdx.x; x < n_w * 4 * RW; x += 256) {
            const int w = x / (4 * RW), i = x % (4 * RW);
            if (i0 + i < ld) Q[(size_t)(q0 * WPQ + w) * ld + i0 + i] = tile[w][i];
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const float e = wave_sum_dpp(err[r]), x = ENT ? 0.f : wave_sum_dpp(excess[r]);
        const int i = i0 + wave * RW + r;
        if (lane == 0 && i < n_rows) {
            if (ENT) {
                slack[i] = slack_steps(e, inv);
            } else {
                base[i] = x * (1.f - SLACK) - e * (1.f + SLACK);
                base[ld + i] = x * (1.f + SLACK) + e * (1.f + SLACK);
                int qlo = 0, qhi = n_queries;
                while (qhi - qlo > 1) {
                    const int mid = (qlo + qhi) >> 1;
                    if (root_off[mid] <= i) qlo = mid; else qhi = mid;
                }
                row_q[i] = qlo;
            }
        }
    }
}
struct QuantiseArgs {
    const float *act, *E, *lo, *grid;
    const uint16_t* E16;
    const int32_t *row_ids, *root_off;
    uint32_t *Yq, *Eq;
    int32_t *slack, *row_q;
    float* base;
    int n_rows, n_ent, n_queries, d, words, ldy, lde, row_blocks;      // row_blocks: workgroups that take branch rows, before those of the entities
};
constexpr int QUANTISE_ROWS = 2;
template <int BITS, int RW>
__global__ __launch_bounds__(256) void quantise_kernel(const QuantiseArgs g) {
    __shared__ uint32_t lds[(BITS == 8 ? 64 : 128) * (4 * (RW > QUANTISE_ROWS ? RW : QUANTISE_ROWS) + 1)];
    if ((int)blockIdx.x < g.row_blocks)                    // uniform
        quantise<BITS, false, QUANTISE_ROWS>(blockIdx.x, g.act, nullptr, g.row_ids, g.n_rows, g.d, g.words, g.lo, g.grid, g.Yq, g.ldy, nullptr, g.base,
                                             g.root_off, g.n_queries, g.row_q, lds);
    else
        quantise<BITS, true, RW>(blockIdx.x - g.row_blocks, g.E, g.E16, nullptr, g.n_ent, g.d, g.words, g.lo, g.grid, g.Eq, g.lde, g.slack, nullptr, nullptr,
                                 0, nullptr, lds);
}

// ---------------------------------------------------------------- integer sums of a tile
template <int BITS>
__device__ __forceinline__ uint32_t sad(uint32_t a, uint32_t b, uint32_t c) {
    return BITS == 8 ? __builtin_amdgcn_sad_u8(a, b, c) : __builtin_amdgcn_sad_u16(a, b, c);
}

// Tile of 16*RPL branch rows x 128 entities, RPL x 8 pairs per lane: rows ty*RPL .., entities
// tx*4 .. +3 and 64 + tx*4 .. +3 (so that the 16-byte LDS reads of neighbouring lanes are adjacent).
// Both operands arrive word-major, SW words are staged at a time, the next ones on their way in
// registers meanwhile.  acc starts at the caller's values.  A launch covers its rows with tiles of 128
// and the remainder with the smallest tile of 32, 64 or 128 rows that holds it (1171 rows: 9 x 128 + 32
// instead of 10 x 128).
constexpr int SW = 8;
constexpr int TILE_LDS = 2 * SW * (128 + 128);      // words
template <int BITS, int RPL>
__device__ __forceinline__ void sad_tile(const uint32_t* __restrict__ Yq, int ldy, int r0, const uint32_t* __restrict__ Eq,
                                         int lde, int e0, int words, uint32_t (&acc)[RPL][8], uint32_t* lds) {
    constexpr int TR = 16 * RPL;
    uint32_t* Ys = lds;                    // [2][SW][TR]
    uint32_t* Es = lds + 2 * SW * TR;      // [2][SW][128]
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    constexpr int YQ = SW * 4 * RPL;       // 16-byte units of the row side of a stage (<= 256)
    const int ew = tid >> 5, ec = (tid & 31) * 4;
    const int yw = tid / (4 * RPL), yc = (tid % (4 * RPL)) * 4;
    const bool has_y = tid < YQ;
    // (words is a multiple of 4 and the rows of both operands are padded to whole tiles)
    uint4 ye = make_uint4(0, 0, 0, 0), ee = make_uint4(0, 0, 0, 0);
    auto issue = [&](int w0) {
        if (has_y) ye = *reinterpret_cast<const uint4*>(Yq + (size_t)min(w0 + yw, words - 1) * ldy + r0 + yc);
        ee = *reinterpret_cast<const uint4*>(Eq + (size_t)min(w0 + ew, words - 1) * lde + e0 + ec);
    };
    auto stage = [&](int buf) {
        if (has_y) *reinterpret_cast<uint4*>(Ys + (buf * SW + yw) * TR + yc) = ye;
        *reinterpret_cast<uint4*>(Es + (buf * SW + ew) * 128 + ec) = ee;
    };
    issue(0);
    stage(0);
    __syncthreads();
    const int ns = (words + SW - 1) / SW;
    for (int s = 0; s < ns; ++s) {
        const int buf = s & 1;
        if (s + 1 < ns) issue((s + 1) * SW);
        const int nw = min(SW, words - s * SW);          // 4 or 8
        for (int h = 0; h < nw; h += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t* yrow = Ys + (buf * SW + h + k) * TR + ty * RPL;
                const uint32_t* erow = Es + (buf * SW + h + k) * 128 + tx * 4;
                uint32_t y[RPL], e[8];
#pragma unroll
                for (int i = 0; i < RPL; i += (RPL < 4 ? 2 : 4)) {
                    if (RPL >= 4) {
                        const uint4 v = *reinterpret_cast<const uint4*>(yrow + i);
                        y[i] = v.x; y[i + 1] = v.y; y[(i + 2) % RPL] = v.z; y[(i + 3) % RPL] = v.w;
                    } else {
                        const uint2 v = *reinterpret_cast<const uint2*>(yrow + i);
                        y[i] = v.x; y[i + 1] = v.y;
                    }
                }
                const uint4 a = *reinterpret_cast<const uint4*>(erow);
                const uint4 b = *reinterpret_cast<const uint4*>(erow + 64);
                e[0] = a.x; e[1] = a.y; e[2] = a.z; e[3] = a.w; e[4] = b.x; e[5] = b.y; e[6] = b.z; e[7] = b.w;
#pragma unroll
                for (int i = 0; i < RPL; ++i)
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[i][j] = sad<BITS>(y[i], e[j], acc[i][j]);
            }
        }
        if (s + 1 < ns) stage(buf ^ 1);
        __syncthreads();
    }
}
// rows of the last tile row: 128, 64 or 32
__host__ __device__ __forceinline__ int tail_rows(int n_rows, int r0) { return n_rows - r0 > 64 ? 128 : (n_rows - r0 > 32 ? 64 : 32); }

struct NearArgs {
    const uint32_t *Yq, *Eq;
    const float *base, *grid, *best;
    const int32_t *row_q, *slack;
    uint32_t *found, *found_pair;
    int ldy, lde, n_rows, n_ent, words, k, parts;
    float rounding;
};
// Pairs that qualify are few (a per cent in the first chunk, one in 10^5 later).  They leave a tile as
// a list of its own, grouped by row, and one word per row that has any: start << 8 | number, at
// [row][tile column] of an array that is zero elsewhere; an entry is the entity's place in the tile (7 bits)
// below its sum less its error (counted from -2^20; 0: below that, where the error of a row far outside the grid may
// lie), i.e. its lower bound.  (Appending them to a list per query takes a
// device-wide atomic each: 140 us for the 300 000 pairs of a first chunk whose sums take 50.)  A tile
// with more than FOUND pairs marks its rows as crowded.
constexpr int FOUND = 2048;
constexpr uint32_t CROWDED = 0xFFFFFFFFu;
constexpr int32_t SUM_BIAS = 1 << 20;
struct NearLds {
    uint32_t tile[TILE_LDS];
    uint32_t pair[FOUND];
    uint8_t row[FOUND];
    int32_t n_row[128], at_row[128];
    int32_t n;
};
template <int RPL>
__device__ __forceinline__ void near_tile(const NearArgs& g, int r0, int e0, NearLds& L) {
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, lane = threadIdx.x & 63;
    uint32_t acc[RPL][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int e = e0 + (j >> 2) * 64 + tx * 4 + (j & 3);
        // the entity's error comes off the sum here; entities past the end never qualify
        int32_t sl = 0;
        for (int p = 0; p < g.parts; ++p) sl += g.slack[(size_t)p * g.lde + min(e, g.n_ent - 1)];
        const uint32_t start = e < g.n_ent ? (uint32_t)-slack_of(sl) : (uint32_t)(INT_MAX / 2);
#pragma unroll
        for (int i = 0; i < RPL; ++i) acc[i][j] = start;
    }
    sad_tile<8, RPL>(g.Yq, g.ldy, r0, g.Eq, g.lde, e0, g.words, acc, L.tile);
    const float inv = g.grid[1];
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int rl = ty * RPL + i, r = r0 + rl;
        int32_t most = INT_MIN;
        if (r < g.n_rows) {
            const float t = (g.best[(size_t)g.row_q[r] * g.k + g.k - 1] * (1.f + g.rounding) - g.base[r]) * inv + 4.f;
            // (no bound yet, or not a number: everything qualifies; rows of unbounded error always do)
            most = t < 5e8f ? (int32_t)fmaxf(t, -(float)(UNBOUNDED - SUM_BIAS)) : INT_MAX / 2 - 1;
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) any |= (int32_t)acc[i][j] <= most;
        if (__ballot(any) == 0ull) continue;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool ok = (int32_t)acc[i][j] <= most;
            const unsigned long long m = __ballot(ok);
            if (m == 0ull) continue;
            int at = 0;
            if (lane == __ffsll(m) - 1) at = atomicAdd(&L.n, __popcll(m));
            at = __builtin_amdgcn_readlane(at, __ffsll(m) - 1) + __popcll(m & ((1ull << lane) - 1ull));
            if (ok) {
                atomicAdd(&L.n_row[rl], 1);
                if (at < FOUND) {
                    L.pair[at] = (uint32_t)(max((int32_t)acc[i][j], -SUM_BIAS) + SUM_BIAS) << 7 | (uint32_t)((j >> 2) * 64 + tx * 4 + (j & 3));
                    L.row[at] = (uint8_t)rl;
                }
            }
        }
    }
    __syncthreads();
    const int n = L.n;
    if (n == 0) return;                              // uniform
    // places of the rows' groups: rows 2 * lane and 2 * lane + 1 of the scan of the first wavefront
    if (threadIdx.x < 64) {
        const int32_t c0 = L.n_row[2 * lane], c1 = L.n_row[2 * lane + 1];
        int32_t inc = c0 + c1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        L.at_row[2 * lane] = inc - c0 - c1;
        L.at_row[2 * lane + 1] = inc - c1;
    }
    __syncthreads();
    const size_t n_tx = gridDim.x;
    if (threadIdx.x < 128 && L.n_row[threadIdx.x] > 0)
        g.found[(r0 + threadIdx.x) * n_tx + blockIdx.x] =
            n > FOUND ? CROWDED : (uint32_t)L.at_row[threadIdx.x] << 8 | (uint32_t)L.n_row[threadIdx.x];
    if (n > FOUND) return;
    __syncthreads();
    uint32_t* out = g.found_pair + (blockIdx.y * n_tx + blockIdx.x) * FOUND;
    for (int x = threadIdx.x; x < n; x += 256) out[atomicAdd(&L.at_row[L.row[x]], 1)] = L.pair[x];
}

// Top-k: the pairs of the chunk whose distance may be at most the k-th distance of the row's query so far.
__global__ __launch_bounds__(256) void near_tile_kernel(const NearArgs g) {
    __shared__ __attribute__((aligned(16))) NearLds L;
    if (threadIdx.x < 128) L.n_row[threadIdx.x] = 0;         // (barriers in the tile loop before their use)
    if (threadIdx.x == 0) L.n = 0;
    const int r0 = blockIdx.y * 128, e0 = blockIdx.x * 128;
    const int rows = tail_rows(g.n_rows, r0);
    if (rows == 128) near_tile<8>(g, r0, e0, L);
    else if (rows == 64) near_tile<4>(g, r0, e0, L);
    else near_tile<2>(g, r0, e0, L);
}

// Filtered ranks, and the top-k of tables taken as a whole: the sums themselves, sums[r * ld + e] = SAD
// (15 000 entities x 585 rows x 400 coordinates by tiles of 64 rows 42 us, of 128 48; 60 000 x 228 x 400 the other way round, 272 and 241 us a ranking.)
// Top-k (8 bits): also edge[r * tiles + tile] = the least of the tile's sums less the entities' errors, and with them
__device__ __forceinline__ int32_t least_of_16(int32_t v) {        // over lanes 16 i .. 16 i + 15, rotated by 8, 4, 2, 1
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xF, 0xF, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xF, 0xF, true));
    return min(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xF, 0xF, true));
}
template <int BITS, int RPL>
__device__ __forceinline__ void sum_tile(const uint32_t* __restrict__ Yq, int ldy, int n_rows, const uint32_t* __restrict__ Eq,
                                         int lde, int n_ent, int words, uint32_t* __restrict__ sums, int ld, int r0, int e0,
                                         const int32_t* __restrict__ slack, int2* __restrict__ edge, uint32_t* lds) {
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    uint32_t acc[RPL][8];
#pragma unroll
    for (int i = 0; i < RPL; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0u;
    sad_tile<BITS, RPL>(Yq, ldy, r0, Eq, lde, e0, words, acc, lds);
    if (BITS == 8) {
        int32_t sl[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = e0 + (j >> 2) * 64 + tx * 4 + (j & 3);
            sl[j] = e < n_ent ? slack_of(slack[e]) : -1;
        }
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            int32_t lo = UNBOUNDED, hi = UNBOUNDED;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                lo = min(lo, sl[j] >= 0 ? (int32_t)acc[i][j] - sl[j] : UNBOUNDED);
                hi = min(hi, sl[j] >= 0 ? (int32_t)acc[i][j] + sl[j] : UNBOUNDED);
            }
            lo = least_of_16(lo);
            hi = least_of_16(hi);
            const int r = r0 + ty * RPL + i;
            if (tx == 0 && r < n_rows) edge[(size_t)r * gridDim.x + blockIdx.x] = make_int2(lo, hi);
        }
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
        const int r = r0 + ty * RPL + i;
        if (r >= n_rows) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = e0 + h * 64 + tx * 4;
            uint32_t* out = sums + (size_t)r * ld + e;
            if (e + 3 < n_ent) {
                *reinterpret_cast<uint4*>(out) = make_uint4(acc[i][4 * h], acc[i][4 * h + 1], acc[i][4 * h + 2], acc[i][4 * h + 3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (e + j < n_ent) out[j] = acc[i][4 * h + j];
            }
        }
    }
}
template <int BITS>
__global__ __launch_bounds__(256) void sum_tile_kernel(const uint32_t* __restrict__ Yq, int ldy, int n_rows,
                                                       const uint32_t* __restrict__ Eq, int lde, int n_ent, int words,
                                                       uint32_t* __restrict__ sums, int ld, int tile_rows,
                                                       const int32_t* __restrict__ slack, int2* __restrict__ edge) {
    __shared__ __attribute__((aligned(16))) uint32_t lds[TILE_LDS];
    const int r0 = blockIdx.y * tile_rows, e0 = blockIdx.x * 128;
    const int rows = min(tile_rows, tail_rows(n_rows, r0));
    if (rows == 128) sum_tile<BITS, 8>(Yq, ldy, n_rows, Eq, lde, n_ent, words, sums, ld, r0, e0, slack, edge, lds);
    else if (rows == 64) sum_tile<BITS, 4>(Yq, ldy, n_rows, Eq, lde, n_ent, words, sums, ld, r0, e0, slack, edge, lds);
    else sum_tile<BITS, 2>(Yq, ldy, n_rows, Eq, lde, n_ent, words, sums, ld, r0, e0, slack, edge, lds);
}

// ---------------------------------------------------------------- fp32 distances of a list
// min over the branch rows r_lo .. r_hi-1 of the fp32 distance to entity row e, one lane per entity,
// coordinates in ascending order: bit for bit what a distance tile holds for the pair.  The 64 rows of
// a wavefront come in slabs of C coordinates, C / 4 lanes a row, through the wavefront's own LDS (a lane
// that read its row itself would touch a cache line for every 16 bytes), PF slabs requested ahead: a list
// is short and the time is the latency of its rows.  The branch row's coordinates of a slab sit in the
// lanes and are broadcast from there.  Whole cache lines (32 coordinates, two ahead) where LDS is not what limits the wavefronts in
// flight: 142 against 150 us in count_open_kernel, but 35 against 29 us a chunk in near_merge_kernel, whose lists then leave room for three
// workgroups a compute unit instead of four.
constexpr int slab_ld(int C) { return C + 4; }
template <bool B16, int SLAB_C, int PF>
__device__ __forceinline__ float exact_distance(const float* __restrict__ act, const int32_t* __restrict__ row_ids, int r_lo,
                                                int r_hi, const float* __restrict__ E, const uint16_t* __restrict__ E16,
                                                int32_t e, int d, float* slab) {
    constexpr int SLAB_LD = slab_ld(SLAB_C), SLAB_PARTS = SLAB_C / 4, SLAB_ROWS = 64 / SLAB_PARTS;
    const int lane = threadIdx.x & 63, part = (lane % SLAB_PARTS) * 4, row = lane / SLAB_PARTS;
    int32_t id[SLAB_PARTS];
#pragma unroll
    for (int i = 0; i < SLAB_PARTS; ++i) id[i] = __shfl(e, row + SLAB_ROWS * i, 64);
    float4 x[PF][SLAB_PARTS];
    float y[PF];
    float best = INFINITY;
    for (int r = r_lo; r < r_hi; ++r) {
        const float* yrow = act + (size_t)row_ids[r] * d;
        auto issue = [&](int u, int c0) {
            const int c = min(c0 + part, d - 4);
            y[u] = yrow[min(c0 + (lane & (SLAB_C - 1)), d - 1)];
#pragma unroll
            for (int i = 0; i < SLAB_PARTS; ++i) {
                const size_t at = (size_t)id[i] * d + c;
                x[u][i] = B16 ? bf16x4_to_f32(*reinterpret_cast<const uint2*>(E16 + at)) : *reinterpret_cast<const float4*>(E + at);
            }
        };
        float acc = 0.f;
#pragma unroll
        for (int u = 0; u < PF; ++u) issue(u, u * SLAB_C);
        for (int c1 = 0; c1 < d; c1 += PF * SLAB_C) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                const int c0 = c1 + u * SLAB_C;
                if (c0 >= d) break;                  // uniform
#pragma unroll
                for (int i = 0; i < SLAB_PARTS; ++i) *reinterpret_cast<float4*>(slab + (row + SLAB_ROWS * i) * SLAB_LD + part) = x[u][i];
                const float yc = y[u];
                __builtin_amdgcn_wave_barrier();
                if (c0 + PF * SLAB_C < d) issue(u, c0 + PF * SLAB_C);
#pragma unroll
                for (int c = 0; c < SLAB_C; c += 4) {
                    if (c0 + c >= d) break;          // uniform
                    const float4 v = *reinterpret_cast<const float4*>(slab + lane * SLAB_LD + c);
                    acc += fabsf(lane_value(yc, c) - v.x);
                    acc += fabsf(lane_value(yc, c + 1) - v.y);
                    acc += fabsf(lane_value(yc, c + 2) - v.z);
                    acc += fabsf(lane_value(yc, c + 3) - v.w);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        best = r == r_lo ? acc : fminf(best, acc);
    }
    return best;
}

__device__ __forceinline__ bool before(float d, int i, float d2, int i2) { return d < d2 || (d == d2 && i < i2); }

struct MergeArgs {
    const float *act, *E, *base, *grid;
    const uint16_t* E16;
    const int32_t *row_ids, *root_off, *slack;
    uint32_t* found;
    const uint32_t* found_pair;
    int32_t *count, *overflowed;
    float* out_dist;
    int32_t* out_ids;
    int n_tx, ent_base, d, k, room, ldb, lde, parts;
    float rounding;
    const int32_t* gave_up;
};
// One workgroup per query: gathers what the tiles left for the query's rows (clearing their words for
// the next chunk) and merges the distances into the running top-k.  In a first chunk a list holds
// hundreds of entities against a bound that the chunk itself would improve: the upper bounds of the
// listed ones give the k-th (a histogram between the smallest and the bound so far), and only what
// can lie below that is computed, a tenth, 64 of them and one branch a wavefront and turn.  Nearly all of these turn out farther than
// the k-th so far; the few that are not are collected, and the first wavefront inserts those that still are before the k-th into the
// list its lanes hold (inserting every one, and a wavefront's branches one after the other: 42 against 28 us for 512 queries x 12 952
// entities x 400 coordinates, 42.5 against 34.5 for 1024 x 262 144 later on).
// What the tiles found goes into one list, or, where that has no room (ROOM entities, or a crowded tile), into one after the other for
// the pieces of the chunk; a query that has no room for a piece is marked (count > room, overflowed) for the fp32 pass of that piece
// alone.  (512 queries x 300 000 entities x 400, 5000 of which lie together near one query: 4.05 ms with the whole chunk in fp32, 2.13 so;
// without such a group 1.06 and 1.08.)  The distances' slabs lie over the lower bounds, which are done with by then: LDS for four
// workgroups a compute unit, all of 1024 queries at once, or three of 256 threads.
// MERGE_T: 128 threads, or 256 where three workgroups a compute unit hold all queries (35.4 and 29.7 us for those 512).  PRUNE_FROM: 64
// entities are one turn, pruned or not (28.5 against 29.7 us from 128 on).
constexpr int PIECE_TILES = RANK_PIECE / 128;
static_assert(PIECE_TILES % 256 == 0, "a thread's words are the same ones by pieces");
constexpr int ROOM = 4096, BINS = 256, MERGE_WIDE_TO = 768, PRUNE_FROM = 64;
template <bool B16, int MERGE_T>
__global__ __launch_bounds__(MERGE_T) void near_merge_kernel(const MergeArgs g) {
    constexpr int SLAB_LDS = 64 * slab_ld(16);
    __shared__ __attribute__((aligned(16))) float lower[ROOM > MERGE_T / 64 * SLAB_LDS ? ROOM : MERGE_T / 64 * SLAB_LDS];
    __shared__ int32_t list[ROOM], hist[BINS];
    __shared__ float sd[MERGE_T], best_hi[MERGE_T / 64];
    __shared__ uint32_t nearest[MERGE_T];
    __shared__ int32_t si[MERGE_T];
    __shared__ int32_t n_list, n_near, n_new, crowded;
    __shared__ float kth_d, bound;
    __shared__ int32_t kth_i;
    const int q = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6, k = g.k;
    if (t == 0) n_list = n_near = n_new = crowded = 0;
    __syncthreads();
    const int r_lo = g.root_off[q], r_hi = g.root_off[q + 1];
    const float step = g.grid[0];
    float my_d = INFINITY;
    int32_t my_i = INT_MAX;
    if (wave == 0 && lane < k) {
        const int32_t id = g.out_ids[(size_t)q * k + lane];
        if (id >= 0) {
            my_d = g.out_dist[(size_t)q * k + lane];
            my_i = id;
        }
        if (lane == k - 1) {
            kth_d = my_d;
            kth_i = my_i;
        }
    }
    // every tile column at once, or a piece after the other (a thread looks at the same words either way; seen: which of them, the last
    // bit for all further ones, are to be cleared)
    const int per_row = (g.n_tx + MERGE_T - 1) / MERGE_T;
    uint32_t seen = 0u;
    auto word_bit = [&](int r, int x) { return 1u << min((r - r_lo) * per_row + x / MERGE_T, 31); };
    for (int x0 = 0, width = g.n_tx;;) {
        const int x1 = min(g.n_tx, x0 + width);
        for (int r = r_lo; r < r_hi; ++r) {
            const uint32_t* words = g.found + (size_t)r * g.n_tx;
            const uint32_t* pairs = g.found_pair + (size_t)(r >> 7) * g.n_tx * FOUND;
            const float b_lo = g.base[r];
            for (int x = x0 + t; x < x1; x += MERGE_T) {
                const uint32_t w = words[x];
                if (w == 0u) continue;
                seen |= word_bit(r, x);
                if (w == CROWDED) {
                    crowded = 1;
                    continue;
                }
                const int n = w & 0xFF, from = w >> 8, at = atomicAdd(&n_list, n);
                for (int i = 0; i < n && at + i < ROOM; ++i) {
                    const uint32_t p = pairs[(size_t)x * FOUND + from + i];
                    list[at + i] = (int32_t)(x * 128 + (p & 127));
                    // (a sum that did not fit its bits bounds nothing)
                    lower[at + i] = p >> 7 ? (float)((int32_t)(p >> 7) - SUM_BIAS - 4) * step + b_lo : -INFINITY;
                }
            }
        }
        __syncthreads();
        int n = n_list;
        const bool over = n > ROOM || crowded;           // uniform
        if (over || x1 < g.n_tx) {                       // (there may be another list)
            __syncthreads();
            if (t == 0) n_list = crowded = 0;
        }
        if (over && width > PIECE_TILES) {
            width = PIECE_TILES;
            __syncthreads();
            continue;
        }
        if (x1 == g.n_tx) {                              // no word is looked at again
            for (int r = r_lo; r < r_hi && seen; ++r)
                for (int x = t; x < g.n_tx; x += MERGE_T)
                    if (seen & word_bit(r, x)) g.found[(size_t)r * g.n_tx + x] = 0u;
            if (n == 0 && !over && width == g.n_tx) return;
        }
        if (over) {
            if (t == 0) {
                const int p = x0 / PIECE_TILES;
                g.overflowed[p] = 1;
                g.count[(size_t)p * gridDim.x + q] = g.room + 1;
            }
            n = 0;
        }
        if (n > PRUNE_FROM && kth_d < INFINITY) {
            // upper bound of a listed entity: its lower one and twice both errors (the widest branch's)
            float both = 0.f;
            for (int r = r_lo; r < r_hi; ++r) both = fmaxf(both, g.base[g.ldb + r] - g.base[r]);
            float hi_min = INFINITY;
            auto upper = [&](int x) {
                int32_t sum = 0;
                for (int p = 0; p < g.parts; ++p) sum += g.slack[(size_t)p * g.lde + list[x]];
                const int32_t sl = slack_of(sum);
                return sl == UNBOUNDED || lower[x] == -INFINITY ? INFINITY : (lower[x] + both + (float)(2 * sl + 8) * step) * (1.f + g.rounding);
            };
            for (int x = t; x < n; x += MERGE_T) hi_min = fminf(hi_min, upper(x));
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) hi_min = fminf(hi_min, __shfl_xor(hi_min, off, 64));
            if (lane == 0) best_hi[wave] = hi_min;
            for (int b = t; b < BINS; b += MERGE_T) hist[b] = 0;
            __syncthreads();
            const float top = kth_d;
            hi_min = best_hi[0];
#pragma unroll
            for (int w = 1; w < MERGE_T / 64; ++w) hi_min = fminf(hi_min, best_hi[w]);
            const float scale = (float)BINS / (top - hi_min);        // (top <= hi_min: nothing falls into a bin)
            for (int x = t; x < n; x += MERGE_T) {
                const float b = (upper(x) - hi_min) * scale;
                if (b >= 0.f && b < (float)BINS) atomicAdd(&hist[(int)b], 1);
            }
            __syncthreads();
            if (wave == 0) {   // the first bin that completes k entities (an entity may be listed by every branch)
                int32_t c[BINS / 64], sum = 0;
#pragma unroll
                for (int i = 0; i < BINS / 64; ++i) {
                    c[i] = hist[lane * (BINS / 64) + i];
                    sum += c[i];
                }
                int32_t inc = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int32_t v = __shfl_up(inc, off, 64);
                    if (lane >= off) inc += v;
                }
                const int want = k * (r_hi - r_lo);
                const unsigned long long m = __ballot(inc >= want);
                if (lane == (m ? __ffsll(m) - 1 : 0)) {
                    int32_t run = inc - sum;
                    int bin = BINS;
#pragma unroll
                    for (int i = BINS / 64 - 1; i >= 0; --i) {
                        int32_t upto = run;
#pragma unroll
                        for (int i2 = 0; i2 <= i; ++i2) upto += c[i2];
                        if (upto >= want) bin = lane * (BINS / 64) + i;
                    }
                    // (one bin of room for the rounding of the bin number)
                    bound = m && bin < BINS - 2 ? fminf(top, hi_min + (float)(bin + 2) / scale) : top;
                }
            }
            __syncthreads();
            // in place: a slot is written by the round that reads it or a later one
            const float most = bound * (1.f + g.rounding);
            for (int base = 0; base < n; base += MERGE_T) {
                const int x = base + t;
                const bool keep = x < n && !(lower[x] > most);
                const int32_t e = x < n ? list[x] : 0;
                __syncthreads();
                const unsigned long long m = __ballot(keep);
                int at = 0;
                if (lane == 0) at = atomicAdd(&n_near, __popcll(m));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
                if (keep) list[at] = e;
                __syncthreads();
            }
            n = n_near;
        }
        for (int base = 0; base < n; base += MERGE_T) {
            // 64 entities and one branch at a time, dealt to the wavefronts (a few entities of a union in one go)
            const int parts = (min(n - base, MERGE_T) + 63) / 64, units = parts * (r_hi - r_lo);
            nearest[t] = 0xFFFFFFFFu;
            __syncthreads();
            for (int u = wave; u < units; u += MERGE_T / 64) {
                const int part = u % parts, r = r_lo + u / parts, x = base + part * 64 + lane;
                const int32_t e = x < n ? list[x] : 0;
                const float dv = exact_distance<B16, 16, 3>(g.act, g.row_ids, r, r + 1, g.E, g.E16, e, g.d, lower + wave * SLAB_LDS);
                atomicMin(&nearest[part * 64 + lane], __builtin_bit_cast(uint32_t, dv));       // (no distance is negative; NaN is above all others)
            }
            __syncthreads();
            if (base + t < n) {
                const float dv = __builtin_bit_cast(float, nearest[t]);
                const int32_t id = g.ent_base + list[base + t];
                if (before(dv, id, kth_d, kth_i)) {
                    const int at = atomicAdd(&n_new, 1);
                    sd[at] = dv;
                    si[at] = id;
                }
            }
            __syncthreads();
            if (wave == 0) {
                // the lanes hold the new distances; whatever is no longer before the k-th falls out at once
                const int m = n_new;
                float dn[MERGE_T / 64];
                int32_t in[MERGE_T / 64];
                bool open[MERGE_T / 64];
                float kd = kth_d;
                int32_t ki = kth_i;
#pragma unroll
                for (int w = 0; w < MERGE_T / 64; ++w) {
                    open[w] = w * 64 + lane < m;
                    dn[w] = open[w] ? sd[w * 64 + lane] : INFINITY;
                    in[w] = open[w] ? si[w * 64 + lane] : INT_MAX;
                }
#pragma unroll
                for (int w = 0; w < MERGE_T / 64; ++w) {
                    for (;;) {
                        const unsigned long long left = __ballot(open[w] && before(dn[w], in[w], kd, ki));
                        if (left == 0ull) break;
                        const int from = __ffsll(left) - 1;
                        const float dv = lane_value(dn[w], from);
                        const int32_t id = lane_value(in[w], from);
                        open[w] = open[w] && lane > from;
                        if (__ballot(my_i == id) != 0ull) continue;      // listed by another branch already
                        const bool stays = before(my_d, my_i, dv, id);
                        const float up_d = __shfl_up(my_d, 1, 64);
                        const int32_t up_i = __shfl_up(my_i, 1, 64);
                        const bool up_stays = lane == 0 || before(up_d, up_i, dv, id);
                        if (!stays) {
                            my_d = up_stays ? dv : up_d;
                            my_i = up_stays ? id : up_i;
                        }
                        if (lane >= k) {
                            my_d = INFINITY;
                            my_i = INT_MAX;
                        }
                        kd = lane_value(my_d, k - 1);
                        ki = lane_value(my_i, k - 1);
                    }
                }
                if (lane == 0) {
                    kth_d = kd;
                    kth_i = ki;
                }
                if (lane == 0) n_new = 0;
            }
            __syncthreads();
        }
        x0 += width;
        if (x0 >= g.n_tx) break;
        __syncthreads();
        if (t == 0) n_near = 0;
        __syncthreads();
    }
    if (wave == 0 && lane < k && !*g.gave_up) {          // (of a pass that gave up there is none from the first chunk on)
        g.out_dist[(size_t)q * k + lane] = my_d;
        g.out_ids[(size_t)q * k + lane] = my_i == INT_MAX ? -1 : my_i;
    }
}

// ---------------------------------------------------------------- filtered ranks
// thr[a] = fp32 distance of answer a to its query, one lane per answer, summed like a distance tile.  The
// lanes of a wavefront may belong to different queries: the branch rows are read from memory (as bound by latency as there are few
// wavefronts: requests of 80 coordinates at a time, 16 us for 8192 answers x 400; 17.4 with 40).  counters[a] and
// counters[n_ans + a] are cleared on the way.
template <bool BOX>
__global__ __launch_bounds__(64) void answer_distance_kernel(const float* __restrict__ act, const float* __restrict__ off, float alpha,
                                                             const int32_t* __restrict__ row_ids, const int32_t* __restrict__ root_off,
                                                             const int32_t* __restrict__ ans_off, int n_queries,
                                                             const int32_t* __restrict__ ans, int a0, int cnt,
                                                             const float* __restrict__ E, const uint16_t* __restrict__ E16, int d,
                                                             const int32_t* __restrict__ gave_up, float* __restrict__ thr, int32_t* __restrict__ counters, int n_ans) {
    const int i = blockIdx.x * 64 + threadIdx.x, a = a0 + i;
    if (i >= cnt) return;
    counters[a] = counters[n_ans + a] = 0;
    int lo = 0, hi = n_queries;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ans_off[mid] <= a) lo = mid; else hi = mid;
    }
    const size_t e = ans ? (size_t)ans[a] : (size_t)i;
    const float shrink = 1.f - alpha;
    float best = INFINITY;
    for (int r = root_off[lo]; r < root_off[lo + 1]; ++r) {
        const size_t yrow = (size_t)row_ids[r] * d;
        float acc = 0.f;
        auto add = [&](float y, float x, float o) {
#pragma clang fp contract(off)
            const float diff = fabsf(y - x);
            acc += BOX ? fmaxf(alpha * diff, diff - shrink * o) : diff;
        };
#pragma unroll 20
        for (int c = 0; c < d; c += 4) {
            const float4 x = E16 ? bf16x4_to_f32(*reinterpret_cast<const uint2*>(E16 + e * d + c)) : *reinterpret_cast<const float4*>(E + e * d + c);
            const float4 y = *reinterpret_cast<const float4*>(act + yrow + c);
            const float4 o = BOX ? *reinterpret_cast<const float4*>(off + yrow + c) : x;
            add(y.x, x.x, o.x);
            add(y.y, x.y, o.y);
            add(y.z, x.z, o.z);
            add(y.w, x.w, o.w);
        }
        best = fminf(best, acc);
    }
    thr[a] = *gave_up ? INFINITY : best;
}

// Bounds of the distance of a (row, entity) pair from its sum, the entity's error in steps and the row's
// constants; every caller gets the same bits.  Every addition of the fp32 distance D errs by at most half a unit in the last
// place of D (its partial sums grow), i.e. 2^-24 of the largest power of two within D, and that of a D below lo is
// no larger than lo's, of any D no larger than that of hi and its relative slack.  (d + 16) 2^-24 of the distance itself left 440 000 entities of 1024
// queries x 63 000 x 400 with 8 answers each undecided: 147 us in count_open_kernel, 131 now.
struct Bounds { float lo, hi; };
__device__ __forceinline__ float power_of_two(float x) { return __uint_as_float(__float_as_uint(x) & 0x7F800000u); }     // of |x|, the largest within
__device__ __forceinline__ Bounds bounds_of(uint32_t sum, int32_t sl, float step, float b_lo, float b_hi, float rounding) {
    sl = min(sl, SLACK_CAP);
    const float lo = fmaf((float)((int32_t)sum - sl), step, b_lo), hi = fmaf((float)((int32_t)sum + sl), step, b_hi);
    const bool none = sl == SLACK_CAP;
    return {none ? -INFINITY : fmaf(-rounding, power_of_two(lo), lo), none ? INFINITY : fmaf(rounding, power_of_two(fmaf(rounding, fabsf(hi), hi)), hi)};
}

// Top-k of a table as a whole: the sums of all its entities are in memory, and one workgroup per query takes its k nearest from them.
// The tiles have left the least upper and lower bound of every row: the k-th smallest upper one of 64 groups of tiles is a bound that k
// entities keep, hardly more than k of them.  Tiles that reach below it are looked through, and whatever may lie within it, some two or
// three times k, is listed and computed; what lies within the same bound on these distances (some k of them, as no two pairs of distance and
// number are alike) is placed by counting.  512 queries x 15 000 entities x 400: 42 us looking through all sums twice, 27 through the tiles.
// 128 registers a lane: four workgroups a compute unit (158, two rounds of 512 queries: 59 us against 42).
// A list has room for ROOM entities (a union lists an entity once, for the first branch that does).  Where more lie within the bound
// (entities that the sums cannot tell apart) the table is taken a piece at a time, and a piece in halves until their lists have room (32
// tiles are ROOM entities), the k nearest so far kept from one to the next; a piece with more than twice ROOM, or a PICK_SHARE-th
// of its entities, goes to the fp32 pass, which is through first then.
// us without such entities, with 300, 1000, 1900, 3000, 5000 of them near many queries' nearest and with nothing else; by chunks from a
// sample on; and with one list of 2048 whose branches' entities were told apart and placed by all pairs, beyond which all pieces went to fp32:
// 15 000 x 584 rows x 400 185 223 294 376 508 560 459; 249 267 325 394 486 527 510; 187 271 655 1272 925 444 461.  60 000 x 228 210 264 373
// 466 571 866 1164; 299 331 374 447 542 699 1175; 208 297 683 1225 1173 1176 1219.  200 000 x 64 292 316 395 464 538 799 3303; 433 442 475
// 521 587 721 3319; 292 370 664 1172 3303 3324 3468.  8000 x 456, which fp32 alone took 178 for, 157 187 253 263 263 263 307.
constexpr int PICK_T = 256, PICK_AT_ONCE = 512, PICK_AHEAD = 4, PICK_WALK = 4, PICK_SHARE = 6;
constexpr int PICK_WAVES = PICK_T / 64;
static_assert(PIECE_TILES % (ROOM / 128) == 0 && (PIECE_TILES / (ROOM / 128) & (PIECE_TILES / (ROOM / 128) - 1)) == 0, "a piece is halved down to tiles that have room");
struct PickArgs {
    const float *act, *E, *base, *grid;
    const uint16_t* E16;
    const int32_t *row_ids, *root_off, *slack;
    const uint32_t* sums;
    const int2* edge;
    int32_t *count, *overflowed;
    float* out_dist;
    int32_t* out_ids;
    int ld, n_ent, d, k, room, ldb;
    float rounding;
    const int32_t* gave_up;
};
template <bool B16>
__global__ __launch_bounds__(PICK_T, 4) void pick_kernel(const PickArgs g) {
    __shared__ __attribute__((aligned(16))) float slab[PICK_WAVES][64 * slab_ld(16)];
    __shared__ int32_t list[ROOM];
    __shared__ uint32_t nearest[PICK_AT_ONCE];
    __shared__ uint64_t s_run[NGDB_MAX_TOPK], s_bound;
    __shared__ float s_far;
    __shared__ int32_t s_most[NGDB_MAX_BRANCH], n_list, n_within;
    uint64_t* const s_least = reinterpret_cast<uint64_t*>(slab);        // [PICK_T], [PICK_AT_ONCE + NGDB_MAX_TOPK]: used when the slabs are not
    uint64_t* const within = s_least + PICK_T;
    static_assert(sizeof(slab) >= (PICK_T + PICK_AT_ONCE + NGDB_MAX_TOPK) * sizeof(uint64_t), "in the place of the slabs");
    constexpr uint64_t NONE = ~0ull;                     // (a distance that is no number comes after all others)
    const int q = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6, k = g.k;
    const int r_lo = g.root_off[q], r_hi = g.root_off[q + 1];
    const float step = g.grid[0];
    const int n_tx = (g.n_ent + 127) / 128;
    float least = INFINITY;
    for (int r = r_lo; r < r_hi; ++r) {
        int32_t sum_least = UNBOUNDED;
        for (int x = t; x < n_tx; x += PICK_T) sum_least = min(sum_least, g.edge[(size_t)r * n_tx + x].y);
        const float hi = fmaf((float)sum_least, step, g.base[g.ldb + r]);
        if (sum_least < UNBOUNDED) least = fminf(least, fmaf(g.rounding, fabsf(hi), hi));
    }
    float* const parts_least = slab[0];
    parts_least[t] = least;
    if (t < k) s_run[t] = NONE;
    __syncthreads();
    if (wave == 0) {                                     // the k-th smallest of the 64 groups' least upper bounds
#pragma unroll
        for (int w = 1; w < PICK_WAVES; ++w) least = fminf(least, parts_least[w * 64 + lane]);
        int smaller = 0;
#pragma unroll
        for (int j = 0; j < 64; ++j) {
            const float o = lane_value(least, j);
            smaller += (o < least || (o == least && j < lane)) ? 1 : 0;
        }
        if (smaller == k - 1) s_far = least;
    }
    __syncthreads();
    if (t < r_hi - r_lo) {
        const float bound = (s_far * (1.f + g.rounding) - g.base[r_lo + t]) * g.grid[1] + 4.f;
        // (no bound, or not a number: everything qualifies; entities of unbounded error always do)
        s_most[t] = bound < 5e8f ? (int32_t)fmaxf(bound, -(float)(UNBOUNDED - SUM_BIAS)) : INT_MAX / 2 - 1;
    }
    for (int x0 = 0, width = n_tx > PIECE_TILES ? RANK_PIECES * PIECE_TILES : PIECE_TILES; x0 < n_tx;) {
        const int x1 = min(n_tx, x0 + width);
        const int most = width == PIECE_TILES ? min(2 * ROOM, (min(g.n_ent, x1 * 128) - x0 * 128) / PICK_SHARE) : ROOM;
        if (t == 0) n_list = 0;
        __syncthreads();
        for (int r = r_lo; r < r_hi; ++r) {
            const int32_t sum_most = s_most[r - r_lo];
            for (int xb = x0; xb < x1; xb += PICK_T) {   // (neighbouring tiles go to different wavefronts)
                const int mine = xb + lane * PICK_WAVES + wave;
                unsigned long long m = __ballot(mine < x1 && g.edge[(size_t)r * n_tx + min(mine, n_tx - 1)].x <= sum_most);
                while (m != 0ull && __builtin_amdgcn_readfirstlane(__hip_atomic_load(&n_list, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) <= most) {
                    int e[PICK_WALK];
                    uint2 sum[PICK_WALK];
                    int2 sl[PICK_WALK];
#pragma unroll
                    for (int i = 0; i < PICK_WALK; ++i) {
                        const int from = m ? __ffsll(m) - 1 : 0;
                        e[i] = m ? (xb + from * PICK_WAVES + wave) * 128 + 2 * lane : g.n_ent;
                        m &= m - 1ull;
                        const int at = min(e[i], (g.n_ent - 1) & ~1);
                        sum[i] = *reinterpret_cast<const uint2*>(g.sums + (size_t)r * g.ld + at);
                        sl[i] = *reinterpret_cast<const int2*>(g.slack + at);
                    }
#pragma unroll
                    for (int i = 0; i < PICK_WALK; ++i) {
                        auto look = [&](int id, uint32_t v, int32_t err) {
                            if (id >= g.n_ent || (int32_t)v - slack_of(err) > sum_most) return;
                            for (int p = r_lo; p < r; ++p)
                                if ((int32_t)g.sums[(size_t)p * g.ld + id] - slack_of(err) <= s_most[p - r_lo]) return;
                            const int at = atomicAdd(&n_list, 1);
                            if (at < ROOM) list[at] = id;
                        };
                        look(e[i], sum[i].x, sl[i].x);
                        look(e[i] + 1, sum[i].y, sl[i].y);
                    }
                }
            }
        }
        __syncthreads();
        const int n = n_list;
        __syncthreads();
        if (n > min(most, ROOM)) {                       // uniform
            if (width == PIECE_TILES && n > most) {
                if (t == 0) {
                    g.count[(size_t)(x0 / PIECE_TILES) * gridDim.x + q] = g.room + 1;
                    g.overflowed[x0 / PIECE_TILES] = 1;
                }
                x0 = x1;
            } else {
                width = width > PIECE_TILES ? PIECE_TILES : width / 2;
            }
            continue;
        }
        for (int l0 = 0; l0 < n; l0 += PICK_AT_ONCE) {
            const int here = min(n - l0, PICK_AT_ONCE), parts = (here + 63) / 64, units = parts * (r_hi - r_lo);
            for (int x = t; x < here; x += PICK_T) nearest[x] = 0xFFFFFFFFu;
            if (t == 0) n_within = 0;
            __syncthreads();
            for (int u = wave; u < units; u += PICK_WAVES) {
                const int r = r_lo + u / parts, x = (u % parts) * 64 + lane;
                const int32_t e = list[l0 + min(x, here - 1)];
                const float dv = exact_distance<B16, 16, PICK_AHEAD>(g.act, g.row_ids, r, r + 1, g.E, g.E16, e, g.d, slab[wave]);
                if (x < here) atomicMin(&nearest[x], __builtin_bit_cast(uint32_t, dv));       // (no distance is negative; NaN is above all others)
            }
            __syncthreads();
            // distance and number as one key, those so far among them
            auto key_of = [&](int x) { return nearest[x] <= 0x7F800000u ? (uint64_t)nearest[x] << 32 | (uint32_t)list[l0 + x] : NONE; };
            uint64_t mine = t < k ? s_run[t] : NONE;
            for (int x = t; x < here; x += PICK_T) mine = min(mine, key_of(x));
            s_least[t] = mine;
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int w = 1; w < PICK_WAVES; ++w) mine = min(mine, s_least[w * 64 + lane]);
                int smaller = 0;
#pragma unroll
                for (int j = 0; j < 64; ++j) {
                    const uint64_t o = (uint64_t)(uint32_t)lane_value((int32_t)(mine >> 32), j) << 32 | (uint32_t)lane_value((int32_t)(uint32_t)mine, j);
                    smaller += (o < mine || (o == mine && j < lane)) ? 1 : 0;
                }
                if (smaller == k - 1) s_bound = mine;
            }
            __syncthreads();
            const uint64_t bound = s_bound;
            auto keep = [&](uint64_t key) {
                if (key <= bound && key != NONE) within[atomicAdd(&n_within, 1)] = key;
            };
            if (t < k) keep(s_run[t]);
            for (int x = t; x < here; x += PICK_T) keep(key_of(x));
            __syncthreads();
            const int m = n_within;
            if (t >= m && t < k) s_run[t] = NONE;
            for (int x = t; x < m; x += PICK_T) {
                const uint64_t key = within[x];
                int place = 0;
                for (int j = 0; j < m; ++j) place += within[j] < key ? 1 : 0;
                if (place < k) s_run[place] = key;
            }
            __syncthreads();
        }
        x0 = x1;
        if (x0 % PIECE_TILES == 0) width = PIECE_TILES;
    }
    __syncthreads();
    if (t < k) {
        const uint64_t key = *g.gave_up ? NONE : s_run[t];
        g.out_dist[(size_t)q * k + t] = key == NONE ? INFINITY : __builtin_bit_cast(float, (uint32_t)(key >> 32));
        g.out_ids[(size_t)q * k + t] = key == NONE ? -1 : (int32_t)(uint32_t)key;
    }
}

// closer[a] += entities that are certainly closer than answer a; an entity that may lie between its bounds from
// some answer of the query is not decided and goes to the query's list.  Grid (parts, queries): a workgroup
// takes every gridDim.x-th slab of 2048 entities, 8 per lane.  The thresholds of a query lie sorted in LDS: an entity looks
// up how many are no larger than its upper bound (a search of log2 steps, 3 vector operations each), which places it in a
// histogram whose running sums are the counts, and it is open if the last of them exceeds its lower bound.  Up to ANS_OWN answers every
// thread has a histogram of its own (lanes that add to one word of LDS take turns); beyond, the workgroup has one (us for 1024 queries x
// 63 000 entities, own and shared: 8 answers 130 and 158, 15 answers 137 and 152; own ones for 31 answers take LDS from all: 8 answers 138, 15
// 145, 16 151 against 157 shared, 20 153 and 153, 24 159 and 155, 31 162 and 158).  The list is
// collected in LDS: one device-wide atomic a workgroup as a rule.  1024 queries x 63 000 entities x 8 answers: 217 us with two
// comparisons per answer whose lanes the scalar unit counts and combines (4 operations at a quarter of the rate), 113 now; reading
// the sums takes 60.  Queries of more than ANS_LDS answers are counted that way, the first 256 of them in LDS (128 queries, 20 of them of 256
// answers: a ranking of 1570 us with a device-wide atomic per answer and slab for all of them, 1534 so).
constexpr int EPT = 8, SLAB = EPT * 256, ANS_LDS = 255, ANS_OWN = 15, OPEN_KEPT = 1024;
static_assert((65536 / SLAB) * EPT < 65536, "own counters of a chunk fit 16 bits");
__global__ __launch_bounds__(256) void count_sure_kernel(const uint32_t* __restrict__ sums, int ld, const int32_t* __restrict__ slack, int parts, int lde,
                                                         const float* __restrict__ base, int ldb, const float* __restrict__ grid,
                                                         const int32_t* __restrict__ root_off, const int32_t* __restrict__ ans_off,
                                                         const float* __restrict__ thr, int n_ent, float rounding,
                                                         int32_t* __restrict__ closer, int32_t* __restrict__ list,
                                                         int32_t* __restrict__ count, int room) {
    __shared__ float s_thr[ANS_LDS + 2], s_raw[ANS_LDS + 1];       // (below the smallest threshold: minus infinity)
    __shared__ int32_t s_of[ANS_LDS + 1], s_sum[ANS_LDS + 1];
    __shared__ uint32_t s_hist[(ANS_OWN + 2) * 128];  // (own ones: two to a word, at most 8 entities times 32 slabs each)
    __shared__ uint16_t s_open[SLAB + OPEN_KEPT];     // (an entity's place in the chunk: at most 65 536 of them)
    __shared__ int32_t n_open, open_at;
    const int q = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int a_lo = ans_off[q], n_a = ans_off[q + 1] - a_lo;
    if (n_a <= 0) return;                                             // uniform
    const int r_lo = root_off[q], r_hi = root_off[q + 1];
    const float step = grid[0];
    const bool searched = n_a <= ANS_LDS, own = n_a <= ANS_OWN;
    const uint32_t mine_one = t & 1 ? 0x10000u : 1u;
    int top = 1;                                     // thresholds with those past the end: the next power of two
    while (top <= n_a) top <<= 1;
    if (searched) {
        // (nothing is closer than an answer whose distance is not a number)
        const float mine = t < n_a ? thr[a_lo + t] : 0.f;
        s_raw[t] = mine == mine ? mine : -INFINITY;
        s_thr[t + 1] = INFINITY;
        if (t == 0) s_thr[0] = -INFINITY;
        for (int x = t; x < (own ? (ANS_OWN + 2) * 128 : 256); x += 256) s_hist[x] = 0u;
        __syncthreads();
        if (t < n_a) {
            const float v = s_raw[t];
            int at = 0;
            for (int i = 0; i < n_a; ++i) at += s_raw[i] < v || (s_raw[i] == v && i < t) ? 1 : 0;
            s_thr[at + 1] = v;
            s_of[at] = t;
        }
    }
    if (!searched) s_sum[t] = 0;
    if (t == 0) n_open = 0;
    __syncthreads();
    for (int e_lo = blockIdx.x * SLAB; e_lo < n_ent; e_lo += gridDim.x * SLAB) {
        const int e_hi = min(n_ent, e_lo + SLAB);
        float vlo[EPT], vhi[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) vlo[j] = vhi[j] = INFINITY;
        for (int r = r_lo; r < r_hi; ++r) {
            const float b_lo = base[r], b_hi = base[ldb + r];
#pragma unroll
            for (int h = 0; h < EPT; h += 4) {       // (rows and errors are padded to groups of four)
                const int e = min(e_lo + h * 256 + t * 4, (e_hi - 1) & ~3);
                const uint4 sum = *reinterpret_cast<const uint4*>(sums + (size_t)r * ld + e);
                int4 sl = *reinterpret_cast<const int4*>(slack + e);
                for (int p = 1; p < parts; ++p) {
                    const int4 x = *reinterpret_cast<const int4*>(slack + (size_t)p * lde + e);
                    sl.x += x.x; sl.y += x.y; sl.z += x.z; sl.w += x.w;
                }
                const Bounds b[4] = {bounds_of(sum.x, sl.x, step, b_lo, b_hi, rounding), bounds_of(sum.y, sl.y, step, b_lo, b_hi, rounding),
                                     bounds_of(sum.z, sl.z, step, b_lo, b_hi, rounding), bounds_of(sum.w, sl.w, step, b_lo, b_hi, rounding)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    vlo[h + i] = fminf(vlo[h + i], b[i].lo);
                    vhi[h + i] = fminf(vhi[h + i], b[i].hi);
                }
            }
        }
        auto place = [&](int j) { return e_lo + (j & 4) * 256 + t * 4 + (j & 3); };
        if (e_hi - e_lo < SLAB) {                    // entities past the end are closer to nothing
#pragma unroll
            for (int j = 0; j < EPT; ++j)
                if (place(j) >= e_hi) vlo[j] = vhi[j] = INFINITY;
        }
        bool open[EPT];
        if (searched) {
            int at[EPT];
#pragma unroll
            for (int j = 0; j < EPT; ++j) at[j] = 0;
            for (int half = top >> 1; half > 0; half >>= 1) {
#pragma unroll
                for (int j = 0; j < EPT; ++j) at[j] += s_thr[at[j] + half] <= vhi[j] ? half : 0;
            }
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                atomicAdd(&s_hist[own ? at[j] * 128 + (t >> 1) : at[j]], own ? mine_one : 1u);
                open[j] = s_thr[at[j]] > vlo[j];
            }
        } else {
            unsigned long long some[EPT];
#pragma unroll
            for (int j = 0; j < EPT; ++j) some[j] = 0ull;
            for (int a = a_lo; a < a_lo + n_a; ++a) {
                const float th = thr[a];
                int c = 0;
#pragma unroll
                for (int j = 0; j < EPT; ++j) {
                    const unsigned long long sure = __ballot(vhi[j] < th);
                    c += __popcll(sure);
                    some[j] |= sure ^ __ballot(vlo[j] < th);
                }
                if (lane == 0 && c) {
                    if (a - a_lo <= ANS_LDS) atomicAdd(&s_sum[a - a_lo], c);
                    else atomicAdd(&closer[a], c);
                }
            }
#pragma unroll
            for (int j = 0; j < EPT; ++j) open[j] = some[j] >> lane & 1ull;
        }
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const unsigned long long m = __ballot(open[j]);
            if (m == 0ull) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&n_open, __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
            if (open[j]) s_open[at] = (uint16_t)place(j);
        }
        __syncthreads();
        const int n = n_open;
        const bool last = e_lo + (int)gridDim.x * SLAB >= n_ent;
        if (n > OPEN_KEPT || (last && n)) {                           // (room for another slab is left otherwise)
            if (t == 0) open_at = atomicAdd(&count[q], n);
            __syncthreads();
            for (int x = t; x < n; x += 256)
                if (open_at + x < room) list[(size_t)q * room + open_at + x] = s_open[x];
            __syncthreads();
            if (t == 0) n_open = 0;
        }
        __syncthreads();
    }
    if (!searched) {                                 // (at least 256 answers)
        if (s_sum[t]) atomicAdd(&closer[a_lo + t], s_sum[t]);
        return;
    }
    if (own) {
        for (int b = wave; b < n_a; b += 4) {
            const uint32_t x = s_hist[b * 128 + lane], y = s_hist[b * 128 + 64 + lane];
            const float c = wave_sum_dpp((float)((x & 0xFFFFu) + (x >> 16) + (y & 0xFFFFu) + (y >> 16)));
            if (lane == 0) s_sum[b] = (int32_t)c;
        }
    } else {
        s_sum[t] = (int32_t)s_hist[t];
    }
    __syncthreads();
    if (t < n_a) {
        int32_t c = 0;
        for (int b = 0; b <= t; ++b) c += s_sum[b];
        if (c) atomicAdd(&closer[a_lo + s_of[t]], c);
    }
}

// The undecided entities of the chunk in fp32 (for the answers that their upper bound has not counted already), and the
// chunk's counts added to the running ones.  Grid (OPEN_PARTS, queries): 64 entities at a time, dealt to the parts in turn (queries
// have up to some hundred entities per answer, and one workgroup per query left the card to those with the longest lists: 198 us
// against 142 for 1024 queries with 1 to 15 answers, some 440 000 rows of 1600 bytes, which is what is left).  Four parts, then one and
// sixteen, us: 1024 queries of 4 answers 98, 97, 294, of 8 143, 166, 297, of 15 256, 294, 319, of 31 491, 565, 472; 64 queries of 8 answers 22,
// 57, 32, of 15 28, 81, 36, of 40 76, 214, 54, of 60 109, 330, 69.  A query whose list overflowed
// drops the chunk's counts (the fp32 pass of the chunk counts for it); its list count stays as the mark for that.
constexpr int OPEN_PARTS = 4;
template <bool B16>
__global__ __launch_bounds__(256) void count_open_kernel(const float* __restrict__ act, const int32_t* __restrict__ row_ids,
                                                         const int32_t* __restrict__ root_off, const int32_t* __restrict__ ans_off,
                                                         const float* __restrict__ thr, const float* __restrict__ E,
                                                         const uint16_t* __restrict__ E16, int d, const uint32_t* __restrict__ sums,
                                                         int ld, const int32_t* __restrict__ slack, int parts, int lde, const float* __restrict__ base,
                                                         int ldb, const float* __restrict__ grid, float rounding,
                                                         const int32_t* __restrict__ list, const int32_t* __restrict__ count, int room,
                                                         int32_t* __restrict__ overflowed, int32_t* __restrict__ chunk_count,
                                                         int32_t* __restrict__ total) {
    __shared__ __attribute__((aligned(16))) float slab[4][64 * slab_ld(32)];
    __shared__ int32_t s_cnt[256];
    const int q = blockIdx.y, part = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int a_lo = ans_off[q], a_hi = ans_off[q + 1];
    const int n = count[q];
    if (a_lo >= a_hi) return;                       // uniform
    if (part == 0) {                                // what count_sure has counted
        for (int a = a_lo + t; a < a_hi; a += 256) {
            const int32_t c = chunk_count[a];
            if (n <= room && c) atomicAdd(&total[a], c);
            chunk_count[a] = 0;
        }
        if (n > room && t == 0) *overflowed = 1;
    }
    if (n > room || part * 64 >= n) return;
    const int r_lo = root_off[q], r_hi = root_off[q + 1];
    const float step = grid[0];
    for (int a0 = a_lo; a0 < a_hi; a0 += 256) {      // (more than 256 answers: the open entities are computed again)
        const int na = min(256, a_hi - a0);
        s_cnt[t] = 0;
        __syncthreads();
        for (int at = (wave * OPEN_PARTS + part) * 64; at < n; at += 256 * OPEN_PARTS) {
            const bool live = at + lane < n;
            const int32_t e = live ? list[(size_t)q * room + at + lane] : 0;
            int32_t sl = 0;
            for (int p = 0; p < parts; ++p) sl += slack[(size_t)p * lde + e];
            float vhi = INFINITY;
            for (int r = r_lo; r < r_hi; ++r)
                vhi = fminf(vhi, bounds_of(sums[(size_t)r * ld + e], sl, step, base[r], base[ldb + r], rounding).hi);
            const float v = exact_distance<B16, 32, 2>(act, row_ids, r_lo, r_hi, E, E16, e, d, slab[wave]);
            for (int a = 0; a < na; ++a) {
                const float limit = thr[a0 + a];
                const int c = __popcll(__ballot(live && v < limit && !(vhi < limit)));
                if (lane == 0 && c) atomicAdd(&s_cnt[a], c);
            }
        }
        __syncthreads();
        if (t < na && s_cnt[t]) atomicAdd(&total[a0 + t], s_cnt[t]);
        __syncthreads();
    }
}

}  // namespace

size_t rank_found_bytes(int ldy, int lde) { return (size_t)(ldy / 128) * (lde / 128) * FOUND * sizeof(uint32_t); }

int rank_filter_words(int d, int bits) { return ((d / 4) * (bits / 8) + 3) / 4 * 4; }

hipError_t launch_rank_grid(const RankFilter& f, const float* E, const uint16_t* E16, int64_t row_step, int n_rows, hipStream_t s) {
    if (n_rows <= 0 || (f.bits != 8 && f.bits != 16) || (f.d & 3) || f.d > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sample_range_kernel, dim3((f.d + 63) / 64, SAMPLE_SLABS), dim3(256), 0, s, E, E16, row_step, n_rows, f.d, f.part,
                       f.found, f.bits == 8 ? f.ldy * (f.lde / 128) : 0);
    hipLaunchKernelGGL(make_grid_kernel, dim3(1), dim3(1024), 0, s, (const float*)f.part, f.d, 1 << f.bits, f.lo, f.grid,
                       f.count, f.n_counters);
    return hipGetLastError();
}

hipError_t launch_quantise(const RankFilter& f, const RankRows* rows, const float* E, const uint16_t* E16, int n_ent, hipStream_t s) {
    QuantiseArgs g{};
    g.lo = f.lo; g.grid = f.grid; g.d = f.d; g.words = f.words; g.ldy = f.ldy; g.lde = f.lde;
    if (rows && rows->n > 0) {
        g.act = rows->act; g.row_ids = rows->ids; g.n_rows = rows->n; g.root_off = rows->root_off; g.n_queries = rows->n_queries;
        g.Yq = f.Yq; g.base = f.base; g.row_q = f.row_q;
        g.row_blocks = (f.ldy + 4 * QUANTISE_ROWS - 1) / (4 * QUANTISE_ROWS);      // (padding rows of the last tile are copies of the last row)
    }
    g.E = E; g.E16 = E16; g.n_ent = n_ent; g.Eq = f.Eq; g.slack = f.slack;
    // 64 rows a workgroup, or 16 where these would be fewer than two a compute unit (12 952 rows of 400 coordinates: 20 and 9.6 us)
    const bool few = n_ent < 32768;
    const dim3 grid(g.row_blocks + (n_ent + 127) / 128 * (few ? 8 : 2)), block(256);
    if (grid.x == 0) return hipSuccess;
    if (f.bits == 8) {
        if (few) hipLaunchKernelGGL((quantise_kernel<8, 4>), grid, block, 0, s, g);
        else hipLaunchKernelGGL((quantise_kernel<8, 16>), grid, block, 0, s, g);
    } else {
        if (few) hipLaunchKernelGGL((quantise_kernel<16, 4>), grid, block, 0, s, g);
        else hipLaunchKernelGGL((quantise_kernel<16, 16>), grid, block, 0, s, g);
    }
    return hipGetLastError();
}

hipError_t launch_near_tile(const RankFilter& f, int n_rows, int n_ent, const float* best, int k, hipStream_t s) {
    if (n_rows <= 0 || n_ent <= 0) return hipSuccess;
    const NearArgs g{f.Yq, f.Eq, f.base, f.grid, best, f.row_q, f.slack, f.found, f.found_pair,
                     f.ldy, f.lde, n_rows, n_ent, f.words, k, f.parts, rounding_of(f.d)};
    hipLaunchKernelGGL(near_tile_kernel, dim3((n_ent + 127) / 128, (n_rows + 127) / 128), dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_near_merge(const RankFilter& f, int piece, const float* act, const int32_t* row_ids, const int32_t* root_off,
                             int n_queries, const float* E, const uint16_t* E16, int ent_base, int n_ent, int k, float* out_dist,
                             int32_t* out_ids, hipStream_t s) {
    if (n_queries <= 0 || n_ent <= 0) return hipSuccess;
    if (!f.gave_up) return hipErrorInvalidValue;
    const MergeArgs g{act, E, f.base, f.grid, E16, row_ids, root_off, f.slack, f.found, f.found_pair, f.count,
                      f.overflowed + piece, out_dist, out_ids, (n_ent + 127) / 128, ent_base, f.d, k, f.room, f.ldy, f.lde, f.parts, rounding_of(f.d), f.gave_up};
    const bool wide = n_queries <= MERGE_WIDE_TO;
    const dim3 grid(n_queries), block(wide ? 256 : 128);
    if (E16 && wide) hipLaunchKernelGGL((near_merge_kernel<true, 256>), grid, block, 0, s, g);
    else if (E16) hipLaunchKernelGGL((near_merge_kernel<true, 128>), grid, block, 0, s, g);
    else if (wide) hipLaunchKernelGGL((near_merge_kernel<false, 256>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((near_merge_kernel<false, 128>), grid, block, 0, s, g);
    return hipGetLastError();
}

hipError_t launch_pick(const RankFilter& f, const uint32_t* sums, int ld, const float* act, const int32_t* row_ids, const int32_t* root_off,
                       int n_queries, const float* E, const uint16_t* E16, int n_ent, int k, float* out_dist, int32_t* out_ids, hipStream_t s) {
    if (n_queries <= 0 || n_ent <= 0) return hipSuccess;
    if (k < 1 || k > NGDB_MAX_TOPK || f.parts != 1 || !f.gave_up || (ld & 3) || n_ent > RANK_PIECES * RANK_PIECE) return hipErrorInvalidValue;      // (NGDB_MAX_BRANCH rows a query: the planner's)
    const PickArgs g{act, E, f.base, f.grid, E16, row_ids, root_off, f.slack, sums, reinterpret_cast<const int2*>(f.found_pair), f.count, f.overflowed, out_dist, out_ids,
                     ld, n_ent, f.d, k, f.room, f.ldy, rounding_of(f.d), f.gave_up};
    if (E16) hipLaunchKernelGGL(pick_kernel<true>, dim3(n_queries), dim3(PICK_T), 0, s, g);
    else hipLaunchKernelGGL(pick_kernel<false>, dim3(n_queries), dim3(PICK_T), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_sum_tile(const RankFilter& f, int n_rows, int n_ent, uint32_t* sums, int ld, hipStream_t s) {
    if (n_rows <= 0 || n_ent <= 0) return hipSuccess;
    // Tiles of 64 rows take more time for the same pairs, 4 where one of 128 takes 7, but go round 256 compute units with less left over:
    // what the busiest one has, either way.  (For 16-bit sums too, always 128, always 64 and so, filtered ranks of 8 answers: 15 000 x 584 x 400
    // 299, 287 and 287 us, 15 000 x 114 182, 169, 171, 63 000 x 1170 883, 893, 884, 200 000 x 584 1554, 1525, 1541, 5000 x 1170 x 512 368, 351, 351.)
    const int tiles_e = (n_ent + 127) / 128;
    auto turns = [&](int tr, int cost) {
        const int rest = n_rows % tr, quarters = n_rows / tr * (tr / 32) + (rest == 0 ? 0 : std::min(tr, tail_rows(rest, 0)) / 32);
        return (int)(((int64_t)tiles_e * quarters / (tr / 32) + 255) / 256) * cost;
    };
    const int tile_rows = turns(64, 4) < turns(128, 7) ? 64 : 128;
    const dim3 grid(tiles_e, (n_rows + tile_rows - 1) / tile_rows), block(256);
    if (f.bits == 8)
        hipLaunchKernelGGL(sum_tile_kernel<8>, grid, block, 0, s, (const uint32_t*)f.Yq, f.ldy, n_rows, (const uint32_t*)f.Eq, f.lde, n_ent,
                           f.words, sums, ld, tile_rows, (const int32_t*)f.slack, reinterpret_cast<int2*>(f.found_pair));
    else
        hipLaunchKernelGGL(sum_tile_kernel<16>, grid, block, 0, s, (const uint32_t*)f.Yq, f.ldy, n_rows, (const uint32_t*)f.Eq, f.lde, n_ent,
                           f.words, sums, ld, tile_rows, (const int32_t*)f.slack, reinterpret_cast<int2*>(f.found_pair));
    return hipGetLastError();
}

hipError_t launch_answer_distance(const float* act, const float* off, float alpha, const int32_t* row_ids, const int32_t* root_off,
                                  const int32_t* ans_off, int n_queries, const int32_t* ans, int a0, int cnt, const float* E,
                                  const uint16_t* E16, int d, const int32_t* gave_up, float* thr, int32_t* counters, int n_ans, hipStream_t s) {
    if (cnt <= 0) return hipSuccess;
    if (!gave_up) return hipErrorInvalidValue;
    const dim3 grid((cnt + 63) / 64), block(64);
    if (off)
        hipLaunchKernelGGL((answer_distance_kernel<true>), grid, block, 0, s, act, off, alpha, row_ids, root_off, ans_off, n_queries, ans,
                           a0, cnt, E, E16, d, gave_up, thr, counters, n_ans);
    else
        hipLaunchKernelGGL((answer_distance_kernel<false>), grid, block, 0, s, act, off, alpha, row_ids, root_off, ans_off, n_queries, ans,
                           a0, cnt, E, E16, d, gave_up, thr, counters, n_ans);
    return hipGetLastError();
}

hipError_t launch_count_sure(const RankFilter& f, const uint32_t* sums, int ld, const int32_t* root_off, const int32_t* ans_off,
                             const float* thr, int n_queries, int n_ent, int32_t* chunk_count, hipStream_t s) {
    if (n_queries <= 0 || n_ent <= 0) return hipSuccess;
    if (n_queries > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(count_sure_kernel, dim3(std::min((n_ent + SLAB - 1) / SLAB, std::max(1, 4096 / n_queries)), n_queries), dim3(256), 0, s, sums, ld,
                       (const int32_t*)f.slack, f.parts, f.lde, (const float*)f.base, f.ldy, (const float*)f.grid, root_off, ans_off, thr, n_ent,
                       rounding_of(f.d), chunk_count, f.list, f.count, f.room);
    return hipGetLastError();
}

hipError_t launch_count_open(const RankFilter& f, int chunk, const uint32_t* sums, int ld, const float* act, const int32_t* row_ids, const int32_t* root_off,
                             const int32_t* ans_off, const float* thr, int n_queries, const float* E, const uint16_t* E16,
                             int32_t* chunk_count, int32_t* total, hipStream_t s) {
    if (n_queries <= 0) return hipSuccess;
    if (n_queries > 65535) return hipErrorInvalidValue;
#define NGDB_OPEN(B16)                                                                                                       \
    hipLaunchKernelGGL((count_open_kernel<B16>), dim3(OPEN_PARTS, n_queries), dim3(256), 0, s, act, row_ids, root_off, ans_off, thr, E, E16, f.d, \
                       sums, ld, (const int32_t*)f.slack, f.parts, f.lde, (const float*)f.base, f.ldy, (const float*)f.grid, rounding_of(f.d),   \
                       (const int32_t*)f.list, (const int32_t*)f.count, f.room, f.overflowed + chunk, chunk_count, total)
    if (E16) NGDB_OPEN(true);
    else NGDB_OPEN(false);
#undef NGDB_OPEN
    return hipGetLastError();
}

}  // namespace ngdb
