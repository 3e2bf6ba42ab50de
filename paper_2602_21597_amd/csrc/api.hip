// C boundary and step orchestration: enqueues, per depth of the batch's operator
// DAG, one grouped launch sequence per operator type (Sec. 4.1 "Batched
// Execution"; Sec. 4.3 cardinality classes), then scoring, the reversed
// frontiers (Alg. 1: gradient nodes are scheduled like forward ones), the
// segmented table updates and Adam (Alg. 1, OptimizerStep).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "common.h"
#include "planner.h"

using namespace ngdb;

static __device__ __align__(256) unsigned char scratch[(size_t)NGDB_NOALLOC_SCRATCH_MIB << 20];

namespace {

struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
};

struct Segment {   // the groups of one (level, type): contiguous MLP rows and references
    int type = 0;
    int rows = 0;          // MLP rows (members for PROJ/NEG, members*inputs for INTER)
    int mlp_base = 0;
    int ref_off = 0;
    int rel_off = -1;
    int out_base = 0;      // PROJ/NEG: first output slot
    int g_lo = 0, g_hi = 0;  // group range (INTER: one combine launch per group)
};

constexpr int T_PROJ = 0, T_INTER = 1, T_NEG = 2;
inline int type_index(int op) { return op == NGDB_OP_PROJ ? T_PROJ : (op == NGDB_OP_INTER ? T_INTER : T_NEG); }

}  // namespace

// Device copy of a plan's arrays plus its pinned staging buffer; recycled through
// the context so that planning allocates nothing in steady state.
struct PlanBlob {
    int32_t* dev = nullptr;
    int32_t* pinned = nullptr;
    size_t cap = 0;               // in int32 elements
    hipEvent_t last_use = nullptr;  // recorded after every step that read the blob
};

struct ngdb_plan_s {
    HostPlan hp;
    ngdb_ctx_t* owner = nullptr;
    PlanBlob blob;
    int32_t* d_blob = nullptr;
    size_t blob_bytes = 0;
    mutable bool uploaded = false;   // else the first call that uses the plan copies it on its own stream
    // device views into the blob
    const int32_t *d_in_ref = nullptr, *d_in_gslot = nullptr, *d_rel = nullptr, *d_root_off = nullptr,
                  *d_root_slot = nullptr, *d_pos = nullptr, *d_ekeys_head = nullptr, *d_r_uniq = nullptr,
                  *d_r_seg_off = nullptr, *d_r_src = nullptr, *d_r_rec = nullptr, *d_n_r_uniq = nullptr;
    // forward-only passes with reclaimed outputs: references, output rows and root rows in storage rows
    const int32_t *d_f_in_ref = nullptr, *d_f_row = nullptr, *d_f_root = nullptr;
    std::vector<std::vector<Segment>> levels;   // levels[l] for l = 1..n_levels (index 0 unused)
    int32_t n_entities = 0;
};

// Looks at a depth's count before a wait gives up: seconds, which no working card comes near.
constexpr int CHAIN_POLLS = 1 << 22;

struct ngdb_ctx_s {
    ngdb_config cfg{};
    ngdb_params prm{};
    bool bound = false;
    bool presized = false;          // workspace allocated once from declared maxima: steps must not grow it
    int64_t n_alloc = 0;            // device / pinned allocations made so far
    int64_t step = 0;
    std::string err;
    hipStream_t side[1]{};          // library stream (num_streams > 1)
    hipEvent_t ev_fork = nullptr;
    hipEvent_t ev_join = nullptr;
    int n_side = 0;
    // workspace
    DevBuf act, dact, Z[3], H[3], dH[3], Att, dAtt, Dx;
    DevBuf score, coef, win, mask, loss_terms, rec_coef, rec_row;
    DevBuf keys_a, keys_b, vals_a, vals_b, hist, scan_tmp, uniq, seg_off, n_uniq;
    DevBuf rank_dist;   // distances of one entity chunk in the all-entity ranking
    DevBuf rank_thr, rank_count;   // filtered ranks: distance of every listed answer, entities closer than it (total, chunk)
    DevBuf rank_filter;            // integer rows, bounds and lists of the filtered passes
    DevBuf gW;          // gradients of the 12 MLP tensors, packed
    // The six weight matrices of the vector family's MLPs as ready-made B operands of the contraction
    // kernel (bf16 pieces in MFMA lane order), in both orientations: rebuilt at the start of every
    // forward pass, so they are never older than the weights the pass reads.
    DevBuf w_pieces;
    bool chained = false;          // the pass under way has a launch of several depths
    bool trains = false;           // ... has a backward half
    bool fuses_beside = false;     // ... fuses many rows beside its forward half, which takes all compute units that are free
    bool rows_chained = false;     // ... its first, which is all of its forward pass (rows_chain)
    bool plan_rides = false;       // the plan comes to the device with the launch of all depths of the forward pass, which reads it where it is
    SmallIndex index_waits{};      // a small gradient index that a launch of the forward pass may take along (n: 0 without one)
    DevBuf sync;        // of the launches of several depths (LevelSync), in device memory
    int32_t* gave_up = nullptr;    // and in pinned host memory: one of them has given up waiting, for good
    int chain_polls = CHAIN_POLLS;       // tests: see ngdb_debug_chain_polls
    int chain_patience = TILE_PATIENCE; // tests: see ngdb_debug_chain_patience
    unsigned long long chain_launch = 0; // number of the last launch whose tiles are taken
    bool chain_odd = false;        // which of two sets of bits the next launch of a few rows finds cleared
    int64_t chain_count[3]{};            // tests: see ngdb_debug_chain_launches
    bool captured = false;         // the pass under way is recorded into a graph: replays have no launch numbers of their own
    const uint16_t* wp[3][4]{};     // per type: Wa forward, Wb forward, Wb backward (dH = dY Wb), Wa backward (dZ = dH Wa)
    bool have_pieces = false;
    int64_t rank_filter_from = -1;       // tests: see ngdb_debug_rank_filter_from
    bool rank_by_chunks = false;         // tests: see ngdb_debug_rank_by_chunks
    const int32_t* rank_overflowed = nullptr;    // the last ranking's marks per piece of a chunk (null: no filter)
    int rank_chunks = 0;
    int near_most = INT32_MAX;     // entities of a filtered chunk for which there was memory, and the memory that was free then
    size_t near_free = 0;
    size_t held = 0, held_limit = SIZE_MAX;      // bytes of the buffers below; tests: see ngdb_debug_device_limit
    // The hidden activations of one depth (forward) or their gradients (backward) once more as bf16
    // pieces in tile order: written by the first launch of a layer pair, read as A operand by the
    // second, then free again.  Only steps whose launches use the small tile get that far.
    DevBuf h_pieces;
    DevBuf gE, gR;      // compact table gradients (ngdb_forward_backward only)
    // text-feature fusion: bf16 copy of Wp, fused rows of the touched entities, position of every
    // contribution's entity in that list, operator references redirected to it, bf16 row gradients,
    // split-wise partial sums and the gradient of Wp, fused rows of one ranking chunk
    DevBuf Wb, Ef, Ea, inv, refs_sem, g_bf16, wp_partial, gWp, rank_ef;
    DevBuf later;       // touched entity rows that wait for the backward pass (positions in uniq)
    // box family: offsets and their gradients by slot (act / dact hold the centres), per-input
    // outputs of the offset MLP with their gradients, direct gradient of the inputs' offsets,
    // compact gradient of Ro.  The offset MLP (V1 c1 V2 c2) uses the Z/H/dH buffers of index T_NEG.
    DevBuf off, doff, Gate, dGate, DxO, gRo;
    DevBuf Eb;          // bf16 copy of E for the scoring and ranking passes (score_bf16)
    size_t gw_off[13]{};
    hipStream_t upload = nullptr;        // plan uploads, independent of the compute streams
    std::vector<PlanBlob> blob_pool;
    std::vector<ngdb_plan_t*> live_plans;   // plans that hold a device buffer of this context
    std::mutex mu;                       // guards blob_pool, live_plans and err: planning may run on a second host thread
    // kernel timing
    uint32_t timing_mask = 0;
    struct Bracket { int cls; hipEvent_t a, b; int route; double flop; };
    std::vector<Bracket> brackets;
    std::vector<hipEvent_t> spare_events;
    ngdb_timing timing{};
    // results of the last step
    bool have_grads = false;
    ngdb_grad_view gv{};
};

namespace {

thread_local std::string g_create_err;

// Scratch of ngdb_score_noalloc: device memory that exists from the moment the library's code
// object is loaded on a GPU until the process ends, one copy per GPU.  In host code the array's
// name only stands for the symbol; its device address on a GPU is asked for once per device
// (noalloc_scratch) and only that address is ever passed to kernels.
constexpr size_t NOALLOC_BYTES = (size_t)NGDB_NOALLOC_SCRATCH_MIB << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

int fail(ngdb_ctx_t* c, int code, const std::string& msg) {
    if (c) {
        std::lock_guard<std::mutex> lk(c->mu);
        c->err = msg;
    }
    return code;
}

#define HIPCHK(c, expr)                                                                        \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail((c), e_ == hipErrorOutOfMemory ? NGDB_ERR_OOM : NGDB_ERR_HIP,          \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                    \
    } while (0)

hipEvent_t take_event(ngdb_ctx_t* c) {
    if (!c->spare_events.empty()) {
        hipEvent_t e = c->spare_events.back();
        c->spare_events.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    return hipEventCreate(&e) == hipSuccess ? e : nullptr;
}

// Brackets one launch (sequence) with an event pair when its class is being timed.
struct Timed {
    ngdb_ctx_t* c;
    hipStream_t s;
    hipEvent_t b = nullptr;
    Timed(ngdb_ctx_t* ctx, int cls, hipStream_t stream) : c(ctx), s(stream) {
        if (!(c->timing_mask >> cls & 1u)) return;
        hipEvent_t a = take_event(c);
        b = take_event(c);
        if (!a || !b) { b = nullptr; return; }
        (void)hipEventRecord(a, s);
        c->brackets.push_back({cls, a, b, -1, 0.0});
    }
    // a contraction launch: the instructions it ran on and its algorithmic work
    void work(int route, double flop) {
        if (!b) return;
        c->brackets.back().route = route == GEMM_SPLIT ? 1 : 0;
        c->brackets.back().flop = flop;
    }
    ~Timed() { if (b) (void)hipEventRecord(b, s); }
};

// One grouped contraction launch, bracketed as class `cls`.
int gemm_timed(ngdb_ctx_t* c, int cls, const GemmArgs* g, int n, hipStream_t s, bool* emitted = nullptr);

void release(ngdb_ctx_t* c, DevBuf& b) {
    if (b.p) (void)hipFree(b.p);
    c->held -= b.cap;
    b.p = nullptr;
    b.cap = 0;
}

// The buffers that the rankings make anew whenever they need them (the device has to be idle).
bool release_rank_buffers(ngdb_ctx_t* c) {
    const bool any = c->rank_dist.p || c->rank_ef.p || c->rank_filter.p;
    release(c, c->rank_dist);
    release(c, c->rank_ef);
    release(c, c->rank_filter);
    c->rank_overflowed = nullptr;
    return any;
}

hipError_t device_alloc(ngdb_ctx_t* c, DevBuf& b, size_t bytes) {
    const hipError_t e = c->held + bytes > c->held_limit ? hipErrorOutOfMemory : hipMalloc(&b.p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();             // (the next launch is not to report it)
        b.p = nullptr;
        return e;
    }
    ++c->n_alloc;
    c->held += b.cap = bytes;
    return e;
}

// What a buffer is for: every call; evaluation only, i.e. the ranking calls or ngdb_forward_backward (allocated on first use also
// under declared maxima); or one that release_rank_buffers gives back.
enum class Use { Any, Evaluation, Ranking };
int ensure(ngdb_ctx_t* c, DevBuf& b, size_t bytes, Use use = Use::Any) {
    if (bytes <= b.cap) return NGDB_OK;
    if (c->presized && use == Use::Any)
        return fail(c, NGDB_ERR_ARG, "the batch needs more workspace than the maxima declared at ngdb_create allow "
                                     "(b_max_queries, k_max, max_nodes_per_query)");
    // growing: nothing may still be using the old allocation
    HIPCHK(c, hipDeviceSynchronize());
    release(c, b);
    const size_t want = bytes + bytes / 4 + 256;
    hipError_t e = device_alloc(c, b, want);
    // (what an earlier ranking has left behind stands in no other call's way; a ranking itself asks for less, see rank_buffers)
    if (e == hipErrorOutOfMemory && use != Use::Ranking && release_rank_buffers(c)) e = device_alloc(c, b, want);
    if (e == hipErrorOutOfMemory && use == Use::Ranking) return NGDB_ERR_OOM;      // (no failure of the call yet, see no_rank_memory)
    HIPCHK(c, e);
    return NGDB_OK;
}

template <class T>
T* ptr(const DevBuf& b) { return static_cast<T*>(b.p); }

// Words of c->sync: LevelSync's counts and the mark of a launch that gave up, the count of tiles that another workgroup computed, then what rows_chain_kernel and
// tile_chain_kernel wait by: bits twice, whose tiles are taken, counts.
constexpr int HELPED_AT = 32, CHAIN_AT = 64, TAKEN_AT = CHAIN_AT + 2 * 2 * CHAIN_SYNC, TILE_AT = TAKEN_AT + 2 * TILE_WORDS, SYNC_WORDS = TILE_AT + TILE_SYNC;
static_assert(LEVEL_SYNC + 1 <= HELPED_AT && CHAIN_AT % 32 == 0 && TAKEN_AT % 32 == 0 && SYNC_WORDS % 32 == 0, "lines of their own");
// ... and behind them the rows of rows_chain_kernel, none of which is used twice: outputs and inputs of intersections, together no more than its words, then hidden
// rows.  They are there from the start, so that no pass has to make the buffers grow that a captured graph may go on using.
bool rows_chain_model(const ngdb_ctx_t* c) {
    return c->cfg.family == NGDB_FAMILY_VEC && c->cfg.d_sem == 0 && std::max(c->cfg.d, c->cfg.h) <= CHAIN_WIDTH && !level_fits(c->cfg.d, c->cfg.h, true);
}
size_t rows_chain_bytes(const ngdb_ctx_t* c) { return rows_chain_model(c) ? (size_t)CHAIN_WORDS * (c->cfg.d + c->cfg.h) * sizeof(float) : 0; }
float* rows_chain_act(const ngdb_ctx_t* c) { return ptr<float>(c->sync) + SYNC_WORDS; }
LevelSync level_sync(const ngdb_ctx_t* c) {
    LevelSync y;
    if (c->chain_polls < 0) return y;            // (a launch per depth)
    y.counts = ptr<int32_t>(c->sync); y.gave_up = y.counts + LEVEL_SYNC; y.host_gave_up = c->gave_up; y.polls = c->chain_polls;
    return y;
}
const int32_t* gave_up_mark(const ngdb_ctx_t* c) { return ptr<int32_t>(c->sync) + LEVEL_SYNC; }
TileHelp tile_help(const ngdb_ctx_t* c) {
    TileHelp t;
    t.helped = ptr<int32_t>(c->sync) + HELPED_AT; t.patience = c->chain_patience;
    return t;
}
// A launch of an earlier call gave up waiting for a depth: nothing is computed on this context any more.
int check_waits(ngdb_ctx_t* c) {
    if (!__atomic_load_n(c->gave_up, __ATOMIC_RELAXED)) return NGDB_OK;
    return fail(c, NGDB_ERR_HIP, "a launch gave up waiting for the operators of a depth: results of that call and of those behind it are not valid "
                                 "(a training step leaves parameters as they were, but for entity rows that were updated beside its backward pass); "
                                 "the context computes nothing any more");
}

int gemm_timed(ngdb_ctx_t* c, int cls, const GemmArgs* g, int n, hipStream_t s, bool* emitted) {
    Timed tm(c, cls, s);
    int route = GEMM_FP32;
    HIPCHK(c, launch_gemm_group(g, n, s, &route, emitted));
    double flop = 0.0;
    for (int i = 0; i < n; ++i)
        if (g[i].M > 0 && g[i].N > 0) flop += 2.0 * g[i].M * g[i].N * g[i].K;
    tm.work(route, flop);
    return NGDB_OK;
}

struct MlpRefs {
    const float *Wa, *ba, *Wb, *bb;
};
MlpRefs mlp_of(const ngdb_params& p, int t) {
    if (t == T_PROJ) return {p.W1.p, p.b1.p, p.W2.p, p.b2.p};
    if (t == T_NEG) return {p.V1.p, p.c1.p, p.V2.p, p.c2.p};
    return {p.U1.p, p.u1.p, p.U2.p, p.u2.p};
}
// order of ngdb_grad_view::g_mlp: W1 b1 W2 b2 | V1 c1 V2 c2 | U1 u1 U2 u2
int gslot_of(int t) { return t == T_PROJ ? 0 : (t == T_NEG ? 4 : 8); }

struct FwdBytes;
FwdBytes forward_bytes(const ngdb_ctx_t* c, const ngdb_plan_t* pl, bool reclaim);
int size_forward_only(ngdb_ctx_t* c, const ngdb_plan_t* pl, int64_t n_tail);
// Whether the weights are split once for a pass, and hidden rows handed on as pieces: with vectors always; the two MLPs of the box family from as many inputs of intersections on as
// some 800 queries have (a step of 4096 boxes at d = 400, h = 800 619 us without and 528 with, of 1024 246 and 226, scoring 1024 108 and 102; a step of 512 takes the host as
// long as the device, with and without; its first pass at d = 300, h = 500 takes 530 to 580 us, with room for both, 18 MB in two allocations, up to 1930).
constexpr int BOX_PIECES_FROM = 768;
bool all_split(const ngdb_ctx_t* c, const HostPlan& hp) { return c->cfg.family == NGDB_FAMILY_VEC || hp.n_int_rows >= BOX_PIECES_FROM; }
// ... or the weights alone, for a launch of several layers (tile_chain_kernel) that the pass may have (first passes 515 to 630 us).
bool weights_split(const ngdb_ctx_t* c, const HostPlan& hp) {
    return all_split(c, hp) || (hp.n_int_rows > 0 && !level_fits(c->cfg.d, c->cfg.h, true) && tile_chain_most(c->cfg.d, c->cfg.h, true, true) > 0);
}
// bytes of the split weights: per MLP two operands of ceil(h/32) x ceil(d/16) tiles and two of ceil(d/32) x ceil(h/16)
size_t weight_pieces_bytes(const ngdb_ctx_t* c, const HostPlan& hp) {
    if (!weights_split(c, hp)) return 0;
    return (c->cfg.family == NGDB_FAMILY_BOX ? 2 : 3) * 2 * (pieces_elems(c->cfg.h, c->cfg.d) + pieces_elems(c->cfg.d, c->cfg.h)) * sizeof(uint16_t);
}
// Room for the hidden rows of one depth as pieces: blocks of 32 rows per segment, k-tiles in pairs.
constexpr size_t H_PIECES_MAX_ROWS = 2048;      // launches over more rows do not write pieces
int h_pieces_kt(const ngdb_ctx_t* c) { return 2 * ((c->cfg.h + 31) / 32); }
size_t h_pieces_bytes(const ngdb_ctx_t* c, const HostPlan& hp) {
    if (!all_split(c, hp)) return 0;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;       // centres and offsets of the intersections' inputs
    const size_t rows = std::min<size_t>(box ? 2 * (size_t)hp.n_int_rows : (size_t)hp.n_proj + hp.n_int_rows + hp.n_neg, H_PIECES_MAX_ROWS);
    return (rows / 32 + 3) * h_pieces_kt(c) * 1536 * sizeof(uint16_t);
}
// Hands the segments of one depth their places in h_pieces (as output of `first`, as A operand of
// `second` once the launch of `first` reports that it wrote them).
struct HiddenPieces {
    uint16_t* at[3] = {};
    int kt = 0;
};
HiddenPieces place_hidden_pieces(ngdb_ctx_t* c, GemmArgs* first, int n) {
    HiddenPieces hpc;
    if (!c->have_pieces || !c->h_pieces.p || n > 3) return hpc;
    hpc.kt = h_pieces_kt(c);
    const size_t tile_row = (size_t)hpc.kt * 1536;
    size_t blocks = 0;
    for (int i = 0; i < n; ++i) blocks += (size_t)(first[i].M + 31) / 32;
    if (blocks * tile_row * sizeof(uint16_t) > c->h_pieces.cap) return hpc;
    uint16_t* at = ptr<uint16_t>(c->h_pieces);
    for (int i = 0; i < n; ++i) {
        hpc.at[i] = first[i].c_pieces = at;
        first[i].c_kt = hpc.kt;
        at += (size_t)((first[i].M + 31) / 32) * tile_row;
    }
    return hpc;
}
void take_hidden_pieces(const HiddenPieces& hpc, GemmArgs* second, int n) {
    for (int i = 0; i < n; ++i) { second[i].a_pieces = hpc.at[i]; second[i].a_kt = hpc.kt; }
}

double level_flop(const ngdb_ctx_t* c, const std::vector<Segment>& segs) {
    double rows = 0.0;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    for (const Segment& sg : segs) rows += box ? (sg.type == T_INTER ? 2.0 * sg.rows : 0.0) : sg.rows;
    return 4.0 * c->cfg.d * c->cfg.h * rows;
}

// The operators of one depth as problems of one launch (level.hip), where the MLPs are small and the depth does not have
// very many rows. 
bool level_problems(const ngdb_ctx_t* c, const ngdb_plan_t* pl, const std::vector<Segment>& segs, LevelArgs* a) {
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    if (!level_fits(c->cfg.d, c->cfg.h, true)) return false;
    const HostPlan& hp = pl->hp;
    *a = LevelArgs{};
    a->d = c->cfg.d; a->h = c->cfg.h;
    for (const Segment& sg : segs) {
        if (box && sg.type != T_INTER) {
            if (sg.type != T_PROJ || !level_add(*a, sg.type, LEVEL_PROJECTION, sg.rows, 1, sg.ref_off, sg.rel_off, 0, sg.out_base)) return false;
            continue;
        }
        if (sg.type != T_INTER) {
            if (!level_add(*a, sg.type, 0, sg.rows, 1, sg.ref_off, sg.rel_off, sg.mlp_base, sg.out_base)) return false;
            continue;
        }
        for (int g = sg.g_lo; g < sg.g_hi; ++g)
            if (!level_add(*a, sg.type, 1, hp.g_n[g], hp.g_nin[g], sg.ref_off + hp.g_mlp_base[g] - sg.mlp_base, -1, hp.g_mlp_base[g], hp.g_out_base[g])) return false;
        for (int g = sg.g_lo; box && g < sg.g_hi; ++g)      // the offsets of the same inputs through the second MLP
            if (!level_add(*a, T_NEG, LEVEL_GATE, hp.g_n[g], hp.g_nin[g], sg.ref_off + hp.g_mlp_base[g] - sg.mlp_base, -1, hp.g_mlp_base[g], hp.g_out_base[g])) return false;
    }
    if (!level_fits(c->cfg.d, c->cfg.h, box) && a->t.tile_start[a->t.count] > LEVEL_FEW) return false;
    if (box) {
        a->act = ptr<float>(c->act); a->off = ptr<float>(c->off); a->dact = ptr<float>(c->dact); a->doff = ptr<float>(c->doff);
        a->Att = ptr<float>(c->Att); a->Gate = ptr<float>(c->Gate); a->dAtt = ptr<float>(c->dAtt); a->dGate = ptr<float>(c->dGate);
        a->refs = pl->d_in_ref; a->rel = pl->d_rel; a->dst_row = pl->d_in_gslot;
        a->E = c->prm.E.p; a->R = c->prm.R.p; a->Ro = c->prm.Ro.p;
        a->keep = true;
    }
    for (int t = 0; t < 3; ++t) {
        const MlpRefs W = mlp_of(c->prm, t);
        a->mlp[t] = LevelMlp{W.Wa, W.ba, W.Wb, W.bb, ptr<float>(c->Z[t]), ptr<float>(c->H[t]), ptr<float>(c->dH[t])};
    }
    return true;
}

// (in a stream capture nothing has run yet: whoever uses the plan outside of it copies again)
void plan_uploaded(const ngdb_ctx_t* c, const ngdb_plan_t* pl) { pl->uploaded = pl->uploaded || !c->captured; }
PlanCopy plan_copy(const ngdb_plan_t* pl) {
    return PlanCopy{reinterpret_cast<const float4*>(pl->blob.pinned), reinterpret_cast<float4*>(pl->blob.dev), (int)(pl->blob_bytes / 16)};
}

// All depths of a direction in one launch, where each would take one and they are few enough.  fill() adds to a depth what the pass knows.
template <class Fill>
bool enqueue_levels(ngdb_ctx_t* c, const ngdb_plan_t* pl, bool backward, Fill fill, const LevelSync& sync, hipStream_t s, int* rc) {
    const int n = pl->hp.n_levels;
    if (n < 2 || n > LEVEL_CHAIN || !sync.counts) return false;
    LevelArgs la[LEVEL_CHAIN];
    double flop = 0.0;
    for (int i = 0; i < n; ++i) {
        const std::vector<Segment>& segs = pl->levels[backward ? n - i : i + 1];
        if (!level_problems(c, pl, segs, &la[i])) return false;
        fill(la[i]);
        flop += level_flop(c, segs);
    }
    if (!levels_chain(la, n)) return false;
    PlanCopy copy;
    if (!backward && c->plan_rides) {
        copy = plan_copy(pl);
        auto there = [&](const int32_t*& p) { if (p) p = pl->blob.pinned + (p - pl->d_blob); };
        for (int i = 0; i < n; ++i) {
            there(la[i].refs); there(la[i].rel); there(la[i].out_row);
        }
        if (c->index_waits.n > 0) there(c->index_waits.head);
    }
    auto launch = [&]() -> int {
        Timed tm(c, backward ? NGDB_TK_GEMM_BWD : NGDB_TK_GEMM_FWD, s);
        HIPCHK(c, launch_levels(la, n, backward, sync, backward ? nullptr : &c->index_waits, copy, s));
        if (!backward) c->index_waits.n = 0;
        c->chained = true;
        tm.work(GEMM_FP32, flop);
        if (!copy.n) return NGDB_OK;
        c->plan_rides = false;
        plan_uploaded(c, pl);
        return NGDB_OK;
    };
    *rc = launch();
    return true;
}

// Whether enqueue_levels will take the forward pass.
bool forward_chained(const ngdb_ctx_t* c, const ngdb_plan_t* pl) {
    const int n = pl->hp.n_levels;
    if (n < 2 || n > LEVEL_CHAIN || !level_sync(c).counts) return false;
    LevelArgs la[LEVEL_CHAIN];
    for (int i = 0; i < n; ++i)
        if (!level_problems(c, pl, pl->levels[i + 1], &la[i])) return false;
    return levels_chain(la, n);
}

// Tiles of the largest layer of a depth in a launch of several (tile_chain_kernel).  0: not a depth that such a launch takes.
int depth_tiles(const ngdb_ctx_t* c, const ngdb_plan_t* pl, const std::vector<Segment>& segs, bool backward) {
    const HostPlan& hp = pl->hp;
    const int d = c->cfg.d, h = c->cfg.h;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    // (forward layers of a few rows are summed in another order: such a depth stays with its launches)
    bool few[2] = {!backward, !backward}, any = false;
    int first = 0, second = 0, plain = 0;
    for (const Segment& sg : segs) {
        if (sg.rows <= 0) continue;
        if (box && sg.type == T_PROJ) {                      // (has no MLP)
            plain += tile_chain_plain(sg.rows, d);
            continue;
        }
        any = true;
        few[0] = few[0] && gemm_takes_rows(sg.rows, d);
        few[1] = few[1] && gemm_takes_rows(sg.rows, h);
        const int sides = box ? 2 : 1;
        for (int g = sg.g_lo; sg.type == T_INTER && g < sg.g_hi; ++g) {
            if (hp.g_nin[g] < 2 || hp.g_nin[g] > TILE_CARD) return 0;
            first += sides * tile_chain_tiles(hp.g_n[g] * hp.g_nin[g], 1, h);
            second += sides * tile_chain_tiles(hp.g_n[g], backward ? 1 : hp.g_nin[g], d);
            if (backward) plain += sides * tile_chain_plain(hp.g_n[g], d);
        }
        if (sg.type == T_INTER) continue;
        first += tile_chain_tiles(sg.rows, 1, h);
        second += tile_chain_tiles(sg.rows, 1, d);
    }
    if (any && (few[0] || few[1])) return 0;
    return std::max(std::max(backward ? first : first + plain, second), plain);
}
// The depths that one launch takes: the last that it can take (depths have fewer rows the deeper they are, as a rule) and those before it.  Looked
// for in every pass, also in those of a few queries, which the host bounds: nothing is laid out here.
// CHAIN_LAUNCHES: what it has to take the place of, two launches a depth with MLPs, three with the pooling of boxes, one of their projections.  One depth of vectors
// alone (1p, 17 to 256 queries), whose time in two launches is 24 to 31 us: at 320, 836, 400, 800 and 512, 1024 0.82 to 1.01 times as fast in one, at 208, 416 and 400, 132
// 0.99 to 1.03, at 128, 256 0.88 to 1.04; two depths of boxes' projections (2p, 26 to 34 us) 1.00 to 1.1.  A training step is the faster for one depth already.
struct ChainDepths { int from = 0, to = 0; };
constexpr int CHAIN_LAUNCHES_TRAIN = 2, CHAIN_LAUNCHES = 4;
// Tiles that wait hold the places of those that fuse rows beside them: forward passes beside more than so many contributions keep their launches.  In one launch, steps of
// 64 to 256 queries at 400, 800 with 1024 and 256 features, 288, 224 with 896, 208, 416 with 512 and 128, 256 with 128 were, with 2600 to 11 000 contributions, 0.98 to 1.07
// times as fast, with 20 000 to 42 000 0.96 to 1.01, with 65 000 to 130 000 0.98 to 1.03; and one of 31 000 at 288, 224 343 us against 379.
constexpr int64_t CHAIN_FUSED = 20000;
bool chain_depths(const ngdb_ctx_t* c, const ngdb_plan_t* pl, bool backward, ChainDepths* out) {
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    const int n = pl->hp.n_levels, most = tile_chain_most(c->cfg.d, c->cfg.h, box, c->trains);
    if (most == 0 || c->captured || level_fits(c->cfg.d, c->cfg.h, box) || (!backward && c->fuses_beside)) return false;
    auto takes = [&](int l) {
        const int tiles = depth_tiles(c, pl, pl->levels[l], backward);
        LevelArgs la;
        return tiles > 0 && tiles <= most && !(level_fits(c->cfg.d, c->cfg.h, true) && level_problems(c, pl, pl->levels[l], &la));
    };
    int l = n;
    while (l > 0 && !takes(l)) --l;
    if (l == 0) return false;
    out->to = l;
    while (l > 1 && out->to - l + 1 < LEVEL_CHAIN && takes(l - 1)) --l;
    out->from = l;
    int launches = 0;
    for (; l <= out->to; ++l) {
        bool mlp = !box;
        for (const Segment& sg : pl->levels[l]) mlp = mlp || sg.type == T_INTER;
        launches += !mlp ? 1 : (box ? 3 : 2);
    }
    return launches >= (c->trains ? CHAIN_LAUNCHES_TRAIN : CHAIN_LAUNCHES);
}
// Splits the weights of the MLPs for a pass, for its backward half too if it has one (at d = 400, h = 800 scoring 1024 queries takes 415 us instead of 423 without it).
// Without the buffer (a context
// that never sized a workspace) the contractions split their B operands themselves.
void add_weight_pieces(ngdb_ctx_t* c, const ngdb_plan_t* pl, bool backward, PieceJobs* J) {
    c->have_pieces = false;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    if (!weights_split(c, pl->hp) || c->w_pieces.cap < weight_pieces_bytes(c, pl->hp) || !c->w_pieces.p) return;
    const int d = c->cfg.d, h = c->cfg.h;
    if ((d & 3) || (h & 3)) return;   // the split reads rows as float4
    if (d < 128 && h < 128) return;   // no contraction of these widths takes the split route
    bool narrow = true;      // every launch of the pass has a few rows only, or takes whole operators
    LevelArgs la;
    for (const std::vector<Segment>& segs : pl->levels) {
        if (level_problems(c, pl, segs, &la)) continue;
        for (const Segment& sg : segs) narrow = narrow && ((box && sg.type == T_PROJ) || gemm_takes_rows(sg.rows, std::max(d, h)));
    }
    ChainDepths depths;
    if (narrow || (!all_split(c, pl->hp) && !chain_depths(c, pl, backward, &depths))) return;
    uint16_t* at = ptr<uint16_t>(c->w_pieces);
    for (int t = 0; t < 3; ++t) {
        if (box && t == T_PROJ) continue;
        const MlpRefs W = mlp_of(c->prm, t);
        // Wa [h][d]: rows as n = forward operand of H = X Wa^T; columns as n = backward operand of dZ = dH Wa
        PieceJob& ja = J->job[J->count++];
        ja.W = W.Wa; ja.R = h; ja.C = d;
        c->wp[t][0] = ja.out_rk = at; at += pieces_elems(h, d);
        c->wp[t][3] = ja.out_ck = backward ? at : nullptr; at += pieces_elems(d, h);
        // Wb [d][h]: rows as n = forward operand of Y = H Wb^T; columns as n = backward operand of dH = dY Wb
        PieceJob& jw = J->job[J->count++];
        jw.W = W.Wb; jw.R = d; jw.C = h;
        c->wp[t][1] = jw.out_rk = at; at += pieces_elems(d, h);
        c->wp[t][2] = jw.out_ck = backward ? at : nullptr; at += pieces_elems(h, d);
    }
    c->have_pieces = true;
    J->clear = ptr<int32_t>(c->sync) + TILE_AT;
    J->clear_n = TILE_SYNC;
}

// All layers of a forward pass in one launch (rows_chain_kernel), where each would be one of a few rows: the same sums in the same order.
// Only passes that keep no rows for others, of the vector family without text features (whose references are made on the device).  Outputs keep a row
// each, by slot, and every depth has rows of its own (TileHelp), in memory that only these launches use: roots are those of passes that keep everything.  False: not such a pass.
bool rows_chain(const ngdb_ctx_t* c, const ngdb_plan_t* pl, RowsChain* r) {
    const HostPlan& hp = pl->hp;
    const int d = c->cfg.d, h = c->cfg.h;
    const LevelSync sync = level_sync(c);
    if (!rows_chain_model(c) || !sync.counts || c->captured || hp.n_levels < 1 || hp.n_levels > LEVEL_CHAIN || hp.n_slots + (int64_t)hp.n_int_rows > CHAIN_WORDS ||
        (int64_t)hp.n_proj + hp.n_int_rows + hp.n_neg > CHAIN_WORDS)
        return false;
    r->d = d; r->h = h; r->depths = hp.n_levels; r->sync = sync;
    auto word = [&](int32_t v) { r->words[r->n_words++] = v; };
    for (int l = 1; l <= hp.n_levels; ++l) {
        int& count = r->count[l - 1];
        count = 0;
        for (const Segment& sg : pl->levels[l]) {
            if (sg.rows <= 0) continue;
            if (!gemm_takes_rows(sg.rows, std::max(d, h))) return false;
            const int classes = sg.type == T_INTER ? sg.g_hi - sg.g_lo : 1;
            for (int i = 0; i < classes; ++i) {
                const int g = sg.g_lo + i;
                const bool inter = sg.type == T_INTER;
                RowsProblem p{sg.type, inter ? hp.g_nin[g] : 1, inter ? hp.g_n[g] : sg.rows, r->n_words, inter ? hp.g_mlp_base[g] : sg.mlp_base};
                if (count == CHAIN_PROBLEMS || p.k > CHAIN_CARD || (inter && p.k < 2) || r->n_words + p.n * (p.k + 2) > CHAIN_WORDS) return false;
                const int ref0 = sg.ref_off + p.row0 - sg.mlp_base, out0 = inter ? hp.g_out_base[g] : sg.out_base;
                for (int x = 0; x < p.n * p.k; ++x) word(hp.in_ref[ref0 + x]);
                for (int x = 0; sg.type == T_PROJ && x < p.n; ++x) word(hp.rel[sg.rel_off + x]);
                for (int x = 0; x < p.n; ++x) word(out0 + x);
                r->p[l - 1][count++] = p;
            }
        }
        if (count == 0) return false;
    }
    const int32_t hidden[3] = {hp.n_proj, hp.n_int_rows, hp.n_neg};
    float* H = rows_chain_act(c) + (size_t)CHAIN_WORDS * d;
    for (int t = 0; t < 3; ++t) {
        const MlpRefs W = mlp_of(c->prm, t);
        r->Wa[t] = W.Wa; r->ba[t] = W.ba; r->Wb[t] = W.Wb; r->bb[t] = W.bb;
        r->H[t] = H;
        H += (size_t)hidden[t] * h;
    }
    r->E = c->prm.E.p; r->R = c->prm.R.p; r->act = rows_chain_act(c); r->Z = r->act + (size_t)hp.n_slots * d;
    return rows_chain_lay_out(*r);
}

// The first launch of a pass: the plan to the device and the weights as pieces.
// A plan of ordinary size reaches the device with the first call that uses it: workgroups of this launch
// read the staging buffer (120 KB: 5 us as a launch of its own), which needs neither a wait on the host (10 us) nor an
// event between streams (9 us of host time).  Large ones are copied when they are planned.
constexpr size_t PLAN_INLINE_BYTES = 256 << 10;
// chain: a forward pass that rows_chain may take; ride: nothing but that pass (and an index it takes along) reads the plan before it is through.
int begin_pass(ngdb_ctx_t* c, const ngdb_plan_t* pl, bool backward, hipStream_t s, bool chain = false, bool ride = false) {
    const int waited = check_waits(c);
    if (waited != NGDB_OK) return waited;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const hipError_t asked = hipStreamIsCapturing(s, &capture);
    if (asked != hipSuccess) {       // (the default stream, while a stream that waits for it is captured)
        if (!pl->uploaded) HIPCHK(c, asked);
        (void)hipGetLastError();
    }
    c->captured = asked != hipSuccess || capture != hipStreamCaptureStatusNone;
    c->chained = c->rows_chained = c->plan_rides = false;
    c->trains = backward;
    c->fuses_beside = false;
    RowsChain r;
    if (chain && rows_chain(c, pl, &r)) {
        if (!pl->uploaded) {
            r.copy = plan_copy(pl);
        }
        unsigned long long* bits = reinterpret_cast<unsigned long long*>(ptr<int32_t>(c->sync) + CHAIN_AT);
        r.through = bits + (c->chain_odd ? CHAIN_SYNC : 0);
        r.clear = bits + (c->chain_odd ? 0 : CHAIN_SYNC);
        r.help = tile_help(c);
        Timed tm(c, NGDB_TK_GEMM_FWD, s);
        HIPCHK(c, launch_rows_chain(r, s));
        ++c->chain_count[0];
        c->chain_odd = !c->chain_odd;
        double flop = 0.0;
        for (const std::vector<Segment>& segs : pl->levels) flop += level_flop(c, segs);
        tm.work(GEMM_FP32, flop);
        c->chained = c->rows_chained = true;
        plan_uploaded(c, pl);
        return NGDB_OK;
    }
    PieceJobs J{};
    if (!pl->uploaded) {
        J.copy_dst = reinterpret_cast<float4*>(pl->blob.dev);
        J.copy_src = reinterpret_cast<const float4*>(pl->blob.pinned);
        J.copy_n = (int)(pl->blob_bytes / 16);
    }
    add_weight_pieces(c, pl, backward, &J);
    // (a launch of the plan alone is 4 of the 62 us of a step of 64 queries x 8 negatives at d = 32, h = 64)
    if (ride && !pl->uploaded && J.count == 0 && forward_chained(c, pl)) {
        c->plan_rides = true;
        return NGDB_OK;
    }
    {
        Timed tm(c, NGDB_TK_GEMM_FWD, s);
        HIPCHK(c, launch_weight_pieces(J, s));
    }
    plan_uploaded(c, pl);
    return NGDB_OK;
}

// The end of a pass, also of one that is refused or fails half way: what it enqueued still reads the plan, whose buffer
// goes to another plan once last_use has passed, and, on the library stream, the caller's tensors, which the caller's
// stream must wait for.
struct PassEnd {
    ngdb_ctx_t* c;
    const ngdb_plan_t* pl;
    hipStream_t s;
    bool forked = false, closed = false;      // forked: the library stream has work that s does not wait for yet
    hipError_t close() {
        closed = true;
        return hipEventRecord(pl->blob.last_use, s);
    }
    ~PassEnd() {
        if (forked && hipEventRecord(c->ev_join, c->side[0]) == hipSuccess) (void)hipStreamWaitEvent(s, c->ev_join, 0);
        if (!closed) (void)close();
    }
};

int size_workspace(ngdb_ctx_t* c, const ngdb_plan_t* pl, int K, bool want_table_grads) {
    const HostPlan& hp = pl->hp;
    const size_t d = c->cfg.d, h = c->cfg.h, f = sizeof(float);
    const size_t rows[3] = {(size_t)hp.n_proj, (size_t)hp.n_int_rows, (size_t)hp.n_neg};
    int rc;
#define ENS(buf, bytes) if ((rc = ensure(c, buf, std::max<size_t>((bytes), 256))) != NGDB_OK) return rc
    ENS(c->w_pieces, weight_pieces_bytes(c, hp));
    ENS(c->h_pieces, h_pieces_bytes(c, hp));
    ENS(c->act, (size_t)hp.n_slots * d * f);
    ENS(c->dact, ((size_t)hp.n_slots + hp.n_anchor) * d * f);
    for (int t = 0; t < 3; ++t) {
        ENS(c->Z[t], rows[t] * d * f);
        ENS(c->H[t], rows[t] * h * f);
        ENS(c->dH[t], rows[t] * h * f);
    }
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    if (box) {
        ENS(c->off, (size_t)hp.n_slots * d * f);
        ENS(c->doff, ((size_t)hp.n_slots + hp.n_anchor) * d * f);
        ENS(c->Z[T_NEG], rows[T_INTER] * d * f);
        ENS(c->H[T_NEG], rows[T_INTER] * h * f);
        ENS(c->dH[T_NEG], rows[T_INTER] * h * f);
        ENS(c->Gate, rows[T_INTER] * d * f);
        ENS(c->dGate, rows[T_INTER] * d * f);
        ENS(c->DxO, rows[T_INTER] * d * f);
    }
    ENS(c->Att, rows[T_INTER] * d * f);
    ENS(c->dAtt, rows[T_INTER] * d * f);
    ENS(c->Dx, rows[T_INTER] * d * f);
    const size_t pairs = (size_t)hp.n_queries * ((size_t)K + 1);
    ENS(c->score, pairs * f);
    ENS(c->coef, pairs * f);
    if (c->cfg.d_sem > 0) {
        ENS(c->mask, pairs * 64 * (d <= 256 ? 1 : (d <= 512 ? 2 : 4)));   // sign codes, per pair and lane
    } else {
        ENS(c->win, pairs * sizeof(int32_t));
    }
    ENS(c->loss_terms, (size_t)hp.n_queries * f);
    ENS(c->rec_coef, ((size_t)hp.n_anchor + pairs) * f);
    ENS(c->rec_row, ((size_t)hp.n_anchor + pairs) * sizeof(int32_t));
    const int64_t nk = (int64_t)hp.n_anchor + hp.n_queries + (int64_t)hp.n_queries * K;
    ENS(c->keys_a, (size_t)nk * 4);
    ENS(c->keys_b, (size_t)nk * 4);
    ENS(c->vals_a, (size_t)nk * 4);
    ENS(c->vals_b, (size_t)nk * 4);
    ENS(c->uniq, (size_t)nk * 4);
    ENS(c->seg_off, ((size_t)nk + 1) * 4);
    ENS(c->hist, index_hist_elems(nk) * 4);
    ENS(c->scan_tmp, index_scan_tmp_elems(nk) * 4);
    ENS(c->n_uniq, 256);       // count, and the number of rows in `later`
    ENS(c->later, (size_t)hp.n_anchor * 4);
    if (!c->gW.p) {
        size_t off = 0;
        for (int t = 0; t < 3; ++t) {
            const size_t sz[4] = {h * d, h, d * h, d};
            for (int k = 0; k < 4; ++k) {
                c->gw_off[t * 4 + k] = off;
                off += (sz[k] + 3) & ~size_t(3);
            }
        }
        c->gw_off[12] = off;
        ENS(c->gW, off * f);
    }
    if (c->cfg.d_sem > 0) {
        const size_t ds = c->cfg.d_sem;
        const size_t urows = (size_t)std::min<int64_t>(nk, c->cfg.n_entities);
        ENS(c->Wb, d * ds * sizeof(uint16_t));
        ENS(c->Ef, urows * d * f);
        ENS(c->inv, (size_t)nk * 4);
        ENS(c->refs_sem, hp.in_ref.size() * 4);
        ENS(c->Ea, (size_t)hp.n_anchor * d * sizeof(float));
        ENS(c->g_bf16, urows * d * sizeof(uint16_t));
        ENS(c->wp_partial, (size_t)sem_wgrad_splits((int64_t)urows, (int)d, (int)ds) * d * ds * f);
        ENS(c->gWp, d * ds * f);
    }
    if (want_table_grads) {
        const size_t urows = (size_t)std::min<int64_t>(nk, c->cfg.n_entities);
        if ((rc = ensure(c, c->gE, urows * d * f, Use::Evaluation)) != NGDB_OK) return rc;
        if ((rc = ensure(c, c->gR, (size_t)std::max<size_t>(hp.r_uniq.size(), 1) * d * f, Use::Evaluation)) != NGDB_OK) return rc;
        if (box && (rc = ensure(c, c->gRo, (size_t)std::max<size_t>(hp.r_uniq.size(), 1) * d * f, Use::Evaluation)) != NGDB_OK) return rc;
    }
#undef ENS
    return NGDB_OK;
}

// Where the entity rows of one call come from: the table itself, or (text-feature fusion) the
// fused rows of the touched entities, addressed by position in that list.
struct EntRows {
    const float* rows;
    const int32_t* refs;   // operator input references (anchors as -1-row)
    const int32_t* pos;    // [B] row of every query's positive
    const int32_t* cand;   // [B, C] rows of the candidates
};

IndexBuffers index_buffers(ngdb_ctx_t* c) {
    return IndexBuffers{ptr<int32_t>(c->keys_a), ptr<int32_t>(c->keys_b), ptr<int32_t>(c->vals_a), ptr<int32_t>(c->vals_b), ptr<int32_t>(c->hist),
                        ptr<int32_t>(c->scan_tmp), ptr<int32_t>(c->uniq), ptr<int32_t>(c->seg_off), ptr<int32_t>(c->n_uniq)};
}

// Index over [anchors | positives | tail], left in the context's buffers; *e_src receives the sorted contribution numbers.
int build_index(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_tail, int64_t n_tail, hipStream_t s, int32_t** e_src) {
    Timed tm(c, NGDB_TK_INDEX, s);
    HIPCHK(c, build_segment_index(pl->d_ekeys_head, pl->hp.n_anchor + pl->hp.n_queries, d_tail, n_tail, c->cfg.n_entities, index_buffers(c), e_src, s));
    return NGDB_OK;
}

// ---- text features: Wp as bf16, the fused rows of the anchors (one per anchor) or of the index's distinct
// entities, and the references to them
int cast_projection(ngdb_ctx_t* c, hipStream_t s) {
    Timed tm(c, NGDB_TK_SEM, s);
    HIPCHK(c, launch_cast_bf16(c->prm.Wp.p, ptr<uint16_t>(c->Wb), (int64_t)c->cfg.d * c->cfg.d_sem, s));
    return NGDB_OK;
}
SemFuseArgs fuse_args(const ngdb_ctx_t* c) {
    SemFuseArgs fa{};
    fa.H = c->prm.H_sem; fa.Wb = ptr<uint16_t>(c->Wb); fa.E = c->prm.E.p; fa.d = c->cfg.d; fa.ds = c->cfg.d_sem;
    return fa;
}
int fuse_anchors(ngdb_ctx_t* c, const ngdb_plan_t* pl, hipStream_t s, EntRows* er, bool reclaim) {
    const HostPlan& hp = pl->hp;
    Timed tm(c, NGDB_TK_SEM, s);
    SemFuseArgs fa = fuse_args(c);
    fa.ids = pl->d_ekeys_head; fa.n_rows = hp.n_anchor; fa.out = ptr<float>(c->Ea);
    HIPCHK(c, launch_sem_fuse(fa, s));
    HIPCHK(c, launch_translate_refs(reclaim ? pl->d_f_in_ref : pl->d_in_ref, pl->d_in_gslot, (int)hp.in_ref.size(), hp.n_slots, nullptr,
                                    ptr<int32_t>(c->refs_sem), s));
    *er = EntRows{ptr<float>(c->Ea), ptr<int32_t>(c->refs_sem), nullptr, nullptr};
    return NGDB_OK;
}
int fuse_indexed(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* e_src, int64_t n_tail, hipStream_t s, EntRows* er) {
    const int n_anchor = pl->hp.n_anchor, B = pl->hp.n_queries;
    const int64_t n_contrib = (int64_t)n_anchor + B + n_tail;
    Timed tm(c, NGDB_TK_SEM, s);
    HIPCHK(c, launch_inverse_index(e_src, ptr<int32_t>(c->seg_off), ptr<int32_t>(c->n_uniq), n_contrib, ptr<int32_t>(c->inv), s));
    SemFuseArgs fa = fuse_args(c);
    fa.ids = ptr<int32_t>(c->uniq); fa.n_rows_dev = ptr<int32_t>(c->n_uniq); fa.n_rows = (int)std::min<int64_t>(n_contrib, c->cfg.n_entities);
    fa.out = ptr<float>(c->Ef);
    HIPCHK(c, launch_sem_fuse(fa, s));
    er->rows = ptr<float>(c->Ef);
    er->pos = ptr<int32_t>(c->inv) + n_anchor;
    er->cand = ptr<int32_t>(c->inv) + n_anchor + B;
    return NGDB_OK;
}
// What a forward-only pass reads: with text features the fused rows of the anchors and, if there are candidates,
// of the distinct entities among them.
int prepare_entities(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_tail, int64_t n_tail, hipStream_t s, EntRows* er, bool reclaim) {
    const HostPlan& hp = pl->hp;
    *er = EntRows{c->prm.E.p, reclaim ? pl->d_f_in_ref : pl->d_in_ref, pl->d_pos, d_tail};
    if (c->cfg.d_sem == 0) return NGDB_OK;
    int rc = cast_projection(c, s);
    if (rc != NGDB_OK || n_tail == 0) return rc != NGDB_OK ? rc : fuse_anchors(c, pl, s, er, reclaim);
    int32_t* e_src = nullptr;
    if ((rc = build_index(c, pl, d_tail, n_tail, s, &e_src)) != NGDB_OK) return rc;
    if ((rc = fuse_indexed(c, pl, e_src, n_tail, s, er)) != NGDB_OK) return rc;
    Timed tm(c, NGDB_TK_SEM, s);
    HIPCHK(c, launch_translate_refs(er->refs, pl->d_in_gslot, (int)hp.in_ref.size(), hp.n_slots, ptr<int32_t>(c->inv), ptr<int32_t>(c->refs_sem), s));
    er->refs = ptr<int32_t>(c->refs_sem);
    return NGDB_OK;
}

// The intersections of one segment as jobs of the pooling kernels: centres (box == false:
// X = Z[T_INTER], logits Att) or offsets of the box family (X = Z[T_NEG], MLP outputs Gate).
// With `pool` the jobs are appended to it and the offset jobs flagged (both kinds in one launch).
int inter_jobs(ngdb_ctx_t* c, const ngdb_plan_t* pl, const Segment& sg, bool offsets, bool backward, InterJobs* ij,
               BoxPoolJobs* pool = nullptr) {
    const HostPlan& hp = pl->hp;
    const int d = c->cfg.d;
    if (pool) ij = &pool->jobs;
    else *ij = InterJobs{};
    ij->d = d;
    for (int g = sg.g_lo; g < sg.g_hi; ++g) {
        const size_t mb = (size_t)hp.g_mlp_base[g] * d, ob = (size_t)hp.g_out_base[g] * d;
        if (ij->count == INTER_MAX_JOBS) return fail(c, NGDB_ERR_UNSUPPORTED, "too many intersection classes in one level");
        InterJob& jb = ij->job[ij->count++];
        jb.X = ptr<float>(c->Z[offsets ? T_NEG : T_INTER]) + mb;
        jb.Att = ptr<float>(offsets ? c->Gate : c->Att) + mb;
        jb.n = hp.g_n[g]; jb.k = hp.g_nin[g];
        if (pool && offsets) pool->gate_mask |= 1u << (ij->count - 1);
        if (!backward) {
            jb.out = ptr<float>(offsets ? c->off : c->act) + ob;
        } else {
            jb.dY = ptr<float>(offsets ? c->doff : c->dact) + ob;
            jb.dAtt = ptr<float>(offsets ? c->dGate : c->dAtt) + mb;
            jb.Dx = ptr<float>(offsets ? c->DxO : c->Dx) + mb;
        }
    }
    return NGDB_OK;
}

BoxProjArgs box_proj_args(ngdb_ctx_t* c, const ngdb_plan_t* pl, const Segment& sg) {
    BoxProjArgs a{};
    a.ref = pl->d_in_ref + sg.ref_off; a.gslot = pl->d_in_gslot + sg.ref_off; a.rel = pl->d_rel + sg.rel_off;
    a.E = c->prm.E.p; a.Rc = c->prm.R.p; a.Ro = c->prm.Ro.p;
    a.act_c = ptr<float>(c->act); a.act_o = ptr<float>(c->off);
    a.dact_c = ptr<float>(c->dact); a.dact_o = ptr<float>(c->doff);
    a.n = sg.rows; a.d = c->cfg.d; a.out_base = sg.out_base;
    return a;
}

// The projection group of a level that can ride in the level's pooling launch (they are
// independent of each other): the first one, if an intersection segment with few enough
// cardinality classes for the joint launch exists.
const Segment* riding_projection(const std::vector<Segment>& segs) {
    const Segment* proj = nullptr;
    bool joint = false;
    for (const Segment& sg : segs) {
        if (sg.type == T_PROJ && !proj) proj = &sg;
        if (sg.type == T_INTER && 2 * (sg.g_hi - sg.g_lo) <= INTER_MAX_JOBS) joint = true;
    }
    return joint ? proj : nullptr;
}

// Device memory the forward pass of the vector family writes: operator outputs by slot, and per
// type the gathered first-layer inputs, the hidden rows and (intersections) the logits.
// reclaim (forward-only passes, Sec. 4.3 eager reference counting): an output is kept only until
// its consumer has run -- act holds n_f_rows storage rows addressed through the plan's f_row map,
// and Z / H / Att hold the rows of one step at a time (sizes: forward_bytes).
struct FwdSpace {
    float* act;
    float* Z[3];
    float* H[3];
    float* Att;
    bool reclaim;
    LevelSync sync;            // (the context's; without: depths in launches of their own)
};
FwdSpace ctx_space(const ngdb_ctx_t* c, bool reclaim = false) {
    return FwdSpace{ptr<float>(c->act), {ptr<float>(c->Z[0]), ptr<float>(c->Z[1]), ptr<float>(c->Z[2])},
                    {ptr<float>(c->H[0]), ptr<float>(c->H[1]), ptr<float>(c->H[2])}, ptr<float>(c->Att), reclaim, level_sync(c)};
}
// Their operators as problems, depth by depth in the order they are computed.  row0: of the type's buffers.  False: too many.
template <class Row0>
bool tile_problems(const ngdb_ctx_t* c, const ngdb_plan_t* pl, const ChainDepths& depths, bool backward, Row0 row0, TileChain* r) {
    const HostPlan& hp = pl->hp;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    const int n = depths.to - depths.from + 1;
    TileProblem problems[LEVEL_CHAIN][TILE_PROBLEMS];
    int counts[LEVEL_CHAIN];
    for (int i = 0; i < n; ++i) {
        int& count = counts[i];
        count = 0;
        for (const Segment& sg : pl->levels[backward ? depths.to - i : depths.from + i]) {
            const bool inter = sg.type == T_INTER;
            if (sg.rows <= 0) continue;
            for (int k = 0; k < (inter ? sg.g_hi - sg.g_lo : 1); ++k) {
                const int g = sg.g_lo + k, at = inter ? hp.g_mlp_base[g] - sg.mlp_base : 0;
                const TileProblem p{sg.type, inter ? hp.g_nin[g] : 1, inter ? hp.g_n[g] : sg.rows, row0(sg) + at, sg.ref_off + at, sg.rel_off,
                                    inter ? hp.g_out_base[g] : sg.out_base};
                for (int side = 0; side < (box && inter ? 2 : 1); ++side) {
                    if (count == TILE_PROBLEMS) return false;
                    problems[i][count] = p;
                    if (side) problems[i][count].type = T_NEG;      // (the offsets of the same inputs through the second MLP)
                    ++count;
                }
            }
        }
    }
    r->d = c->cfg.d; r->h = c->cfg.h;
    return tile_chain_lay_out(*r, problems, counts, n, backward, box);
}
// (the box family's own buffers; null with vectors)
void chain_boxes(const ngdb_ctx_t* c, TileChain* r) {
    r->Ro = c->prm.Ro.p; r->off = ptr<float>(c->off); r->Gate = ptr<float>(c->Gate);
    r->doff = ptr<float>(c->doff); r->dGate = ptr<float>(c->dGate); r->DxO = ptr<float>(c->DxO);
}
// All layers of some depths in one launch (tile_chain_kernel), where their launches would be small ones: the same sums in the same order.  False: no such depths.
bool tile_chain(const ngdb_ctx_t* c, const ngdb_plan_t* pl, const EntRows& er, const FwdSpace& w, ChainDepths* depths, TileChain* r) {
    if (!w.sync.counts || !c->have_pieces || !chain_depths(c, pl, false, depths) ||
        !tile_problems(c, pl, *depths, false, [&](const Segment& sg) { return w.reclaim ? 0 : sg.mlp_base; }, r))
        return false;
    r->keep = w.reclaim ? 0 : 1;
    for (int t = 0; t < 3; ++t) {
        const MlpRefs W = mlp_of(c->prm, t);
        r->W[0][t] = c->wp[t][0]; r->W[1][t] = c->wp[t][1]; r->bias[0][t] = W.ba; r->bias[1][t] = W.bb;
        r->Z[t] = w.Z[t]; r->H[t] = w.H[t]; r->dH[t] = nullptr;
    }
    r->E = er.rows; r->R = c->prm.R.p; r->refs = er.refs; r->rel = pl->d_rel; r->out_row = w.reclaim ? pl->d_f_row : nullptr;
    r->act = w.act; r->Att = w.Att; r->dact = r->dAtt = r->Dx = nullptr;
    chain_boxes(c, r);
    r->sync = w.sync; r->chain = w.sync.counts + TILE_AT;
    return true;
}
// ... of the backward pass, the deepest first.
bool tile_chain_backward(const ngdb_ctx_t* c, const ngdb_plan_t* pl, ChainDepths* depths, TileChain* r) {
    const LevelSync sync = level_sync(c);
    if (!sync.counts || !c->have_pieces || !chain_depths(c, pl, true, depths) ||
        !tile_problems(c, pl, *depths, true, [](const Segment& sg) { return sg.mlp_base; }, r))
        return false;
    r->keep = 0;
    for (int t = 0; t < 3; ++t) {
        r->W[0][t] = c->wp[t][2]; r->W[1][t] = c->wp[t][3]; r->bias[0][t] = r->bias[1][t] = nullptr;
        r->Z[t] = ptr<float>(c->Z[t]); r->H[t] = ptr<float>(c->H[t]); r->dH[t] = ptr<float>(c->dH[t]);
    }
    r->E = r->R = nullptr; r->refs = pl->d_in_gslot; r->rel = r->out_row = nullptr;
    chain_boxes(c, r);
    r->act = nullptr; r->Att = ptr<float>(c->Att); r->dact = ptr<float>(c->dact); r->dAtt = ptr<float>(c->dAtt); r->Dx = ptr<float>(c->Dx);
    r->sync = sync; r->chain = sync.counts + TILE_AT + TILE_LAYERS * TILE_LAYER;
    return true;
}
int enqueue_chain(ngdb_ctx_t* c, const ngdb_plan_t* pl, TileChain& chain, const ChainDepths& depths, bool backward, hipStream_t s) {
    chain.taken = reinterpret_cast<unsigned long long*>(ptr<int32_t>(c->sync) + TAKEN_AT);
    chain.launch = ++c->chain_launch;
    chain.help = tile_help(c);
    Timed tm(c, backward ? NGDB_TK_GEMM_BWD : NGDB_TK_GEMM_FWD, s);
    HIPCHK(c, launch_tile_chain(chain, backward, c->cfg.family == NGDB_FAMILY_BOX, s));
    ++c->chain_count[backward ? 2 : 1];
    double flop = 0.0;
    for (int l = depths.from; l <= depths.to; ++l) flop += level_flop(c, pl->levels[l]);
    tm.work(GEMM_SPLIT, flop);
    c->chained = true;
    return NGDB_OK;
}

// Box family, forward: projections are one elementwise launch per group; an intersection runs two
// MLPs over its inputs (attention logits from the centres, gate inputs from the offsets), grouped
// into one launch per layer, then the two pooling kernels.
int enqueue_forward_box(ngdb_ctx_t* c, const ngdb_plan_t* pl, hipStream_t s) {
    const int d = c->cfg.d, h = c->cfg.h;
    int rc_l = NGDB_OK;
    if (enqueue_levels(c, pl, false, [](LevelArgs&) {}, level_sync(c), s, &rc_l)) return rc_l;
    TileChain chain;
    ChainDepths depths;
    const EntRows er{c->prm.E.p, pl->d_in_ref, nullptr, nullptr};
    const FwdSpace w = ctx_space(c);
    const bool in_one = tile_chain(c, pl, er, w, &depths, &chain);
    for (int l = 1; l <= pl->hp.n_levels; ++l) {
        const std::vector<Segment>& segs = pl->levels[l];
        if (in_one && l == depths.from) {
            if ((rc_l = enqueue_chain(c, pl, chain, depths, false, s)) != NGDB_OK) return rc_l;
            l = depths.to;
            continue;
        }
        LevelArgs la;
        if (level_problems(c, pl, segs, &la)) {
            Timed tm(c, NGDB_TK_GEMM_FWD, s);
            HIPCHK(c, launch_level(la, false, s));
            tm.work(GEMM_FP32, level_flop(c, segs));
            continue;
        }
        GemmArgs g1[GEMM_MAX_GROUP], g2[GEMM_MAX_GROUP];
        int n = 0;
        const Segment* ride = riding_projection(segs);
        for (const Segment& sg : segs) {
            if (sg.type == T_PROJ) {
                if (&sg == ride) continue;
                Timed tm(c, NGDB_TK_INTER, s);
                HIPCHK(c, launch_box_proj(box_proj_args(c, pl, sg), false, s));
                continue;
            }
            if (sg.type != T_INTER || n + 2 > GEMM_MAX_GROUP) return fail(c, NGDB_ERR_UNSUPPORTED, "operator not available in the box family");
            for (int part = 0; part < 2; ++part) {
                const int t = part ? T_NEG : T_INTER;
                const MlpRefs W = mlp_of(c->prm, t);
                float* Hh = ptr<float>(c->H[t]) + (size_t)sg.mlp_base * h;
                GemmArgs& a = g1[n];
                a.a_ref = pl->d_in_ref + sg.ref_off; a.a_base0 = ptr<float>(part ? c->off : c->act);
                a.a_base1 = c->prm.E.p;       // never taken: the plan holds no anchor below an intersection
                a.a_copy = ptr<float>(c->Z[t]) + (size_t)sg.mlp_base * d; a.lda = d; a.B = W.Wa; a.ldb = d;
                a.C = Hh; a.ldc = h; a.M = sg.rows; a.N = h; a.K = d; a.bias = W.ba; a.relu = true;
                GemmArgs& b = g2[n];
                b.A = Hh; b.lda = h; b.B = W.Wb; b.ldb = h; b.M = sg.rows; b.N = d; b.K = h; b.bias = W.bb; b.ldc = d;
                b.C = ptr<float>(part ? c->Gate : c->Att) + (size_t)sg.mlp_base * d;
                if (c->have_pieces) {
                    a.b_pieces = c->wp[t][0]; a.b_kt = (d + 15) / 16;
                    b.b_pieces = c->wp[t][1]; b.b_kt = (h + 15) / 16;
                }
                ++n;
            }
        }
        if (n == 0) continue;
        int rc_g;
        const HiddenPieces hpc = place_hidden_pieces(c, g1, n);
        bool emitted = false;
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_FWD, g1, n, s, &emitted)) != NGDB_OK) return rc_g;
        if (emitted) take_hidden_pieces(hpc, g2, n);
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_FWD, g2, n, s)) != NGDB_OK) return rc_g;
        for (const Segment& sg : segs) {
            if (sg.type != T_INTER) continue;
            Timed tm(c, NGDB_TK_INTER, s);
            InterJobs ij;
            int rc;
            if (2 * (sg.g_hi - sg.g_lo) <= INTER_MAX_JOBS) {     // centre and offset jobs fit one launch
                BoxPoolJobs pool{};
                if ((rc = inter_jobs(c, pl, sg, false, false, nullptr, &pool)) != NGDB_OK) return rc;
                if ((rc = inter_jobs(c, pl, sg, true, false, nullptr, &pool)) != NGDB_OK) return rc;
                if (ride) { pool.has_proj = 1; pool.proj = box_proj_args(c, pl, *ride); ride = nullptr; }
                HIPCHK(c, launch_box_pool(pool, false, s));
                continue;
            }
            if ((rc = inter_jobs(c, pl, sg, false, false, &ij)) != NGDB_OK) return rc;
            HIPCHK(c, launch_inter(ij, false, s));
            if ((rc = inter_jobs(c, pl, sg, true, false, &ij)) != NGDB_OK) return rc;
            HIPCHK(c, launch_box_offset(ij, false, s));
        }
    }
    return NGDB_OK;
}

// Bytes of the buffers of a forward-only pass, in the order act, Att, then Z and H per type.
struct FwdBytes { size_t act, att, z[3], h[3]; };
FwdBytes forward_bytes(const ngdb_ctx_t* c, const ngdb_plan_t* pl, bool reclaim) {
    const HostPlan& hp = pl->hp;
    const size_t d = c->cfg.d, h = c->cfg.h, f = sizeof(float);
    const size_t all[3] = {(size_t)hp.n_proj, (size_t)hp.n_int_rows, (size_t)hp.n_neg};
    FwdBytes b{};
    b.act = (size_t)(reclaim ? hp.n_f_rows : hp.n_slots) * d * f;
    for (int t = 0; t < 3; ++t) {
        const size_t rows = reclaim ? (size_t)hp.f_step_rows[t] : all[t];
        b.z[t] = rows * d * f;
        b.h[t] = rows * h * f;
        if (t == T_INTER) b.att = rows * d * f;
    }
    return b;
}

// Workspace of a forward-only pass of the vector family: the activation buffers at their
// reclaimed sizes; with text features also the index over [anchors | tail] and the fused rows.
int size_forward_only(ngdb_ctx_t* c, const ngdb_plan_t* pl, int64_t n_tail) {
    const HostPlan& hp = pl->hp;
    const FwdBytes fb = forward_bytes(c, pl, true);
    int rc;
#define ENS(buf, bytes) if ((rc = ensure(c, buf, std::max<size_t>((bytes), 256))) != NGDB_OK) return rc
    ENS(c->w_pieces, weight_pieces_bytes(c, hp));
    ENS(c->h_pieces, h_pieces_bytes(c, hp));
    ENS(c->act, fb.act);
    ENS(c->Att, fb.att);
    for (int t = 0; t < 3; ++t) {
        ENS(c->Z[t], fb.z[t]);
        ENS(c->H[t], fb.h[t]);
    }
    if (c->cfg.d_sem > 0) {
        const size_t d = c->cfg.d, ds = c->cfg.d_sem;
        const int64_t nk = (int64_t)hp.n_anchor + hp.n_queries + n_tail;
        const size_t urows = (size_t)std::min<int64_t>(nk, c->cfg.n_entities);
        ENS(c->keys_a, (size_t)nk * 4);
        ENS(c->keys_b, (size_t)nk * 4);
        ENS(c->vals_a, (size_t)nk * 4);
        ENS(c->vals_b, (size_t)nk * 4);
        ENS(c->uniq, (size_t)nk * 4);
        ENS(c->seg_off, ((size_t)nk + 1) * 4);
        ENS(c->hist, index_hist_elems(nk) * 4);
        ENS(c->scan_tmp, index_scan_tmp_elems(nk) * 4);
        ENS(c->n_uniq, 256);
        ENS(c->Wb, d * ds * sizeof(uint16_t));
        ENS(c->Ef, urows * d * sizeof(float));
        ENS(c->inv, (size_t)nk * 4);
        ENS(c->refs_sem, hp.in_ref.size() * 4);
        ENS(c->Ea, (size_t)hp.n_anchor * d * sizeof(float));
    }
#undef ENS
    return NGDB_OK;
}

// forward over the plan's frontiers; results in w.act.  The type segments of one
// depth are independent: they share one grouped launch per MLP layer.
int enqueue_forward(ngdb_ctx_t* c, const ngdb_plan_t* pl, const EntRows& er, hipStream_t s, const FwdSpace& w) {
    if (c->cfg.family == NGDB_FAMILY_BOX) return enqueue_forward_box(c, pl, s);   // (always on the context's buffers)
    if (c->rows_chained) return NGDB_OK;       // (the launch that began the pass)
    const int d = c->cfg.d, h = c->cfg.h;
    auto forward_level = [&](LevelArgs& la) {
        la.refs = er.refs; la.rel = pl->d_rel; la.E = er.rows; la.R = c->prm.R.p;
        la.act = w.act; la.Att = w.Att; la.out_row = w.reclaim ? pl->d_f_row : nullptr;
        la.keep = !w.reclaim;
    };
    int rc_l = NGDB_OK;
    if (enqueue_levels(c, pl, false, forward_level, w.sync, s, &rc_l)) return rc_l;
    TileChain chain;
    ChainDepths depths;
    const bool in_one = tile_chain(c, pl, er, w, &depths, &chain);
    for (int l = 1; l <= pl->hp.n_levels; ++l) {
        const std::vector<Segment>& segs = pl->levels[l];
        if (in_one && l == depths.from) {
            if ((rc_l = enqueue_chain(c, pl, chain, depths, false, s)) != NGDB_OK) return rc_l;
            l = depths.to;
            continue;
        }
        LevelArgs la;
        if (level_problems(c, pl, segs, &la)) {
            forward_level(la);
            Timed tm(c, NGDB_TK_GEMM_FWD, s);
            HIPCHK(c, launch_level(la, false, s));
            tm.work(GEMM_FP32, level_flop(c, segs));
            continue;
        }
        GemmArgs g1[3], g2[3];
        int n = 0;
        for (const Segment& sg : segs) {
            const MlpRefs W = mlp_of(c->prm, sg.type);
            // (with reclaimed outputs the per-type buffers hold this step's rows only)
            const size_t row0 = w.reclaim ? 0 : (size_t)sg.mlp_base;
            float* Z = w.Z[sg.type] + row0 * d;
            float* Hh = w.H[sg.type] + row0 * h;
            GemmArgs& a = g1[n];
            // first layer reads its rows through the plan's references and leaves a copy in Z for who reads them again: the weight
            // gradients, and the pooling of intersections
            a.a_ref = er.refs + sg.ref_off; a.a_base0 = w.act; a.a_base1 = er.rows;
            if (sg.rel_off >= 0) { a.a_add_idx = pl->d_rel + sg.rel_off; a.a_add = c->prm.R.p; }
            a.a_copy = w.reclaim && sg.type != T_INTER ? nullptr : Z;
            a.lda = d; a.B = W.Wa; a.ldb = d; a.C = Hh; a.ldc = h;
            a.M = sg.rows; a.N = h; a.K = d; a.bias = W.ba; a.relu = true;
            GemmArgs& b = g2[n];
            b.A = Hh; b.lda = h; b.B = W.Wb; b.ldb = h; b.M = sg.rows; b.N = d; b.K = h; b.bias = W.bb; b.ldc = d;
            if (c->have_pieces) {
                a.b_pieces = c->wp[sg.type][0]; a.b_kt = (d + 15) / 16;
                b.b_pieces = c->wp[sg.type][1]; b.b_kt = (h + 15) / 16;
            }
            if (sg.type == T_INTER) {
                b.C = w.Att + row0 * d;
            } else if (w.reclaim) {         // outputs go to their storage rows
                b.C = w.act;
                b.dst_row = pl->d_f_row + sg.out_base;
            } else {
                b.C = w.act + (size_t)sg.out_base * d;
            }
            ++n;
        }
        int rc_g;
        const HiddenPieces hpc = place_hidden_pieces(c, g1, n);
        bool emitted = false;
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_FWD, g1, n, s, &emitted)) != NGDB_OK) return rc_g;
        if (emitted) take_hidden_pieces(hpc, g2, n);
        // second layer with the pooling in its epilogue: the intersections class by class
        GemmArgs gp[GEMM_MAX_GROUP];
        int np = 0;
        bool pooled = false;
        for (int i = 0; i < n && np <= GEMM_MAX_GROUP; ++i) {
            const Segment& sg = segs[i];
            const int classes = sg.type == T_INTER ? sg.g_hi - sg.g_lo : 1;
            pooled = pooled || sg.type == T_INTER;
            for (int k = 0; k < classes; ++k, ++np) {
                if (np == GEMM_MAX_GROUP) { np = GEMM_MAX_GROUP + 1; break; }
                GemmArgs& b = gp[np] = g2[i];
                if (sg.type != T_INTER) continue;
                const int g = sg.g_lo + k, r0 = pl->hp.g_mlp_base[g] - sg.mlp_base, out0 = pl->hp.g_out_base[g];
                b.A += (size_t)r0 * h; b.a_row0 = r0; b.M = pl->hp.g_n[g] * pl->hp.g_nin[g];
                b.C = w.reclaim ? nullptr : b.C + (size_t)r0 * d;      // (the backward pass reads the logits)
                b.pool_k = pl->hp.g_nin[g];
                b.pool_X = w.Z[T_INTER] + ((w.reclaim ? 0 : (size_t)sg.mlp_base) + r0) * d;
                b.pool_out = w.reclaim ? w.act : w.act + (size_t)out0 * d;
                b.pool_row = w.reclaim ? pl->d_f_row + out0 : nullptr;
            }
        }
        if (pooled && np <= GEMM_MAX_GROUP) {
            Timed tm(c, NGDB_TK_GEMM_FWD, s);
            int route = GEMM_FP32;
            const hipError_t e = launch_gemm_group(gp, np, s, &route);
            if (e == hipSuccess) {
                double flop = 0.0;
                for (int i = 0; i < np; ++i) flop += 2.0 * gp[i].M * gp[i].N * gp[i].K;
                tm.work(route, flop);
                continue;
            }
            if (e != hipErrorNotSupported) HIPCHK(c, e);
        }
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_FWD, g2, n, s)) != NGDB_OK) return rc_g;
        for (const Segment& sg : segs) {
            if (sg.type != T_INTER) continue;
            Timed tm(c, NGDB_TK_INTER, s);
            InterJobs ij{};
            ij.d = d;
            for (int g = sg.g_lo; g < sg.g_hi; ++g) {
                const size_t mb = (size_t)(pl->hp.g_mlp_base[g] - (w.reclaim ? sg.mlp_base : 0)) * d;
                if (ij.count == INTER_MAX_JOBS) return fail(c, NGDB_ERR_UNSUPPORTED, "too many intersection classes in one level");
                InterJob& jb = ij.job[ij.count++];
                jb.X = w.Z[T_INTER] + mb; jb.Att = w.Att + mb;
                if (w.reclaim) {
                    jb.out = w.act;
                    jb.out_row = pl->d_f_row + pl->hp.g_out_base[g];
                } else {
                    jb.out = w.act + (size_t)pl->hp.g_out_base[g] * d;
                }
                jb.n = pl->hp.g_n[g]; jb.k = pl->hp.g_nin[g];
            }
            HIPCHK(c, launch_inter(ij, false, s));
        }
    }
    return NGDB_OK;
}

struct WgradJob {   // what enqueue_weight_grads needs after a backward chain
    int nt = 0;
    int types[3]{};
    size_t rows[3]{};
    const float* dY[3]{};
};

// Gradients of the MLP tensors of the given types (their Z / H / dH buffers, dY = gradient of
// the second layer's output): weights and biases of both layers of every type in one launch.
int enqueue_weight_grads(ngdb_ctx_t* c, const WgradJob& wj, hipStream_t s, bool aside) {
    const int d = c->cfg.d, h = c->cfg.h, nt = wj.nt;
    float* gW = ptr<float>(c->gW);
    Timed tm(c, NGDB_TK_WGRAD, s);
    WgradArgs w[6];
    double flop = 0.0;
    for (int i = 0; i < nt; ++i) {
        const int t = wj.types[i], gs = gslot_of(t), r = (int)wj.rows[i];
        // dWa[h,d] = dH^T Z, dba = column sums of dH; dWb[d,h] = dY^T H, dbb = column sums of dY
        w[2 * i] = WgradArgs{ptr<float>(c->dH[t]), ptr<float>(c->Z[t]), gW + c->gw_off[gs + 0], gW + c->gw_off[gs + 1], h, d, r, h, d, d};
        w[2 * i + 1] = WgradArgs{wj.dY[i], ptr<float>(c->H[t]), gW + c->gw_off[gs + 2], gW + c->gw_off[gs + 3], d, h, r, d, h, h};
        flop += 4.0 * h * d * r;
    }
    HIPCHK(c, launch_wgrad_group(w, 2 * nt, s, aside));
    tm.work(GEMM_SPLIT, flop);
    return NGDB_OK;
}

// reversed frontiers; *wj receives the inputs of the weight gradients (one grouped launch, later)
int enqueue_backward_box(ngdb_ctx_t* c, const ngdb_plan_t* pl, hipStream_t s, WgradJob* wj);
int enqueue_backward(ngdb_ctx_t* c, const ngdb_plan_t* pl, hipStream_t s, WgradJob* wj) {
    if (c->cfg.family == NGDB_FAMILY_BOX) return enqueue_backward_box(c, pl, s, wj);
    const int d = c->cfg.d, h = c->cfg.h;
    const HostPlan& hp = pl->hp;
    float* dact = ptr<float>(c->dact);
    auto backward_level = [&](LevelArgs& la) {
        la.dst_row = pl->d_in_gslot; la.Att = ptr<float>(c->Att); la.dact = dact; la.dAtt = ptr<float>(c->dAtt);
    };
    int rc_l = NGDB_OK;
    const bool chained = enqueue_levels(c, pl, true, backward_level, level_sync(c), s, &rc_l);
    if (rc_l != NGDB_OK) return rc_l;
    TileChain chain;
    ChainDepths depths;
    const bool in_one = !chained && tile_chain_backward(c, pl, &depths, &chain);
    for (int l = chained ? 0 : hp.n_levels; l >= 1; --l) {
        const std::vector<Segment>& segs = pl->levels[l];
        if (in_one && l == depths.to) {
            if ((rc_l = enqueue_chain(c, pl, chain, depths, true, s)) != NGDB_OK) return rc_l;
            l = depths.from;
            continue;
        }
        LevelArgs la;
        if (level_problems(c, pl, segs, &la)) {
            backward_level(la);
            Timed tm(c, NGDB_TK_GEMM_BWD, s);
            HIPCHK(c, launch_level(la, true, s));
            tm.work(GEMM_FP32, level_flop(c, segs));
            continue;
        }
        GemmArgs b2[3], b1[3];
        int n = 0;
        for (const Segment& sg : segs) {
            const MlpRefs W = mlp_of(c->prm, sg.type);
            const float* dOut;
            const float* addend = nullptr;
            if (sg.type == T_INTER) {
                Timed tm(c, NGDB_TK_INTER, s);
                InterJobs ij{};
                ij.d = d;
                for (int g = sg.g_lo; g < sg.g_hi; ++g) {
                    const size_t mb = (size_t)hp.g_mlp_base[g] * d;
                    if (ij.count == INTER_MAX_JOBS) return fail(c, NGDB_ERR_UNSUPPORTED, "too many intersection classes in one level");
                    InterJob& jb = ij.job[ij.count++];
                    jb.X = ptr<float>(c->Z[T_INTER]) + mb; jb.Att = ptr<float>(c->Att) + mb;
                    jb.dY = dact + (size_t)hp.g_out_base[g] * d;
                    jb.dAtt = ptr<float>(c->dAtt) + mb; jb.Dx = ptr<float>(c->Dx) + mb;
                    jb.n = hp.g_n[g]; jb.k = hp.g_nin[g];
                }
                HIPCHK(c, launch_inter(ij, true, s));
                dOut = ptr<float>(c->dAtt) + (size_t)sg.mlp_base * d;
                addend = ptr<float>(c->Dx) + (size_t)sg.mlp_base * d;
            } else {
                dOut = dact + (size_t)sg.out_base * d;
            }
            const float* Hh = ptr<float>(c->H[sg.type]) + (size_t)sg.mlp_base * h;
            float* dHh = ptr<float>(c->dH[sg.type]) + (size_t)sg.mlp_base * h;
            GemmArgs& x = b2[n];   // dH = (dOut * Wb) masked by relu
            x.A = dOut; x.lda = d; x.B = W.Wb; x.ldb = h; x.b_kcontig = false;
            x.C = dHh; x.ldc = h; x.M = sg.rows; x.N = h; x.K = d; x.mask = Hh; x.ldmask = h;
            GemmArgs& y = b1[n];   // dZ = dH * Wa, scattered to the gradient rows of the inputs
            y.A = dHh; y.lda = h; y.B = W.Wa; y.ldb = d; y.b_kcontig = false;
            y.C = dact; y.ldc = d; y.M = sg.rows; y.N = d; y.K = h;
            y.addend = addend; y.ldadd = d; y.dst_row = pl->d_in_gslot + sg.ref_off;
            if (c->have_pieces) {
                x.b_pieces = c->wp[sg.type][2]; x.b_kt = (d + 15) / 16;
                y.b_pieces = c->wp[sg.type][3]; y.b_kt = (h + 15) / 16;
            }
            ++n;
        }
        int rc_g;
        const HiddenPieces hpc = place_hidden_pieces(c, b2, n);
        bool emitted = false;
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_BWD, b2, n, s, &emitted)) != NGDB_OK) return rc_g;
        if (emitted) take_hidden_pieces(hpc, b1, n);
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_BWD, b1, n, s)) != NGDB_OK) return rc_g;
    }
    // weight gradients: one contraction per tensor over all rows of the type
    wj->nt = 3;
    const int types[3] = {T_PROJ, T_INTER, T_NEG};
    const size_t rows[3] = {(size_t)hp.n_proj, (size_t)hp.n_int_rows, (size_t)hp.n_neg};
    const float* dY[3] = {dact, ptr<float>(c->dAtt), dact + ((size_t)hp.n_proj + hp.n_inter) * d};
    for (int i = 0; i < 3; ++i) { wj->types[i] = types[i]; wj->rows[i] = rows[i]; wj->dY[i] = dY[i]; }
    return NGDB_OK;
}

// Box family, backward: the reverse of enqueue_forward_box; the gradient of a projection's
// input is the gradient of its output (copied to the input's rows, where the relation tables
// pick it up too).
int enqueue_backward_box(ngdb_ctx_t* c, const ngdb_plan_t* pl, hipStream_t s, WgradJob* wj) {
    const int d = c->cfg.d, h = c->cfg.h;
    const HostPlan& hp = pl->hp;
    int rc_l = NGDB_OK;
    const bool chained = enqueue_levels(c, pl, true, [](LevelArgs&) {}, level_sync(c), s, &rc_l);
    if (rc_l != NGDB_OK) return rc_l;
    TileChain chain;
    ChainDepths depths;
    const bool in_one = !chained && tile_chain_backward(c, pl, &depths, &chain);
    for (int l = chained ? 0 : hp.n_levels; l >= 1; --l) {
        const std::vector<Segment>& segs = pl->levels[l];
        if (in_one && l == depths.to) {
            if ((rc_l = enqueue_chain(c, pl, chain, depths, true, s)) != NGDB_OK) return rc_l;
            l = depths.from;
            continue;
        }
        LevelArgs la;
        if (level_problems(c, pl, segs, &la)) {
            Timed tm(c, NGDB_TK_GEMM_BWD, s);
            HIPCHK(c, launch_level(la, true, s));
            tm.work(GEMM_FP32, level_flop(c, segs));
            continue;
        }
        GemmArgs b2[GEMM_MAX_GROUP], b1[GEMM_MAX_GROUP];
        int n = 0;
        const Segment* ride = riding_projection(segs);
        for (const Segment& sg : segs) {
            if (sg.type == T_PROJ) {
                if (&sg == ride) continue;
                Timed tm(c, NGDB_TK_INTER, s);
                HIPCHK(c, launch_box_proj(box_proj_args(c, pl, sg), true, s));
                continue;
            }
            if (sg.type != T_INTER || n + 2 > GEMM_MAX_GROUP) return fail(c, NGDB_ERR_UNSUPPORTED, "operator not available in the box family");
            {
                Timed tm(c, NGDB_TK_INTER, s);
                InterJobs ij;
                int rc;
                if (2 * (sg.g_hi - sg.g_lo) <= INTER_MAX_JOBS) {
                    BoxPoolJobs pool{};
                    if ((rc = inter_jobs(c, pl, sg, false, true, nullptr, &pool)) != NGDB_OK) return rc;
                    if ((rc = inter_jobs(c, pl, sg, true, true, nullptr, &pool)) != NGDB_OK) return rc;
                    if (ride) { pool.has_proj = 1; pool.proj = box_proj_args(c, pl, *ride); ride = nullptr; }
                    HIPCHK(c, launch_box_pool(pool, true, s));
                } else {
                    if ((rc = inter_jobs(c, pl, sg, false, true, &ij)) != NGDB_OK) return rc;
                    HIPCHK(c, launch_inter(ij, true, s));
                    if ((rc = inter_jobs(c, pl, sg, true, true, &ij)) != NGDB_OK) return rc;
                    HIPCHK(c, launch_box_offset(ij, true, s));
                }
            }
            for (int part = 0; part < 2; ++part) {
                const int t = part ? T_NEG : T_INTER;
                const MlpRefs W = mlp_of(c->prm, t);
                const size_t mb = (size_t)sg.mlp_base;
                const float* Hh = ptr<float>(c->H[t]) + mb * h;
                float* dHh = ptr<float>(c->dH[t]) + mb * h;
                GemmArgs& x = b2[n];
                x.A = ptr<float>(part ? c->dGate : c->dAtt) + mb * d; x.lda = d; x.B = W.Wb; x.ldb = h; x.b_kcontig = false;
                x.C = dHh; x.ldc = h; x.M = sg.rows; x.N = h; x.K = d; x.mask = Hh; x.ldmask = h;
                GemmArgs& y = b1[n];
                y.A = dHh; y.lda = h; y.B = W.Wa; y.ldb = d; y.b_kcontig = false;
                y.C = ptr<float>(part ? c->doff : c->dact); y.ldc = d; y.M = sg.rows; y.N = d; y.K = h;
                y.addend = ptr<float>(part ? c->DxO : c->Dx) + mb * d; y.ldadd = d; y.dst_row = pl->d_in_gslot + sg.ref_off;
                if (c->have_pieces) {
                    x.b_pieces = c->wp[t][2]; x.b_kt = (d + 15) / 16;
                    y.b_pieces = c->wp[t][3]; y.b_kt = (h + 15) / 16;
                }
                ++n;
            }
        }
        if (n == 0) continue;
        int rc_g;
        const HiddenPieces hpc = place_hidden_pieces(c, b2, n);
        bool emitted = false;
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_BWD, b2, n, s, &emitted)) != NGDB_OK) return rc_g;
        if (emitted) take_hidden_pieces(hpc, b1, n);
        if ((rc_g = gemm_timed(c, NGDB_TK_GEMM_BWD, b1, n, s)) != NGDB_OK) return rc_g;
    }
    wj->nt = 2;
    wj->types[0] = T_INTER; wj->types[1] = T_NEG;
    wj->rows[0] = wj->rows[1] = (size_t)hp.n_int_rows;
    wj->dY[0] = ptr<float>(c->dAtt); wj->dY[1] = ptr<float>(c->dGate);
    return NGDB_OK;
}

// (streaming: plain rows of a table that the 256 MB last-level cache cannot hold; with text features rows fused for the call are read instead)
void candidate_table(const ngdb_ctx_t* c, ScoreArgs* sa) {
    const size_t values = (size_t)c->cfg.n_entities * c->cfg.d;
    sa->table_bytes = values * (c->cfg.score_bf16 ? sizeof(uint16_t) : sizeof(float));
    sa->streaming = c->cfg.d_sem == 0 && values * sizeof(float) > ((size_t)256 << 20);
}

int run_step(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_neg, int K, hipStream_t stream, float* d_loss,
             bool apply) {
    if (!c || !pl) return NGDB_ERR_ARG;
    if (!c->bound) return fail(c, NGDB_ERR_STATE, "parameters not bound");
    if (K < 1 || (pl->hp.n_queries > 0 && !d_neg) || !d_loss)
        return fail(c, NGDB_ERR_ARG, "bad negatives (K >= 1 is required) / loss pointer");
    if (pl->n_entities != c->cfg.n_entities || !pl->d_blob)
        return fail(c, NGDB_ERR_ARG, "plan belongs to another configuration or was built without a device");
    const HostPlan& hp = pl->hp;
    const int d = c->cfg.d, B = hp.n_queries;
    if (c->presized && (K > c->cfg.k_max || B > c->cfg.b_max_queries))
        return fail(c, NGDB_ERR_ARG, "batch beyond the maxima declared at ngdb_create (b_max_queries, k_max)");
    c->have_grads = false;
    int rc = size_workspace(c, pl, K, !apply);
    if (rc != NGDB_OK) return rc;
    PassEnd end{c, pl, stream};

    // 1. entity gradient index (depends only on the plan and the negatives).  With a library stream the index build, and with
    // text features the fusion of all rows that are scored, run beside the forward pass, which needs the anchors' rows only.
    int32_t* e_src = nullptr;
    const bool sem = c->cfg.d_sem > 0;
    const int64_t n_contrib = (int64_t)hp.n_anchor + B + (int64_t)B * K, max_rows = std::min<int64_t>(n_contrib, c->cfg.n_entities);
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    // The three waits between streams cost the host some 30 us a step.  Steps that are bound by the host either way stay on
    // the caller's stream: an index of one launch, or small MLPs with few rows to update (64 queries x 32 negatives 119
    // against 133 us at d = 64 and 211 against 220 at d = 400; 256 x 64 at d = 64 145 against 175, 1024 x 64 187 against 202, but
    // 1024 x 256 237 against 222; at d = 128, h = 256 256 x 64 196 against 184, as boxes, with fewer depths, 141 against 167).
    const bool host_bound = !sem && (n_contrib <= 4096 || (level_fits(d, c->cfg.h, box) && (box || d * c->cfg.h <= 16384) &&
                                                          n_contrib <= 70000 && max_rows * d <= 2000000));
    const bool aside = c->n_side > 0 && !host_bound;
    hipStream_t s_idx = aside ? c->side[0] : stream;
    // (a small index on the caller's stream: the launch of a small forward pass takes it along, or it follows)
    c->index_waits.n = 0;
    const bool index_rides = !aside && !sem && small_index_job(pl->d_ekeys_head, hp.n_anchor + B, d_neg, (int64_t)B * K, c->cfg.n_entities,
                                                               index_buffers(c), &c->index_waits);
    if ((rc = begin_pass(c, pl, true, stream, false, index_rides)) != NGDB_OK) {
        c->index_waits.n = 0;
        return rc;
    }
    c->fuses_beside = aside && sem && n_contrib > CHAIN_FUSED;
    if (sem && (rc = cast_projection(c, stream)) != NGDB_OK) return rc;
    if (aside) {
        HIPCHK(c, hipEventRecord(c->ev_fork, stream));
        HIPCHK(c, hipStreamWaitEvent(s_idx, c->ev_fork, 0));
        end.forked = true;
    }
    EntRows er{c->prm.E.p, pl->d_in_ref, pl->d_pos, d_neg}, scored = er;
    if (index_rides) e_src = c->index_waits.vals_out;
    else if ((rc = build_index(c, pl, d_neg, (int64_t)B * K, s_idx, &e_src)) != NGDB_OK) return rc;
    if (sem) {
        if ((rc = fuse_indexed(c, pl, e_src, (int64_t)B * K, s_idx, &scored)) != NGDB_OK) return rc;
        if (aside) HIPCHK(c, hipEventRecord(c->ev_join, s_idx));
        if ((rc = fuse_anchors(c, pl, stream, &er, false)) != NGDB_OK) return rc;
    }

    // 2. forward frontiers
    rc = enqueue_forward(c, pl, er, stream, ctx_space(c));
    const bool index_left = c->index_waits.n > 0;
    c->index_waits.n = 0;
    if (rc != NGDB_OK) return rc;
    if (index_left && (rc = build_index(c, pl, d_neg, (int64_t)B * K, stream, &e_src)) != NGDB_OK) return rc;

    // 3. scores, loss terms, dL/ds, gradients of the branch embeddings
    if (sem && aside) HIPCHK(c, hipStreamWaitEvent(stream, c->ev_join, 0));
    ScoreArgs sa{};
    sa.act = ptr<float>(c->act); sa.E = scored.rows; candidate_table(c, &sa);
    sa.root_off = pl->d_root_off; sa.root_slot = pl->d_root_slot;
    sa.pos = scored.pos; sa.cand = scored.cand; sa.B = B; sa.C = K; sa.d = d; sa.max_branch = std::max(1, hp.max_branch);
    sa.gamma = c->cfg.gamma; sa.score = ptr<float>(c->score); sa.coef = ptr<float>(c->coef);
    sa.win = sem ? nullptr : ptr<int32_t>(c->win); sa.mask = sem ? c->mask.p : nullptr; sa.dact = ptr<float>(c->dact); sa.loss_terms = ptr<float>(c->loss_terms);
    if (box) { sa.off = ptr<float>(c->off); sa.doff = ptr<float>(c->doff); sa.alpha = c->cfg.box_alpha; }
    if (c->cfg.score_bf16) sa.E16 = ptr<uint16_t>(c->Eb);
    {
        Timed tm(c, NGDB_TK_SCORE, stream);
        hipError_t e = launch_score(sa, true, stream);
        if (e == hipErrorInvalidValue) return fail(c, NGDB_ERR_UNSUPPORTED, "embedding width / union branch count too large for the scoring kernel");
        HIPCHK(c, e);
    }

    // 4. entity rows whose contributions are (query, candidate) pairs only need nothing of the backward pass: with a
    // library stream they are updated beside it, and only the rows that anchors refer to are left to the end of the
    // step.  (All rows after the backward pass, beside the weight gradients: 307 against 290 us a step at 512 queries over
    // 15 000 entities, 507 against 457 at 1024 over 63 000, 6.64 against 6.46 ms at 4096 over 2.5 million.)
    hipStream_t s_tab = aside ? c->side[0] : stream;     // after the index on the same stream
    // A pass that ends before the backward pass does even on few wavefronts is kept to few of them: at full width it
    // takes the compute units and caches from the launches that the step waits for.  Estimates in us: by 1024 wavefronts three
    // rows read and written at 2.7 TB/s, but 2 us a row, and 0.2 us a contribution; a chain of launches and its contractions.
    const double mlp_rows = (double)hp.n_proj + (box ? 2.0 : 1.0) * hp.n_int_rows + hp.n_neg;
    const double pass_us = std::max(24.0 * max_rows * d / 2.7e6, 2.0 * max_rows / 1024.0) + 0.2 * n_contrib / 1024.0;
    const double chain_us = level_fits(d, c->cfg.h, box) ? 25.0 + 18.0 * hp.n_levels : 100.0 + 12.0 * c->cfg.h * d * mlp_rows / 1e8;
    const bool short_pass = aside ? pass_us <= chain_us : max_rows <= 65536;
    const int64_t t = c->step + 1;
    AdamHyper ah{c->cfg.lr, c->cfg.beta1, c->cfg.beta2, c->cfg.eps,
                 (float)(1.0 - std::pow((double)c->cfg.beta1, (double)t)),
                 (float)(1.0 - std::pow((double)c->cfg.beta2, (double)t))};
    if (c->chained) ah.gave_up = gave_up_mark(c);
    TableArgs te{};
    te.P = c->prm.E.p; te.Mo = c->prm.E.m; te.Vo = c->prm.E.v;
    te.uniq = ptr<int32_t>(c->uniq); te.seg_off = ptr<int32_t>(c->seg_off);
    te.n_uniq_dev = ptr<int32_t>(c->n_uniq); te.d = d;
    te.rec_coef = ptr<float>(c->rec_coef); te.rec_row = ptr<int32_t>(c->rec_row);
    te.dact = ptr<float>(c->dact); te.act = ptr<float>(c->act); te.g_out = apply ? nullptr : ptr<float>(c->gE);
    if (sem) { te.mask = c->mask.p; te.g_bf16 = ptr<uint16_t>(c->g_bf16); }
    TableArgs tr = te;
    // parameters + two moments beyond what the 256 MB last-level cache could keep between steps (300 MB of them: 489
    // against 463 us a step; 72 MB: 304 with the hint against 296)
    te.streaming = (size_t)c->cfg.n_entities * d * 3 * sizeof(float) > ((size_t)256 << 20);
    if (c->cfg.score_bf16) te.shadow = ptr<uint16_t>(c->Eb);   // signs against the rounded rows; written only when updating
    if (box) { te.off = ptr<float>(c->off); te.alpha = c->cfg.box_alpha; }
    // the sum of the loss terms rides in the launch that resolves the records
    auto resolve_records = [&]() -> int {
        HIPCHK(c, launch_resolve(e_src, n_contrib, hp.n_anchor, hp.n_slots, B, K, ptr<float>(c->coef),
                                 sem ? nullptr : ptr<int32_t>(c->win), ptr<float>(c->rec_coef), ptr<int32_t>(c->rec_row),
                                 ptr<float>(c->loss_terms), B > 0 ? 1.f / (2.f * B) : 0.f, d_loss, gave_up_mark(c), s_tab));
        return NGDB_OK;
    };
    // who updates the rows resolves for itself: the launch that ends the step, or plain rows' own wavefronts
    const bool unresolved = (!aside && short_pass) || (!sem && table_takes_once(te, short_pass, max_rows));
    LossSum loss_sum{};
    if (unresolved) {
        te.src = e_src; te.pair_coef = ptr<float>(c->coef); te.pair_win = sem ? nullptr : ptr<int32_t>(c->win);
        te.n_rowsrc = hp.n_anchor; te.row_base = hp.n_slots; te.B = B; te.K = K;
        loss_sum = LossSum{ptr<float>(c->loss_terms), B, B > 0 ? 1.f / (2.f * B) : 0.f, d_loss, gave_up_mark(c)};
    }
    if (aside) {
        HIPCHK(c, hipEventRecord(c->ev_fork, stream));
        HIPCHK(c, hipStreamWaitEvent(s_tab, c->ev_fork, 0));
        if (!unresolved && (rc = resolve_records()) != NGDB_OK) return rc;
        te.later = ptr<int32_t>(c->later); te.n_later = ptr<int32_t>(c->n_uniq) + 1;
        {
            Timed tm(c, NGDB_TK_TABLE_E, s_tab);
            HIPCHK(c, launch_table_update(te, ah, short_pass, max_rows, s_tab));
        }
        HIPCHK(c, hipEventRecord(c->ev_join, s_tab));
        te.pick = te.later; te.n_uniq_dev = te.n_later;
        te.later = te.n_later = nullptr;
    }

    // 5. reversed frontiers, weight gradients
    WgradJob wj;
    rc = enqueue_backward(c, pl, stream, &wj);
    if (rc != NGDB_OK) return rc;
    if (c->chained) ah.gave_up = gave_up_mark(c);

    rc = enqueue_weight_grads(c, wj, stream, aside && !short_pass);
    if (rc != NGDB_OK) return rc;

    // 6. the other table rows, relation tables, dense Adam
    if (!aside && !unresolved && (rc = resolve_records()) != NGDB_OK) return rc;
    tr.g_bf16 = nullptr; tr.mask = nullptr;
    tr.P = c->prm.R.p; tr.Mo = c->prm.R.m; tr.Vo = c->prm.R.v;
    tr.uniq = pl->d_r_uniq; tr.seg_off = pl->d_r_seg_off; tr.n_uniq_dev = pl->d_n_r_uniq;
    tr.rec_coef = nullptr; tr.rec_row = pl->d_r_rec; tr.g_out = apply ? nullptr : ptr<float>(c->gR);
    TableArgs small[2] = {tr, tr};
    int n_small = 1;
    if (box) {   // relation offsets: the same segments over the offset gradients, gated by relu
        TableArgs& to = small[n_small++];
        to.P = c->prm.Ro.p; to.Mo = c->prm.Ro.m; to.Vo = c->prm.Ro.v;
        to.dact = ptr<float>(c->doff); to.relu_gate = true; to.g_out = apply ? nullptr : ptr<float>(c->gRo);
    }
    DenseAdamJob job{};
    if (apply) {
        const ngdb_tensor* ts[12] = {&c->prm.W1, &c->prm.b1, &c->prm.W2, &c->prm.b2, &c->prm.V1, &c->prm.c1,
                                     &c->prm.V2, &c->prm.c2, &c->prm.U1, &c->prm.u1, &c->prm.U2, &c->prm.u2};
        const int64_t hd = (int64_t)c->cfg.h * d;
        const int64_t sz[4] = {hd, c->cfg.h, hd, d};
        for (int i = box ? 4 : 0; i < 12; ++i) {   // the box family has no projection MLP
            const int k = job.count++;
            job.p[k] = ts[i]->p; job.m[k] = ts[i]->m; job.v[k] = ts[i]->v;
            job.g[k] = ptr<float>(c->gW) + c->gw_off[i];
            job.n[k] = sz[i % 4];
        }
    }
    if (!short_pass) {    // the passes that run long on their own: not in the launch that ends the step
        if (!aside) {
            Timed tm(c, NGDB_TK_TABLE_E, stream);
            HIPCHK(c, launch_table_update(te, ah, false, max_rows, stream));
        }
        Timed tm(c, NGDB_TK_ADAM, stream);
        HIPCHK(c, launch_dense_adam(job, ah, stream));
        job.count = 0;
    }
    if (aside) {
        HIPCHK(c, hipStreamWaitEvent(stream, c->ev_join, 0));
        end.forked = false;
    }
    {
        Timed tm(c, short_pass ? NGDB_TK_ADAM : NGDB_TK_TABLE_R, stream);
        const int64_t left = aside ? std::min<int64_t>(hp.n_anchor, max_rows) : (short_pass ? max_rows : 0);
        HIPCHK(c, launch_step_tail(te, left, small, n_small, c->cfg.n_relations, job, loss_sum, ah, stream));
    }
    if (sem) {
        // gradient of the text projection over the touched rows, then its Adam step
        Timed tm(c, NGDB_TK_SEM, stream);
        const int ds = c->cfg.d_sem;
        SemWgradArgs wa{};
        wa.H = c->prm.H_sem; wa.ids = ptr<int32_t>(c->uniq); wa.G = ptr<uint16_t>(c->g_bf16);
        wa.n_rows_dev = ptr<int32_t>(c->n_uniq); wa.n_rows = (int)std::min<int64_t>(n_contrib, c->cfg.n_entities);
        wa.d = d; wa.ds = ds; wa.n_splits = sem_wgrad_splits(wa.n_rows, d, ds); wa.partial = ptr<float>(c->wp_partial);
        HIPCHK(c, launch_sem_wgrad(wa, ptr<float>(c->gWp), stream));
        if (apply) {
            DenseAdamJob job{};
            job.p[0] = c->prm.Wp.p; job.m[0] = c->prm.Wp.m; job.v[0] = c->prm.Wp.v;
            job.g[0] = ptr<float>(c->gWp); job.n[0] = (int64_t)d * ds; job.count = 1;
            HIPCHK(c, launch_dense_adam(job, ah, stream));
        }
    }

    HIPCHK(c, end.close());
    if (apply) c->step = t;
    // describe the results
    ngdb_grad_view& gv = c->gv;
    std::memset(&gv, 0, sizeof(gv));
    gv.n_e_contrib = hp.n_anchor + B + B * K;
    gv.n_r_uniq = (int32_t)hp.r_uniq.size();
    gv.n_slots = hp.n_slots;
    gv.n_pairs = B * (K + 1);
    gv.e_uniq = ptr<int32_t>(c->uniq);
    gv.e_seg_off = ptr<int32_t>(c->seg_off);
    gv.e_src = e_src;
    gv.gE = apply ? nullptr : ptr<float>(c->gE);
    gv.gR = apply ? nullptr : ptr<float>(c->gR);
    for (int i = box ? 4 : 0; i < 12; ++i) gv.g_mlp[i] = ptr<float>(c->gW) + c->gw_off[i];
    if (box) {
        gv.gRo = apply ? nullptr : ptr<float>(c->gRo);
        gv.off = ptr<float>(c->off);
        gv.doff = ptr<float>(c->doff);
    }
    gv.e_shadow = c->cfg.score_bf16 ? ptr<uint16_t>(c->Eb) : nullptr;
    gv.g_Wp = sem ? ptr<float>(c->gWp) : nullptr;
    gv.act = ptr<float>(c->act);
    gv.dact = ptr<float>(c->dact);
    gv.n_grad_rows = hp.n_slots + hp.n_anchor;
    gv.pair_score = ptr<float>(c->score);
    gv.loss_terms = ptr<float>(c->loss_terms);
    c->have_grads = true;
    return NGDB_OK;
}

bool new_blob(ngdb_ctx_t* c, size_t cap, PlanBlob* pb) {
    pb->cap = cap;
    if (hipMalloc((void**)&pb->dev, cap * 4) != hipSuccess ||
        hipHostMalloc((void**)&pb->pinned, cap * 4, hipHostMallocDefault) != hipSuccess ||
        hipEventCreateWithFlags(&pb->last_use, hipEventDisableTiming) != hipSuccess) {
        if (pb->dev) (void)hipFree(pb->dev);
        if (pb->pinned) (void)hipHostFree(pb->pinned);
        *pb = PlanBlob{};
        return false;
    }
    c->n_alloc += 2;
    return true;
}

// The whole workspace and four plan buffers for the largest batch the configuration declares
// (b_max_queries queries of at most max_nodes_per_query nodes, k_max negatives): every count a plan
// can reach is bounded by the number of nodes.
int presize(ngdb_ctx_t* c) {
    const size_t B = (size_t)c->cfg.b_max_queries, cap = B * (size_t)c->cfg.max_nodes_per_query;
    if (cap > (size_t)INT32_MAX / 4 || B * ((size_t)c->cfg.k_max + 1) > (size_t)INT32_MAX)
        return fail(c, NGDB_ERR_ARG, "declared maxima too large");
    ngdb_plan_s most;
    HostPlan& hp = most.hp;
    hp.n_queries = (int32_t)B;
    hp.n_slots = hp.n_anchor = hp.n_proj = hp.n_int_rows = hp.n_neg = hp.n_roots = (int32_t)cap;
    hp.n_f_rows = (int32_t)cap;
    for (int t = 0; t < 3; ++t) hp.f_step_rows[t] = (int32_t)cap;
    hp.in_ref.resize(cap);
    int rc = size_workspace(c, &most, c->cfg.k_max, false);
    if (rc != NGDB_OK) return rc;
    const size_t blob_cap = 10 * cap + 4 * B + 2 * (size_t)std::min<size_t>(cap, c->cfg.n_relations) + 256;
    for (int i = 0; i < 4; ++i) {
        PlanBlob pb;
        if (!new_blob(c, blob_cap, &pb)) return fail(c, NGDB_ERR_OOM, "allocation of the plan buffers failed");
        c->blob_pool.push_back(pb);
    }
    c->presized = true;
    return NGDB_OK;
}

// ---- all-entity passes: the entity rows chunk by chunk
constexpr int RANK_CHUNK = RANK_PIECE;
// A filtered top-k takes chunks of up to NEAR_CHUNK: what a chunk costs beside its sums (merging, the launches of an fp32 pass that
// finds nothing to do) is 50 us whatever its size.  5 million fused entities x 1024 queries 28.5 ms in chunks of 65 536, 27.7 of twice
// that, 26.6 of four times that; a table of 2.5 million x 512 queries 7.7, 7.06, 6.8.  NEAR_PAIRS bounds the (branch row, entity) pairs of a
// chunk, for which the tiles need half a byte each to say what they found (256 MiB).  The fp32 pass walks a chunk by as many pieces of RANK_CHUNK
// as have distances of 256 MiB (NEAR_DIST of them), at least one, so that the distances take no more memory than those of an unfiltered pass of 1024 rows;
// its launches, which normally find nothing to do, cost 2.2 us each (345 queries x 717 000 entities x 292: 1314 us a piece at a time, 1304 two).
constexpr int NEAR_CHUNK = RANK_PIECES * RANK_CHUNK;
constexpr int64_t NEAR_PAIRS = 1 << 29, NEAR_DIST = 1 << 26;
constexpr int RANK_SAMPLE = 2048;      // most rows ranked in fp32 first (top-k of several pieces); rows the integer grid is made from
constexpr int RANK_ROOM = 4096;        // entities per query and chunk that the filtered ranks may leave undecided (top-k: rank_filter.hip)

// Where a chunk of entity rows lies: in the table (or its bf16 copy), or, with text features, fused
// into the context's chunk buffer by this call.  sample: there, too, RANK_SAMPLE rows spread over the table (a launch
// of its own for so few workgroups takes 100 us).  grid: rows fused here are also put on it.
struct ChunkRows { const float* rows; const uint16_t* rows16; const float* sample; };
int rank_chunk_rows(ngdb_ctx_t* c, int e0, int cnt, bool sample, const RankFilter* grid, hipStream_t s, ChunkRows* out) {
    const int d = c->cfg.d;
    *out = ChunkRows{c->prm.E.p + (size_t)e0 * d, c->cfg.score_bf16 ? ptr<uint16_t>(c->Eb) + (size_t)e0 * d : nullptr, nullptr};
    if (c->cfg.d_sem == 0) return NGDB_OK;
    SemFuseArgs fa = fuse_args(c);
    fa.id_base = e0; fa.n_rows = cnt; fa.out = ptr<float>(c->rank_ef);
    if (sample) {
        fa.n_seq = cnt; fa.n_rows += RANK_SAMPLE; fa.spread = c->cfg.n_entities / RANK_SAMPLE;
        out->sample = fa.out + (size_t)cnt * d;
    }
    if (grid) { fa.bits = grid->bits; fa.ldq = grid->lde; fa.words = grid->words; fa.lo = grid->lo; fa.grid = grid->grid; fa.Q = grid->Eq; fa.err = grid->slack; }
    HIPCHK(c, launch_sem_fuse(fa, s));
    out->rows = ptr<float>(c->rank_ef);
    return NGDB_OK;
}

// Lays the buffers of a filtered pass over R branch rows of B queries out from `base` (null: only for their size, in bytes).
size_t rank_filter_layout(const ngdb_ctx_t* c, int bits, int R, int B, int chunk, void* base, RankFilter* f) {
    *f = RankFilter{};
    f->d = c->cfg.d; f->bits = bits; f->words = rank_filter_words(f->d, bits);
    f->ldy = (R + 127) / 128 * 128; f->lde = (chunk + 127) / 128 * 128; f->room = RANK_ROOM;
    f->parts = c->cfg.d_sem > 0 ? sem_fuse_parts(f->d) : 1;
    const int n_lists = B * (bits == 8 ? (chunk + RANK_CHUNK - 1) / RANK_CHUNK : 1);
    f->n_counters = n_lists + c->cfg.n_entities / RANK_CHUNK + 32;
    size_t at = 0;
    auto place = [&](auto*& p, size_t words) {
        p = base ? reinterpret_cast<std::remove_reference_t<decltype(p)>>(static_cast<uint32_t*>(base) + at) : nullptr;
        at += (words + 63) / 64 * 64;
    };
    place(f->part, (size_t)32 * f->d);
    place(f->lo, f->d);
    place(f->grid, 2);
    place(f->Yq, (size_t)f->words * f->ldy);
    place(f->base, 2 * (size_t)f->ldy);
    place(f->row_q, f->ldy);
    place(f->Eq, (size_t)f->words * f->lde);
    place(f->slack, (size_t)f->parts * f->lde);
    place(f->list, bits == 16 ? (size_t)B * f->room : 0);
    place(f->found, bits == 8 ? (size_t)f->ldy * (f->lde / 128) : 0);
    place(f->found_pair, bits == 8 ? rank_found_bytes(f->ldy, f->lde) / 4 : 0);
    place(f->count, f->n_counters);
    f->overflowed = base ? f->count + n_lists : nullptr;
    f->gave_up = gave_up_mark(c);
    return at * 4;
}

// Buffers of a ranking: distances [R, ld] of a piece, fused rows (text features), and those of a filter of `bits` over chunks of `chunk` entities (0: none).
int rank_buffers(ngdb_ctx_t* c, int R, int B, int ld, int64_t fused_rows, int bits, int chunk, RankFilter* f) {
    int rc = ensure(c, c->rank_dist, std::max<size_t>((size_t)R * ld * sizeof(float), 256), Use::Ranking);
    if (rc == NGDB_OK && c->cfg.d_sem > 0) rc = ensure(c, c->rank_ef, ((size_t)fused_rows + RANK_SAMPLE) * c->cfg.d * sizeof(float), Use::Ranking);
    if (rc == NGDB_OK && bits) {
        rc = ensure(c, c->rank_filter, rank_filter_layout(c, bits, R, B, chunk, nullptr, f), Use::Ranking);
        if (rc == NGDB_OK) rank_filter_layout(c, bits, R, B, chunk, c->rank_filter.p, f);
    }
    return rc;
}

int no_rank_memory(ngdb_ctx_t* c) { return fail(c, NGDB_ERR_OOM, "no device memory for the buffers of a ranking"); }

// Device memory that an allocation of this context can have.
size_t device_free(const ngdb_ctx_t* c) {
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return std::min(avail, c->held_limit > c->held ? c->held_limit - c->held : 0);
}

// The filter serves the plain distance (vector family).  It replaces two operations per coordinate by a quarter (top-k) or a
// half of one, for launches and lists of its own and for rounding the entity rows: below `from` the fp32 pass is through first.
// Top-k: the fp32 tiles take 32, 64 or 128 rows at a time, filled or not, and rounding the table costs about as much as 48
// rows.  (These rows - 48) x entities x coordinates in 1e9, then us in fp32 and with the filter: 15 000 entities x 584 rows
// x 256 coordinates (2.3) 228 and 220, 60 000 x 228 x 256 (3.2) 253 and 269, 15 000 x 584 x 400 (3.6) 322 and 284,
// 30 000 x 292 x 400 (4.0) 305 and 315, 100 000 x 114 x 400 (3.2) 364 and 428, 200 000 x 114 x 256 (4.1) 434 and 415,
// 300 000 x 114 x 400 (9.6) 801 and 767; 500 000 x 56 x 400 (3.2) 817 and 909, 500 000 x 72 x 400 (16) 1201 and 1026;
// with 8 to 18 rows (below 0) the filter was 6 to 25 % slower from 500 000 to 2.5 million entities.
// Answers: the filter's counting takes as long per pair as 64 coordinates save, and each chunk has launches of its own:
// 502 us in fp32 and 602 with the filter at 200 000 x 585 x 64, 250 and 230 at 15 000 x 585 x 256, 439 and 586 at 200 000 x 114 x
// 256 (four chunks), 1357 and 1180 at 200 000 x 585 x 256.
// A table of one piece, or of up to four whose sums fit 256 MiB, needs no fp32 rows, lists or chunks (pick_kernel), and the filter pays from less on, in the same units and order:
// 8000 x 228 x 400 (0.67) 130 and 137, 30 000 x 114 x 400 (0.96) 160 and 147, 15 000 x 585 x 128 (1.1) 157 and 131, 5000 x 585 x 400 (1.2) 168 and
// 157, 60 000 x 114 x 400 (1.9) 228 and 177, 65 000 x 1171 x 400 (32) 1402 and 447; with chunks from a sample of 2048 rows on the filter took
// 184, 261, 151, 192, 291 and 540.  60 000 x 28 x 400 (below 0) 127 and 143.  Several pieces, from a sample on and as a whole: 70 000 x 585 x 400 396 and
// 309, 100 000 x 114 x 400 301 and 217, 200 000 x 57 x 400 352 and 266, 262 144 x 228 x 400 602 and 477 (not with text features, whose rows are rounded as they
// are fused in the chunks, and here would be by a launch that reads them again).
constexpr double NEAR_FROM = 3.3e9, WHOLE_FROM = 0.8e9;
double near_work(const ngdb_ctx_t* c, int n_rows) {
    const int tile_rows = n_rows <= 32 ? 32 : (n_rows <= 64 ? 64 : (n_rows + 127) / 128 * 128);
    return (double)(tile_rows - 48) * c->cfg.n_entities * c->cfg.d;
}
bool rank_filtered(const ngdb_ctx_t* c, int n_rows, double work, double from) {
    if (c->cfg.family != NGDB_FAMILY_VEC || c->cfg.n_entities <= 2 * RANK_SAMPLE) return false;
    if (c->rank_filter_from >= 0) return (double)n_rows * c->cfg.n_entities * c->cfg.d >= (double)c->rank_filter_from;
    return work >= from;
}

// The grid of a filtered pass, from rows spread over the table (the first rows alone would leave a table that is ordered
// by kind with most of its rows off the grid, every list overflowing and every chunk paid twice).
int rank_filter_begin(ngdb_ctx_t* c, const RankFilter& f, const float* fused_sample, hipStream_t s) {
    HIPCHK(c, launch_rank_grid(f, fused_sample ? fused_sample : c->prm.E.p, c->cfg.score_bf16 ? ptr<uint16_t>(c->Eb) : nullptr,
                               fused_sample ? 1 : c->cfg.n_entities / RANK_SAMPLE, RANK_SAMPLE, s));
    return NGDB_OK;
}

int rank_nearest(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* roots, int topk, int32_t* d_ids, float* d_dist, hipStream_t s) {
    const int N = c->cfg.n_entities, d = c->cfg.d, R = pl->hp.n_roots, B = pl->hp.n_queries;
    const float* act = c->rows_chained ? rows_chain_act(c) : ptr<float>(c->act);
    const float* box_off = c->cfg.family == NGDB_FAMILY_BOX ? ptr<float>(c->off) : nullptr;
    const bool whole = !c->rank_by_chunks && (N <= RANK_CHUNK || (c->cfg.d_sem == 0 && N <= NEAR_CHUNK && (int64_t)R * N <= NEAR_DIST));
    bool filtered = rank_filtered(c, R, near_work(c, R), whole ? WHOLE_FROM : NEAR_FROM);
    const bool needed = c->rank_filter_from >= 0 || near_work(c, R) >= NEAR_FROM;
    RankFilter f{};
    int most = RANK_CHUNK, chunk, at_once, ld, rc;
    while (filtered && most < std::min(N, NEAR_CHUNK) && 2ll * most * R <= NEAR_PAIRS) most *= 2;
    if (most > c->near_most) {
        // There was no memory for such chunks.  They are tried again once as much more is free as one needs (not while the
        // stream is captured: nothing may be allocated then).
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        const size_t more = (size_t)NEAR_DIST * sizeof(float) + (c->cfg.d_sem > 0 ? (size_t)most * d * sizeof(float) : 0) + rank_filter_layout(c, 8, R, B, most, nullptr, &f);
        if (hipStreamIsCapturing(s, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone && device_free(c) >= c->near_free + more + more / 4) c->near_most = INT32_MAX;
        (void)hipGetLastError();
        most = std::min(most, c->near_most);
    }
    for (bool emptied = false, shorter = false;; emptied = true) {
        chunk = std::min(N, most);
        at_once = RANK_CHUNK;                // (short of memory: a piece)
        while (!emptied && at_once < chunk && (2ll * at_once * R <= NEAR_DIST || (whole && filtered))) at_once *= 2;
        ld = (std::min(chunk, at_once) + 3) & ~3;
        rc = rank_buffers(c, R, B, ld, chunk, filtered ? 8 : 0, chunk, &f);
        if (rc == NGDB_ERR_OOM && emptied && filtered && !needed) {      // (fp32 takes little longer, and the distances only)
            filtered = false;
            most = RANK_CHUNK;
        } else if (rc != NGDB_ERR_OOM || (emptied && most == RANK_CHUNK)) {
            if (rc == NGDB_OK && shorter) c->near_free = device_free(c);
            break;
        }
        // a buffer that is larger than the next attempt needs would stay and take the memory from the others
        release_rank_buffers(c);
        if (most > RANK_CHUNK) {
            c->near_most = most /= 2;
            shorter = true;
        }
    }
    c->rank_overflowed = rc == NGDB_OK ? f.overflowed : nullptr;
    if (rc != NGDB_OK) return rc == NGDB_ERR_OOM ? no_rank_memory(c) : rc;
    float* dist = ptr<float>(c->rank_dist);
    Overflowed only{f.row_q, f.count, f.room, f.overflowed, B};
    const RankRows rows{act, roots, R, pl->d_root_off, B};
    Timed tm(c, NGDB_TK_SCORE, s);
    if (filtered && whole && ld >= N) {      // (a table of several pieces: unless short of memory) the sums of all entities, the nearest of these, and what had no room in fp32
        ChunkRows er;
        if ((rc = rank_chunk_rows(c, 0, N, true, nullptr, s, &er)) != NGDB_OK) return rc;
        if ((rc = rank_filter_begin(c, f, er.sample, s)) != NGDB_OK) return rc;
        f.parts = 1;                         // (the rows are fused with those of the sample, and rounded after them)
        uint32_t* sums = reinterpret_cast<uint32_t*>(dist);
        HIPCHK(c, launch_quantise(f, &rows, er.rows, er.rows16, N, s));
        HIPCHK(c, launch_sum_tile(f, R, N, sums, ld, s));
        HIPCHK(c, launch_pick(f, sums, ld, act, roots, pl->d_root_off, B, er.rows, er.rows16, N, topk, d_dist, d_ids, s));
        only.any = f.overflowed;
        HIPCHK(c, launch_l1_tile(act, box_off, c->cfg.box_alpha, roots, R, er.rows, N, d, dist, ld, s, er.rows16, &only));
        HIPCHK(c, launch_topk_merge(dist, ld, pl->d_root_off, B, 0, N, topk, false, d_dist, d_ids, gave_up_mark(c), s, &only));
        c->rank_chunks = (N + RANK_CHUNK - 1) / RANK_CHUNK;
        return NGDB_OK;
    }
    // filtered: the sample's k-th distance lets k / sample of the first chunk pass, and chunks grow with what has
    // been ranked (each at most 12 times that), so that a list holds 12 k entities and some that are only near it
    const int sample = std::min(RANK_SAMPLE, std::max(512, 128 * topk));
    int i_piece = 0;
    for (int e0 = 0; e0 < N;) {
        const int want = !filtered ? chunk : (e0 == 0 ? sample : (int)std::min<int64_t>(chunk, 12ll * e0));
        const int cnt = std::min(want, N - e0);
        ChunkRows er;
        const bool rounded = filtered && e0 > 0;
        if ((rc = rank_chunk_rows(c, e0, cnt, filtered && e0 == 0, rounded ? &f : nullptr, s, &er)) != NGDB_OK) return rc;
        if (!rounded) {
            HIPCHK(c, launch_l1_tile(act, box_off, c->cfg.box_alpha, roots, R, er.rows, cnt, d, dist, ld, s, er.rows16));
            HIPCHK(c, launch_topk_merge(dist, ld, pl->d_root_off, B, e0, cnt, topk, e0 == 0, d_dist, d_ids, gave_up_mark(c), s));
            if (filtered && (rc = rank_filter_begin(c, f, er.sample, s)) != NGDB_OK) return rc;
            ++i_piece;
        } else {
            const bool fused = c->cfg.d_sem > 0;
            if (!fused || e0 == sample) HIPCHK(c, launch_quantise(f, e0 == sample ? &rows : nullptr, er.rows, er.rows16, fused ? 0 : cnt, s));
            HIPCHK(c, launch_near_tile(f, R, cnt, d_dist, topk, s));
            HIPCHK(c, launch_near_merge(f, i_piece, act, roots, pl->d_root_off, B, er.rows, er.rows16, e0, cnt, topk, d_dist, d_ids, s));
            for (int p0 = 0; p0 < cnt; p0 += at_once) {
                const int n = std::min(at_once, cnt - p0);
                const size_t at = (size_t)p0 * d;
                only.count = f.count + (size_t)(p0 / RANK_CHUNK) * B;
                only.any = f.overflowed + i_piece;
                HIPCHK(c, launch_l1_tile(act, box_off, c->cfg.box_alpha, roots, R, er.rows + at, n, d, dist, ld, s, er.rows16 ? er.rows16 + at : nullptr, &only));
                HIPCHK(c, launch_topk_merge(dist, ld, pl->d_root_off, B, e0 + p0, n, topk, false, d_dist, d_ids, gave_up_mark(c), s, &only));
                i_piece += (n + RANK_CHUNK - 1) / RANK_CHUNK;
            }
        }
        e0 += cnt;
    }
    c->rank_chunks = i_piece;
    return NGDB_OK;
}

int rank_listed(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* roots, const int32_t* d_ans_off, const int32_t* d_ans, int n_ans,
                int32_t* d_rank, float* d_ans_dist, hipStream_t s) {
    const int N = c->cfg.n_entities, d = c->cfg.d, R = pl->hp.n_roots, B = pl->hp.n_queries;
    const float* act = c->rows_chained ? rows_chain_act(c) : ptr<float>(c->act);
    const float* box_off = c->cfg.family == NGDB_FAMILY_BOX ? ptr<float>(c->off) : nullptr;
    const bool sem = c->cfg.d_sem > 0;
    // (with very many answers per query most entities are undecided for one of them)
    const int chunk = std::min(N, RANK_CHUNK), ld = (chunk + 3) & ~3;
    const bool filtered = rank_filtered(c, R, (double)R * N * (d - 64), 1.4e9 + 3.7e9 * ((N - 1) / chunk)) && n_ans <= 64ll * B;
    RankFilter f{};
    int rc = ensure(c, c->rank_count, (size_t)n_ans * 8, Use::Evaluation);
    if (rc == NGDB_OK && !d_ans_dist) rc = ensure(c, c->rank_thr, (size_t)n_ans * 4, Use::Evaluation);
    for (bool emptied = false; rc == NGDB_OK; emptied = true) {
        rc = rank_buffers(c, R, B, ld, std::max(chunk, std::min(n_ans, RANK_CHUNK)), filtered ? 16 : 0, chunk, &f);
        if (rc != NGDB_ERR_OOM || emptied) break;
        release_rank_buffers(c);             // (a top-k has left larger ones)
        rc = NGDB_OK;
    }
    c->rank_overflowed = rc == NGDB_OK ? f.overflowed : nullptr;
    c->rank_chunks = (N + chunk - 1) / chunk;
    if (rc != NGDB_OK) return rc == NGDB_ERR_OOM ? no_rank_memory(c) : rc;
    float* dist = ptr<float>(c->rank_dist);
    float* thr = d_ans_dist ? d_ans_dist : ptr<float>(c->rank_thr);
    int32_t* total = ptr<int32_t>(c->rank_count);
    int32_t* in_chunk = total + n_ans;
    const RankRows rows{act, roots, R, pl->d_root_off, B};
    Overflowed only{f.row_q, f.count, f.room, f.overflowed, B};
    Timed tm(c, NGDB_TK_SCORE, s);
    // distance of every listed answer to its query (the arithmetic of the all-entity pass, so an answer
    // compares equal to itself there)
    for (int a0 = 0; a0 < n_ans; a0 += RANK_CHUNK) {
        const int cnt = std::min(RANK_CHUNK, n_ans - a0);
        const float* ans_rows = c->prm.E.p;
        if (sem) {
            SemFuseArgs fa{};
            fa.H = c->prm.H_sem; fa.Wb = ptr<uint16_t>(c->Wb); fa.E = c->prm.E.p; fa.ids = d_ans + a0; fa.n_rows = cnt;
            fa.d = d; fa.ds = c->cfg.d_sem; fa.out = ptr<float>(c->rank_ef);
            HIPCHK(c, launch_sem_fuse(fa, s));
            ans_rows = ptr<float>(c->rank_ef);
        }
        HIPCHK(c, launch_answer_distance(act, box_off, c->cfg.box_alpha, roots, pl->d_root_off, d_ans_off, B, sem ? nullptr : d_ans, a0, cnt,
                                         ans_rows, c->cfg.score_bf16 ? ptr<uint16_t>(c->Eb) : nullptr, d, gave_up_mark(c), thr, total, n_ans, s));
    }
    // entities strictly closer than each answer, chunk by chunk
    for (int e0 = 0; e0 < N; e0 += chunk) {
        const int cnt = std::min(chunk, N - e0);
        ChunkRows er;
        const bool rounded = filtered && sem && e0 > 0;      // (the first chunk's rows hold the sample that the grid comes from)
        if ((rc = rank_chunk_rows(c, e0, cnt, filtered && e0 == 0, rounded ? &f : nullptr, s, &er)) != NGDB_OK) return rc;
        if (filtered) {
            if (e0 == 0 && (rc = rank_filter_begin(c, f, er.sample, s)) != NGDB_OK) return rc;
            f.parts = rounded ? sem_fuse_parts(d) : 1;
            if (!rounded) HIPCHK(c, launch_quantise(f, e0 == 0 ? &rows : nullptr, er.rows, er.rows16, cnt, s));
            HIPCHK(c, launch_sum_tile(f, R, cnt, reinterpret_cast<uint32_t*>(dist), ld, s));
            HIPCHK(c, launch_count_sure(f, reinterpret_cast<const uint32_t*>(dist), ld, pl->d_root_off, d_ans_off, thr, B, cnt, in_chunk, s));
            HIPCHK(c, launch_count_open(f, e0 / chunk, reinterpret_cast<const uint32_t*>(dist), ld, act, roots, pl->d_root_off, d_ans_off, thr, B, er.rows, er.rows16, in_chunk, total, s));
            only.any = f.overflowed + e0 / chunk;
        }
        HIPCHK(c, launch_l1_tile(act, box_off, c->cfg.box_alpha, roots, R, er.rows, cnt, d, dist, ld, s, er.rows16, filtered ? &only : nullptr));
        HIPCHK(c, launch_count_less(dist, ld, pl->d_root_off, d_ans_off, thr, B, cnt, total, s, filtered ? &only : nullptr));
        if (filtered && e0 + cnt < N) HIPCHK(c, launch_fill_zero_i32(f.count, B, s));
    }
    HIPCHK(c, launch_finish_rank(total, thr, d_ans_off, B, n_ans, gave_up_mark(c), d_rank, s));
    return NGDB_OK;
}

// Device address of the scratch array on the current GPU (looked up on first use per device).
hipError_t noalloc_scratch(unsigned char** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        unsigned char* p = nullptr;
        e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

// ------------------------------------------------------------------------ C ABI
extern "C" {

int ngdb_create(const ngdb_config* cfg, ngdb_ctx_t** out) {
    if (!cfg || !out) return NGDB_ERR_ARG;
    *out = nullptr;
    if (cfg->n_entities <= 0 || cfg->n_relations <= 0 || cfg->d <= 0 || cfg->h <= 0 || (cfg->d & 3) ||
        (cfg->h & 3) || cfg->d > 1024 || cfg->num_streams < 1 || cfg->num_streams > 4 || cfg->d_sem < 0)
        return NGDB_ERR_ARG;
    if (cfg->d_sem != 0 && ((cfg->d_sem & 63) || (cfg->d & 7))) return NGDB_ERR_ARG;
    if ((cfg->schedule != NGDB_SCHED_LEVEL && cfg->schedule != NGDB_SCHED_MAX_FILL) || cfg->b_max < 0) return NGDB_ERR_ARG;
    if (cfg->family != NGDB_FAMILY_VEC && cfg->family != NGDB_FAMILY_BOX) return NGDB_ERR_ARG;
    if (cfg->family == NGDB_FAMILY_BOX && (cfg->d_sem != 0 || !(cfg->box_alpha >= 0.f && cfg->box_alpha <= 1.f)))
        return NGDB_ERR_ARG;
    if ((cfg->score_bf16 != 0 && cfg->score_bf16 != 1) || (cfg->score_bf16 && (cfg->family != NGDB_FAMILY_VEC || cfg->d_sem != 0 || (cfg->d & 7))))
        return NGDB_ERR_ARG;
    if (cfg->b_max_queries < 0 || cfg->k_max < 0 || cfg->max_nodes_per_query < 0 ||
        (cfg->b_max_queries > 0 && cfg->k_max < 1) || (cfg->b_max_queries == 0 && (cfg->k_max || cfg->max_nodes_per_query)))
        return NGDB_ERR_ARG;
    ngdb_ctx_t* c = new (std::nothrow) ngdb_ctx_s();
    if (!c) return NGDB_ERR_OOM;
    c->cfg = *cfg;
    if (c->cfg.b_max_queries > 0 && c->cfg.max_nodes_per_query == 0) c->cfg.max_nodes_per_query = 12;
    c->n_side = cfg->num_streams > 1 ? 1 : 0;
    bool ok = true;
    if (c->n_side) ok = hipStreamCreateWithFlags(&c->side[0], hipStreamNonBlocking) == hipSuccess;
    // (they order work of this GPU only: no fence towards the host, 2 us of a launch queue and of host time each)
    const unsigned ev_flags = hipEventDisableTiming | hipEventDisableSystemFence;
    ok = ok && hipEventCreateWithFlags(&c->ev_join, ev_flags) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->ev_fork, ev_flags) == hipSuccess;
    ok = ok && hipStreamCreateWithFlags(&c->upload, hipStreamNonBlocking) == hipSuccess;
    unsigned char* sp = nullptr;
    ok = ok && noalloc_scratch(&sp) == hipSuccess;     // address of the static scratch on this GPU
    ok = ok && device_alloc(c, c->sync, SYNC_WORDS * sizeof(int32_t) + rows_chain_bytes(c)) == hipSuccess && launch_fill_zero_i32(ptr<int32_t>(c->sync), SYNC_WORDS, nullptr) == hipSuccess &&
         hipStreamSynchronize(nullptr) == hipSuccess;
    ok = ok && hipHostMalloc((void**)&c->gave_up, sizeof(int32_t), hipHostMallocDefault) == hipSuccess;
    if (ok) {
        *c->gave_up = 0;
        ++c->n_alloc;
    }
    if (!ok) {
        ngdb_destroy(c);
        return NGDB_ERR_HIP;
    }
    if (c->cfg.b_max_queries > 0) {
        const int rc = presize(c);
        if (rc != NGDB_OK) {
            ngdb_destroy(c);
            return rc;
        }
    }
    *out = c;
    return NGDB_OK;
}

void ngdb_destroy(ngdb_ctx_t* c) {
    if (!c) return;
    (void)hipDeviceSynchronize();
    DevBuf* all[] = {&c->act, &c->dact, &c->Z[0], &c->Z[1], &c->Z[2], &c->H[0], &c->H[1], &c->H[2], &c->dH[0],
                     &c->dH[1], &c->dH[2], &c->Att, &c->dAtt, &c->Dx, &c->score, &c->coef, &c->win, &c->mask,
                     &c->loss_terms, &c->rec_coef, &c->rec_row, &c->keys_a, &c->keys_b, &c->vals_a, &c->vals_b, &c->hist, &c->scan_tmp,
                     &c->uniq, &c->seg_off, &c->n_uniq, &c->gW, &c->w_pieces, &c->sync, &c->h_pieces, &c->gE, &c->gR, &c->rank_dist, &c->rank_thr, &c->rank_count, &c->rank_filter,
                     &c->Wb, &c->Ef, &c->Ea, &c->inv, &c->refs_sem, &c->g_bf16, &c->wp_partial, &c->gWp, &c->rank_ef,
                     &c->off, &c->doff, &c->Gate, &c->dGate, &c->DxO, &c->gRo, &c->Eb, &c->later};
    for (DevBuf* b : all) release(c, *b);
    if (c->gave_up) (void)hipHostFree(c->gave_up);
    if (c->side[0]) (void)hipStreamDestroy(c->side[0]);
    if (c->ev_join) (void)hipEventDestroy(c->ev_join);
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    if (c->upload) (void)hipStreamDestroy(c->upload);
    // plans that outlive the context keep their host arrays (export, free) and lose their device buffer
    for (ngdb_plan_t* pl : c->live_plans) {
        c->blob_pool.push_back(pl->blob);
        pl->blob = PlanBlob{};
        pl->d_blob = nullptr;
        pl->owner = nullptr;
    }
    c->live_plans.clear();
    for (PlanBlob& b : c->blob_pool) {
        if (b.dev) (void)hipFree(b.dev);
        if (b.pinned) (void)hipHostFree(b.pinned);
        if (b.last_use) (void)hipEventDestroy(b.last_use);
    }
    for (const ngdb_ctx_s::Bracket& b : c->brackets) {
        (void)hipEventDestroy(b.a);
        (void)hipEventDestroy(b.b);
    }
    for (hipEvent_t e : c->spare_events) (void)hipEventDestroy(e);
    delete c;
}

int ngdb_bind_params(ngdb_ctx_t* c, const ngdb_params* p) {
    if (!c || !p) return NGDB_ERR_ARG;
    const bool box = c->cfg.family == NGDB_FAMILY_BOX;
    const ngdb_tensor* ts[14] = {&p->E, &p->R, &p->V1, &p->c1, &p->V2, &p->c2, &p->U1, &p->u1, &p->U2, &p->u2,
                                 box ? &p->Ro : &p->W1, box ? &p->Ro : &p->b1, box ? &p->Ro : &p->W2,
                                 box ? &p->Ro : &p->b2};
    for (const ngdb_tensor* t : ts) {
        if (!t->p || !t->m || !t->v) return fail(c, NGDB_ERR_ARG, "null parameter or moment tensor");
        if (((uintptr_t)t->p | (uintptr_t)t->m | (uintptr_t)t->v) & 15)
            return fail(c, NGDB_ERR_ARG, "tensors must be 16-byte aligned");
    }
    if (c->cfg.d_sem > 0) {
        if (!p->Wp.p || !p->Wp.m || !p->Wp.v || !p->H_sem)
            return fail(c, NGDB_ERR_ARG, "text features configured: Wp (with moments) and H_sem are required");
        if (((uintptr_t)p->Wp.p | (uintptr_t)p->Wp.m | (uintptr_t)p->Wp.v | (uintptr_t)p->H_sem) & 15)
            return fail(c, NGDB_ERR_ARG, "tensors must be 16-byte aligned");
    }
    if (p->step < 0) return fail(c, NGDB_ERR_ARG, "negative step count");
    if (c->cfg.score_bf16) {   // the bf16 copy of the entity table
        const size_t n = (size_t)c->cfg.n_entities * c->cfg.d;
        int rc = ensure(c, c->Eb, n * sizeof(uint16_t), Use::Evaluation);
        if (rc != NGDB_OK) return rc;
        HIPCHK(c, launch_cast_bf16(p->E.p, ptr<uint16_t>(c->Eb), (int64_t)n, nullptr));
        HIPCHK(c, hipDeviceSynchronize());
    }
    c->prm = *p;
    c->step = p->step;
    c->bound = true;
    c->have_grads = false;
    return NGDB_OK;
}

// host part of planning: frontiers, index arrays, level/type segments
static int plan_host(const ngdb_query_batch* qb, int32_t n_entities, int32_t n_relations, int32_t schedule,
                     int32_t b_max, ngdb_plan_t** out, std::string& err) {
    *out = nullptr;
    ngdb_plan_t* pl = new (std::nothrow) ngdb_plan_s();
    if (!pl) {
        err = "host allocation failed";
        return NGDB_ERR_OOM;
    }
    int rc = NGDB_OK;
    try {
        rc = build_plan(*qb, n_entities, n_relations, schedule, b_max, pl->hp, err);
    } catch (const std::bad_alloc&) {
        rc = NGDB_ERR_OOM;
        err = "host allocation failed";
    }
    if (rc != NGDB_OK) {
        delete pl;
        return rc;
    }
    HostPlan& hp = pl->hp;
    pl->n_entities = n_entities;
    pl->levels.assign(hp.n_levels + 1, {});
    for (int g = 0; g < hp.n_groups; ++g) {
        std::vector<Segment>& segs = pl->levels[hp.g_level[g]];
        const int t = type_index(hp.g_type[g]);
        const int rows = hp.g_n[g] * (t == T_INTER ? hp.g_nin[g] : 1);
        if (!segs.empty() && segs.back().type == t) {   // further intersection class of the same level
            segs.back().rows += rows;
            segs.back().g_hi = g + 1;
        } else {
            Segment sg;
            sg.type = t; sg.rows = rows; sg.mlp_base = hp.g_mlp_base[g]; sg.ref_off = hp.g_ref_off[g];
            sg.rel_off = hp.g_rel_off[g]; sg.out_base = hp.g_out_base[g]; sg.g_lo = g; sg.g_hi = g + 1;
            segs.push_back(sg);
        }
    }
    *out = pl;
    return NGDB_OK;
}

int ngdb_plan_host(int32_t n_entities, int32_t n_relations, const ngdb_query_batch* qb, ngdb_plan_t** out) {
    return ngdb_plan_host_sched(n_entities, n_relations, qb, NGDB_SCHED_LEVEL, 0, out);
}

int ngdb_plan_host_sched(int32_t n_entities, int32_t n_relations, const ngdb_query_batch* qb, int32_t schedule,
                         int32_t b_max, ngdb_plan_t** out) {
    if (!qb || !out || n_entities <= 0 || n_relations <= 0) return NGDB_ERR_ARG;
    std::string err;
    return plan_host(qb, n_entities, n_relations, schedule, b_max, out, err);
}

int ngdb_plan(ngdb_ctx_t* c, const ngdb_query_batch* qb, ngdb_plan_t** out) {
    if (!c || !qb || !out) return NGDB_ERR_ARG;
    std::string err;
    ngdb_plan_t* pl = nullptr;
    int rc = plan_host(qb, c->cfg.n_entities, c->cfg.n_relations, c->cfg.schedule, c->cfg.b_max, &pl, err);
    if (rc != NGDB_OK) return fail(c, rc, err);
    HostPlan& hp = pl->hp;
    if (c->presized && (hp.n_queries > c->cfg.b_max_queries ||
                        (size_t)hp.n_slots + hp.n_anchor > (size_t)c->cfg.b_max_queries * c->cfg.max_nodes_per_query)) {
        delete pl;
        return fail(c, NGDB_ERR_ARG, "batch beyond the maxima declared at ngdb_create (b_max_queries, max_nodes_per_query)");
    }
    if (c->cfg.family == NGDB_FAMILY_BOX) {
        bool ok = hp.n_neg == 0;
        for (int g = 0; g < hp.n_groups && ok; ++g) {
            if (hp.g_type[g] != NGDB_OP_INTER) continue;
            const int n_ref = hp.g_n[g] * hp.g_nin[g];
            for (int i = 0; i < n_ref && ok; ++i) ok = hp.in_ref[hp.g_ref_off[g] + i] >= 0;
        }
        if (!ok) {
            delete pl;
            return fail(c, NGDB_ERR_UNSUPPORTED, "box family: no negation, and an intersection input must be an operator output");
        }
    }

    // one upload: every device-side array, each padded to 16 bytes (at least 16)
    size_t blob_size = 0;
    auto place = [&](size_t n) {
        const size_t off = blob_size;
        blob_size += std::max<size_t>((n + 3) & ~size_t(3), 4);
        return off;
    };
    const size_t n_ekeys = hp.anchor_ent.size() + hp.pos.size();
    const size_t o_ref = place(hp.in_ref.size()), o_gs = place(hp.in_gslot.size()), o_rel = place(hp.rel.size()),
                 o_ro = place(hp.root_off.size()), o_rs = place(hp.root_slot.size()), o_pos = place(hp.pos.size()),
                 o_ek = place(n_ekeys), o_ru = place(hp.r_uniq.size()), o_rso = place(hp.r_seg_off.size()),
                 o_rsrc = place(hp.r_src.size()), o_rrec = place(hp.r_src.size()), o_nru = place(1),
                 o_fref = place(hp.in_ref.size()), o_frow = place(hp.f_row.size()), o_froot = place(hp.root_slot.size());
    // A recycled buffer whose last reader has finished; else a new one, as long as the context has few; else the
    // one that has been waiting longest.  (With a single buffer planning would wait for the step before.)
    PlanBlob pb;
    bool busy = false;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        size_t fits = c->blob_pool.size(), pick = fits;
        for (size_t i = 0; i < c->blob_pool.size() && pick == c->blob_pool.size(); ++i) {
            if (c->blob_pool[i].cap < blob_size) continue;
            if (fits == c->blob_pool.size()) fits = i;
            if (hipEventQuery(c->blob_pool[i].last_use) == hipSuccess) pick = i;
        }
        const bool enough = c->presized || c->blob_pool.size() + c->live_plans.size() >= 4;
        if (pick == c->blob_pool.size() && fits < pick && enough) {
            pick = fits;
            busy = true;
        }
        if (pick < c->blob_pool.size()) {
            pb = c->blob_pool[pick];
            c->blob_pool.erase(c->blob_pool.begin() + pick);
        } else {
            // one of those that are too small makes room once there are several
            for (size_t i = 0; enough && !c->presized && i < c->blob_pool.size(); ++i)
                if (c->blob_pool[i].cap < blob_size) {
                    PlanBlob& old = c->blob_pool[i];
                    (void)hipEventSynchronize(old.last_use);
                    (void)hipFree(old.dev);
                    (void)hipHostFree(old.pinned);
                    (void)hipEventDestroy(old.last_use);
                    c->blob_pool.erase(c->blob_pool.begin() + i);
                    break;
                }
            if (!new_blob(c, blob_size + blob_size / 2 + 1024, &pb)) pb = PlanBlob{};
        }
    }
    if (!pb.dev) {
        delete pl;
        return fail(c, NGDB_ERR_OOM, "allocation for the plan failed");
    }
    if (busy && hipEventSynchronize(pb.last_use) != hipSuccess) {
        delete pl;
        return fail(c, NGDB_ERR_HIP, "waiting for a recycled plan buffer failed");
    }
    {   // straight into the staging buffer
        int32_t* at = pb.pinned;
        auto put = [&](size_t off, const std::vector<int32_t>& v) {
            if (!v.empty()) std::memcpy(at + off, v.data(), v.size() * sizeof(int32_t));
        };
        put(o_ref, hp.in_ref); put(o_gs, hp.in_gslot); put(o_rel, hp.rel); put(o_ro, hp.root_off); put(o_rs, hp.root_slot);
        put(o_pos, hp.pos); put(o_ek, hp.anchor_ent); put(o_ek + hp.anchor_ent.size(), hp.pos); put(o_ru, hp.r_uniq);
        put(o_rso, hp.r_seg_off); put(o_rsrc, hp.r_src); put(o_frow, hp.f_row);
        for (size_t i = 0; i < hp.r_src.size(); ++i) at[o_rrec + i] = -1 - hp.r_src[i];   // relation contributions are gradient rows
        at[o_nru] = (int32_t)hp.r_uniq.size();
        for (size_t i = 0; i < hp.in_ref.size(); ++i) at[o_fref + i] = hp.in_ref[i] >= 0 ? hp.f_row[hp.in_ref[i]] : hp.in_ref[i];
        for (size_t i = 0; i < hp.root_slot.size(); ++i) at[o_froot + i] = hp.f_row[hp.root_slot[i]];
    }
    pl->blob_bytes = blob_size * 4;
    if (pl->blob_bytes > PLAN_INLINE_BYTES &&
        (hipMemcpyAsync(pb.dev, pb.pinned, pl->blob_bytes, hipMemcpyHostToDevice, c->upload) != hipSuccess ||
         hipStreamSynchronize(c->upload) != hipSuccess)) {
        {
            std::lock_guard<std::mutex> lk(c->mu);
            c->blob_pool.push_back(pb);
        }
        delete pl;
        return fail(c, NGDB_ERR_HIP, "plan upload failed");
    }
    pl->uploaded = pl->blob_bytes > PLAN_INLINE_BYTES;
    pl->owner = c;
    pl->blob = pb;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        c->live_plans.push_back(pl);
    }
    pl->d_blob = pb.dev;
    pl->d_in_ref = pl->d_blob + o_ref; pl->d_in_gslot = pl->d_blob + o_gs; pl->d_rel = pl->d_blob + o_rel;
    pl->d_root_off = pl->d_blob + o_ro; pl->d_root_slot = pl->d_blob + o_rs; pl->d_pos = pl->d_blob + o_pos;
    pl->d_ekeys_head = pl->d_blob + o_ek; pl->d_r_uniq = pl->d_blob + o_ru; pl->d_r_seg_off = pl->d_blob + o_rso;
    pl->d_r_src = pl->d_blob + o_rsrc; pl->d_r_rec = pl->d_blob + o_rrec; pl->d_n_r_uniq = pl->d_blob + o_nru;
    pl->d_f_in_ref = pl->d_blob + o_fref; pl->d_f_row = pl->d_blob + o_frow; pl->d_f_root = pl->d_blob + o_froot;
    *out = pl;
    return NGDB_OK;
}

int ngdb_plan_export(const ngdb_plan_t* pl, ngdb_plan_view* v) {
    if (!pl || !v) return NGDB_ERR_ARG;
    const HostPlan& hp = pl->hp;
    v->n_queries = hp.n_queries; v->n_groups = hp.n_groups; v->n_levels = hp.n_levels; v->n_slots = hp.n_slots;
    v->n_anchor = hp.n_anchor; v->n_proj = hp.n_proj; v->n_inter = hp.n_inter; v->n_neg = hp.n_neg;
    v->n_int_rows = hp.n_int_rows; v->n_roots = hp.n_roots; v->n_refs = (int32_t)hp.in_ref.size();
    v->n_r_uniq = (int32_t)hp.r_uniq.size();
    v->peak_live = hp.peak_live;
    v->lvl_off = hp.lvl_off.data(); v->g_level = hp.g_level.data(); v->g_type = hp.g_type.data();
    v->g_nin = hp.g_nin.data(); v->g_n = hp.g_n.data(); v->g_out_base = hp.g_out_base.data();
    v->g_mlp_base = hp.g_mlp_base.data(); v->g_ref_off = hp.g_ref_off.data(); v->g_rel_off = hp.g_rel_off.data();
    v->in_ref = hp.in_ref.data(); v->in_gslot = hp.in_gslot.data(); v->rel = hp.rel.data();
    v->root_off = hp.root_off.data(); v->root_slot = hp.root_slot.data(); v->anchor_ent = hp.anchor_ent.data();
    v->pos = hp.pos.data(); v->r_uniq = hp.r_uniq.data(); v->r_seg_off = hp.r_seg_off.data();
    v->r_src = hp.r_src.data();
    v->n_f_rows = hp.n_f_rows;
    for (int k = 0; k < 3; ++k) v->f_step_rows[k] = hp.f_step_rows[k];
    v->f_row = hp.f_row.data();
    return NGDB_OK;
}

void ngdb_plan_free(ngdb_plan_t* pl) {
    if (!pl) return;
    if (pl->owner) {   // the device buffer goes back to its context (reused once last_use has passed)
        ngdb_ctx_t* c = pl->owner;
        std::lock_guard<std::mutex> lk(c->mu);
        c->live_plans.erase(std::remove(c->live_plans.begin(), c->live_plans.end(), pl), c->live_plans.end());
        if (pl->blob.dev) c->blob_pool.push_back(pl->blob);
    }
    delete pl;
}

int ngdb_train_step(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_neg, int32_t K, void* stream,
                    float* d_loss) {
    return run_step(c, pl, d_neg, K, static_cast<hipStream_t>(stream), d_loss, true);
}

int ngdb_forward_backward(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_neg, int32_t K, void* stream,
                          float* d_loss) {
    return run_step(c, pl, d_neg, K, static_cast<hipStream_t>(stream), d_loss, false);
}

int ngdb_get_grads(ngdb_ctx_t* c, ngdb_grad_view* out) {
    if (!c || !out) return NGDB_ERR_ARG;
    if (!c->have_grads) return fail(c, NGDB_ERR_STATE, "no step has been run on this context");
    HIPCHK(c, hipDeviceSynchronize());
    const int rc = check_waits(c);
    if (rc != NGDB_OK) return rc;
    HIPCHK(c, hipMemcpy(&c->gv.n_e_uniq, c->n_uniq.p, sizeof(int32_t), hipMemcpyDeviceToHost));
    *out = c->gv;
    return NGDB_OK;
}

int ngdb_score(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_cand, int32_t C, int32_t topk,
               float* d_scores, int32_t* d_topk_ids, float* d_topk_dist, void* stream) {
    if (!c || !pl) return NGDB_ERR_ARG;
    if (!c->bound) return fail(c, NGDB_ERR_STATE, "parameters not bound");
    if (pl->n_entities != c->cfg.n_entities || !pl->d_blob)
        return fail(c, NGDB_ERR_ARG, "plan belongs to another configuration or was built without a device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d_cand) {
        if (C <= 0 || !d_scores) return fail(c, NGDB_ERR_ARG, "candidate mode needs C > 0 and d_scores");
    } else if (topk < 1 || topk > NGDB_MAX_TOPK || !d_topk_ids || !d_topk_dist) {
        return fail(c, NGDB_ERR_ARG, "all-entity mode needs 1 <= topk <= NGDB_MAX_TOPK and both output arrays");
    }
    c->have_grads = false;
    // forward only: an operator output is reclaimed as soon as its consumer has run (Sec. 4.3);
    // the box family keeps one row per output
    const bool reclaim = c->cfg.family == NGDB_FAMILY_VEC;
    const int64_t n_tail = d_cand ? (int64_t)pl->hp.n_queries * C : 0;
    if (c->presized && d_cand && C > c->cfg.k_max)
        return fail(c, NGDB_ERR_ARG, "more candidates per query than the k_max declared at ngdb_create");
    int rc = reclaim ? size_forward_only(c, pl, n_tail) : size_workspace(c, pl, d_cand ? C : 0, false);
    if (rc != NGDB_OK) return rc;
    PassEnd end{c, pl, s};
    if ((rc = begin_pass(c, pl, false, s, reclaim, c->cfg.d_sem == 0)) != NGDB_OK) return rc;
    const int32_t* roots = reclaim && !c->rows_chained ? pl->d_f_root : pl->d_root_slot;
    EntRows er{};
    rc = prepare_entities(c, pl, d_cand, n_tail, s, &er, reclaim);
    if (rc != NGDB_OK) return rc;
    rc = enqueue_forward(c, pl, er, s, ctx_space(c, reclaim));
    if (rc != NGDB_OK) return rc;
    if (d_cand) {
        ScoreArgs sa{};
        sa.act = c->rows_chained ? rows_chain_act(c) : ptr<float>(c->act); sa.E = er.rows; candidate_table(c, &sa);
        sa.root_off = pl->d_root_off; sa.root_slot = roots;
        sa.pos = nullptr; sa.cand = er.cand; sa.B = pl->hp.n_queries; sa.C = C; sa.d = c->cfg.d;
        sa.max_branch = std::max(1, pl->hp.max_branch); sa.gave_up = gave_up_mark(c); sa.gamma = c->cfg.gamma; sa.score = d_scores;
        if (c->cfg.family == NGDB_FAMILY_BOX) { sa.off = ptr<float>(c->off); sa.alpha = c->cfg.box_alpha; }
        if (c->cfg.score_bf16) sa.E16 = ptr<uint16_t>(c->Eb);
        hipError_t e;
        { Timed tm(c, NGDB_TK_SCORE, s); e = launch_score(sa, false, s); }
        if (e == hipErrorInvalidValue) return fail(c, NGDB_ERR_UNSUPPORTED, "embedding width / union branch count too large for the scoring kernel");
        HIPCHK(c, e);
    } else {
        rc = rank_nearest(c, pl, roots, topk, d_topk_ids, d_topk_dist, s);
        if (rc != NGDB_OK) return rc;
    }
    HIPCHK(c, end.close());
    return NGDB_OK;
}

size_t ngdb_score_noalloc_bytes(const ngdb_ctx_t* c, const ngdb_plan_t* pl) {
    if (!c || !pl) return 0;
    const FwdBytes fb = forward_bytes(c, pl, true);
    auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    size_t need = up(fb.act) + up(fb.att);
    for (int t = 0; t < 3; ++t) need += up(fb.z[t]) + up(fb.h[t]);
    return need;
}

int ngdb_score_noalloc(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_cand, int32_t C, float* d_scores,
                       void* stream) {
    if (!c || !pl) return NGDB_ERR_ARG;
    if (!c->bound) return fail(c, NGDB_ERR_STATE, "parameters not bound");
    if (pl->n_entities != c->cfg.n_entities || !pl->d_blob)
        return fail(c, NGDB_ERR_ARG, "plan belongs to another configuration or was built without a device");
    if (c->cfg.family != NGDB_FAMILY_VEC || c->cfg.d_sem != 0)
        return fail(c, NGDB_ERR_UNSUPPORTED, "ngdb_score_noalloc: vector family without text features only");
    if (!d_cand || C <= 0 || !d_scores) return fail(c, NGDB_ERR_ARG, "ngdb_score_noalloc needs candidates, C > 0 and d_scores");
    const size_t need = ngdb_score_noalloc_bytes(c, pl);
    if (need > NOALLOC_BYTES)
        return fail(c, NGDB_ERR_ARG, "ngdb_score_noalloc: this batch needs " + std::to_string(need) +
                                         " bytes of forward workspace, the static scratch holds " +
                                         std::to_string(NOALLOC_BYTES) + " (NGDB_NOALLOC_SCRATCH_MIB)");
    unsigned char* base = nullptr;
    HIPCHK(c, noalloc_scratch(&base));
    // carve the forward buffers out of the scratch (outputs reclaimed once their consumer has run,
    // per-step buffers: as in ngdb_score); every row that is read was written earlier in this call
    // (operator outputs before their consumers, copies and hidden rows by the launch before the
    // one that reads them), so nothing has to be cleared
    const HostPlan& hp = pl->hp;
    const FwdBytes fb = forward_bytes(c, pl, true);
    size_t at = 0;
    auto take = [&](size_t bytes) {
        float* p = reinterpret_cast<float*>(base + at);
        at += (bytes + 255) & ~size_t(255);
        return p;
    };
    FwdSpace w{};
    w.reclaim = true;
    w.act = take(fb.act);
    w.Att = take(fb.att);
    for (int t = 0; t < 3; ++t) {
        w.Z[t] = take(fb.z[t]);
        w.H[t] = take(fb.h[t]);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    c->have_grads = false;
    const uint32_t timing = c->timing_mask;     // event brackets would create events: off for this call
    c->timing_mask = 0;
    const EntRows er{c->prm.E.p, pl->d_f_in_ref, pl->d_pos, d_cand};
    PassEnd end{c, pl, s};
    int rc = begin_pass(c, pl, false, s);
    if (rc == NGDB_OK) rc = enqueue_forward(c, pl, er, s, w);
    if (rc == NGDB_OK) {
        ScoreArgs sa{};
        sa.act = w.act; sa.E = er.rows; candidate_table(c, &sa);
        sa.root_off = pl->d_root_off; sa.root_slot = pl->d_f_root;
        sa.pos = nullptr; sa.cand = d_cand; sa.B = hp.n_queries; sa.C = C; sa.d = c->cfg.d;
        sa.max_branch = std::max(1, hp.max_branch); sa.gave_up = gave_up_mark(c); sa.gamma = c->cfg.gamma; sa.score = d_scores;
        if (c->cfg.score_bf16) sa.E16 = ptr<uint16_t>(c->Eb);
        const hipError_t e = launch_score(sa, false, s);
        if (e == hipErrorInvalidValue) rc = fail(c, NGDB_ERR_UNSUPPORTED, "embedding width / union branch count too large for the scoring kernel");
        else if (e != hipSuccess) rc = fail(c, NGDB_ERR_HIP, std::string("scoring launch: ") + hipGetErrorString(e));
    }
    c->timing_mask = timing;
    if (rc != NGDB_OK) return rc;
    HIPCHK(c, end.close());
    return NGDB_OK;
}

int ngdb_rank_answers(ngdb_ctx_t* c, const ngdb_plan_t* pl, const int32_t* d_ans_off, const int32_t* d_ans,
                      int32_t n_ans, int32_t* d_rank, float* d_ans_dist, void* stream) {
    if (!c || !pl) return NGDB_ERR_ARG;
    if (!c->bound) return fail(c, NGDB_ERR_STATE, "parameters not bound");
    if (pl->n_entities != c->cfg.n_entities || !pl->d_blob)
        return fail(c, NGDB_ERR_ARG, "plan belongs to another configuration or was built without a device");
    if (n_ans < 0 || !d_ans_off || (n_ans > 0 && (!d_ans || !d_rank)))
        return fail(c, NGDB_ERR_ARG, "answer lists / rank output missing");
    if (pl->hp.n_queries > 65535) return fail(c, NGDB_ERR_UNSUPPORTED, "more than 65535 queries in one ranking call");
    hipStream_t s = static_cast<hipStream_t>(stream);
    c->have_grads = false;
    const bool reclaim = c->cfg.family == NGDB_FAMILY_VEC;     // as in ngdb_score
    int rc = reclaim ? size_forward_only(c, pl, 0) : size_workspace(c, pl, 0, false);
    if (rc != NGDB_OK) return rc;
    PassEnd end{c, pl, s};
    if ((rc = begin_pass(c, pl, false, s, reclaim, c->cfg.d_sem == 0)) != NGDB_OK) return rc;
    const int32_t* roots = reclaim && !c->rows_chained ? pl->d_f_root : pl->d_root_slot;
    EntRows er{};
    rc = prepare_entities(c, pl, nullptr, 0, s, &er, reclaim);
    if (rc != NGDB_OK) return rc;
    rc = enqueue_forward(c, pl, er, s, ctx_space(c, reclaim));
    if (rc != NGDB_OK) return rc;
    if (n_ans > 0) {
        rc = rank_listed(c, pl, roots, d_ans_off, d_ans, n_ans, d_rank, d_ans_dist, s);
        if (rc != NGDB_OK) return rc;
    }
    HIPCHK(c, end.close());
    return NGDB_OK;
}

int ngdb_rank_metrics(const int32_t* d_rank, const int32_t* d_ans_off, const int32_t* d_n_take, int32_t n_queries,
                      float* d_out, void* stream) {
    if (!d_ans_off || !d_out || n_queries < 0 || (n_queries > 0 && !d_rank)) return NGDB_ERR_ARG;
    const hipError_t e = launch_rank_metrics(d_rank, d_ans_off, d_n_take, n_queries, d_out,
                                             static_cast<hipStream_t>(stream));
    return e == hipSuccess ? NGDB_OK : NGDB_ERR_HIP;
}

int ngdb_debug_gemm(const float* A, const float* B, float* C, int32_t M, int32_t N, int32_t K, int32_t lda,
                    int32_t ldb, int32_t ldc, int32_t a_kcontig, int32_t b_kcontig, const float* bias, int32_t relu,
                    const float* mask, int32_t ldmask, const float* addend, int32_t ldadd, const int32_t* dst_row,
                    int32_t arith, void* stream) {
    if (!A || !B || !C || M < 0 || N < 0 || K < 0 || arith < 0 || arith > 2) return NGDB_ERR_ARG;
    GemmArgs g;
    g.A = A; g.B = B; g.C = C; g.M = M; g.N = N; g.K = K; g.lda = lda; g.ldb = ldb; g.ldc = ldc;
    g.a_kcontig = a_kcontig != 0; g.b_kcontig = b_kcontig != 0; g.bias = bias; g.relu = relu != 0;
    g.mask = mask; g.ldmask = ldmask; g.addend = addend; g.ldadd = ldadd; g.dst_row = dst_row;
    g.arith = arith;
    // (as the step chooses: weight gradients have a kernel of their own)
    const bool wgrad = arith == 0 && !g.a_kcontig && !g.b_kcontig && !bias && !relu && !mask && !addend && !dst_row &&
                       ((M | N | lda | ldb | ldc) & 3) == 0 && (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15) == 0;
    const WgradArgs w{A, B, C, nullptr, M, N, K, lda, ldb, ldc};
    const hipError_t e = wgrad ? launch_wgrad_group(&w, 1, static_cast<hipStream_t>(stream)) : launch_gemm(g, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? NGDB_OK : (e == hipErrorInvalidValue ? NGDB_ERR_ARG : NGDB_ERR_HIP);
}

int ngdb_debug_gemm_group(int32_t count, const float* const* A, const float* const* B, float* const* C, const int32_t* M,
                          const int32_t* N, const int32_t* K, void* stream) {
    if (count < 1 || count > GEMM_MAX_GROUP || !A || !B || !C || !M || !N || !K) return NGDB_ERR_ARG;
    GemmArgs g[GEMM_MAX_GROUP];
    for (int i = 0; i < count; ++i) {
        if (!A[i] || !B[i] || !C[i] || M[i] < 1 || N[i] < 1 || K[i] < 4) return NGDB_ERR_ARG;
        g[i].A = A[i]; g[i].B = B[i]; g[i].C = C[i]; g[i].M = M[i]; g[i].N = N[i]; g[i].K = K[i];
        g[i].lda = g[i].ldb = K[i]; g[i].ldc = N[i];
    }
    const hipError_t e = launch_gemm_group(g, count, static_cast<hipStream_t>(stream), nullptr);
    return e == hipSuccess ? NGDB_OK : (e == hipErrorInvalidValue ? NGDB_ERR_ARG : NGDB_ERR_HIP);
}

int ngdb_debug_mlp(const float* X, const float* W1, const float* b1, const float* W2, const float* b2, const float* mask,
                   float* H, float* Y, int32_t M, int32_t d, int32_t h, int32_t backward, int32_t* used, void* stream) {
    if (!X || !W1 || !W2 || !H || !Y || M < 1 || d < 4 || h < 4 || (d & 3) || (h & 3) || (backward && !mask)) return NGDB_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int kt = 2 * ((h + 31) / 32);
    const size_t w_elems = 2 * (pieces_elems(h, d) + pieces_elems(d, h));
    const size_t h_elems = (size_t)((M + 31) / 32) * kt * 1536;
    uint16_t* buf = nullptr;
    if (hipMalloc(&buf, (w_elems + h_elems) * sizeof(uint16_t)) != hipSuccess) return NGDB_ERR_OOM;
    PieceJobs J{};
    J.count = 2;
    J.job[0].W = W1; J.job[0].R = h; J.job[0].C = d;
    J.job[0].out_rk = buf; J.job[0].out_ck = buf + pieces_elems(h, d);
    J.job[1].W = W2; J.job[1].R = d; J.job[1].C = h;
    J.job[1].out_rk = J.job[0].out_ck + pieces_elems(d, h); J.job[1].out_ck = J.job[1].out_rk + pieces_elems(d, h);
    uint16_t* hp = buf + w_elems;
    GemmArgs first, second;
    first.A = X; first.lda = d; first.M = M; first.N = h; first.K = d; first.C = H; first.ldc = h;
    second.A = H; second.lda = h; second.M = M; second.N = d; second.K = h; second.C = Y; second.ldc = d;
    first.arith = second.arith = GEMM_SPLIT;
    first.c_pieces = hp; first.c_kt = kt;
    if (!backward) {
        first.B = W1; first.ldb = d; first.bias = b1; first.relu = true; first.b_pieces = J.job[0].out_rk; first.b_kt = (d + 15) / 16;
        second.B = W2; second.ldb = h; second.bias = b2; second.b_pieces = J.job[1].out_rk; second.b_kt = (h + 15) / 16;
    } else {
        first.B = W2; first.ldb = h; first.b_kcontig = false; first.mask = mask; first.ldmask = h;
        first.b_pieces = J.job[1].out_ck; first.b_kt = (d + 15) / 16;
        second.B = W1; second.ldb = d; second.b_kcontig = false; second.b_pieces = J.job[0].out_ck; second.b_kt = (h + 15) / 16;
    }
    bool emitted = false;
    int kernel[2] = {};
    hipError_t e = launch_weight_pieces(J, s);
    if (e == hipSuccess) e = launch_gemm_group(&first, 1, s, nullptr, &emitted, &kernel[0]);
    if (e == hipSuccess && emitted) { second.a_pieces = hp; second.a_kt = kt; }
    if (e == hipSuccess) e = launch_gemm_group(&second, 1, s, nullptr, nullptr, &kernel[1]);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(buf);
    if (used) *used = 1 | (emitted ? 2 : 0) | kernel[0] << 2 | kernel[1] << 4;
    return e == hipSuccess ? NGDB_OK : (e == hipErrorInvalidValue ? NGDB_ERR_ARG : NGDB_ERR_HIP);
}

int ngdb_debug_copy(void* d_dst, const void* d_src, size_t bytes, void* stream) {
    if (!d_dst || !d_src) return NGDB_ERR_ARG;
    const hipError_t e = launch_copy(d_dst, d_src, bytes, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? NGDB_OK : (e == hipErrorInvalidValue ? NGDB_ERR_ARG : NGDB_ERR_HIP);
}

int ngdb_debug_stream(int32_t mode, void* d_dst, const void* d_src, size_t bytes, const int32_t* d_rows, int64_t n_rows,
                      int32_t row_floats, void* stream) {
    if (!d_dst || (mode != NGDB_STREAM_WRITE && mode != NGDB_STREAM_UPDATE && mode != NGDB_STREAM_UPDATE_NT && !d_src)) return NGDB_ERR_ARG;
    const hipError_t e = launch_stream_pattern(mode, d_dst, d_src, bytes, d_rows, n_rows, row_floats,
                                               static_cast<hipStream_t>(stream));
    return e == hipSuccess ? NGDB_OK : (e == hipErrorInvalidValue ? NGDB_ERR_ARG : NGDB_ERR_HIP);
}

int ngdb_set_timing(ngdb_ctx_t* c, uint32_t class_mask) {
    if (!c) return NGDB_ERR_ARG;
    c->timing_mask = class_mask & ((1u << NGDB_TK_COUNT) - 1u);
    return NGDB_OK;
}

int ngdb_get_timing(ngdb_ctx_t* c, ngdb_timing* out, int reset) {
    if (!c || !out) return NGDB_ERR_ARG;
    HIPCHK(c, hipDeviceSynchronize());
    for (const ngdb_ctx_s::Bracket& b : c->brackets) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, b.a, b.b) == hipSuccess) {
            c->timing.ms[b.cls] += ms;
            c->timing.brackets[b.cls] += 1;
            if (b.route >= 0) {
                c->timing.route_ms[b.cls][b.route] += ms;
                c->timing.route_launches[b.cls][b.route] += 1;
                c->timing.route_flop[b.cls][b.route] += b.flop;
            }
        }
        c->spare_events.push_back(b.a);
        c->spare_events.push_back(b.b);
    }
    c->brackets.clear();
    *out = c->timing;
    if (reset) c->timing = ngdb_timing{};
    return NGDB_OK;
}

int ngdb_copy_to_host(void* h_dst, const void* d_src, size_t bytes) {
    if (bytes == 0) return NGDB_OK;
    if (!h_dst || !d_src) return NGDB_ERR_ARG;
    if (hipDeviceSynchronize() != hipSuccess) return NGDB_ERR_HIP;
    return hipMemcpy(h_dst, d_src, bytes, hipMemcpyDeviceToHost) == hipSuccess ? NGDB_OK : NGDB_ERR_HIP;
}

int64_t ngdb_debug_alloc_count(const ngdb_ctx_t* c) { return c ? c->n_alloc : -1; }

int64_t ngdb_debug_device_bytes(const ngdb_ctx_t* c) { return c ? (int64_t)c->held : -1; }

int ngdb_debug_device_limit(ngdb_ctx_t* c, int64_t bytes) {
    if (!c) return NGDB_ERR_ARG;
    c->held_limit = bytes < 0 ? SIZE_MAX : (size_t)bytes;
    return NGDB_OK;
}

int ngdb_debug_chain_polls(ngdb_ctx_t* c, int32_t polls) {
    if (!c) return NGDB_ERR_ARG;
    HIPCHK(c, hipDeviceSynchronize());
    HIPCHK(c, launch_fill_zero_i32(ptr<int32_t>(c->sync), SYNC_WORDS, nullptr));
    HIPCHK(c, hipDeviceSynchronize());
    *c->gave_up = 0;
    c->chain_polls = polls;
    return NGDB_OK;
}

int ngdb_debug_chain_patience(ngdb_ctx_t* c, int32_t looks) {
    if (!c) return NGDB_ERR_ARG;
    c->chain_patience = looks;
    return NGDB_OK;
}

int64_t ngdb_debug_chain_launches(ngdb_ctx_t* c, int32_t kind) {
    if (!c || kind < 0 || kind > 3) return -1;
    if (kind < 3) return c->chain_count[kind];
    int32_t helped = 0;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(&helped, ptr<int32_t>(c->sync) + HELPED_AT, sizeof(helped), hipMemcpyDeviceToHost) != hipSuccess) return -1;
    return helped;
}

int ngdb_debug_rank_filter_from(ngdb_ctx_t* c, int64_t work) {
    if (!c) return NGDB_ERR_ARG;
    c->rank_filter_from = work;
    return NGDB_OK;
}

int ngdb_debug_rank_by_chunks(ngdb_ctx_t* c, int32_t on) {
    if (!c) return NGDB_ERR_ARG;
    c->rank_by_chunks = on != 0;
    return NGDB_OK;
}

int ngdb_debug_rank_overflows(ngdb_ctx_t* c) {
    if (!c) return -1;
    if (!c->rank_overflowed) return 0;
    int n = 0;
    for (int i = 0; i < c->rank_chunks; ++i) {
        int32_t mark = 0;
        if (hipMemcpy(&mark, c->rank_overflowed + i, sizeof(mark), hipMemcpyDeviceToHost) != hipSuccess) return -1;
        n += mark != 0;
    }
    return n;
}

int64_t ngdb_step_count(const ngdb_ctx_t* c) { return c ? c->step : -1; }

const char* ngdb_strerror(int code) {
    switch (code) {
        case NGDB_OK: return "ok";
        case NGDB_ERR_ARG: return "invalid argument";
        case NGDB_ERR_UNSUPPORTED: return "unsupported query or configuration";
        case NGDB_ERR_RANGE: return "entity or relation id out of range";
        case NGDB_ERR_OOM: return "out of memory";
        case NGDB_ERR_HIP: return "HIP runtime error";
        case NGDB_ERR_STATE: return "call order error";
        default: return "unknown error";
    }
}

const char* ngdb_last_error(const ngdb_ctx_t* c) { return c ? c->err.c_str() : ""; }

}  // extern "C"
