// Host planner.  Turns a batch of query trees into the paper's operator pools
// (Sec. 4.1) resolved ahead of time into a sequence of execution steps.  Two
// schedules: level-synchronous -- at every depth, the operators of one type
// (and, for intersections, one input count: the classes C_k of Sec. 4.3) from
// all queries form one group, all groups of a depth are one step; and the
// paper's Max-Fillness loop (Sec. 4.1 "Dynamic Scheduling", Alg. 1) -- ready
// operators wait in one pool per class, every step runs up to B_max operators
// of the fullest pool.  All gather / scatter positions are resolved here, ahead
// of the step (Sec. 4.2 "Efficient Tensor Indexing").  The numbering rules are
// stated in ngdb.h (ngdb_plan_view).
#include "planner.h"

#include <algorithm>
#include <climits>
#include <numeric>

namespace ngdb {
namespace {

struct Tree {          // node of a union-free branch (no heap: at most NGDB_MAX_CARD inputs)
    int32_t type, arg, n_kids;   // arg: the node of the query whose argument it takes (-1: none)
    int32_t kids[NGDB_MAX_CARD];
};

struct Expander {
    const ngdb_query_batch& qb;
    int32_t base;                 // first node of the current query
    int32_t n_local;
    std::vector<Tree>& pool;
    std::string& err;
    int code = NGDB_OK;

    int32_t make(int32_t type, int32_t arg, const int32_t* kids, int32_t n_kids) {
        Tree t;
        t.type = type; t.arg = arg; t.n_kids = n_kids;
        for (int32_t k = 0; k < n_kids; ++k) t.kids[k] = kids[k];
        pool.push_back(t);
        return (int32_t)pool.size() - 1;
    }

    // Appends the conjunctive branches of the sub-query rooted at local node j to `out`.
    void expand(int32_t j, int depth, std::vector<int32_t>& out) {
        if (code != NGDB_OK) return;
        if (depth > NGDB_MAX_LEVELS + 1) {
            code = NGDB_ERR_UNSUPPORTED;
            err = "query deeper than NGDB_MAX_LEVELS";
            return;
        }
        const int32_t n = base + j;
        const int32_t lo = qb.in_off[n], hi = qb.in_off[n + 1];
        const int op = qb.op[n];
        const size_t first = out.size();
        switch (op) {
            case NGDB_OP_ANCHOR:
                out.push_back(make(NGDB_OP_ANCHOR, j, nullptr, 0));
                break;
            case NGDB_OP_PROJ: {
                expand(qb.in_idx[lo], depth + 1, out);          // one projection on top of every branch of the input
                for (size_t i = first; i < out.size() && code == NGDB_OK; ++i) {
                    const int32_t kid = out[i];
                    out[i] = make(NGDB_OP_PROJ, j, &kid, 1);
                }
                break;
            }
            case NGDB_OP_UNION: {
                for (int32_t k = lo; k < hi; ++k) expand(qb.in_idx[k], depth + 1, out);
                break;
            }
            default: {   // INTER, NEG: every input must be union-free
                int32_t kids[NGDB_MAX_CARD];
                int32_t n_kids = 0;
                for (int32_t k = lo; k < hi; ++k) {
                    const size_t before = out.size();
                    expand(qb.in_idx[k], depth + 1, out);
                    if (code != NGDB_OK) return;
                    if (out.size() != before + 1) {
                        code = NGDB_ERR_UNSUPPORTED;
                        err = "union below an intersection or a negation";
                        return;
                    }
                    kids[n_kids++] = out.back();                // validate() bounds the input count
                    out.pop_back();
                }
                out.push_back(make(op, -1, kids, n_kids));
            }
        }
        if (out.size() - first > (size_t)NGDB_MAX_BRANCH && code == NGDB_OK) {
            code = NGDB_ERR_UNSUPPORTED;
            err = "query has more than NGDB_MAX_BRANCH conjunctive branches";
        }
    }
};

struct Flat {   // nodes after DNF, numbered in post-order
    std::vector<int32_t> type, arg, level, in_off, in;
    int32_t size() const { return (int32_t)type.size(); }
    int32_t add(int32_t t, int32_t a, int32_t lvl, const int32_t* ins, int32_t n_ins) {
        type.push_back(t);
        arg.push_back(a);
        level.push_back(lvl);
        in.insert(in.end(), ins, ins + n_ins);
        in_off.push_back((int32_t)in.size());
        return (int32_t)type.size() - 1;
    }
    int32_t nin(int32_t g) const { return in_off[g + 1] - in_off[g]; }
};

int32_t number_postorder(const std::vector<Tree>& pool, int32_t t, Flat& flat) {
    const Tree& node = pool[t];
    int32_t ins[NGDB_MAX_CARD];
    int32_t lvl = 0;
    for (int32_t k = 0; k < node.n_kids; ++k) {
        ins[k] = number_postorder(pool, node.kids[k], flat);
        lvl = std::max(lvl, flat.level[ins[k]] + 1);
    }
    return flat.add(node.type, node.arg, lvl, ins, node.n_kids);
}

// Max-Fillness schedule (Alg. 1 without the gradient nodes, which mirror it): returns the step
// (1-based) in which every operator node runs.  One pool per class (type, input count), in
// the order PROJ < INTER by input count < NEG.  A cycle files the newly ready operators into
// their pools in node order, picks the pool with the most entries (fillness = entries / B_max
// with one B_max for all classes; ties to the first class), and runs its first min(size,
// B_max) entries; consumers whose inputs are all done become ready for the next cycle.  The
// loop runs until every pool is empty (the printed loop condition, "ready set not empty",
// would strand the remainder of a pool that was cut at B_max).  Also returns the largest
// number of operator outputs alive at once under eager reference counting (Sec. 4.3): an
// output dies when its consumer has run; the outputs of roots stay for scoring.
void max_fillness_steps(const Flat& flat, int32_t b_max, std::vector<int32_t>& step, int32_t& peak_live) {
    const int32_t n = (int32_t)flat.type.size();
    auto cls = [&](int32_t g) {
        const int32_t t = flat.type[g];
        return t == NGDB_OP_PROJ ? 0 : (t == NGDB_OP_INTER ? flat.nin(g) - 1 : NGDB_MAX_CARD);   // 0, 1..7, 8
    };
    constexpr int N_CLS = NGDB_MAX_CARD + 1;
    std::vector<int32_t> consumer(n, -1), waiting(n, 0);
    for (int32_t g = 0; g < n; ++g)
        for (int32_t k = flat.in_off[g]; k < flat.in_off[g + 1]; ++k) {
            consumer[flat.in[k]] = g;
            if (flat.type[flat.in[k]] != NGDB_OP_ANCHOR) ++waiting[g];
        }
    std::vector<std::vector<int32_t>> pool(N_CLS);
    std::vector<size_t> head(N_CLS, 0);
    std::vector<int32_t> ready;
    for (int32_t g = 0; g < n; ++g)
        if (flat.type[g] != NGDB_OP_ANCHOR && waiting[g] == 0) ready.push_back(g);
    step.assign(n, 0);
    int32_t s = 0, live = 0;
    peak_live = 0;
    for (;;) {
        std::sort(ready.begin(), ready.end());
        for (int32_t g : ready) pool[cls(g)].push_back(g);
        ready.clear();
        int best = -1;
        size_t best_n = 0;
        for (int c = 0; c < N_CLS; ++c) {
            const size_t cnt = pool[c].size() - head[c];
            if (cnt > best_n) { best_n = cnt; best = c; }
        }
        if (best < 0) break;
        const size_t take = b_max > 0 ? std::min<size_t>(best_n, (size_t)b_max) : best_n;
        ++s;
        live += (int32_t)take;                       // outputs of this step exist next to their inputs
        peak_live = std::max(peak_live, live);
        for (size_t i = 0; i < take; ++i) {
            const int32_t g = pool[best][head[best] + i];
            step[g] = s;
            for (int32_t k = flat.in_off[g]; k < flat.in_off[g + 1]; ++k)
                if (flat.type[flat.in[k]] != NGDB_OP_ANCHOR) --live;   // its only consumer has run
            const int32_t c = consumer[g];
            if (c >= 0 && --waiting[c] == 0) ready.push_back(c);
        }
        head[best] += take;
    }
}

// Checks the queries q_lo .. q_hi - 1 (and the batch as a whole).
int validate(const ngdb_query_batch& qb, int32_t N, int32_t R, int32_t q_lo, int32_t q_hi, std::string& err) {
    if (qb.n_queries < 0) { err = "n_queries < 0"; return NGDB_ERR_ARG; }
    if (qb.n_queries == 0) return NGDB_OK;
    if (!qb.node_off || !qb.op || !qb.arg || !qb.in_off || !qb.pos) {
        err = "null array in query batch";
        return NGDB_ERR_ARG;
    }
    if (qb.node_off[0] != 0 || qb.in_off[0] != 0) { err = "offsets must start at 0"; return NGDB_ERR_ARG; }
    for (int32_t q = q_lo; q < q_hi; ++q) {
        const int32_t lo = qb.node_off[q], hi = qb.node_off[q + 1];
        if (hi <= lo) { err = "query without nodes"; return NGDB_ERR_ARG; }
        if (qb.pos[q] < 0 || qb.pos[q] >= N) { err = "positive entity id out of range"; return NGDB_ERR_RANGE; }
        for (int32_t n = lo; n < hi; ++n) {
            const int32_t a = qb.in_off[n], b = qb.in_off[n + 1];
            if (b < a) { err = "in_off not monotone"; return NGDB_ERR_ARG; }
            const int32_t nin = b - a;
            if (nin > 0 && !qb.in_idx) { err = "null in_idx"; return NGDB_ERR_ARG; }
            for (int32_t k = a; k < b; ++k)
                if (qb.in_idx[k] < 0 || qb.in_idx[k] >= n - lo) {
                    err = "input must be an earlier node of the same query";
                    return NGDB_ERR_ARG;
                }
            switch (qb.op[n]) {
                case NGDB_OP_ANCHOR:
                    if (nin != 0) { err = "anchor with inputs"; return NGDB_ERR_ARG; }
                    if (qb.arg[n] < 0 || qb.arg[n] >= N) { err = "anchor entity id out of range"; return NGDB_ERR_RANGE; }
                    break;
                case NGDB_OP_PROJ:
                    if (nin != 1) { err = "projection needs one input"; return NGDB_ERR_ARG; }
                    if (qb.arg[n] < 0 || qb.arg[n] >= R) { err = "relation id out of range"; return NGDB_ERR_RANGE; }
                    break;
                case NGDB_OP_NEG:
                    if (nin != 1) { err = "negation needs one input"; return NGDB_ERR_ARG; }
                    break;
                case NGDB_OP_INTER:
                    if (nin < 2) { err = "intersection needs at least two inputs"; return NGDB_ERR_ARG; }
                    if (nin > NGDB_MAX_CARD) { err = "intersection with more than NGDB_MAX_CARD inputs"; return NGDB_ERR_UNSUPPORTED; }
                    break;
                case NGDB_OP_UNION:
                    if (nin < 1) { err = "union without inputs"; return NGDB_ERR_ARG; }
                    break;
                default:
                    err = "unknown operator code";
                    return NGDB_ERR_ARG;
            }
        }
    }
    return NGDB_OK;
}

// Stable grouping of values by key (keys in [0, key_bound)): the keys that occur in ascending order, segment offsets, and
// the values segment by segment in input order.  A counting sort where the key range allows it, else a merge sort.
void group_by_key(const std::vector<int32_t>& key, int32_t key_bound, const std::vector<int32_t>& value, std::vector<int32_t>& uniq,
                  std::vector<int32_t>& seg_off, std::vector<int32_t>& grouped) {
    const size_t n = key.size();
    uniq.clear();
    seg_off.clear();
    grouped.resize(n);
    if (key_bound <= (int64_t)(4 * n + 1024)) {
        std::vector<int32_t> at((size_t)key_bound, 0);
        for (size_t i = 0; i < n; ++i) ++at[key[i]];
        int32_t sum = 0;
        for (int32_t k = 0; k < key_bound; ++k) {
            const int32_t c = at[k];
            at[k] = sum;
            if (c == 0) continue;
            uniq.push_back(k);
            seg_off.push_back(sum);
            sum += c;
        }
        for (size_t i = 0; i < n; ++i) grouped[at[key[i]]++] = value[i];
    } else {
        std::vector<int32_t> order(n);
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return key[a] < key[b]; });
        for (size_t i = 0; i < n; ++i) {
            if (i == 0 || key[order[i]] != key[order[i - 1]]) {
                uniq.push_back(key[order[i]]);
                seg_off.push_back((int32_t)i);
            }
            grouped[i] = value[order[i]];
        }
    }
    seg_off.push_back((int32_t)n);
}

// A structure of queries: everything the plan needs to know of a query but its arguments.  A batch has thousands of
// queries and few structures, so each is checked, expanded (DNF) and numbered once and the queries only look up theirs:
// expanding and checking every query by itself was more than half of the planner's time, most of it mispredicted branches
// (450 us for 4096 queries of 14 structures, 50 for 512; 170 and 30 now).
struct Shape {
    uint64_t ops, n_ins;                 // four bits a node: operator, input count
    int32_t n, m, in0;                   // nodes and inputs as given; its inputs in given_in
    int32_t count;                       // queries
    // ranges of the table's arrays
    struct Range { int32_t at, n; } node, op, ref, anchor, root, ent, rel;
};

// The structures of a batch and their nodes (numbered from 0 in each structure).
struct ShapeTable {
    static constexpr int SLOTS = 256;
    static constexpr int32_t NODES = 16, INPUTS = 32;      // of the queries that are looked up; larger ones get a structure each
    struct Op { int32_t node, cls, rel; };            // an operator, its class; rel: node of the query that names the relation (-1: none)
    struct Ref { int32_t op, k, kid; };               // input k of the op-th operator is node kid
    std::vector<Shape> shapes;
    Flat flat;                           // arg: node of the query; in: numbered over all structures
    std::vector<Op> op;
    std::vector<Ref> ref;
    std::vector<int32_t> anchor, root, ent, rel, given_in;  // ent, rel: nodes of the query whose arguments are entities, relations
    std::vector<Tree> pool;              // scratch
    std::vector<int32_t> branches;
    int16_t slot[SLOTS];

    ShapeTable() {
        std::fill(slot, slot + SLOTS, (int16_t)-1);
        shapes.reserve(32);
        flat.type.reserve(256); flat.arg.reserve(256); flat.level.reserve(256); flat.in_off.reserve(257); flat.in.reserve(256);
        flat.in_off.push_back(0);
        op.reserve(256); ref.reserve(256);
        anchor.reserve(128); root.reserve(64); ent.reserve(128); rel.reserve(128); given_in.reserve(256);
        pool.reserve(32); branches.reserve(16);
    }
    int32_t level(const Shape& sh, const Op& o) const { return flat.level[sh.node.at + o.node]; }
    int32_t type(const Shape& sh, int32_t node) const { return flat.type[sh.node.at + node]; }
    int32_t nin(const Shape& sh, const Op& o) const { return flat.nin(sh.node.at + o.node); }

    // The structure of query q, or -1 if it is new: key then holds what it looks like and *at its free place among
    // the slots, or -1 if it is not to be looked up.  A query that is found passes every check but those of its arguments and
    // its positive.
    int32_t find(const ngdb_query_batch& qb, int32_t q, Shape& key, int32_t* at) const {
        const int32_t lo = qb.node_off[q], n = qb.node_off[q + 1] - lo;
        *at = -1;
        if (n < 1 || n > NODES) return -1;
        uint64_t ops = 0, n_ins = 0;
        uint32_t large = 0;
        const int32_t in_lo = qb.in_off[lo];
        int32_t before = in_lo;
        for (int32_t i = 0; i < n; ++i) {
            const int32_t next = qb.in_off[lo + i + 1];
            const uint32_t o = qb.op[lo + i], e = (uint32_t)next - (uint32_t)before;
            before = next;
            large |= o | e;
            ops |= (uint64_t)(o & 15u) << (4 * i);
            n_ins |= (uint64_t)(e & 15u) << (4 * i);
        }
        if (large > 15u) return -1;
        const int32_t m = before - in_lo;
        if (m > INPUTS || (m > 0 && !qb.in_idx)) return -1;
        const int32_t* in = qb.in_idx + in_lo;
        int32_t h = (int32_t)((ops * 0x9E3779B97F4A7C15ull ^ n_ins * 0xC2B2AE3D27D4EB4Full) >> 56);
        for (int probe = 0; probe < 8; ++probe, h = (h + 1) & (SLOTS - 1)) {
            const int32_t s = slot[h];
            if (s < 0) {
                *at = h;
                key.ops = ops; key.n_ins = n_ins; key.n = n; key.m = m;
                return -1;
            }
            const Shape& c = shapes[s];
            if (c.ops != ops || c.n_ins != n_ins || c.n != n) continue;
            const int32_t* want = given_in.data() + c.in0;
            int32_t differ = 0;
            for (int32_t k = 0; k < m; ++k) differ |= want[k] ^ in[k];
            if (differ == 0) return s;
        }
        return -1;
    }

    // Adds the structure of query q, which has been validated; its number in *s.
    int add(const ngdb_query_batch& qb, int32_t q, Shape sh, int32_t at, int32_t* s, std::string& err) {
        const int32_t lo = qb.node_off[q], hi = qb.node_off[q + 1];
        pool.clear();
        branches.clear();
        Expander ex{qb, lo, hi - lo, pool, err};
        ex.expand(ex.n_local - 1, 0, branches);
        if (ex.code != NGDB_OK) return ex.code;
        sh.count = 0;
        sh.in0 = (int32_t)given_in.size();
        given_in.insert(given_in.end(), qb.in_idx + qb.in_off[lo], qb.in_idx + qb.in_off[hi]);
        const int32_t base = flat.size();
        auto open = [](const auto& v) { return Shape::Range{(int32_t)v.size(), 0}; };
        auto close = [](Shape::Range& r, const auto& v) { r.n = (int32_t)v.size() - r.at; };
        sh.root = open(root); sh.op = open(op); sh.ref = open(ref); sh.anchor = open(anchor); sh.ent = open(ent); sh.rel = open(rel);
        for (const int32_t b : branches) {
            if (pool[b].type == NGDB_OP_ANCHOR) {
                err = "a query must contain at least one operator";
                return NGDB_ERR_UNSUPPORTED;
            }
            const int32_t g = number_postorder(pool, b, flat);
            if (flat.level[g] > NGDB_MAX_LEVELS) {
                err = "query deeper than NGDB_MAX_LEVELS";
                return NGDB_ERR_UNSUPPORTED;
            }
            root.push_back(g - base);
        }
        for (int32_t g = base; g < flat.size(); ++g) {
            if (flat.type[g] == NGDB_OP_ANCHOR) {
                anchor.push_back(g - base);
                continue;
            }
            const int32_t i = (int32_t)op.size() - sh.op.at;
            for (int32_t k = 0; k < flat.nin(g); ++k) ref.push_back({i, k, flat.in[flat.in_off[g] + k] - base});
            op.push_back({g - base, 0, flat.type[g] == NGDB_OP_PROJ ? flat.arg[g] : -1});
        }
        for (int32_t n = lo; n < hi; ++n) {
            if (qb.op[n] == NGDB_OP_ANCHOR) ent.push_back(n - lo);
            if (qb.op[n] == NGDB_OP_PROJ) rel.push_back(n - lo);
        }
        sh.node = {base, flat.size() - base};
        close(sh.root, root); close(sh.op, op); close(sh.ref, ref); close(sh.anchor, anchor); close(sh.ent, ent); close(sh.rel, rel);
        *s = (int32_t)shapes.size();
        shapes.push_back(sh);
        if (at >= 0 && *s <= INT16_MAX) slot[at] = (int16_t)*s;
        return NGDB_OK;
    }
};
template <class V>
struct Span {            // a range of one of the table's arrays
    const V *b, *e;
    Span(const std::vector<V>& v, Shape::Range r) : b(v.data() + r.at), e(b + r.n) {}
    const V* begin() const { return b; }
    const V* end() const { return e; }
};

}  // namespace

int build_plan(const ngdb_query_batch& qb, int32_t N, int32_t R, int32_t schedule, int32_t b_max, HostPlan& P,
               std::string& err) {
    if ((schedule != NGDB_SCHED_LEVEL && schedule != NGDB_SCHED_MAX_FILL) || b_max < 0) {
        err = "unknown schedule or negative b_max";
        return NGDB_ERR_ARG;
    }
    int rc = validate(qb, N, R, 0, 0, err);
    if (rc != NGDB_OK) return rc;
    P = HostPlan{};
    const int32_t B = qb.n_queries;
    P.n_queries = B;

    // 1. the structure of every query (DNF + numbering), its arguments checked
    ShapeTable tab;
    std::vector<int32_t> shape_of(B);
    P.root_off.resize((size_t)B + 1);
    P.root_off[0] = 0;
    for (int32_t q = 0; q < B; ++q) {
        Shape key;
        int32_t at, s = tab.find(qb, q, key, &at);
        bool bad = (uint32_t)qb.pos[q] >= (uint32_t)N;
        if (s < 0) {
            std::string why;
            int code = validate(qb, N, R, q, q + 1, why);
            if (code == NGDB_OK) code = tab.add(qb, q, key, at, &s, why);
            if (code != NGDB_OK) {           // what is wrong with any query outranks what is not supported
                rc = validate(qb, N, R, 0, B, err);
                if (rc != NGDB_OK) return rc;
                err = why;
                return code;
            }
        } else {
            const int32_t* arg = qb.arg + qb.node_off[q];
            for (const int32_t n : Span(tab.ent, tab.shapes[s].ent)) bad |= (uint32_t)arg[n] >= (uint32_t)N;
            for (const int32_t n : Span(tab.rel, tab.shapes[s].rel)) bad |= (uint32_t)arg[n] >= (uint32_t)R;
        }
        if (bad) return validate(qb, N, R, 0, B, err);
        Shape& sh = tab.shapes[s];
        ++sh.count;
        shape_of[q] = s;
        P.root_off[q + 1] = P.root_off[q] + sh.root.n;
    }
    P.pos.assign(qb.pos, qb.pos + B);
    int32_t n_nodes = 0, n_anchor = 0, n_ref = 0, max_level = 0;
    for (const Shape& sh : tab.shapes) {
        n_nodes += sh.count * sh.node.n;
        n_anchor += sh.count * sh.anchor.n;
        n_ref += sh.count * sh.ref.n;
        for (const ShapeTable::Op& o : Span(tab.op, sh.op)) max_level = std::max(max_level, tab.level(sh, o));
        P.max_branch = std::max(P.max_branch, sh.root.n);
    }
    P.n_anchor = n_anchor;
    P.n_slots = n_nodes - n_anchor;
    P.n_roots = P.root_off[B];

    // 1b. execution step of every operator: its depth, or its Max-Fillness step.  From here
    // on "level" means execution step.  The eager-reclamation peak of the level-synchronous
    // order is computed the same way: outputs of a step appear, then their inputs die.
    std::vector<int32_t> step;               // Max-Fillness: of every node
    int32_t top_level = max_level;
    if (schedule == NGDB_SCHED_MAX_FILL) {
        Flat all;
        all.type.reserve(n_nodes); all.in.reserve(n_ref); all.in_off.reserve(n_nodes + 1);
        all.in_off.push_back(0);
        for (int32_t q = 0; q < B; ++q) {
            const Shape& sh = tab.shapes[shape_of[q]];
            const int32_t base = all.size();
            for (int32_t g = sh.node.at; g < sh.node.at + sh.node.n; ++g) {
                all.type.push_back(tab.flat.type[g]);
                for (int32_t k = tab.flat.in_off[g]; k < tab.flat.in_off[g + 1]; ++k) all.in.push_back(tab.flat.in[k] - sh.node.at + base);
                all.in_off.push_back((int32_t)all.in.size());
            }
        }
        max_fillness_steps(all, b_max, step, P.peak_live);
        for (const int32_t l : step) top_level = std::max(top_level, l);
    } else {
        std::vector<int32_t> born(max_level + 2, 0), dead(max_level + 2, 0);
        for (const Shape& sh : tab.shapes) {
            for (const ShapeTable::Op& o : Span(tab.op, sh.op)) born[tab.level(sh, o)] += sh.count;
            for (const ShapeTable::Ref& r : Span(tab.ref, sh.ref))
                if (tab.type(sh, r.kid) != NGDB_OP_ANCHOR) dead[tab.level(sh, tab.op[sh.op.at + r.op])] += sh.count;
        }
        int32_t live = 0;
        for (int32_t l = 1; l <= max_level; ++l) {
            live += born[l];
            P.peak_live = std::max(P.peak_live, live);
            live -= dead[l];
        }
    }

    // 2. the class (type, level, input count) of every operator; the classes in order (type-major, then level, input
    // count) give the slots, a class's in node order
    auto type_rank = [](int32_t t) { return t == NGDB_OP_PROJ ? 0 : (t == NGDB_OP_INTER ? 1 : 2); };
    const int64_t n_lvl = (int64_t)top_level + 1, n_card = NGDB_MAX_CARD + 1;
    const int64_t n_class = 3 * n_lvl * n_card;
    if (n_class > INT32_MAX) {
        err = "too many execution steps";
        return NGDB_ERR_UNSUPPORTED;
    }
    auto class_of = [&](int32_t t, int32_t level, int32_t nin) { return (int32_t)((type_rank(t) * n_lvl + level) * n_card + nin); };
    std::vector<int32_t> start((size_t)n_class + 1, 0);
    for (const Shape& sh : tab.shapes)
        for (int32_t i = sh.op.at; i < sh.op.at + sh.op.n; ++i) {
            ShapeTable::Op& o = tab.op[i];
            o.cls = class_of(tab.type(sh, o.node), tab.level(sh, o), tab.nin(sh, o));
            if (step.empty()) start[o.cls + 1] += sh.count;
        }
    std::vector<int32_t> cls;                // Max-Fillness: of every operator, in node order
    if (!step.empty()) {
        cls.reserve(P.n_slots);
        int32_t base = 0;
        for (int32_t q = 0; q < B; ++q) {
            const Shape& sh = tab.shapes[shape_of[q]];
            for (const ShapeTable::Op& o : Span(tab.op, sh.op)) {
                cls.push_back(class_of(tab.type(sh, o.node), step[base + o.node], tab.nin(sh, o)));
                ++start[cls.back() + 1];
            }
            base += sh.node.n;
        }
    }
    for (int64_t c = 0; c < n_class; ++c) start[c + 1] += start[c];
    P.n_proj = start[n_lvl * n_card];
    P.n_inter = start[2 * n_lvl * n_card] - P.n_proj;
    P.n_neg = P.n_slots - P.n_proj - P.n_inter;
    const int32_t type_base[3] = {0, P.n_proj, P.n_proj + P.n_inter};

    // 3. groups: the classes that have members, by level, type, input count; members are a class's slots
    struct Class { int32_t next, ref0, n; };             // next slot; reference k of slot s is at ref0 + k * n + s
    std::vector<Class> at_class(n_class);
    int32_t ref_off = 0;
    for (int64_t l = 1; l < n_lvl; ++l)
        for (int32_t tr = 0; tr < 3; ++tr)
            for (int32_t nin = 1; nin < n_card; ++nin) {
                const int64_t c = (tr * n_lvl + l) * n_card + nin;
                const int32_t s0 = start[c], n = start[c + 1] - s0;
                if (n == 0) continue;
                const int32_t t = tr == 0 ? NGDB_OP_PROJ : (tr == 1 ? NGDB_OP_INTER : NGDB_OP_NEG);
                P.g_level.push_back((int32_t)l);
                P.g_type.push_back(t);
                P.g_nin.push_back(nin);
                P.g_n.push_back(n);
                P.g_out_base.push_back(s0);
                P.g_ref_off.push_back(ref_off);
                if (t == NGDB_OP_INTER) {
                    P.g_mlp_base.push_back(P.n_int_rows);
                    P.n_int_rows += n * nin;
                } else {
                    P.g_mlp_base.push_back(s0 - type_base[tr]);
                }
                P.g_rel_off.push_back(t == NGDB_OP_PROJ ? s0 : -1);      // (projections have the first slots)
                at_class[c] = Class{s0, ref_off - s0, n};
                ref_off += n * nin;
            }
    P.in_ref.resize(n_ref);
    P.in_gslot.resize(n_ref);
    P.rel.resize(P.n_proj);
    P.anchor_ent.resize(n_anchor);
    P.root_slot.resize(P.n_roots);
    {
        int32_t widest = 1;
        for (const Shape& sh : tab.shapes) widest = std::max(widest, sh.node.n);
        struct Place { int32_t ref, grad; };             // how operators refer to a node, and its gradient row
        std::vector<Place> place(widest);
        struct Out { int32_t at, stride; };
        std::vector<Out> out(widest);                    // where an operator's references go
        int32_t a = 0, r = 0;
        const int32_t* own = cls.data();
        for (int32_t q = 0; q < B; ++q) {
            const Shape& sh = tab.shapes[shape_of[q]];
            const int32_t* arg = qb.arg + qb.node_off[q];
            const int32_t* src = tab.flat.arg.data() + sh.node.at;
            for (const int32_t g : Span(tab.anchor, sh.anchor)) {
                const int32_t e = arg[src[g]];
                P.anchor_ent[a] = e;
                place[g] = Place{-1 - e, P.n_slots + a++};
            }
            const ShapeTable::Op* op = tab.op.data() + sh.op.at;
            for (int32_t i = 0; i < sh.op.n; ++i) {
                const ShapeTable::Op& o = op[i];
                Class& c = at_class[step.empty() ? o.cls : own[i]];
                const int32_t s = c.next++;
                place[o.node] = Place{s, s};
                out[i] = Out{c.ref0 + s, c.n};
                if (o.rel >= 0) P.rel[s] = arg[o.rel];
            }
            for (const ShapeTable::Ref& x : Span(tab.ref, sh.ref)) {
                const int32_t at = out[x.op].at + x.k * out[x.op].stride;
                P.in_ref[at] = place[x.kid].ref;
                P.in_gslot[at] = place[x.kid].grad;
            }
            for (const int32_t g : Span(tab.root, sh.root)) P.root_slot[r++] = place[g].ref;
            if (!step.empty()) own += sh.op.n;
        }
    }
    P.n_groups = (int32_t)P.g_level.size();
    P.n_levels = P.n_groups ? P.g_level.back() : 0;
    P.lvl_off.assign(P.n_levels + 2, 0);
    for (int32_t l : P.g_level) P.lvl_off[l + 1] += 1;
    for (size_t l = 1; l < P.lvl_off.size(); ++l) P.lvl_off[l] += P.lvl_off[l - 1];

    // 4. relation gradient index over the projections in slot order
    std::vector<int32_t> rsrc(P.n_proj);
    for (int32_t g = 0; g < P.n_groups; ++g)
        if (P.g_type[g] == NGDB_OP_PROJ)
            std::copy_n(P.in_gslot.begin() + P.g_ref_off[g], P.g_n[g], rsrc.begin() + P.g_out_base[g]);
    group_by_key(P.rel, R, rsrc, P.r_uniq, P.r_seg_off, P.r_src);

    // 5. rows of a forward-only pass under eager reference counting (Sec. 4.3, Reclaim(T); Alg. 1,
    // DecrementRefCounts): the steps in order; every output of a step takes, in group and member
    // order, the lowest free row (a new one if none is free); when the step has run, the rows of
    // the outputs it consumed are free again.  Every output has one consumer (queries are trees);
    // roots have none and keep their rows.  Free rows are bits; the search for the lowest goes on from
    // where the last one was found, and starts over when rows were freed.
    P.f_row.resize(P.n_slots);
    std::vector<uint64_t> free_bits((size_t)P.n_slots / 64 + 1, 0);
    size_t n_free = 0, word = 0;
    P.n_f_rows = 0;
    for (int32_t l = 1; l <= P.n_levels; ++l) {
        int32_t rows_now[3] = {0, 0, 0};
        for (int32_t g = P.lvl_off[l]; g < P.lvl_off[l + 1]; ++g) {
            const int32_t t = P.g_type[g];
            rows_now[type_rank(t)] += P.g_n[g] * (t == NGDB_OP_INTER ? P.g_nin[g] : 1);
            for (int32_t m = 0; m < P.g_n[g]; ++m) {
                int32_t row;
                if (n_free > 0) {
                    while (free_bits[word] == 0) ++word;
                    row = (int32_t)(word * 64 + __builtin_ctzll(free_bits[word]));
                    free_bits[word] &= free_bits[word] - 1;
                    --n_free;
                } else {
                    row = P.n_f_rows++;
                }
                P.f_row[P.g_out_base[g] + m] = row;
            }
        }
        for (int32_t g = P.lvl_off[l]; g < P.lvl_off[l + 1]; ++g) {
            const int32_t n_ref = P.g_n[g] * P.g_nin[g];
            for (int32_t k = 0; k < n_ref; ++k) {
                const int32_t ref = P.in_ref[P.g_ref_off[g] + k];
                if (ref < 0) continue;
                const int32_t row = P.f_row[ref];
                free_bits[row >> 6] |= 1ull << (row & 63);
                ++n_free;
            }
        }
        word = 0;
        for (int k = 0; k < 3; ++k) P.f_step_rows[k] = std::max(P.f_step_rows[k], rows_now[k]);
    }
    return NGDB_OK;
}

}  // namespace ngdb
