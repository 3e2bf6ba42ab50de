// Online query sampler (App. "Stochastic Online Query Sampling"): batches of
// first-order-logic queries are synthesised on the fly from the graph instead
// of being read from a pre-computed set.  A query is a template (one of the 14
// patterns of Sec. 3.1) instantiated by a restricted random walk that runs
// backwards from the answer -- a projection reaching entity v takes a uniform
// in-edge of v, the children of an intersection all reach v, a negated or a
// second union branch is grown toward an unrelated entity -- followed by
// rejection: walks that hit an entity without in-edges, intersections with two
// identical children, and queries whose end point is not an answer (it may lie
// in a negated branch) are drawn again, so every query has a non-empty answer
// set that contains its positive.  Host only, C++ threads; every query draws
// from its own counter-based random stream (seed, batch number, query number),
// so a batch does not depend on the number of threads.
#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "ngdb.h"

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define NGDB_WIDE_DRAWS 1
#include <immintrin.h>
#endif

namespace {

// ---------------------------------------------------------------- random stream
struct Rng {   // splitmix64 over a per-query counter
    uint64_t s;
    Rng(uint64_t seed, uint64_t batch, uint64_t query) {
        s = seed ^ (batch * 0x9E3779B97F4A7C15ull) ^ (query * 0xC2B2AE3D27D4EB4Full + 0x165667B19E3779F9ull);
        next();
        next();
    }
    uint64_t next() {
        uint64_t z = (s += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
    // uniform in [0, n), n > 0 (multiply-shift with rejection of the biased tail, which is shorter than n: the
    // division is left to the draws that might lie in it)
    uint64_t below(uint64_t n) {
        for (;;) {
            const uint64_t x = next();
            const unsigned __int128 m = (unsigned __int128)x * n;
            if ((uint64_t)m >= n || (uint64_t)m >= (uint64_t)(-n) % n) return (uint64_t)(m >> 64);
        }
    }
    double unit() { return (double)(next() >> 11) * (1.0 / 9007199254740992.0); }
    // two uniform draws in [0, n), n < 2^31, from one 64-bit word (each half: multiply-shift,
    // redrawn together if either falls into the biased tail = 2^32 mod n)
    void below32x2(uint32_t n, uint32_t tail, int32_t* out) {
        for (;;) {
            const uint64_t x = next();
            const uint64_t a = (uint64_t)(uint32_t)x * n, b = (x >> 32) * n;
            if ((uint32_t)a >= tail && (uint32_t)b >= tail) {
                out[0] = (int32_t)(a >> 32);
                out[1] = (int32_t)(b >> 32);
                return;
            }
        }
    }
};

// Rng::below32x2 eight times at once, for as long as none of the eight is redrawn: the counters after s, results as it leaves them.
// Returns the pairs drawn, a multiple of eight.  Batches on four threads, one by one against this: 512 queries x 256 negatives 60 and
// 48 us, 1500 x 100 117 and 106, 2048 x 256 222 and 208 (with the structures' names in one call); below 16 negatives nothing changes.
#ifdef NGDB_WIDE_DRAWS
__attribute__((target("avx512f,avx512dq"))) int draw_wide(uint64_t s, uint32_t n, uint32_t tail, int pairs, int32_t* out) {
    constexpr uint64_t G = 0x9E3779B97F4A7C15ull;
    const __m512i lanes = _mm512_set_epi64(8, 7, 6, 5, 4, 3, 2, 1);
    const __m512i c1 = _mm512_set1_epi64((long long)0xBF58476D1CE4E5B9ull), c2 = _mm512_set1_epi64((long long)0x94D049BB133111EBull);
    const __m512i low = _mm512_set1_epi64(0xFFFFFFFFll), of = _mm512_set1_epi64(n), least = _mm512_set1_epi64(tail);
    __m512i counter = _mm512_add_epi64(_mm512_set1_epi64((long long)s), _mm512_mullo_epi64(lanes, _mm512_set1_epi64((long long)G)));
    int p = 0;
    for (; p + 8 <= pairs; p += 8) {
        __m512i z = counter;
        z = _mm512_mullo_epi64(_mm512_xor_si512(z, _mm512_srli_epi64(z, 30)), c1);
        z = _mm512_mullo_epi64(_mm512_xor_si512(z, _mm512_srli_epi64(z, 27)), c2);
        z = _mm512_xor_si512(z, _mm512_srli_epi64(z, 31));
        const __m512i a = _mm512_mul_epu32(z, of), b = _mm512_mul_epu32(_mm512_srli_epi64(z, 32), of);
        if (_mm512_cmplt_epu64_mask(_mm512_and_si512(a, low), least) | _mm512_cmplt_epu64_mask(_mm512_and_si512(b, low), least)) break;
        _mm512_storeu_si512(out + 2 * p, _mm512_or_si512(_mm512_srli_epi64(a, 32), _mm512_andnot_si512(low, b)));
        counter = _mm512_add_epi64(counter, _mm512_set1_epi64((long long)(8 * G)));
    }
    return p;
}
bool draws_wide() { return __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512dq"); }
#else
int draw_wide(uint64_t, uint32_t, uint32_t, int, int32_t*) { return 0; }
bool draws_wide() { return false; }
#endif

// K uniform draws in [0, n)
void draw_row(Rng& rng, uint32_t n, uint32_t tail, int K, int32_t* out) {
    static const bool wide = draws_wide();
    int k = 0;
    while (k + 2 <= K) {
        if (wide && K - k >= 16) {
            const int pairs = draw_wide(rng.s, n, tail, (K - k) / 2, out + k);
            rng.s += (uint64_t)pairs * 0x9E3779B97F4A7C15ull;
            k += 2 * pairs;
            if (k + 2 > K) break;
        }
        rng.below32x2(n, tail, out + k);
        k += 2;
    }
    if (k < K) out[k] = (int32_t)rng.below((uint64_t)n);
}

// ---------------------------------------------------------------- graph
struct Graph {
    int32_t N = 0, R = 0;
    int64_t T = 0;
    std::vector<int64_t> in_off, out_off;          // [N+1]
    struct InEdge { int32_t head, rel; };
    struct OutEdge { int32_t rel, tail; };
    std::vector<InEdge> in_edge;                   // in-edges of every entity, any fixed order
    struct RelEdge { int32_t rel, at, head; };
    std::vector<RelEdge> rel_edge;                 // the same sorted by relation; at: place among the entity's in-edges
    std::vector<OutEdge> out_edge;                 // out-edges sorted by (relation, tail)
    std::vector<int32_t> tails;                    // tail of every triple (answers are drawn from it)

    bool has_triple(int32_t h, int32_t r, int32_t t) const {
        int64_t lo = out_off[h], hi = out_off[h + 1];
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            const OutEdge e = out_edge[mid];
            if (e.rel < r || (e.rel == r && e.tail < t)) lo = mid + 1; else hi = mid;
        }
        return lo < out_off[h + 1] && out_edge[lo].rel == r && out_edge[lo].tail == t;
    }
};

// ---------------------------------------------------------------- templates
struct Tmpl {            // node of a template tree
    char kind;           // 'e' 'p' 'i' 'n' 'u'
    std::vector<int> kids;
};
struct Template {
    std::string name;
    std::vector<Tmpl> nodes;   // root last
};

// shapes in a small prefix notation: e, p(x), i(x,..), n(x), u(x,..)
int parse(const char*& s, std::vector<Tmpl>& out) {
    Tmpl t;
    t.kind = *s++;
    if (t.kind != 'e') {
        ++s;   // '('
        for (;;) {
            t.kids.push_back(parse(s, out));
            if (*s == ',') { ++s; continue; }
            ++s;   // ')'
            break;
        }
    }
    out.push_back(t);
    return (int)out.size() - 1;
}

const char* shape_of(const std::string& name) {
    static const char* const table[][2] = {
        {"1p", "p(e)"}, {"2p", "p(p(e))"}, {"3p", "p(p(p(e)))"}, {"2i", "i(p(e),p(e))"}, {"3i", "i(p(e),p(e),p(e))"},
        {"ip", "p(i(p(e),p(e)))"}, {"pi", "i(p(p(e)),p(e))"}, {"2u", "u(p(e),p(e))"}, {"up", "p(u(p(e),p(e)))"},
        {"2in", "i(p(e),n(p(e)))"}, {"3in", "i(p(e),p(e),n(p(e)))"}, {"inp", "p(i(p(e),n(p(e))))"},
        {"pin", "i(p(p(e)),n(p(e)))"}, {"pni", "i(n(p(p(e))),p(e))"}};
    for (const auto& row : table)
        if (name == row[0]) return row[1];
    return nullptr;
}

// ---------------------------------------------------------------- one query
constexpr int MAX_NODES = 16;   // of a query, and inputs of all its nodes: more than any template has
struct Query {           // nodes in post-order, root last
    int n = 0;
    uint8_t op[MAX_NODES];
    int32_t arg[MAX_NODES], in_off[MAX_NODES + 1] = {0}, in_idx[MAX_NODES];
    void clear() { n = 0; }
    int add(uint8_t o, int32_t a, const int* ins, int n_in) {
        op[n] = o;
        arg[n] = a;
        for (int k = 0; k < n_in; ++k) in_idx[in_off[n] + k] = ins[k];
        in_off[n + 1] = in_off[n] + n_in;
        return n++;
    }
    void truncate(int n_nodes) { n = n_nodes; }
};

struct Builder {
    const Graph& g;
    const Template& tp;
    Rng& rng;
    Query& q;
    long budget = 0;     // membership tests: edge visits left

    // Is v an answer of the sub-query rooted at node n?  Exact, by walking in-edges; gives
    // up (treated as "cannot tell") when the budget runs out.
    int contains(int n, int32_t v) {
        const uint8_t o = q.op[n];
        const int32_t* ins = q.in_idx + q.in_off[n];
        const int nin = q.in_off[n + 1] - q.in_off[n];
        if (o == NGDB_OP_ANCHOR) return q.arg[n] == v;
        if (o == NGDB_OP_NEG) {
            const int c = contains(ins[0], v);
            return c < 0 ? c : !c;
        }
        if (o == NGDB_OP_INTER || o == NGDB_OP_UNION) {
            for (int k = 0; k < nin; ++k) {
                const int c = contains(ins[k], v);
                if (c < 0) return c;
                if (o == NGDB_OP_INTER && !c) return 0;
                if (o == NGDB_OP_UNION && c) return 1;
            }
            return o == NGDB_OP_INTER;
        }
        // projection by relation r: some m with (m, r, v) in the graph and m an answer of the input
        const int32_t r = q.arg[n];
        if (q.op[ins[0]] == NGDB_OP_ANCHOR) return g.has_triple(q.arg[ins[0]], r, v);
        // The budget counts in-edges in their fixed order, whatever their relation; those of relation r are looked up
        // (entities that answers are drawn at have thousands of in-edges, few of them of one relation).
        const Graph::RelEdge *e = g.rel_edge.data() + g.in_off[v], *end = g.rel_edge.data() + g.in_off[v + 1];
        const long degree = (long)(end - e);
        e = std::lower_bound(e, end, r, [](const Graph::RelEdge& x, int32_t rel) { return x.rel < rel; });
        long seen = 0;
        for (; e < end && e->rel == r; ++e) {
            budget -= e->at + 1 - seen;
            seen = e->at + 1;
            if (budget < 0) return -1;
            const int c = contains(ins[0], e->head);
            if (c) return c;
        }
        budget -= degree - seen;
        if (budget < 0) return -1;
        return 0;
    }

    bool same_subtree(int a0, int a1, int b0, int b1) const {
        if (a1 - a0 != b1 - b0) return false;
        for (int i = 0; i < a1 - a0; ++i) {
            if (q.op[a0 + i] != q.op[b0 + i] || q.arg[a0 + i] != q.arg[b0 + i]) return false;
            const int na = q.in_off[a0 + i + 1] - q.in_off[a0 + i], nb = q.in_off[b0 + i + 1] - q.in_off[b0 + i];
            if (na != nb) return false;
            for (int k = 0; k < na; ++k)
                if (q.in_idx[q.in_off[a0 + i] + k] - a0 != q.in_idx[q.in_off[b0 + i] + k] - b0)
                    return false;
        }
        return true;
    }

    int32_t random_tail() { return g.tails[rng.below((uint64_t)g.T)]; }

    // instantiate template node t so that v is one of its answers; -1 = draw the query again
    int grow(int t, int32_t v) {
        const Tmpl& node = tp.nodes[t];
        switch (node.kind) {
            case 'e':
                return q.add(NGDB_OP_ANCHOR, v, nullptr, 0);
            case 'p': {
                const int64_t lo = g.in_off[v], hi = g.in_off[v + 1];
                if (hi == lo) return -1;
                const int64_t j = lo + (int64_t)rng.below((uint64_t)(hi - lo));
                const Graph::InEdge e = g.in_edge[j];
                const int c = grow(node.kids[0], e.head);
                if (c < 0) return -1;
                return q.add(NGDB_OP_PROJ, e.rel, &c, 1);
            }
            case 'n': {
                const int c = grow(node.kids[0], random_tail());
                if (c < 0) return -1;
                return q.add(NGDB_OP_NEG, 0, &c, 1);
            }
            case 'i': {
                int kids[MAX_NODES], span[MAX_NODES], n = 0;      // roots and first nodes of the children
                for (int kt : node.kids) {
                    int c = -1;
                    for (int attempt = 0; attempt < 8; ++attempt) {
                        const int start = q.n;
                        c = grow(kt, v);
                        if (c < 0) return -1;
                        bool dup = false;
                        for (int k = 0; k < n; ++k) dup = dup || same_subtree(span[k], kids[k] + 1, start, q.n);
                        if (!dup) {
                            span[n] = start;
                            break;
                        }
                        q.truncate(start);
                        c = -1;
                    }
                    if (c < 0) return -1;
                    kids[n++] = c;
                }
                return q.add(NGDB_OP_INTER, 0, kids, n);
            }
            case 'u': {
                int kids[MAX_NODES], n = 0;
                for (int kt : node.kids) {
                    const int c = grow(kt, n == 0 ? v : random_tail());
                    if (c < 0) return -1;
                    kids[n++] = c;
                }
                return q.add(NGDB_OP_UNION, 0, kids, n);
            }
        }
        return -1;
    }
};

}  // namespace

// A batch is drawn in chunks of 32 queries, which the threads take in turn; each chunk leaves its queries one after
// the other in arrays of its own, and whoever ends the last one strings them together.  (Equal shares per thread, queries
// in vectors strung together by one thread, in-edges of hubs scanned for a relation: 107 us a batch of 512 queries with
// 128 negatives over 310 000 triples on four threads, 57 now; one thread alone 235, now 169.)
constexpr int CHUNK = 32;
struct Chunk {
    int n_nodes, n_idx, failed;           // failed: first query that could not be drawn, or -1
    int32_t node_end[CHUNK];
    uint8_t op[CHUNK * MAX_NODES];
    int32_t arg[CHUNK * MAX_NODES], in_end[CHUNK * MAX_NODES], in_idx[CHUNK * MAX_NODES];
};

struct BatchArrays {   // what ngdb_sampler_next hands out
    std::vector<int32_t> node_off, arg, in_off, in_idx, pos, neg;
    std::vector<uint8_t> op, tmpl;
    std::vector<Chunk> chunk;
};

struct ngdb_sampler_s {
    Graph g;
    std::vector<Template> templates;
    std::vector<double> cdf;
    uint64_t seed = 0, batch_no = 0;
    BatchArrays out[3];                 // three sets taking turns: a batch stays valid over the next call
                                        // while the one after it is already being drawn
    std::string err;
    // The batch being drawn.  Read-ahead: after a call has returned batch t, the threads draw batch t+1 (same
    // sizes), so that the next call usually finds its batch ready.  The batches
    // are functions of (seed, batch number, query number): reading ahead changes nothing in them.
    std::vector<std::thread> threads;
    std::mutex mu;
    std::condition_variable work, done;
    bool stop = false, posted = false, ahead = false;       // from here on guarded by mu (ahead: batch `no` is the next call's)
    uint64_t no = 0;
    int B = 0, K = 0, n_chunks = 0, next = 0, ended = 0, rc = NGDB_OK;
    std::string draw_err;
    std::atomic<uint64_t> posts{0}, finished{0};            // batches posted / complete so far (also read without mu)

    ~ngdb_sampler_s() {
        {
            std::lock_guard<std::mutex> lk(mu);
            stop = true;
        }
        work.notify_all();
        for (std::thread& t : threads) t.join();
    }
};

namespace {

void draw_chunk(const ngdb_sampler_s& s, uint64_t batch_no, int lo, int hi, int K, BatchArrays& o, Chunk& c) {
    c.n_nodes = c.n_idx = 0;
    c.failed = -1;
    const uint32_t n = (uint32_t)s.g.N, tail = (uint32_t)(-n) % n;
    Query q;
    for (int i = lo; i < hi; ++i) {
        Rng rng(s.seed, batch_no, (uint64_t)i);
        const double u = rng.unit();
        size_t t = 0;
        while (t + 1 < s.cdf.size() && u >= s.cdf[t]) ++t;
        o.tmpl[i] = (uint8_t)t;
        const Template& tp = s.templates[t];
        bool ok = false;
        int32_t v = 0;
        for (int attempt = 0; attempt < 1000 && !ok; ++attempt) {
            q.clear();
            v = s.g.tails[rng.below((uint64_t)s.g.T)];
            Builder b{s.g, tp, rng, q};
            if (b.grow((int)tp.nodes.size() - 1, v) < 0) continue;
            b.budget = 20000;
            ok = b.contains(q.n - 1, v) == 1;   // (not if e.g. the end point lies in a negated branch)
        }
        o.pos[i] = ok ? v : 0;
        if (!ok && c.failed < 0) c.failed = i;
        for (int k = 0; k < q.n; ++k) {
            c.op[c.n_nodes + k] = q.op[k];
            c.arg[c.n_nodes + k] = q.arg[k];
            c.in_end[c.n_nodes + k] = c.n_idx + q.in_off[k + 1];
        }
        for (int k = 0; k < q.in_off[q.n]; ++k) c.in_idx[c.n_idx + k] = q.in_idx[k];
        c.n_nodes += q.n;
        c.n_idx += q.in_off[q.n];
        c.node_end[i - lo] = c.n_nodes;
        draw_row(rng, n, tail, K, o.neg.data() + (size_t)i * K);
    }
}

// the chunks of a batch one after the other
int join_chunks(const ngdb_sampler_s& s, int B, int n_chunks, BatchArrays& o, std::string* err) {
    size_t nodes = 0, idx = 0;
    for (int c = 0; c < n_chunks; ++c) {
        if (o.chunk[c].failed >= 0) {
            *err = "query instantiation kept failing for template " + s.templates[o.tmpl[o.chunk[c].failed]].name;
            return NGDB_ERR_UNSUPPORTED;
        }
        nodes += o.chunk[c].n_nodes;
        idx += o.chunk[c].n_idx;
    }
    auto room = [](auto& v, size_t n) { if (v.size() < n) v.resize(n + n / 8); };
    try {
        room(o.node_off, (size_t)B + 1);
        room(o.op, nodes); room(o.arg, nodes); room(o.in_off, nodes + 1); room(o.in_idx, idx);
    } catch (const std::bad_alloc&) {
        return NGDB_ERR_OOM;
    }
    int32_t nb = 0, ib = 0, q = 0;
    o.node_off[0] = o.in_off[0] = 0;
    for (int c = 0; c < n_chunks; ++c) {
        const Chunk& ch = o.chunk[c];
        memcpy(o.op.data() + nb, ch.op, ch.n_nodes);
        memcpy(o.arg.data() + nb, ch.arg, (size_t)ch.n_nodes * 4);
        memcpy(o.in_idx.data() + ib, ch.in_idx, (size_t)ch.n_idx * 4);
        int32_t* off = o.in_off.data() + nb + 1;
        for (int k = 0; k < ch.n_nodes; ++k) off[k] = ib + ch.in_end[k];
        const int nq = std::min(CHUNK, B - q);
        for (int k = 0; k < nq; ++k) o.node_off[q + 1 + k] = nb + ch.node_end[k];
        nb += ch.n_nodes;
        ib += ch.n_idx;
        q += nq;
    }
    return NGDB_OK;
}

inline void relax() {
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
}
constexpr int SPINS = 1000;      // about 20 us: a thread that has just drawn (or a caller that finds its batch
                                 // under way) is not put to sleep and woken for a wait shorter than that

// Draws chunks of the posted batch until none is left to take; mu is held on entry and on return.
void help(ngdb_sampler_s* s, std::unique_lock<std::mutex>& lk) {
    while (!s->stop && s->posted && s->next < s->n_chunks) {
        const int c = s->next++, B = s->B, K = s->K, n_chunks = s->n_chunks;
        const uint64_t no = s->no;
        BatchArrays& o = s->out[no % 3];
        lk.unlock();
        draw_chunk(*s, no, c * CHUNK, std::min(B, (c + 1) * CHUNK), K, o, o.chunk[c]);
        lk.lock();
        if (++s->ended < n_chunks) continue;      // (the batch stays posted until its last chunk has ended)
        lk.unlock();
        std::string err;
        const int rc = join_chunks(*s, B, n_chunks, o, &err);
        lk.lock();
        s->rc = rc;
        s->draw_err = err;
        s->posted = false;
        s->finished.fetch_add(1);
        s->done.notify_all();
    }
}

void thread_loop(ngdb_sampler_s* s) {
    std::unique_lock<std::mutex> lk(s->mu);
    for (;;) {
        help(s, lk);
        if (s->stop) return;
        const uint64_t seen = s->posts.load();
        lk.unlock();
        for (int i = 0; i < SPINS && s->posts.load(std::memory_order_relaxed) == seen; ++i) relax();
        lk.lock();
        s->work.wait(lk, [&] { return s->stop || s->posts.load() != seen || (s->posted && s->next < s->n_chunks); });
        if (s->stop) return;
    }
}

// hands batch number no to the threads; mu held, nothing posted
int post(ngdb_sampler_s* s, uint64_t no, int B, int K) {
    BatchArrays& o = s->out[no % 3];
    s->n_chunks = (B + CHUNK - 1) / CHUNK;
    try {
        if (o.pos.size() < (size_t)B) { o.pos.resize(B); o.tmpl.resize(B); }
        if (o.neg.size() < (size_t)B * K) o.neg.resize((size_t)B * K);
        if (o.chunk.size() < (size_t)s->n_chunks) o.chunk.resize(s->n_chunks);
        if (B == 0) { o.node_off.assign(1, 0); o.in_off.assign(1, 0); }
    } catch (const std::bad_alloc&) {
        return NGDB_ERR_OOM;
    }
    s->no = no; s->B = B; s->K = K;
    s->next = s->ended = 0;
    s->rc = NGDB_OK;
    s->posted = s->n_chunks > 0;
    s->posts.fetch_add(1);
    if (!s->posted) s->finished.fetch_add(1);
    return NGDB_OK;
}

}  // namespace

extern "C" {

int ngdb_sampler_create(int32_t N, int32_t R, int64_t T, const int32_t* head, const int32_t* rel,
                        const int32_t* tail, const char* template_names, const float* weights, uint64_t seed,
                        int32_t n_threads, ngdb_sampler_t** out) {
    if (!out) return NGDB_ERR_ARG;
    *out = nullptr;
    if (N <= 0 || R <= 0 || T <= 0 || !head || !rel || !tail || !template_names || n_threads < 1 || n_threads > 256)
        return NGDB_ERR_ARG;
    for (int64_t i = 0; i < T; ++i)
        if (head[i] < 0 || head[i] >= N || tail[i] < 0 || tail[i] >= N || rel[i] < 0 || rel[i] >= R)
            return NGDB_ERR_RANGE;
    ngdb_sampler_t* s = new (std::nothrow) ngdb_sampler_s();
    if (!s) return NGDB_ERR_OOM;
    try {
        // templates: comma separated names
        std::string names(template_names), cur;
        names.push_back(',');
        for (char ch : names) {
            if (ch != ',') { cur.push_back(ch); continue; }
            if (cur.empty()) continue;
            const char* shape = shape_of(cur);
            if (!shape) { delete s; return NGDB_ERR_ARG; }
            Template tp;
            tp.name = cur;
            parse(shape, tp.nodes);          // (at most 9 nodes with 8 inputs: MAX_NODES)
            s->templates.push_back(std::move(tp));
            cur.clear();
        }
        if (s->templates.empty()) { delete s; return NGDB_ERR_ARG; }
        double tot = 0.0;
        for (size_t i = 0; i < s->templates.size(); ++i) {
            const double w = weights ? (double)weights[i] : 1.0;
            if (!(w >= 0.0)) { delete s; return NGDB_ERR_ARG; }
            tot += w;
            s->cdf.push_back(tot);
        }
        if (!(tot > 0.0)) { delete s; return NGDB_ERR_ARG; }
        for (double& c : s->cdf) c /= tot;
        // adjacency by tail (in-edges) and by head (out-edges, sorted by relation and tail)
        Graph& g = s->g;
        g.N = N; g.R = R; g.T = T;
        g.tails.assign(tail, tail + T);
        g.in_off.assign((size_t)N + 1, 0);
        g.out_off.assign((size_t)N + 1, 0);
        for (int64_t i = 0; i < T; ++i) { ++g.in_off[tail[i] + 1]; ++g.out_off[head[i] + 1]; }
        for (int32_t v = 0; v < N; ++v) { g.in_off[v + 1] += g.in_off[v]; g.out_off[v + 1] += g.out_off[v]; }
        g.in_edge.resize(T); g.out_edge.resize(T);
        std::vector<int64_t> in_fill(g.in_off.begin(), g.in_off.end() - 1), out_fill(g.out_off.begin(), g.out_off.end() - 1);
        for (int64_t i = 0; i < T; ++i) {
            const int64_t a = in_fill[tail[i]]++, b = out_fill[head[i]]++;
            g.in_edge[a] = {head[i], rel[i]};
            g.out_edge[b] = {rel[i], tail[i]};
        }
        // (relations in ascending order: every entity's list fills up sorted)
        std::vector<int64_t> rel_off((size_t)R + 1, 0), by_rel(T);
        for (int64_t j = 0; j < T; ++j) ++rel_off[g.in_edge[j].rel + 1];
        for (int32_t r = 0; r < R; ++r) rel_off[r + 1] += rel_off[r];
        std::vector<int32_t> tail_of(T);
        for (int32_t v = 0; v < N; ++v)
            for (int64_t j = g.in_off[v]; j < g.in_off[v + 1]; ++j) {
                tail_of[j] = v;
                by_rel[rel_off[g.in_edge[j].rel]++] = j;
            }
        g.rel_edge.resize(T);
        in_fill.assign(g.in_off.begin(), g.in_off.end() - 1);
        for (const int64_t j : by_rel) {
            const int32_t v = tail_of[j];
            g.rel_edge[in_fill[v]++] = {g.in_edge[j].rel, (int32_t)(j - g.in_off[v]), g.in_edge[j].head};
        }
        for (int32_t v = 0; v < N; ++v)
            std::sort(g.out_edge.begin() + g.out_off[v], g.out_edge.begin() + g.out_off[v + 1],
                      [](const Graph::OutEdge& x, const Graph::OutEdge& y) { return x.rel != y.rel ? x.rel < y.rel : x.tail < y.tail; });
    } catch (const std::bad_alloc&) {
        delete s;
        return NGDB_ERR_OOM;
    }
    s->seed = seed;
    try {
        for (int i = 0; i < n_threads; ++i) s->threads.emplace_back(thread_loop, s);
    } catch (...) {
        delete s;
        return NGDB_ERR_OOM;
    }
    *out = s;
    return NGDB_OK;
}

void ngdb_sampler_destroy(ngdb_sampler_t* s) { delete s; }

int ngdb_sampler_next(ngdb_sampler_t* s, int32_t B, int32_t K, ngdb_query_batch* batch, const int32_t** neg,
                      const uint8_t** template_id) {
    if (!s || !batch || B < 0 || K < 0 || (K > 0 && !neg)) return NGDB_ERR_ARG;
    const uint64_t batch_no = s->batch_no++;
    BatchArrays& o = s->out[batch_no % 3];
    {
        std::unique_lock<std::mutex> lk(s->mu);
        auto wait = [&] {          // for the batch posted last
            const uint64_t want = s->posts.load();
            lk.unlock();
            for (int i = 0; i < SPINS && s->finished.load(std::memory_order_relaxed) < want; ++i) relax();
            lk.lock();
            s->done.wait(lk, [&] { return s->finished.load() >= want; });
        };
        if (s->posted) wait();
        if (!s->ahead || s->no != batch_no || s->B != B || s->K != K) {     // first call, or other sizes than read ahead
            const int rc = post(s, batch_no, B, K);
            if (rc != NGDB_OK) return rc;
            s->work.notify_all();
            help(s, lk);
            if (s->posted) wait();
        }
        s->ahead = false;
        if (s->rc != NGDB_OK) {
            s->err = s->draw_err;
            return s->rc;
        }
        // read ahead: the next batch with the same sizes (left to the next call if there is no memory for it)
        s->ahead = post(s, batch_no + 1, B, K) == NGDB_OK;
    }
    s->work.notify_all();
    batch->n_queries = B;
    batch->node_off = o.node_off.data();
    batch->op = o.op.data();
    batch->arg = o.arg.data();
    batch->in_off = o.in_off.data();
    batch->in_idx = o.in_idx.data();
    batch->pos = o.pos.data();
    if (neg) *neg = o.neg.data();
    if (template_id) *template_id = o.tmpl.data();
    return NGDB_OK;
}

const char* ngdb_sampler_last_error(const ngdb_sampler_t* s) { return s ? s->err.c_str() : ""; }

}  // extern "C"
