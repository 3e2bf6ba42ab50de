"""What a program built on this framework has it do, as cases that can be timed and compared.

A case is a dict of plain values: which path is taken, the sizes of the knowledge graph (N entities, R
relations), of the model (d, h, d_sem) and of the call (B queries, K negatives, C candidates, k results).
`prepare` makes what such a program holds before the call, `run` is one pass through the public entry points
(planning of the batch included: every batch of a program is a new one), `work` what no implementation can do
without, `tolerance` what another correct one may differ by.

Inputs follow the workloads of this repository: the 14 query structures, uniform negatives, entities of queries
drawn with the heavy-tailed frequencies of a knowledge graph. Tables and weights are those of a training run
under way: entity rows of the size they start with, weights scaled so that an operator keeps the size of what it
is given (distances then lie about the margin), moments of the size the gradients of such a batch have.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2602_21597_amd as ngdb
from paper_2602_21597_amd import binding

_KIND = {"e": 0, "p": 1, "i": 2, "n": 3, "u": 4}
# structure -> its operators, each with the positions of its inputs, the root last
_STRUCTURES = {
    "1p": "e p0", "2p": "e p0 p1", "3p": "e p0 p1 p2",
    "2i": "e p0 e p2 i1,3", "3i": "e p0 e p2 e p4 i1,3,5",
    "ip": "e p0 e p2 i1,3 p4", "pi": "e p0 p1 e p3 i2,4",
    "2u": "e p0 e p2 u1,3", "up": "e p0 e p2 u1,3 p4",
    "2in": "e p0 e p2 n3 i1,4", "3in": "e p0 e p2 e p4 n5 i1,3,6",
    "inp": "e p0 e p2 n3 i1,4 p5", "pin": "e p0 p1 e p3 n4 i2,5", "pni": "e p0 p1 n2 e p4 i3,5",
}
_ALL = ("1p", "2p", "3p", "2i", "3i", "ip", "pi", "2u", "up", "2in", "3in", "inp", "pin", "pni")
_POSITIVE = _ALL[:9]
_MIXES = {
    "five": {n: 0.2 for n in ("1p", "2p", "2i", "2in", "2u")},
    "all": {n: 1 / 14 for n in _ALL},
    "positive": {n: 1 / 9 for n in _POSITIVE},           # what box embeddings can express
    "weighted": {n: w / len(g) for g, w in ((_ALL[:3], 0.4), (_ALL[3:7], 0.3), (_ALL[9:], 0.2), (_ALL[7:9], 0.1))
                 for n in g},
    # for the sampler: structures of one size, so that a batch of B queries always has as many nodes
    "small": {n: 0.5 for n in ("2i", "2u")},
    "middle": {n: 0.25 for n in ("ip", "pi", "up", "2in")},
}


def _parsed(name):
    """(kind, inputs) of every node of a structure, the root last."""
    return [(_KIND[w[0]], [int(x) for x in w[1:].split(",") if x]) for w in _STRUCTURES[name].split()]


def _census(name):
    """branches, projections, intersection inputs, intersections, negations, anchors of one query of a structure
    (a projection above a union is repeated in each of its branches)."""
    nodes = _parsed(name)
    n = {k: sum(1 for kind, _ in nodes if kind == k) for k in range(5)}
    inputs = sum(len(i) for kind, i in nodes if kind == 2)
    branches = 2 if n[4] else 1
    return branches, n[1] + (1 if name == "up" else 0), inputs, n[2], n[3], n[0]


def _mean_census(case):
    mix = _MIXES[case["mix"]]
    return [sum(w * _census(name)[i] for name, w in mix.items()) for i in range(6)]


# ---------------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest training job: a graph of a thousand entities; a step is launches and host work
        dict(name="train_tiny", path="train", family="vec", N=1000, R=20, d=32, h=64, d_sem=0, B=64, K=8, mix="five",
             gamma=12.0, streams=1),
        # the everyday training step: FB15k-237-sized graph, tables that fit the caches
        dict(name="train_fb15k237", path="train", family="vec", N=15000, R=474, d=400, h=800, d_sem=0, B=512, K=128,
             mix="all", gamma=24.0, streams=2),
        # NELL-sized graph, a larger batch
        dict(name="train_nell", path="train", family="vec", N=63000, R=400, d=400, h=800, d_sem=0, B=1024, K=128,
             mix="all", gamma=24.0, streams=4),
        # a graph of millions of entities trained on one card: bound by the table rows that a step touches
        dict(name="train_wikikg2", path="train", family="vec", N=2500000, R=1070, d=400, h=800, d_sem=0, B=4096,
             K=1024, mix="weighted", gamma=24.0, streams=2),
        # the same with frozen text features projected into every entity row that is read
        dict(name="train_semantic", path="train", family="vec", N=5000000, R=2000, d=400, h=800, d_sem=1024, B=4096,
             K=1024, mix="all", gamma=24.0, streams=2),
        # box embeddings on a mid-size graph, at sizes that fill no tile
        dict(name="train_box_ragged", path="train", family="box", N=15000, R=474, d=300, h=500, d_sem=0, B=509, K=77,
             mix="positive", gamma=24.0, streams=2),
        # one user's question answered from a list of candidates: the latency of a call
        dict(name="serve_one", path="score", family="vec", N=15000, R=474, d=400, h=800, d_sem=0, B=1, C=1000,
             mix="all", gamma=24.0, streams=1),
        # candidate lists of an evaluation on a large graph
        dict(name="score_wikikg2", path="score", family="vec", N=2500000, R=1070, d=400, h=800, d_sem=0, B=1024,
             C=1000, mix="weighted", gamma=24.0, streams=1),
        # the ten nearest entities of a batch of queries
        dict(name="rank_fb15k237", path="rank", family="vec", N=15000, R=474, d=400, h=800, d_sem=0, B=512, k=10,
             mix="all", gamma=24.0, streams=1),
        # the same over five million entities with text features: the largest call of the framework
        dict(name="rank_semantic", path="rank", family="vec", N=5000000, R=2000, d=400, h=800, d_sem=1024, B=1024,
             k=10, mix="all", gamma=24.0, streams=1),
        # filtered ranks of known answers (the MRR and Hit@k of a validation pass)
        dict(name="answers_nell", path="answers", family="vec", N=63000, R=400, d=400, h=800, d_sem=0, B=1024, A=8,
             mix="all", gamma=24.0, streams=1),
        # a batch of queries and negatives drawn from the graph on the host
        dict(name="sample_fb15k237", path="sample", N=15000, R=474, T=310000, B=512, K=128,
             mix="middle"),
    ]


def _log(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / multiple) * multiple)))


def draw(rng):
    path = rng.choice(("train", "train", "train", "score", "rank", "answers", "sample"))
    if path == "sample":
        N = _log(rng, 1000, 60000)
        return dict(path=path, N=N, R=_log(rng, 20, 1000), T=_log(rng, 8 * N, 20 * N), B=_log(rng, 32, 2048),
                    K=_log(rng, 4, 256), mix=rng.choice(("small", "middle")))
    family = rng.choice(("vec", "vec", "vec", "box"))
    d_sem = rng.choice((0, 0, 0, 64 * rng.randint(2, 16))) if family == "vec" else 0
    d = _log(rng, 32, 512, 8 if d_sem else 4)
    c = dict(path=path, family=family, R=_log(rng, 20, 2000), d=d, h=_log(rng, 64, 1024, 4), d_sem=d_sem,
             mix="positive" if family == "box" else rng.choice(("five", "all", "weighted")),
             gamma=rng.choice((12.0, 24.0)), streams=rng.choice((1, 2, 4)) if path == "train" else 1)
    c["N"] = _log(rng, 1000, 1000000 if d_sem else 2500000)
    if path == "train":
        c["B"] = _log(rng, 16, 4096)
        c["K"] = _log(rng, 4, 1024)
    elif path == "score":
        c["B"] = _log(rng, 1, 1024)
        c["C"] = _log(rng, 10, 2000)
    else:
        c["B"] = _log(rng, 8, 1024)
        if path == "rank":
            c["k"] = rng.randint(1, 16)
        else:
            c["A"] = rng.randint(1, 12)
        if family == "box":                 # several times the arithmetic of the plain distance
            c["N"] = min(c["N"], 1000000)
    return c


# ------------------------------------------------------------------------------------------------- inputs

_HUB = 1.0 / 11.0     # entity frequencies fall as rank^-(1 - 1/11): a degree exponent of 2.1
_HEAD = 5.0           # the head of that law is cut off here: no entity takes more than a few per cent


def _entities(rng, N, n, stride):
    """n entity ids with heavy-tailed frequencies; `stride` scatters the frequent ones over the table."""
    lo, hi = _HEAD ** _HUB, (N + _HEAD) ** _HUB
    rank = np.minimum((rng.random(n) * (hi - lo) + lo) ** (1.0 / _HUB) - _HEAD, N - 1).astype(np.int64)
    return ((np.maximum(rank, 0) * stride + 7) % N).astype(np.int32)


def _strides(N):
    """Two different numbers without a common factor with N."""
    out = [p for p in range(int(N * 0.6180339) | 1, 4 * N + 8, 2) if math.gcd(p, N) == 1]
    return out[0], out[min(len(out) - 1, max(1, len(out) // 3))]


def _batch(case, rng):
    """A batch of queries in the flat arrays of the C boundary."""
    mix, B = _MIXES[case["mix"]], case["B"]
    names = sorted(mix)
    share = np.array([mix[n] for n in names])
    # shares met as nearly as B allows, the rest drawn
    count = np.floor(share * B + 1e-9).astype(np.int64)
    for i in rng.choice(len(names), size=int(B - count.sum()), p=share / share.sum()):
        count[i] += 1
    order = rng.permutation(np.repeat(np.arange(len(names)), count))
    shapes = []
    for n in names:
        nodes = _parsed(n)
        shapes.append((np.array([k for k, _ in nodes], np.uint8), np.array([len(i) for _, i in nodes], np.int32),
                       np.array([x for _, i in nodes for x in i], np.int32)))
    op = np.concatenate([shapes[t][0] for t in order])
    n_in = np.concatenate([shapes[t][1] for t in order])
    off = lambda lens: np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    s_head, s_tail = _strides(case["N"])
    arg = np.zeros(op.size, np.int32)
    arg[op == 0] = _entities(rng, case["N"], int((op == 0).sum()), s_head)
    arg[op == 1] = rng.integers(0, case["R"], int((op == 1).sum()), dtype=np.int32)
    return SimpleNamespace(B=B, node_off=off([shapes[t][0].size for t in order]), op=op, arg=arg, in_off=off(n_in),
                           in_idx=np.concatenate([shapes[t][2] for t in order]),
                           pos=_entities(rng, case["N"], B, s_tail))


def _tables(case, eng, gen):
    """Parameters, moments and text features on the GPU, bound to the engine."""
    dev = eng.device
    N, R, d, h, d_sem = case["N"], case["R"], case["d"], case["h"], case["d_sem"]
    near = lambda shape, a, lo=None: torch.empty(shape, device=dev).uniform_(-a if lo is None else lo, a, generator=gen)
    shapes = {"E": ((N, d), 0.1), "R": ((R, d), 0.1), "Ro": ((R, d), 0.1), "Wp": ((d, d_sem), 0.1)}
    for a, b, c, e in (("W1", "b1", "W2", "b2"), ("V1", "c1", "V2", "c2"), ("U1", "u1", "U2", "u2")):
        shapes.update({a: ((h, d), math.sqrt(6.0 / d)), b: ((h,), 0.02), c: ((d, h), math.sqrt(3.0 / h)), e: ((d,), 0.02)})
    size = 0.2 / case["B"]
    eng.tensors = {}
    for name in eng.tensor_names():
        shape, a = shapes[name]
        p = near(shape, a, -a / 4 if name == "Ro" else None)
        if case["path"] == "train":
            m = near(shape, 1.7 * size)
            v = torch.empty(shape, device=dev).uniform_(0.2 * size * size, 2 * size * size, generator=gen)
        else:
            m = v = torch.zeros(1, device=dev)        # an inference program has no moments
        eng.tensors[name] = (p, m, v)
    eng.H_sem = None
    if d_sem:
        sem = torch.empty((N, d_sem), dtype=torch.bfloat16, device=dev)
        for lo in range(0, N, 1 << 19):
            x = torch.empty((min(N - lo, 1 << 19), d_sem), device=dev).normal_(generator=gen)
            sem[lo:lo + x.shape[0]] = x / x.norm(dim=1, keepdim=True)
        eng.H_sem = sem.view(torch.int16)
    eng.bind(step=1000 if case["path"] == "train" else 0)


def _graph(case, rng):
    """T triples of a graph with hubs, heads and tails over two different sets of them."""
    N, R, T = case["N"], case["R"], case["T"]
    s_head, s_tail = _strides(N)
    keys = np.zeros(0, np.int64)
    for _ in range(50):
        n = int((T - keys.size) * 1.3) + 16
        h, t = _entities(rng, N, n, s_head), _entities(rng, N, n, s_tail)
        r = rng.integers(0, R, n)
        ok = h != t
        keys = np.unique(np.concatenate([keys, (h[ok].astype(np.int64) * R + r[ok]) * N + t[ok]]))
        if keys.size >= T:
            break
    keys = rng.permutation(keys)[:T]
    return ((keys // N // R).astype(np.int32), (keys // N % R).astype(np.int32), (keys % N).astype(np.int32))


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["path"] == "sample":
        mix = _MIXES[case["mix"]]
        names = sorted(mix)
        sampler = ngdb.Sampler(case["N"], case["R"], *_graph(case, rng), names, [mix[n] for n in names], seed=int(seed),
                               n_threads=4)
        return SimpleNamespace(case=case, sampler=sampler)
    eng = ngdb.Engine(case["N"], case["R"], case["d"], case["h"], case["gamma"], d_sem=case["d_sem"],
                      num_streams=case["streams"],
                      family=binding.FAMILY_BOX if case["family"] == "box" else binding.FAMILY_VEC)
    gen = torch.Generator(device=eng.device)
    gen.manual_seed(int(seed))
    _tables(case, eng, gen)
    s = SimpleNamespace(case=case, eng=eng, batch=_batch(case, rng))
    dev, N, B = eng.device, case["N"], case["B"]
    if case["path"] == "train":
        s.neg = torch.randint(0, N, (B, case["K"]), dtype=torch.int32, device=dev, generator=gen)
        s.state = {name + suffix: t for name, ts in eng.tensors.items() for suffix, t in zip((".p", ".m", ".v"), ts)}
    elif case["path"] == "score":
        s.cand = torch.randint(0, N, (B, case["C"]), dtype=torch.int32, device=dev, generator=gen)
    elif case["path"] == "answers":
        # 1 to 2A - 1 answers a query, A of them on average
        n = rng.permutation(1 + np.arange(B) * (2 * case["A"] - 1) // B)
        off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
        ans = _entities(rng, N, int(off[-1]), _strides(N)[1])
        ans[off[:-1]] = s.batch.pos
        s.ans_off, s.ans = torch.from_numpy(off).to(dev), torch.from_numpy(ans).to(dev)
    return s


# --------------------------------------------------------------------------------------------- one pass

def run(s):
    case = s.case
    if case["path"] == "sample":
        b = s.sampler.next(case["B"], case["K"])
        return [b.node_off, b.op, b.arg, b.in_off, b.in_idx, b.pos, b.negs]
    plan = s.eng.plan(s.batch)
    if case["path"] == "train":
        out = {"loss": s.eng.train_step(plan, s.neg), **s.state}
    elif case["path"] == "score":
        out = s.eng.score(plan, s.cand)
    elif case["path"] == "rank":
        out = s.eng.rank_all(plan, case["k"])
    else:
        # ranks as numbers: an entity within rounding of an answer's distance may count or not
        ranks, dist, metrics = s.eng.rank_answers(plan, s.ans_off, s.ans)
        out = [ranks.to(torch.float32), dist, metrics]
    plan.free()
    return out


def work(case):
    B = case["B"]
    branches, proj, inputs, inter, neg, anchors = _mean_census(case)
    if case["path"] == "sample":      # a batch and its negatives written, the triples it is made of read once
        nodes = B * (anchors + proj + inter + neg)
        return {"bytes": B * case["K"] * 4 + nodes * (1 + 4 + 4 + 4 + 12) + 2 * 4 * B, "flops": 0}
    N, R, d, h, d_sem = case["N"], case["R"], case["d"], case["h"], case["d_sem"]
    box = case["family"] == "box"
    rows = B * (2 * inputs if box else proj + inputs + neg)       # rows that pass through a two-layer MLP
    weights = (2 if box else 3) * (2 * d * h + d + h)
    distinct = lambda n, of: of * -math.expm1(n * math.log1p(-1.0 / of)) if of > 1 else min(n, of)
    if case["path"] == "train":
        pairs = B * (case["K"] + 1)
        e = distinct(B * (case["K"] + anchors + 1), N)
        r = distinct(B * proj, R) * (2 if box else 1)
        sem = 2 * e * d_sem + (24 * d * d_sem if d_sem else 0)
        return {"bytes": 24 * d * (e + r) + 24 * weights + sem + 4 * B * case["K"],
                "flops": 12 * d * h * rows + (10 if box else 5) * pairs * branches * d + 4 * e * d * d_sem}
    forward = 4 * d * h * rows
    if case["path"] == "score":
        pairs = B * case["C"]
        e = distinct(pairs + B * anchors, N)
        return {"bytes": e * (4 * d + 2 * d_sem) + 4 * d * min(R, B * proj) + 4 * weights + 8 * pairs,
                "flops": forward + (5 if box else 2) * pairs * branches * d + 2 * e * d * d_sem}
    out = 8 * B * case["k"] if case["path"] == "rank" else 12 * B * case["A"]
    return {"bytes": N * (4 * d + 2 * d_sem) + 4 * d * min(R, B * proj) + 4 * weights + out,
            "flops": forward + (5 if box else 2) * B * branches * N * d + 2 * N * d * d_sem}


def tolerance(case):
    path = case["path"]
    if path == "sample":
        return "exact"
    if path == "train":
        # fp32 sums and their order give 1e-6 to 1e-5. Beyond that a hidden unit or a coordinate whose sign hangs on
        # the last bit switches one element of one row's gradient, which shows in the moments: inputs moved by one
        # unit in the last place give up to 4e-4 (0.04 at one element) on the large graph, and 1.8e-3 (0.54 at one
        # element) with text features, whose projection and its gradient are products of bf16 rows
        return {"rel": 4e-3, "max": 0.9} if case["d_sem"] else {"rel": 1e-3, "max": 0.6}
    if path == "score":
        return {"rel": 1e-5, "max": 1e-3}
    if path == "rank":
        # ids of entities at equal distance within rounding may change places
        return {"rel": 1e-5, "max": 1e-3, "differ": 5e-3}
    # distances to rounding; an entity within rounding of an answer moves its rank by one
    return {"rel": 1e-3, "max": 0.1}
