"""Kernels chosen by size, at the sizes where the choice changes: matrix-vector forward layers, candidate lists shared by
several workgroups, weight gradients, the gradient index of one workgroup, of a short and of a long histogram."""
import numpy as np
import pytest

import workloads as wl
from oracle import model as om
from oracle import plan as oplan
from oracle import rank as orank
from . import parity as par

pytestmark = pytest.mark.gpu


def chain_launches(eng):
    """Launches of several layers so far (few rows, forward, backward), and their tiles that were computed by a workgroup with another one."""
    from paper_2602_21597_amd import binding
    n = [binding.lib().ngdb_debug_chain_launches(eng.ctx, kind) for kind in range(4)]
    assert min(n) >= 0
    return np.array(n)


@pytest.mark.parametrize("M,N,K", [(1, 5, 4), (1, 800, 400), (2, 401, 260), (3, 36, 1024), (8, 17, 800), (9, 72, 100),
                                   (16, 33, 1024), (17, 33, 64), (1, 9, 16384), (3, 8, 5460), (4, 16, 1028), (5, 12, 400)])
def test_forward_layers_of_few_rows(M, N, K):
    import torch
    from paper_2602_21597_amd import binding
    rng = np.random.default_rng(M * 1000 + N)
    A, B, bias = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N,)))
    perm = rng.permutation(M + 3)[:M].astype(np.int32)
    f = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = binding.debug_gemm(f(A), f(B), M, N, K, bias=f(bias), relu=True, dst_row=f(perm), out_rows=M + 3).cpu().numpy()
    want = np.maximum(A.astype(np.float64) @ B.T.astype(np.float64) + bias, 0.0)
    scale = np.abs(A).astype(np.float64) @ np.abs(B.T) + np.abs(bias)
    assert (np.abs(got[perm] - want) / scale).max() < 0.1 * 2e-6 * max(1.0, np.sqrt(K) / 8)
    assert not np.any(np.delete(got, perm, axis=0))


# problems of one launch that differ in rows and k: the longest input row is not that of the most rows
@pytest.mark.parametrize("sizes", [[(1, 24, 16384), (16, 40, 1024)], [(4, 8, 4096), (1, 9, 16000), (3, 17, 4)], [(2, 8, 8192), (1, 12, 400)]])
def test_forward_layers_of_few_rows_and_several_sizes(sizes):
    import torch
    from paper_2602_21597_amd import binding
    rng = np.random.default_rng(len(sizes))
    A, B = ([rng.standard_normal(s).astype(np.float32) for s in shapes] for shapes in ([(M, K) for M, N, K in sizes], [(N, K) for M, N, K in sizes]))
    f = lambda a: torch.from_numpy(a).cuda()
    for a, b, got in zip(A, B, binding.debug_gemm_group([f(a) for a in A], [f(b) for b in B])):
        want, scale = a.astype(np.float64) @ b.T.astype(np.float64), np.abs(a).astype(np.float64) @ np.abs(b.T)
        assert (np.abs(got.cpu().numpy() - want) / scale).max() < 0.1 * 2e-6 * max(1.0, np.sqrt(a.shape[1]) / 8)


# rows: none, one, below and above a block of 16, a block of every wavefront and one more, several rounds
@pytest.mark.parametrize("K", [0, 1, 15, 17, 64, 65, 127, 500])
@pytest.mark.parametrize("M,N", [(4, 4), (64, 60), (68, 132), (200, 64)])
def test_weight_gradients_by_rows(M, N, K):
    import torch
    from paper_2602_21597_amd import binding
    rng = np.random.default_rng(M * 1000 + K)
    A, B = (rng.standard_normal((K, n)).astype(np.float32) for n in (M, N))
    f = lambda a: torch.from_numpy(a if K else np.zeros((1, a.shape[1]), np.float32)).cuda()
    got = binding.debug_gemm(f(A), f(B), M, N, K, a_kcontig=False, b_kcontig=False).cpu().numpy()
    want = A.astype(np.float64).T @ B.astype(np.float64)
    scale = np.abs(A).astype(np.float64).T @ np.abs(B) + 1e-30
    assert (np.abs(got - want) / scale).max() < 0.1 * 2e-6 * max(1.0, np.sqrt(K) / 8)


# The kernel's products are sums of bf16 products: they may be no further from fp64 than those of the fp32 matrix
# instructions, which the yardstick (arith=1) is made of.  Hidden rows of one sign make partial sums large, and an accumulator's
# rounding counts as often as it is added to.  (5 %: the spread of the ratio over draws of 76 800 sums.  With both operands of
# one sign, which no gradient is over thousands of rows, the four partial sums here are 9 % worse than the yardstick's eight
# at 5000 rows.)
@pytest.mark.parametrize("K", [16, 64, 182, 300, 730, 1356, 5000])
@pytest.mark.parametrize("hidden", [False, True])
def test_weight_gradients_are_as_exact_as_fp32_products(K, hidden):
    import torch
    from paper_2602_21597_amd import binding
    M, N = 240, 320
    rng = np.random.default_rng(K)
    A, B = (rng.standard_normal((K, n)).astype(np.float32) for n in (M, N))
    if hidden:                                   # gradients of rows of different size, and hidden rows
        A, B = A * np.exp(rng.standard_normal((K, 1))).astype(np.float32), np.maximum(B, 0)
    want = A.astype(np.float64).T @ B.astype(np.float64)
    f = lambda a: torch.from_numpy(a).cuda()
    rms = [np.sqrt(np.mean((binding.debug_gemm(f(A), f(B), M, N, K, a_kcontig=False, b_kcontig=False, arith=arith).cpu().numpy() - want) ** 2))
           for arith in (0, 1)]
    assert rms[0] <= 1.05 * rms[1], rms


# (the last: a table beyond the caches)
@pytest.mark.parametrize("B,C,N", [(1, 1, 3000), (1, 15, 3000), (1, 17, 3000), (1, 1000, 3000), (3, 4097, 3000), (40, 33, 3000),
                                   (128, 1920, 3000), (128, 1919, 3000), (24, 50, 1200000)])
def test_candidate_lists_shared_by_workgroups(B, C, N):
    import torch
    case = par.Case(N, 10, 60, 40, B, 2, 8.0, seed=17, T=3 * N)
    cand = np.random.default_rng(C).integers(0, case.N, (B, C)).astype(np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    got = eng.score(plan, torch.from_numpy(cand).cuda()).cpu().numpy()
    par.assert_close(got, orank.score_candidates(case.qb, cand, om.Model(case.params, case.gamma)), "scores %d x %d" % (B, C))
    plan.free()


# long lists, on both sides of the lines from which on half as many workgroups share them (bytes of a row by kind, of the table,
# 1024 and more workgroups, queries): a pair's score does not depend on the list that it stands in
@pytest.mark.parametrize("kind,N,d,B,C", [("plain", 11000, 196, 130, 1900), ("plain", 11000, 200, 130, 1900), ("plain", 10000, 200, 130, 1900),
                                          ("plain", 11000, 200, 128, 1920), ("plain", 4100, 512, 1024, 240), ("plain", 5000, 516, 130, 1900),
                                          ("plain", 9000, 256, 1025, 240), ("box", 6000, 396, 130, 1900), ("box", 6000, 400, 130, 1900),
                                          ("box", 6000, 400, 128, 1920), ("bf16", 9000, 504, 130, 1900), ("bf16", 9000, 512, 130, 1900),
                                          ("bf16", 8000, 512, 130, 1900)])
def test_long_candidate_lists_by_workgroups(kind, N, d, B, C):
    import torch
    from paper_2602_21597_amd import Engine, binding
    box = kind == "box"
    qb = wl.make_batch(wl.make_kg(N, 5, 4 * N, 2.1, 3), B, {n: 1.0 for n in ("1p", "2i", "2u")}, 4)
    eng = Engine(N, 5, d, 40, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC, score_bf16=kind == "bf16")
    eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, 5, d, 40, 6))
    plan = eng.plan(qb)
    cand = torch.from_numpy(np.random.default_rng(C).integers(0, N, (B, C)).astype(np.int32)).cuda()
    got = eng.score(plan, cand).clone()
    step = 61
    for lo in range(0, C, step):
        assert torch.equal(eng.score(plan, cand[:, lo:lo + step].contiguous()), got[:, lo:lo + step]), lo
    plan.free()


# keys: one; 4096 and more (one workgroup / tiles); 80 000 and more (tiles of 2048 and 4096 keys, heads counted by every workgroup / from
# sums); 262 144 and more (tiles of 8192 keys); 524 288 and more (histogram scanned by every workgroup / once); a bound of one digit, of
# two and of three; a few keys all of the time
@pytest.mark.parametrize("N,B,n_keys", [(50, 1, 3), (200, 8, 4096), (200, 8, 4104), (200, 8, 16384), (70000, 8, 16392),
                                        (70000, 8, 32768), (3000, 8, 32776), (70000, 64, 4096), (70000, 64, 262144),
                                        (300, 64, 262208), (1000, 700, 300000), (70000, 64, 79936), (70000, 64, 80064), (5000, 64, 131136),
                                        (70000, 64, 524288), (70000, 64, 524352), (20, 64, 600000)])
def test_gradient_index_by_size(N, B, n_keys):
    import torch
    from paper_2602_21597_amd import Engine
    kg = wl.make_kg(N, 5, 4 * N, 2.1, 3)
    qb = wl.make_batch(kg, B, {"1p": 1.0}, 4)                # one anchor per query
    K = (n_keys - 2 * B) // B
    negs = wl.make_negatives(N, B, K, 5)
    eng = Engine(N, 5, 4, 4, 8.0)
    eng.bind_numpy(wl.make_params(N, 5, 4, 4, 6))
    plan = eng.plan(qb)
    eng.forward_backward(plan, torch.from_numpy(negs).cuda())
    g = eng.grads()
    assert g["e_src"].size == 2 * B + B * K
    u, off, src = oplan.entity_index(plan.export(), qb.pos, negs)
    for name, want in (("e_uniq", u), ("e_seg_off", off), ("e_src", src)):
        assert np.array_equal(g[name], want), name
    plan.free()


# table rows beside the backward pass, rows of anchors after it: every row an anchor's, nearly none, a pass kept to few
# wavefronts, one at full width over a table beyond the caches, text features, a bf16 copy of the table (hidden layers wide
# enough, and contributions many enough, that the second stream is used)
@pytest.mark.parametrize("N,d,B,K,d_sem,bf16", [(20, 32, 60, 80, 0, False), (9000, 64, 3, 1500, 0, False), (9000, 260, 40, 200, 0, False),
                                                (60000, 400, 60, 1000, 0, False), (3000, 40, 50, 90, 64, False),
                                                (60000, 520, 60, 1000, 64, False), (3000, 40, 50, 90, 0, True)])
def test_tables_beside_the_backward_pass(N, d, B, K, d_sem, bf16):
    import torch
    from paper_2602_21597_amd import Engine
    qb = wl.make_batch(wl.make_kg(N, 7, 5 * N, 2.1, 1), B, {n: 1.0 for n in wl.configs.ALL14}, 2)
    params = wl.make_params(N, 7, d, 520, 3, d_sem=d_sem)
    sem = wl.make_sem_features(N, d_sem, 4) if d_sem else None
    negs = torch.from_numpy(wl.make_negatives(N, B, K, 5)).cuda()
    out = []
    for streams in (1, 2):
        eng = Engine(N, 7, d, 520, 12.0, num_streams=streams, d_sem=d_sem, score_bf16=bf16)
        eng.bind_numpy(params, sem_bits=sem)
        plan = eng.plan(qb)
        eng.forward_backward(plan, negs)
        grads = {k: np.copy(v) for k, v in eng.grads().items()}
        losses = [float(eng.train_step(plan, negs)) for _ in range(3)]
        out.append((grads, losses, [t for name in eng.tensor_names() for t in eng.tensors[name]]))
        plan.free()
    for name, want in out[0][0].items():
        assert np.array_equal(out[1][0][name], want), name
    assert out[0][1] == out[1][1]
    assert all(torch.equal(a, b) for a, b in zip(out[0][2], out[1][2]))


# tables beyond the caches, a wavefront a row (second stream) against the rows walked at the end of the step (one stream, up to
# 65 536 rows): rows that fill part of a 256 B piece, of one, two and four pieces; touched rows of less than a window of workgroups
# and of many; boxes; a bf16 copy, which is read and written with the rows; rows with no pair, with one and with hundreds (the workload's
# heavy-tailed positives)
@pytest.mark.parametrize("N,d,B,K,kind", [(200000, 120, 70, 700, "plain"), (65000, 384, 61, 1000, "plain"), (24000, 1024, 40, 1200, "plain"),
                                          (65000, 384, 61, 1000, "box"), (120000, 200, 65, 900, "box"), (65000, 384, 61, 1000, "bf16"),
                                          (120000, 200, 65, 900, "bf16")])
def test_tables_beyond_the_caches_a_wavefront_a_row(N, d, B, K, kind):
    import torch
    from paper_2602_21597_amd import Engine, binding
    box = kind == "box"
    names = wl.configs.EPFO9 if box else wl.configs.ALL14
    qb = wl.make_batch(wl.make_kg(N, 7, 5 * N, 2.1, 1), B, {n: 1.0 for n in names}, 2)
    negs = torch.from_numpy(wl.make_negatives(N, B, K, 5)).cuda()
    out = []
    for streams in (1, 2):
        eng = Engine(N, 7, d, 520, 12.0, num_streams=streams, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC, score_bf16=kind == "bf16")
        eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, 7, d, 520, 3))
        plan = eng.plan(qb)
        losses = [float(eng.train_step(plan, negs)) for _ in range(2)]
        out.append((losses, [t for name in eng.tensor_names() for t in eng.tensors[name]], []))
        if kind == "bf16":
            eng.forward_backward(plan, negs)
            out[-1][2].append(eng.grads()["e_shadow"])
            rounded = eng.tensors["E"][0].to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
            assert np.array_equal(out[-1][2][0], rounded)
        plan.free()
    assert out[0][0] == out[1][0]
    assert all(torch.equal(a, b) for a, b in zip(out[0][1], out[1][1]))
    assert all(np.array_equal(a, b) for a, b in zip(out[0][2], out[1][2]))


# a table of 280 MB, whose rows are scored by non-temporal loads, against its first rows as a table of their own: both families, both
# directions
@pytest.mark.parametrize("box", [False, True])
def test_rows_of_a_table_beyond_the_caches_are_scored_alike(box):
    import torch
    from paper_2602_21597_amd import Engine, binding
    few, N, d, B, K = 3000, 700000, 100, 40, 60
    qb = wl.make_batch(wl.make_kg(few, 7, 5 * few, 2.1, 1), B, {n: 1.0 for n in (wl.configs.EPFO9 if box else wl.configs.ALL14)}, 2)
    negs = torch.from_numpy(wl.make_negatives(few, B, K, 5)).cuda()
    params = (wl.make_box_params if box else wl.make_params)(few, 7, d, 520, 3)
    out = []
    for n in (few, N):
        eng = Engine(n, 7, d, 520, 12.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
        E = np.zeros((n, d), np.float32)
        E[:few] = params["E"]
        eng.bind_numpy(dict(params, E=E))
        plan = eng.plan(qb)
        got = [eng.score(plan, negs)] + [eng.train_step(plan, negs).clone() for _ in range(2)]
        out.append(got + [t[:few] if name == "E" else t for name in eng.tensor_names() for t in eng.tensors[name]])
        plan.free()
    assert all(torch.equal(a, b) for a, b in zip(*out))


# operators of a depth in one launch: widths that fill no tile, the widest hidden layer, the limit of weights a layer (for any
# depth, for depths of few row blocks) and beyond it; one query, row blocks that are nearly empty, intersections of two to eight inputs
@pytest.mark.parametrize("d,h,B", [(4, 4, 5), (20, 36, 1), (36, 100, 30), (64, 512, 40), (128, 256, 90), (132, 256, 40), (256, 128, 17),
                                   (40, 512, 60), (128, 160, 40), (128, 164, 3), (128, 164, 14), (128, 256, 4)])
def test_operators_of_a_depth_in_one_launch(d, h, B):
    rng = np.random.default_rng(d)
    N, R = 300, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    trees = []
    for i in range(2 * B):
        k = 2 + i % 7
        trees.append([proj(), proj(proj()), proj(("i",) + tuple(proj() for _ in range(k))),
                      ("i", proj(), ("n", proj(proj()))), ("u", proj(), proj())][(i // 2) % 5])
    case = par.Case(N, R, d, h, B, 7, 6.0, seed=d + h, trees=trees, pos=[int(x) for x in rng.integers(0, N, len(trees))])
    par.check_forward_backward(case)
    import torch
    cand = rng.integers(0, N, (case.B, 9)).astype(np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    par.assert_close(eng.score(plan, torch.from_numpy(cand).cuda()).cpu().numpy(),
                     orank.score_candidates(case.qb, cand, om.Model(case.params, case.gamma)), "scores d=%d h=%d" % (d, h))
    plan.free()


# all depths of a pass in one launch against a launch each (the entry point without allocations): nearly empty tiles, up to 256
# workgroups and beyond, calls in a row; and with the gradient index taken along, up to 4096 keys and beyond
@pytest.mark.parametrize("B,d,h", [(1, 36, 52), (64, 36, 52), (300, 128, 160), (1200, 36, 52), (1900, 36, 52)])
def test_depths_of_a_pass_in_one_launch(B, d, h):
    import torch
    case = par.Case(900, 9, d, h, B, 2, 6.0, seed=B)
    eng = case.engine()
    cand = torch.from_numpy(np.random.default_rng(B).integers(0, 900, (B, 5)).astype(np.int32)).cuda()
    for n in (B, max(1, B // 3), B):
        plan = eng.plan(case.qb.select(np.arange(n)))
        want = eng.score_noalloc(plan, cand[:n].contiguous(), torch.empty((n, 5), dtype=torch.float32, device="cuda")).clone()
        for _ in range(3):
            assert torch.equal(eng.score(plan, cand[:n].contiguous()), want)
        plan.free()


# A pass of a handful of queries, all layers in one launch against a launch each, bit for bit: one row and rows that fill no tile, widths
# that fill no chunk of a wavefront up to the widest, every cardinality it pools and one more, as many depths as it takes and one more, more
# words than its arguments hold; from a plan that it brings to the device itself, and for what reads that plan afterwards; on context after another
@pytest.mark.parametrize("d,h,B", [(400, 800, 1), (400, 800, 5), (132, 260, 3), (260, 1024, 7), (1024, 36, 4), (516, 132, 16), (400, 800, 40)])
def test_layers_of_a_few_rows_in_one_launch(d, h, B):
    import torch
    from paper_2602_21597_amd import Engine, binding
    rng = np.random.default_rng(d + B)
    N, R = 900, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    inter = lambda k: ("i",) + tuple(proj() for _ in range(k))
    kinds = [lambda: proj(), lambda: inter(2), lambda: proj(inter(3)), lambda: ("i", proj(), ("n", proj(proj()))), lambda: ("u", proj(), proj(proj())),
             lambda: proj(("i", proj(), ("n", proj()))), lambda: inter(4), lambda: inter(5), lambda: proj(proj(proj(proj(proj()))))]
    batches = [[kinds[(first + i) % len(kinds)]() for i in range(B)] for first in range(len(kinds))]
    eng = Engine(N, R, d, h, 8.0)
    eng.bind_numpy(wl.make_params(N, R, d, h, 6))
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    ans = cand[:, :2].contiguous().view(-1)
    off = torch.arange(0, 2 * B + 1, 2, dtype=torch.int32, device="cuda")
    taken = {}
    for trees in batches:
        qb = wl.batch_from_trees(trees, [0] * B)
        out = []
        for polls in (-1, 1 << 22):
            before = chain_launches(eng)
            assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
            got = []
            for call in (lambda p: [eng.score(p, cand)], lambda p: list(eng.rank_all(p, 3)), lambda p: list(eng.rank_answers(p, off, ans))):
                plan = eng.plan(qb)
                got += [t.clone() for _ in range(2) for t in call(plan)]
                plan.free()
            plan = eng.plan(qb)
            got.append(eng.score(plan, cand).clone())
            got.append(eng.score_noalloc(plan, cand, torch.empty_like(got[0])).clone())
            got.append(eng.forward_backward(plan, cand).clone())
            plan.free()
            out.append(got)
            taken[polls] = taken.get(polls, 0) + (chain_launches(eng) - before)[0]
        assert all(torch.equal(a, b) for a, b in zip(*out)), trees
    # (seven calls without allocations or gradients, for the batches of which no query is of the last two kinds)
    assert taken == {-1: 0, 1 << 22: 7 * max(0, 8 - B)}


# ... one that gives up waiting (here at once): nobody can take what it leaves for results, the next call is refused, and what is computed
# after that is as if nothing had been
def test_layers_of_a_few_rows_that_give_up_waiting():
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R, B = 900, 9, 3
    eng = Engine(N, R, 400, 800, 8.0)
    eng.bind_numpy(wl.make_params(N, R, 400, 800, 6))
    qb = wl.batch_from_trees([("p", 1, ("e", 5)), ("i", ("p", 2, ("e", 7)), ("p", 3, ("e", 9))), ("p", 4, ("p", 5, ("e", 6)))], [0] * B)
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9)
    off = torch.arange(0, 2 * B + 1, 2, dtype=torch.int32, device="cuda")
    calls = [lambda p: [eng.score(p, cand)], lambda p: list(eng.rank_all(p, 3)), lambda p: list(eng.rank_answers(p, off, cand[:, :2].contiguous().view(-1)))]
    invalid = [lambda out: bool((out[0] == -np.inf).all()), lambda out: bool((out[0] == -1).all()), lambda out: bool((out[0] == 0).all())]
    polls = lambda n: binding.lib().ngdb_debug_chain_polls(eng.ctx, n)
    plan = eng.plan(qb)
    want = [[t.clone() for t in call(plan)] for call in calls]
    for call, ok in zip(calls, invalid):
        assert polls(0) == 0
        assert ok(call(plan))
        torch.cuda.synchronize()
        with pytest.raises(binding.NgdbError) as e:
            eng.score(plan, cand)
        assert e.value.code == binding.ERR_HIP, str(e.value)
    assert polls(1 << 22) == 0
    for call, ok in zip(calls, want):
        assert all(torch.equal(a, b) for a, b in zip(call(plan), ok))
    plan.free()


# Passes of more rows, the layers of their depths in one launch of tiles a direction against a launch each, bit for bit: rows that fill no tile, widths that
# fill no block of k and no column tile, one chunk of k and two, the widest and one more, classes of two to four inputs and one more, as many
# depths as it takes and one more, depths of too many rows before those it takes and of too few behind them
@pytest.mark.parametrize("d,h,B", [(400, 800, 40), (132, 260, 33), (512, 1024, 50), (128, 1024, 70), (404, 132, 90), (400, 800, 300), (208, 416, 900), (400, 800, 140),
                                   (256, 512, 170), (516, 132, 60)])
def test_layers_of_some_rows_in_one_launch(d, h, B):
    import torch
    from paper_2602_21597_amd import Engine, binding
    rng = np.random.default_rng(d + B)
    N, R = 900, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    inter = lambda k: ("i",) + tuple(proj() for _ in range(k))
    kinds = [lambda: proj(), lambda: inter(2), lambda: proj(inter(3)), lambda: ("i", proj(), ("n", proj(proj()))), lambda: ("u", proj(), proj(proj())),
             lambda: proj(("i", proj(), ("n", proj()))), lambda: inter(4)]
    batches = [kinds[:6], kinds, kinds + [lambda: inter(5)], kinds[:2] + [lambda: proj(proj(proj(proj(proj()))))], kinds[2:4], [lambda: proj(proj())]]
    eng = Engine(N, R, d, h, 8.0)
    params = wl.make_params(N, R, d, h, 6)
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    count = np.zeros(4, int)
    for some in batches:
        qb = wl.batch_from_trees([some[i % len(some)]() for i in range(B)], [int(x) for x in rng.integers(0, N, B)])
        out = []
        for polls in (-1, 1 << 22):
            assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
            eng.bind_numpy(params)
            plan = eng.plan(qb)
            got = [eng.score(plan, cand).clone() for _ in range(3)]
            assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
            got += [eng.forward_backward(plan, cand).clone()] + [eng.train_step(plan, cand).clone() for _ in range(2)]
            got += [t[0].clone() for t in eng.tensors.values()] + [t[2].clone() for t in eng.tensors.values()]
            plan.free()
            out.append(got[2:])
            if polls < 0:
                assert (chain_launches(eng) == count).all()
        assert all(torch.equal(a, b) for a, b in zip(*out)), [i for i, (a, b) in enumerate(zip(*out)) if not torch.equal(a, b)]
        count = chain_launches(eng)
    # (forward and backward passes of most batches, where the widths are taken)
    assert (count[0], count[1] >= 12, count[2] >= 12) == (0, d <= 512, d <= 512), count


# ... of boxes: projections and both sides of intersections, classes of two to four inputs and one more, depths without intersections, of too few
# rows and of too many
@pytest.mark.parametrize("d,h,B", [(300, 500, 40), (400, 800, 130), (132, 260, 33), (512, 1024, 50), (160, 320, 700), (404, 132, 90)])
def test_layers_of_some_boxes_in_one_launch(d, h, B):
    import torch
    from paper_2602_21597_amd import Engine, binding
    rng = np.random.default_rng(d + B)
    N, R = 900, 9
    params = wl.make_box_params(N, R, d, h, 5)
    eng = Engine(N, R, d, h, 8.0, family=binding.FAMILY_BOX)
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    inter = lambda k: ("i",) + tuple(proj() for _ in range(k))
    kinds = [lambda: proj(), lambda: inter(2), lambda: proj(inter(3)), lambda: ("i", proj(), proj(proj())), lambda: ("u", proj(), proj(proj())), lambda: inter(4)]
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    count = np.zeros(4, int)
    for some in (kinds, kinds[:4], kinds + [lambda: inter(5)], kinds[:2] + [lambda: proj(proj(proj(proj(proj()))))], kinds[:1] + kinds[4:5], kinds[2:4]):
        qb = wl.batch_from_trees([some[i % len(some)]() for i in range(B)], [int(x) for x in rng.integers(0, N, B)])
        out = []
        for polls in (-1, 1 << 22):
            assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
            eng.bind_numpy(params)
            plan = eng.plan(qb)
            got = [eng.score(plan, cand).clone() for _ in range(3)]
            assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
            got += [eng.forward_backward(plan, cand).clone()] + [eng.train_step(plan, cand).clone() for _ in range(2)]
            got += [t[0].clone() for t in eng.tensors.values()] + [t[2].clone() for t in eng.tensors.values()]
            plan.free()
            out.append(got[2:])
            if polls < 0:
                assert (chain_launches(eng) == count).all()
        assert all(torch.equal(a, b) for a, b in zip(*out)), [i for i, (a, b) in enumerate(zip(*out)) if not torch.equal(a, b)]
        count = chain_launches(eng)
    # (forward and backward passes of most batches, where the widths are taken)
    assert (count[0], count[1] >= 12, count[2] >= 12) == (0, d <= 512, d <= 512), count


# Memory of contexts of few boxes: room for split weights where a launch of several layers may read them (both widths from 128 on), and for nothing else of that kind
def test_few_boxes_hold_what_their_passes_read():
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R, B, h = 200, 5, 40, 600
    qb = wl.batch_from_trees([("p", 1, ("i", ("p", 2, ("e", i)), ("p", 3, ("e", i + 1)))) for i in range(B)], [0] * B)
    cand = torch.arange(B * 3, dtype=torch.int32, device="cuda").view(B, 3)
    held = {}
    for d in (124, 128):
        eng = Engine(N, R, d, h, 8.0, family=binding.FAMILY_BOX)
        eng.bind_numpy(wl.make_box_params(N, R, d, h, 5))
        plan = eng.plan(qb)
        eng.train_step(plan, cand)
        torch.cuda.synchronize()
        held[d] = binding.lib().ngdb_debug_device_bytes(eng.ctx)
        plan.free()
    tiles = lambda n, k: -(-n // 32) * -(-k // 16) * 1536
    pieces = 2 * 2 * 2 * (tiles(h, 128) + tiles(128, h))        # two MLPs, both orientations of both layers, two bytes a value
    without = held[124] * 128 / 124                              # (buffers have a quarter more than is needed)
    assert without + pieces < held[128] < without + 1.25 * pieces + (1 << 18), (held, pieces)


# ... with text features, whose anchors' rows are fused by the pass itself; and beside many rows that are fused on the library's stream, where forward passes keep their launches
@pytest.mark.parametrize("K,beside", [(9, False), (400, True)])
def test_layers_of_some_rows_with_text_features(K, beside):
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R, d, h, ds, B = 30000, 9, 128, 256, 64, 60
    rng = np.random.default_rng(8)
    e = lambda: ("e", int(rng.integers(N)))
    qb = wl.batch_from_trees([("p", 1, ("i", ("p", 2, e()), ("p", 3, e()))) for _ in range(B)], [int(x) for x in rng.integers(0, N, B)])
    cand = torch.from_numpy(rng.integers(0, N, (B, K)).astype(np.int32)).cuda()
    params = wl.make_params(N, R, d, h, 6, ds)
    eng = Engine(N, R, d, h, 8.0, d_sem=ds, num_streams=2)
    out = []
    for polls in (-1, 1 << 22):
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
        eng.bind_numpy(params, sem_bits=wl.make_sem_features(N, ds, 7))
        before = chain_launches(eng)
        plan = eng.plan(qb)
        got = [eng.score(plan, cand).clone()] + [eng.train_step(plan, cand).clone() for _ in range(2)] + [t[0].clone() for t in eng.tensors.values()]
        plan.free()
        out.append(got)
        assert list((chain_launches(eng) - before)[:3]) == ([0, 0, 0] if polls < 0 else [0, 1 if beside else 3, 2])
    assert all(torch.equal(a, b) for a, b in zip(*out))


# ... one that gives up waiting (here at once): the rows of its depths are nobody's results, parameters stay as they were, and the next call is refused
def test_layers_of_some_rows_that_give_up_waiting():
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R, B = 900, 9, 60
    rng = np.random.default_rng(3)
    eng = Engine(N, R, 400, 800, 8.0)
    eng.bind_numpy(wl.make_params(N, R, 400, 800, 6))
    qb = wl.batch_from_trees([("p", int(rng.integers(R)), ("p", 1, ("e", int(rng.integers(N))))) for _ in range(B)], [0] * B)
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
    polls = lambda n: binding.lib().ngdb_debug_chain_polls(eng.ctx, n)
    plan = eng.plan(qb)
    want = eng.score(plan, cand).clone()
    before = {k: t[0].clone() for k, t in eng.tensors.items()}
    for call in (lambda: eng.score(plan, cand), lambda: eng.train_step(plan, cand)):
        assert polls(0) == 0
        got = call()
        torch.cuda.synchronize()
        assert got.numel() == 1 or bool((got == -np.inf).all())
        with pytest.raises(binding.NgdbError) as e:
            eng.score(plan, cand)
        assert e.value.code == binding.ERR_HIP, str(e.value)
        assert all(torch.equal(before[k], eng.tensors[k][0]) for k in before)
    assert polls(1 << 22) == 0
    assert torch.equal(eng.score(plan, cand), want)
    plan.free()


# ... nothing of such a pass can be taken for a result, whatever follows it: deeper depths of few rows in launches of their own, whose relu makes a number of what is none, unions
# one branch of which is valid, the filter of rankings, in chunks and as a whole; passes of a few rows, of more and of small models; both families
@pytest.mark.parametrize("box,d,h,B,N", [(False, 400, 800, 60, 900), (False, 400, 800, 60, 5000), (False, 400, 800, 60, 70000), (False, 400, 800, 4, 900), (False, 36, 52, 60, 900),
                                         (False, 36, 52, 60, 5000), (True, 300, 500, 60, 900), (True, 36, 52, 60, 900)])
def test_nothing_of_a_pass_that_gave_up_is_a_result(box, d, h, B, N):
    import torch
    from paper_2602_21597_amd import Engine, binding
    rng = np.random.default_rng(B)
    R = 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    trees = [(proj(), proj(proj()), ("i", proj(), proj(proj())), ("u", proj(), proj(proj())))[i % 4] for i in range(B - 2)] + [proj(proj(proj())), ("u", proj(), proj(proj(proj())))]
    eng = Engine(N, R, d, h, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
    eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, R, d, h, 6))
    if N > 900:
        assert binding.lib().ngdb_debug_rank_filter_from(eng.ctx, 0) == 0
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    off = torch.arange(0, 2 * B + 1, 2, dtype=torch.int32, device="cuda")
    ans = cand[:, :2].contiguous().view(-1)
    polls = lambda n: binding.lib().ngdb_debug_chain_polls(eng.ctx, n)
    chunks = lambda on: binding.lib().ngdb_debug_rank_by_chunks(eng.ctx, on)
    plan = eng.plan(wl.batch_from_trees(trees, [0] * B))

    def ranked(on):
        assert chunks(on) == 0
        return eng.rank_all(plan, 3)

    calls = [(lambda: eng.score(plan, cand), lambda s: bool((s == -np.inf).all())),
             (lambda: ranked(0), lambda r: bool((r[0] == -1).all()) and bool((r[1] == np.inf).all())),
             (lambda: ranked(1), lambda r: bool((r[0] == -1).all()) and bool((r[1] == np.inf).all())),
             (lambda: eng.rank_answers(plan, off, ans), lambda r: bool((r[0] == 0).all()) and bool((r[1] == np.inf).all()))]
    if B > 16 or box or d < 128:
        calls.append((lambda: eng.train_step(plan, cand), lambda loss: float(loss) == np.inf))
    before = {k: t[0].clone() for k, t in eng.tensors.items()}
    want = eng.score(plan, cand).clone()
    for call, nothing in calls:
        assert polls(0) == 0
        got = call()
        assert nothing(got), got
        torch.cuda.synchronize()
        with pytest.raises(binding.NgdbError) as e:
            eng.score(plan, cand)
        assert e.value.code == binding.ERR_HIP, str(e.value)
    assert all(torch.equal(before[k], eng.tensors[k][0]) for k in before)
    assert polls(1 << 22) == 0
    assert torch.equal(eng.score(plan, cand), want)
    plan.free()


# ... every eighth workgroup late (some milliseconds, or until its tile is taken): the others compute its tiles, each once, and the results are the same bits.  A
# handful of queries and more, both families and directions, launches of more workgroups than the card holds; and as it is by default, calls in a row
@pytest.mark.parametrize("box,d,h,B", [(False, 400, 800, 3), (False, 132, 260, 5), (False, 400, 800, 40), (False, 260, 516, 170), (False, 512, 1024, 50),
                                       (True, 300, 500, 40), (True, 160, 320, 130)])
def test_tiles_of_workgroups_that_start_late(box, d, h, B):
    import torch
    from paper_2602_21597_amd import Engine, binding
    rng = np.random.default_rng(d + B)
    N, R = 900, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    kinds = [lambda: proj(proj()), lambda: proj(("i", proj(), proj())), lambda: ("i", proj(), proj(proj()), proj()), lambda: ("u", proj(), proj(proj()))]
    qb = wl.batch_from_trees([kinds[i % 4]() for i in range(B)], [int(x) for x in rng.integers(0, N, B)])
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    params = (wl.make_box_params if box else wl.make_params)(N, R, d, h, 6)
    eng = Engine(N, R, d, h, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
    few = not box and B <= 16
    out, helped = [], []
    for polls, patience in ((-1, 1024), (1 << 22, -4096), (1 << 22, 0), (1 << 22, 1024)):
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
        assert binding.lib().ngdb_debug_chain_patience(eng.ctx, patience) == 0
        eng.bind_numpy(params)
        plan = eng.plan(qb)
        before = chain_launches(eng)
        got = [eng.score(plan, cand).clone() for _ in range(3)]
        if not few:
            got += [eng.train_step(plan, cand).clone() for _ in range(2)] + [t[0].clone() for t in eng.tensors.values()]
        torch.cuda.synchronize()
        plan.free()
        out.append(got)
        new = chain_launches(eng) - before
        assert list(new[:3]) == ([0, 0, 0] if polls < 0 else [3, 0, 0] if few else [0, 5, 2])
        helped.append(new[3])
    assert all(torch.equal(a, b) for got in out[1:] for a, b in zip(got, out[0]))
    assert helped[0] == 0 and helped[1] > 0


# ... passes that keep a launch a layer: more tiles than one launch takes, captures; nothing is counted that was not launched
@pytest.mark.parametrize("box,d,h,B,captured", [(False, 1024, 1024, 24, False), (False, 400, 800, 3, True), (True, 300, 500, 40, True)])
def test_passes_that_keep_a_launch_a_layer(box, d, h, B, captured):
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R = 200, 5
    eng = Engine(N, R, d, h, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
    eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, R, d, h, 5))
    p = lambda t: ("p", 1, t)
    e = lambda i: ("e", i % N)
    # (24: few rows a layer, but 2304 tiles in all)
    kinds = [lambda i: p(("i", p(e(i)), p(e(i + 1))))] if box or B < 16 else [lambda i: p(("n", ("i", e(i), e(i + 1)))), lambda i: p(("n", ("n", e(i)))), lambda i: p(p(e(i)))]
    plan = eng.plan(wl.batch_from_trees([kinds[i * len(kinds) // B](i) for i in range(B)], [0] * B))
    cand = torch.arange(B * 3, dtype=torch.int32, device="cuda").view(B, 3) % N
    counts, out = [], []
    for polls in (-1, 1 << 22):
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
        eng.score(plan, cand)
        before = chain_launches(eng)
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                got = eng.score(plan, cand)
            counts.append(None)
            graph.replay()
            torch.cuda.synchronize()
            out.append(got.clone())
        else:
            eng.set_timing(("gemm_fwd", "inter"))
            eng.get_timing(reset=True)
            out.append(eng.score(plan, cand).clone())
            counts.append({k: v[1] for k, v in eng.get_timing(reset=True).items()})
            eng.set_timing(())
        assert (chain_launches(eng) == before).all()
    assert counts[0] == counts[1] and torch.equal(out[0], out[1]), counts
    plan.free()


# ... the first ones of a context, whose memory an earlier context's launches have left their marks in
def test_first_layers_of_a_context():
    import torch
    from paper_2602_21597_amd import Engine
    N, R, d, h = 900, 9, 260, 516
    params = wl.make_params(N, R, d, h, 6)
    qb = wl.batch_from_trees([("p", 1, ("i", ("p", 2, ("e", i)), ("p", 3, ("e", i + 1)))) for i in range(60)], [0] * 60)
    cand = torch.arange(60 * 9, dtype=torch.int32, device="cuda").view(60, 9)
    got = []
    for first in (60, 2, 60, 2):
        eng = Engine(N, R, d, h, 8.0)
        eng.bind_numpy(params)
        for n in (first, 62 - first, 60, 2):
            plan = eng.plan(qb.select(np.arange(n)))
            got.append((n, eng.score(plan, cand[:n].contiguous()).clone()))
            plan.free()
        assert list(chain_launches(eng)[:2]) == [2, 2]
        del eng
    want = {n: s for n, s in got[:2]}
    assert all(torch.equal(s, want[n]) for n, s in got)


# ... two contexts on two streams, calls of both under way at a time: each as it is alone, in launches of several layers all the same
@pytest.mark.parametrize("patience", [1024, 0])
@pytest.mark.parametrize("B", [60, 2])
def test_layers_of_some_rows_on_two_streams(B, patience):
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R = 900, 9
    rng = np.random.default_rng(6)
    proj = lambda: ("p", int(rng.integers(R)), ("p", int(rng.integers(R)), ("e", int(rng.integers(N)))))
    cand = torch.from_numpy(rng.integers(0, N, (B, 9)).astype(np.int32)).cuda()
    sides = []
    for d, h in ((260, 516), (300, 400)):
        eng = Engine(N, R, d, h, 8.0)
        eng.bind_numpy(wl.make_params(N, R, d, h, 6))
        assert binding.lib().ngdb_debug_chain_patience(eng.ctx, patience) == 0
        plan = eng.plan(wl.batch_from_trees([("i", proj(), proj()) for _ in range(B)], [0] * B))
        sides.append((eng, plan, torch.cuda.Stream(), eng.score(plan, cand).clone()))
    torch.cuda.synchronize()
    before = [chain_launches(eng)[:2].sum() for eng, _, _, _ in sides]
    got = []
    for _ in range(20):
        for eng, plan, stream, want in sides:
            with torch.cuda.stream(stream):
                got.append((eng.score(plan, cand), want))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in got)
    assert [chain_launches(eng)[:2].sum() - n for (eng, _, _, _), n in zip(sides, before)] == [20, 20]
    for eng, plan, _, _ in sides:
        plan.free()


# ... two processes on the card, both with such launches: each as it is by launches of a layer
_PROCESS = """
import sys
import numpy as np, torch
import workloads as wl
from paper_2602_21597_amd import Engine, binding
B, N, R = int(sys.argv[1]), 900, 9
eng = Engine(N, R, 300, 400, 8.0)
eng.bind_numpy(wl.make_params(N, R, 300, 400, 6))
plan = eng.plan(wl.batch_from_trees([("p", 1, ("i", ("p", 2, ("e", i)), ("p", 3, ("e", i + 1)))) for i in range(B)], [0] * B))
cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
assert binding.lib().ngdb_debug_chain_polls(eng.ctx, -1) == 0
want = eng.score(plan, cand).clone()
assert binding.lib().ngdb_debug_chain_polls(eng.ctx, 1 << 22) == 0
for _ in range(150):
    got = [eng.score(plan, cand) for _ in range(20)]
    torch.cuda.synchronize()
    assert all(torch.equal(g, want) for g in got)
assert sum(binding.lib().ngdb_debug_chain_launches(eng.ctx, kind) for kind in (0, 1)) == 3000
"""


def test_layers_of_some_rows_in_two_processes():
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    children = [subprocess.Popen([sys.executable, "-c", _PROCESS, str(B)], cwd=root, stderr=subprocess.PIPE, text=True) for B in (160, 2)]
    ends = [child.communicate(timeout=100)[1][-2000:] for child in children]
    assert [child.returncode for child in children] == [0, 0], ends


# ... captured: every replay as the call, with other launches of the kind in between
def test_layers_of_some_rows_captured():
    import torch
    from paper_2602_21597_amd import Engine
    N, R, B = 900, 9, 60
    rng = np.random.default_rng(4)
    eng = Engine(N, R, 260, 516, 8.0)
    eng.bind_numpy(wl.make_params(N, R, 260, 516, 6))
    e = lambda: ("e", int(rng.integers(N)))
    qb = wl.batch_from_trees([("p", 3, ("i", ("p", 1, e()), ("p", 2, e()))) for _ in range(B)], [0] * B)
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
    plan, other = eng.plan(qb), eng.plan(qb.select(np.arange(25)))
    want = eng.score(plan, cand).clone()
    before = chain_launches(eng)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = eng.score(plan, cand)
    assert (chain_launches(eng) == before).all()           # (replays have no launch numbers of their own)
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        eng.score(other, cand[:25].contiguous())
    plan.free()
    other.free()


# ... a stream that has run such a launch is captured while another context has one on a stream of its own: neither notices the other
def test_layers_of_some_rows_beside_a_capture():
    import torch
    from paper_2602_21597_amd import Engine
    N, R, B = 900, 9, 60
    rng = np.random.default_rng(4)
    e = lambda: ("e", int(rng.integers(N)))
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
    sides = []
    for seed in (6, 7):
        eng, stream = Engine(N, R, 260, 516, 8.0), torch.cuda.Stream()
        eng.bind_numpy(wl.make_params(N, R, 260, 516, seed))
        plan = eng.plan(wl.batch_from_trees([("p", 3, ("i", ("p", 1, e()), ("p", 2, e()))) for _ in range(B)], [0] * B))
        with torch.cuda.stream(stream):
            sides.append((eng, plan, stream, eng.score(plan, cand).clone()))
    torch.cuda.synchronize()
    (a, plan_a, stream_a, want_a), (b, plan_b, stream_b, want_b) = sides
    with torch.cuda.stream(stream_a):
        a.score(plan_a, cand)
    before = chain_launches(b)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream_a, capture_error_mode="relaxed"):
        out = a.score(plan_a, cand)
        with torch.cuda.stream(stream_b):
            got = b.score(plan_b, cand)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want_a) and torch.equal(got, want_b)
    assert list((chain_launches(b) - before)[:3]) == [0, 1, 0]
    for _, plan, _, _ in sides:
        plan.free()


# ... a pass over some of its queries, or over a handful, makes no buffer grow that the graph uses
def test_fewer_queries_after_a_capture():
    import torch
    from paper_2602_21597_amd import Engine, binding
    N, R, B = 900, 9, 60
    rng = np.random.default_rng(4)
    eng = Engine(N, R, 260, 516, 8.0)
    eng.bind_numpy(wl.make_params(N, R, 260, 516, 6))
    qb = wl.batch_from_trees([("p", 3, ("p", 1, ("p", 2, ("e", int(rng.integers(N)))))) for _ in range(B)], [0] * B)
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
    plan = eng.plan(qb)
    want = eng.score(plan, cand).clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = eng.score(plan, cand)
    few = [(n, eng.plan(qb.select(np.arange(n)))) for n in (53, 16, 2)]
    allocs = binding.lib().ngdb_debug_alloc_count(eng.ctx)
    for n, some in few:
        got = eng.score(some, cand[:n].contiguous())
        assert binding.lib().ngdb_debug_alloc_count(eng.ctx) == allocs, n
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, -1) == 0
        assert torch.equal(got, eng.score(some, cand[:n].contiguous()))
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, 1 << 22) == 0
        some.free()
    plan.free()


# ... a call on the default stream, whose state cannot be asked for while a stream that waits for it is captured, and whose plan is on the device
def test_layers_of_some_rows_beside_a_capture_of_a_blocking_stream():
    import ctypes
    import torch
    from paper_2602_21597_amd import Engine
    N, R, B = 900, 9, 60
    rng = np.random.default_rng(4)
    e = lambda: ("e", int(rng.integers(N)))
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9) % N
    eng = Engine(N, R, 260, 516, 8.0)
    eng.bind_numpy(wl.make_params(N, R, 260, 516, 6))
    plan = eng.plan(wl.batch_from_trees([("p", 3, ("i", ("p", 1, e()), ("p", 2, e()))) for _ in range(B)], [0] * B))
    want = eng.score(plan, cand).clone()
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    assert hip.hipStreamBeginCapture(stream, 2) == 0               # (2: relaxed)
    try:
        got = eng.score(plan, cand)
    finally:
        ended = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
    torch.cuda.synchronize()
    assert ended == 0 and torch.equal(got, want)
    assert torch.equal(eng.score(plan, cand), want)
    if graph.value:
        assert hip.hipGraphDestroy(graph) == 0
    assert hip.hipStreamDestroy(stream) == 0
    plan.free()


# ... captured, and so the launch of all depths of a small model, which copies the plan too: every replay as the call
@pytest.mark.parametrize("d,h", [(400, 800), (36, 52)])
def test_layers_of_a_few_rows_captured(d, h):
    import torch
    from paper_2602_21597_amd import Engine
    N, R, B = 900, 9, 3
    eng = Engine(N, R, d, h, 8.0)
    eng.bind_numpy(wl.make_params(N, R, d, h, 6))
    qb = wl.batch_from_trees([("p", 1, ("e", 5)), ("i", ("p", 2, ("e", 7)), ("p", 3, ("e", 9))), ("p", 4, ("p", 5, ("e", 6)))], [0] * B)
    cand = torch.arange(B * 9, dtype=torch.int32, device="cuda").view(B, 9)
    plan, other = eng.plan(qb), eng.plan(qb.select(np.arange(2)))
    want = eng.score(plan, cand).clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = eng.score(plan, cand)
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        eng.score(other, cand[:2].contiguous())
    plan.free()
    other.free()


# both directions of both families, all depths in one launch against a launch each
@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("B,d,h", [(1, 36, 52), (64, 32, 64), (300, 128, 160), (700, 64, 128), (1900, 36, 52)])
def test_depths_of_a_step_in_one_launch(B, d, h, box):
    import torch
    from paper_2602_21597_amd import Engine, binding
    N = 900
    qb = wl.make_batch(wl.make_kg(N, 5, 4 * N, 2.1, 3), B, {n: 1.0 for n in (wl.configs.EPFO9 if box else wl.configs.ALL14)}, 4)
    negs = torch.from_numpy(wl.make_negatives(N, B, 6, 5)).cuda()
    out = []
    for polls in (-1, 1 << 22):
        eng = Engine(N, 5, d, h, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
        eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, 5, d, h, 6))
        assert binding.lib().ngdb_debug_chain_polls(eng.ctx, polls) == 0
        plan = eng.plan(qb)
        got = [eng.score(plan, negs)] + [eng.train_step(plan, negs).clone() for _ in range(3)]
        out.append(got + [t for name in eng.tensor_names() for t in eng.tensors[name]])
        plan.free()
    assert all(torch.equal(a, b) for a, b in zip(*out))


# such launches of two contexts beside one another on two streams, up to all workgroups that one may have: each as if alone
@pytest.mark.parametrize("B,d,h", [(64, 32, 64), (300, 128, 160)])
def test_depths_of_two_contexts_at_once(B, d, h):
    import torch
    from paper_2602_21597_amd import Engine
    N, steps = 900, 20
    qb = wl.make_batch(wl.make_kg(N, 5, 4 * N, 2.1, 3), B, {n: 1.0 for n in wl.configs.ALL14}, 4)
    negs = torch.from_numpy(wl.make_negatives(N, B, 6, 5)).cuda()
    out = []
    for together in (False, True):
        engs, plans, losses = [], [], [[], []]
        for seed in (6, 7):
            engs.append(Engine(N, 5, d, h, 8.0))
            engs[-1].bind_numpy(wl.make_params(N, 5, d, h, seed))
            plans.append(engs[-1].plan(qb))
        streams = [torch.cuda.Stream() for _ in engs] if together else [torch.cuda.current_stream()] * 2
        torch.cuda.synchronize()
        for _ in range(steps):
            for eng, plan, stream, loss in zip(engs, plans, streams, losses):
                at = torch.empty(1, dtype=torch.float32, device="cuda")
                at.record_stream(stream)
                loss.append(eng.train_step(plan, negs, stream=stream, loss_out=at))
                if not together:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        out.append([l for ls in losses for l in ls] + [t for eng in engs for name in eng.tensor_names() for t in eng.tensors[name]])
        for plan in plans:
            plan.free()
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("B,n_keys", [(2, 40), (30, 4096), (30, 4126)])
def test_index_taken_along_by_a_forward_pass(B, n_keys, box):
    import torch
    from paper_2602_21597_amd import Engine, binding
    N = 700
    qb = wl.make_batch(wl.make_kg(N, 5, 4 * N, 2.1, 3), B, {"2i": 1.0}, 4)                  # two anchors a query, two depths
    K = (n_keys - 3 * B) // B
    negs = wl.make_negatives(N, B, K, 5)
    eng = Engine(N, 5, 20, 36, 8.0, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
    eng.bind_numpy((wl.make_box_params if box else wl.make_params)(N, 5, 20, 36, 6))
    plan = eng.plan(qb)
    u, off, src = oplan.entity_index(plan.export(), qb.pos, negs)
    for _ in range(2):
        eng.forward_backward(plan, torch.from_numpy(negs).cuda())
        g = eng.grads()
        for name, want in (("e_uniq", u), ("e_seg_off", off), ("e_src", src)):
            assert np.array_equal(g[name], want), name
    plan.free()


# A launch of several depths that gives up waiting (here at once): nobody can take what it leaves for results, parameters and moments stay as
# they were, the next call is refused, and what is computed after that is as if nothing had been.  Both families; rankings by the
# fp32 pass and by the filter; the entity table updated with the end of the step and beside the backward pass
@pytest.mark.parametrize("box,N,B,streams", [(False, 700, 20, 1), (True, 700, 20, 1), (False, 5000, 200, 1), (False, 80000, 300, 2)])
def test_depths_that_give_up_waiting(box, N, B, streams):
    import torch
    from paper_2602_21597_amd import Engine, binding
    names = ["2p", "2i", "2u", "pi"] if box else ["2p", "2i", "2in", "pi", "2u", "inp"]
    qb = wl.make_batch(wl.make_kg(N, 5, 4 * N, 2.1, 3), B, {n: 1.0 for n in names}, 4)
    d, h, K = 36, 52, 500 if streams > 1 else 7
    negs = torch.from_numpy(wl.make_negatives(N, B, K, 5)).cuda()
    cand = negs[:, :5].contiguous()
    off = torch.arange(0, 2 * B + 1, 2, dtype=torch.int32, device="cuda")
    ans = negs[:, :2].contiguous().view(-1)
    eng = Engine(N, 5, d, h, 8.0, num_streams=streams, family=binding.FAMILY_BOX if box else binding.FAMILY_VEC)
    if N == 5000:
        assert binding.lib().ngdb_debug_rank_filter_from(eng.ctx, 0) == 0
    params = (wl.make_box_params if box else wl.make_params)(N, 5, d, h, 6)
    polls = lambda n: binding.lib().ngdb_debug_chain_polls(eng.ctx, n)
    state = lambda: [t.clone() for name in eng.tensor_names() for t in eng.tensors[name]]
    same = lambda a, b: all(torch.equal(x, y) for x, y in zip(a, b))

    def calls(plan):
        out = [eng.score(plan, cand)] + list(eng.rank_all(plan, 3)) + list(eng.rank_answers(plan, off, ans))
        return [t.clone() for t in out + [eng.train_step(plan, negs), eng.train_step(plan, negs)] + state()]

    def fresh():
        eng.bind_numpy(params)
        return eng.plan(qb)

    assert polls(-1) == 0                              # a launch per depth
    want = calls(fresh())
    plan = fresh()
    before = state()

    def gives_up(call, *results):
        assert polls(0) == 0
        out = call()
        for got, ok in zip(out if isinstance(out, tuple) else (out,), results):
            assert ok(got), got
        torch.cuda.synchronize()
        for again in (lambda: eng.train_step(plan, negs), lambda: eng.score(plan, cand)):
            with pytest.raises(binding.NgdbError) as e:
                again()
            assert e.value.code == binding.ERR_HIP, str(e.value)
        torch.cuda.synchronize()
        assert same(state(), before)

    nowhere = lambda t: bool((t == -np.inf).all())
    gives_up(lambda: eng.score(plan, cand), nowhere)
    gives_up(lambda: eng.rank_all(plan, 3), lambda t: bool((t == -1).all()))
    gives_up(lambda: eng.rank_answers(plan, off, ans), lambda t: bool((t == 0).all()))
    gives_up(lambda: eng.train_step(plan, negs), lambda t: not bool(torch.isfinite(t)))
    assert polls(0) == 0
    eng.forward_backward(plan, negs)
    with pytest.raises(binding.NgdbError) as e:
        eng.grad_view()
    assert e.value.code == binding.ERR_HIP
    plan.free()
    for n in (1 << 22, -1):
        assert polls(n) == 0
        plan = fresh()
        assert same(calls(plan), want)
        plan.free()


# Rounding errors of a layer over k: chains of 16 products, four of them as a tree, these sums one after the other.  In units of
# the variance of one relative rounding (at most 2^-48 / 3), for products of random sign: 8.5 + 2 + (k / 64 + 1) / 2.  (Two
# chains over all of k have k / 4.)  The errors of both layers add up in quadrature.
@pytest.mark.parametrize("d,h", [(40, 512), (128, 160), (256, 80)])
def test_rounding_of_operators_of_a_depth_in_one_launch(d, h):
    def live(P):                     # rows keep their size through a layer
        for a, b in (("W1", "W2"), ("V1", "V2"), ("U1", "U2")):
            P[a] *= np.float32(np.sqrt(6.0 / d) / 0.1)
            P[b] *= np.float32(np.sqrt(3.0 / h) / 0.1)
    case = par.Case(2000, 20, d, h, 100, 4, 12.0, mix={"1p": 1.0}, seed=d + h, params_edit=live)
    eng = case.engine()
    plan = eng.plan(case.qb)
    eng.forward_backward(plan, case.neg_dev())
    slots, act, M = plan.export()["root_slot"], eng.grads()["act"], case.model()
    want = np.stack([orank.query_embeddings(case.qb, q, M)[0] for q in range(case.B)])
    err = np.linalg.norm(act[slots] - want) / np.linalg.norm(want)
    assert err <= np.sqrt(sum(10.5 + (k / 64 + 1) / 2 for k in (d, h)) / 3) * 2.0 ** -24, err
    plan.free()


# the pooling in the second layer's launch: widths that fill no tile, one member a tile and sixteen, rows of both layers
# few and many, more classes than a launch takes
@pytest.mark.parametrize("d,h,B,cards", [(132, 256, 40, (2, 3, 5, 8)), (400, 100, 150, (2, 3)), (200, 200, 12, (8,)), (260, 132, 90, (2, 3, 4, 5, 6, 7, 8)),
                                         (256, 800, 400, (3,))])
def test_pooling_in_the_second_layer(d, h, B, cards):
    import torch
    rng = np.random.default_rng(d + B)
    N, R = 300, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    trees = []
    for i in range(2 * B):
        both = ("i",) + tuple(proj() for _ in range(cards[i % len(cards)]))
        trees.append([both, proj(both), ("i", proj(), ("n", proj(proj())))][(i // len(cards)) % 3 if 2 in cards else (i // len(cards)) % 2])
    case = par.Case(N, R, d, h, B, 5, 6.0, seed=d + h, trees=trees, pos=[int(x) for x in rng.integers(0, N, len(trees))])
    par.check_forward_backward(case)
    cand = rng.integers(0, N, (case.B, 9)).astype(np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    par.assert_close(eng.score(plan, torch.from_numpy(cand).cuda()).cpu().numpy(),
                     orank.score_candidates(case.qb, cand, om.Model(case.params, case.gamma)), "scores d=%d h=%d" % (d, h))
    plan.free()


@pytest.mark.parametrize("d,h,B", [(8, 12, 20), (36, 100, 40), (64, 512, 40), (128, 256, 60), (132, 256, 30)])
def test_box_operators_of_a_depth_in_one_launch(d, h, B):
    from . import parity_box as pb
    pb.check_forward_backward(pb.BoxCase(500, 9, d, h, B, 6, 4.0, alpha=0.2, seed=d + h))


# both layers over many rows; the kernel of each (0: few tiles, 1: many rows, k split over eight wavefronts, 2: pairs of them).  Tiles of 32 x 64
# on both sides of the lines, 140 and 256 (k from 256 on) and 256 (shorter k); widths that fill no tile and k that fills no block, fewer
# blocks of k than groups of wavefronts
@pytest.mark.parametrize("M,d,h,kernels", [(4480, 260, 36, (0, 2)), (4481, 260, 36, (1, 2)), (8192, 260, 36, (1, 2)), (8193, 260, 36, (2, 2)), (8192, 132, 36, (0, 2)),
                                           (8193, 132, 36, (2, 2)), (1633, 132, 260, (2, 1)), (4100, 148, 68, (2, 2)), (4513, 36, 68, (2, 0))])
def test_layers_of_many_rows(M, d, h, kernels):
    import torch
    from paper_2602_21597_amd import binding
    rng = np.random.default_rng(M)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    X, W1, W2, b1, b2, mask = f(M, d), f(h, d), f(d, h), f(h), f(d), f(M, h)
    dev = [torch.from_numpy(a).cuda() for a in (X, W1, b1, W2, b2)]
    bar = lambda k: 0.1 * 2e-6 * max(1.0, np.sqrt(k) / 8)
    for backward in (False, True):
        H, Y, used = binding.debug_mlp(*dev, mask=torch.from_numpy(mask).cuda(), backward=backward)
        assert (used >> 2 & 3, used >> 4 & 3) == kernels
        H, Y = (t.cpu().numpy().astype(np.float64) for t in (H, Y))
        A, B = (W2, W1) if backward else (W1.T, W2.T)
        pre = X.astype(np.float64) @ A + (0 if backward else b1)
        scale = np.abs(X).astype(np.float64) @ np.abs(A) + (0 if backward else np.abs(b1))
        want = np.where(mask > 0, pre, 0) if backward else np.maximum(pre, 0)
        assert (np.abs(H - want) / scale).max() < bar(d)
        add = 0 if backward else b2
        assert (np.abs(Y - (H @ B + add)) / (np.abs(H) @ np.abs(B) + np.abs(add) + 1e-30)).max() < bar(h)


# gathered rows with and without relations, rows kept, pooling and scattered gradients in launches of many rows
@pytest.mark.parametrize("d,h,B", [(132, 260, 300), (260, 516, 400)])
def test_operators_over_many_rows(d, h, B):
    import torch
    rng = np.random.default_rng(d + B)
    N, R = 300, 9
    proj = lambda t=None: ("p", int(rng.integers(R)), t or ("e", int(rng.integers(N))))
    trees = []
    for i in range(2 * B):
        both = ("i",) + tuple(proj() for _ in range(2 + i % 2))
        trees.append([both, proj(both), ("i", proj(), ("n", proj(proj())))][i % 3])
    case = par.Case(N, R, d, h, B, 5, 6.0, seed=d + h, trees=trees, pos=[int(x) for x in rng.integers(0, N, len(trees))])
    par.check_forward_backward(case)
    cand = rng.integers(0, N, (case.B, 9)).astype(np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    par.assert_close(eng.score(plan, torch.from_numpy(cand).cuda()).cpu().numpy(),
                     orank.score_candidates(case.qb, cand, om.Model(case.params, case.gamma)), "scores d=%d h=%d" % (d, h))
    plan.free()


# rows of text features by list, several tiles a workgroup: a column tile, two of which one holds 8 columns, three; feature stages that
# leave the ring of stages at another place after every tile; a second launch of fewer rows
@pytest.mark.parametrize("d,d_sem", [(24, 1024), (216, 256), (432, 320)])
def test_fused_rows_of_many_tiles(d, d_sem):
    import torch
    N, B, A = 3001, 60, 1201
    par.say("fused rows: d=%d d_sem=%d, %d rows" % (d, d_sem, B * A))
    case = par.Case(N, 12, d, 32, B, 2, 8.0, seed=5 + d, T=2 * N, d_sem=d_sem)
    M = case.model()
    rng = np.random.default_rng(d)
    answers = np.stack([rng.choice(N, A, replace=False) for _ in range(B)])
    off = np.arange(0, B * A + 1, A).astype(np.int32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda()
    eng = case.engine()
    plan = eng.plan(case.qb)
    dist = eng.rank_answers(plan, dev(off), dev(answers.reshape(-1)))[1].cpu().numpy().reshape(B, A)
    for q in range(B):
        want = case.distances_all(case.qb, q, M)[answers[q]]
        np.testing.assert_allclose(dist[q], want, rtol=1e-5)     # (fp32 distances, as in the oracle's band of ranks)
    plan.free()


# the projection's gradient over nearly all of N rows: a part of a 32-row stage, a whole one, one row more, fewer stages than are requested
# ahead, as many, several splits of them with a ragged end; coordinates and features of two tiles
@pytest.mark.parametrize("N,B,K,d,d_sem", [(20, 3, 2, 8, 64), (32, 12, 9, 24, 128), (33, 12, 9, 24, 128), (130, 20, 30, 216, 320),
                                           (193, 20, 40, 216, 64), (1500, 60, 90, 40, 320)])
def test_projection_gradient_by_rows(N, B, K, d, d_sem):
    par.say("projection gradient: N=%d d=%d d_sem=%d" % (N, d, d_sem))
    par.check_forward_backward(par.Case(N, 6, d, 32, B, K, 8.0, seed=N + d, T=4 * N, d_sem=d_sem))


def test_a_step_after_passes_without_a_backward_half():
    """Weights are split for the forward half only where nothing else follows: a step on the same context has both."""
    case = par.Case(1200, 12, 128, 160, 60, 5, 8.0, seed=91, T=2400)
    eng = case.engine()
    plan = eng.plan(case.qb)
    eng.rank_all(plan, 5)
    plan.free()
    par.check_forward_backward(case, eng)
