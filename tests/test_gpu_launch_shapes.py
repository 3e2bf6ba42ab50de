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


@pytest.mark.parametrize("M,N,K", [(1, 5, 4), (1, 800, 400), (2, 401, 260), (3, 36, 1024), (8, 17, 800), (9, 72, 100),
                                   (16, 33, 1024), (17, 33, 64)])
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


@pytest.mark.parametrize("B,C", [(1, 1), (1, 15), (1, 17), (1, 1000), (3, 4097), (40, 33)])
def test_candidate_lists_shared_by_workgroups(B, C):
    import torch
    case = par.Case(3000, 10, 60, 40, B, 2, 8.0, seed=17, T=9000)
    cand = np.random.default_rng(C).integers(0, case.N, (B, C)).astype(np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    got = eng.score(plan, torch.from_numpy(cand).cuda()).cpu().numpy()
    par.assert_close(got, orank.score_candidates(case.qb, cand, om.Model(case.params, case.gamma)), "scores %d x %d" % (B, C))
    plan.free()


# keys: one; 4096 and one more (one workgroup / tiles); 262 144 and more (short / long histogram); a bound of one digit, of
# two and of three
@pytest.mark.parametrize("N,B,n_keys", [(50, 1, 3), (200, 8, 4096), (200, 8, 4104), (70000, 64, 4096), (70000, 64, 262144),
                                        (300, 64, 262208), (1000, 700, 300000)])
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
