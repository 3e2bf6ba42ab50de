"""Helpers of the GPU parity tests: build a seeded workload, run the oracle and
the HIP library on it, compare under the stated tolerances.

Tolerances (fp32 path): loss |d|/|L| <= 1e-4; every tensor both
max|d|/max|ref| <= 1e-4 and ||d||_2/||ref||_2 <= 1e-4.  Table gradients are
additionally checked row by row at 1e-3 (rows whose largest entry is below
1e-30 are compared absolutely), so that an error confined to the tiny rows of
saturated negatives cannot hide behind the large rows.
"""
import numpy as np

import workloads as wl
from oracle import model as om
from oracle import plan as oplan
from oracle import rank as orank

TOL = 1e-4
PYTEST_CONFIG = None


def say(msg):
    """Names the case (and the stage of a long one) on the terminal right away, also under
    pytest's output capture: a GPU run that dies leaves the name of its last case behind."""
    line = "[case] " + msg
    capman = PYTEST_CONFIG.pluginmanager.getplugin("capturemanager") if PYTEST_CONFIG is not None else None
    if capman is None:
        print(line, flush=True)
        return
    with capman.global_and_fixture_disabled():
        print("\n" + line, flush=True)
# Distance the seeded inputs keep from the kinks of the model (ReLU at 0, |.| at 0,
# ties of the min over union branches): there the result is decided by the last
# bits of an fp32 sum, two correct implementations may differ, and the paper's
# method says nothing about which side to take.  fp32 rounding moves a
# pre-activation or a coordinate difference by about 1e-7 on these workloads.
TAU_PRE, TAU_ABS, TAU_TIE = 1e-6, 5e-7, 1e-4
# Text-feature fusion: products of bf16 values are exact in fp32 and are summed in fp32, so
# fused rows, scores, loss and table gradients stay under the fp32 bar.  Only the gradient of
# the projection Wp passes through bf16 (every touched row's gradient is rounded to bf16,
# relative error <= 2^-9 per element, before the contraction with the bf16 features) and is
# held to the bf16 bar.
TOL_BF16 = 2e-2


def tol_of(name, tol):
    return TOL_BF16 if name == "Wp" else tol


class Case:
    def __init__(self, N, R, d, h, B, K, gamma, mix=None, seed=0, T=None, alpha=2.1, trees=None, pos=None,
                 d_sem=0, schedule="level", b_max=0, score_bf16=False, params_edit=None, exact_kinks=False):
        self.N, self.R, self.d, self.h, self.B, self.K, self.gamma = N, R, d, h, B, K, gamma
        self.d_sem = d_sem
        # exact_kinks: inputs that sit exactly on a kink (a pre-activation or a coordinate difference
        # that is 0.0 on both sides, two branches at bit-identical distance) are allowed: there the
        # stated rules decide (relu'(0) = 0, sign(0) = 0, lowest branch) and both sides must follow
        # them; the margins still apply to everything that is merely close to a kink
        self.exact_kinks = exact_kinks
        self.score_bf16 = score_bf16                     # candidate rows from a bf16 copy of E
        self.schedule, self.b_max = schedule, b_max      # order of execution: values must not depend on it
        self.hp = dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, gamma=gamma)
        self.params = wl.make_params(N, R, d, h, seed + 3, d_sem=d_sem)
        if params_edit is not None:
            params_edit(self.params)
        self.sem_bits = wl.make_sem_features(N, d_sem, seed + 5) if d_sem else None
        if trees is not None:
            qb = wl.batch_from_trees(trees, pos)
            want = B or qb.B                             # B > 0: the first B of the trees that are clear of kinks
        else:
            kg = wl.make_kg(N, R, T or 10 * N, alpha, seed)
            want = B
            qb = wl.make_batch(kg, B + B // 4 + 8, mix or {n: 1.0 for n in wl.configs.ALL14}, seed + 1)
        negs = wl.make_negatives(N, qb.B, K, seed + 2)
        self.qb, self.negs, self.n_redrawn = keep_clear_of_kinks(qb, negs, self.params, gamma, N, want, seed + 4,
                                                                 strict=trees is None or B > 0, sem_bits=self.sem_bits,
                                                                 score_bf16=score_bf16, exact_kinks=exact_kinks)
        self.B = self.qb.B

    @classmethod
    def from_config(cls, idx, B=None, K=None, seed_offset=0):
        c = wl.get_config(idx)
        return cls(c.N, c.R, c.d, c.h, B or c.B, K or c.K, c.gamma, mix=c.mix, seed=c.seed + seed_offset,
                   T=c.T, alpha=c.alpha)

    def fresh_negs(self, seed):
        """Another [B, K] draw of negatives, kept clear of the |.| kinks like the first."""
        negs = wl.make_negatives(self.N, self.B, self.K, seed)
        _, negs, _ = keep_clear_of_kinks(self.qb, negs, self.params, self.gamma, self.N, self.B, seed + 1,
                                         strict=False, queries_are_clean=True, sem_bits=self.sem_bits,
                                         score_bf16=self.score_bf16, exact_kinks=self.exact_kinks)
        return negs

    def engine(self, num_streams=1):
        from paper_2602_21597_amd import Engine
        eng = Engine(self.N, self.R, self.d, self.h, self.gamma, num_streams=num_streams, d_sem=self.d_sem,
                     schedule={"level": 0, "max_fill": 1}[self.schedule], b_max=self.b_max, score_bf16=self.score_bf16)
        eng.bind_numpy(self.params, sem_bits=self.sem_bits)
        return eng

    def neg_dev(self, negs=None):
        import torch
        return torch.from_numpy(np.ascontiguousarray(self.negs if negs is None else negs, np.int32)).cuda()

    distances_all = staticmethod(orank.distances_all)    # query -> distance to every entity

    def model(self):
        return om.Model(self.params, self.gamma, self.sem_bits, self.score_bf16)

    def oracle_grads(self, negs=None):
        M = self.model()
        return (M,) + om.batch_loss_and_grads(self.qb, self.negs if negs is None else negs, M)


def min_abs_preactivation(tape, skip_zero=False):
    """Smallest |pre-activation| of any hidden unit met while the oracle evaluated a tree (`tape`
    is what oracle.model.forward returns beside the embedding): the distance of the evaluation
    from a ReLU kink.  skip_zero: units whose pre-activation is exactly 0.0 do not count."""
    def least(pre):
        a = np.abs(pre)
        if skip_zero:
            a = a[a > 0.0]
        return float(a.min()) if a.size else np.inf

    kind = tape[0]
    if kind == "e":
        return np.inf
    if kind == "p":
        return min(least(tape[3][1]), min_abs_preactivation(tape[2], skip_zero))
    if kind == "n":
        return min(least(tape[2][1]), min_abs_preactivation(tape[1], skip_zero))
    return min(min(least(t[1]) for t in tape[2]),
               min(min_abs_preactivation(t, skip_zero) for t in tape[1]))


def keep_clear_of_kinks(qb, negs, params, gamma, N, want, seed, strict=True, queries_are_clean=False,
                        sem_bits=None, score_bf16=False, exact_kinks=False):
    """First `want` queries of qb that stay clear of every kink, with negatives
    that sit on an |.| kink redrawn.  Uses the oracle's forward pass only.
    exact_kinks: values exactly on a kink (0.0, or two equal branch distances) are let through."""
    M = om.Model(params, gamma, sem_bits, score_bf16)
    rng = np.random.default_rng(seed)
    negs = negs.copy()
    keep, redrawn = [], 0
    for i in range(qb.B):
        if len(keep) == want:
            break
        fw = [om.forward(b, M) for b in om.dnf(qb.tree(i))]
        Y = np.stack([y for y, _ in fw])
        ok = min(min_abs_preactivation(t, exact_kinks) for _, t in fw) >= TAU_PRE

        def clear(e):
            dist = np.abs(Y - M.candidate(e)[None]).sum(axis=1)
            w = int(np.argmin(dist))
            gap = np.sort(dist)[1] - dist[w] if len(dist) > 1 else np.inf
            tie = gap < TAU_TIE and not (exact_kinks and gap == 0.0)
            diff = np.abs(Y[w] - M.candidate(e))
            if exact_kinks:
                diff = diff[diff > 0.0]
            return (not tie) and (diff.size == 0 or diff.min() >= TAU_ABS)

        ok = queries_are_clean or (ok and clear(int(qb.pos[i])))
        if ok:
            for j in range(negs.shape[1]):
                tries = 0
                while not clear(int(negs[i, j])):
                    negs[i, j] = rng.integers(0, N)
                    redrawn += 1
                    tries += 1
                    assert tries < 100
            keep.append(i)
        elif not strict:
            raise AssertionError("hand-built query %d sits on a kink; change the test's constants" % i)
    assert len(keep) == want, "not enough kink-free queries: %d of %d" % (len(keep), want)
    return qb.select(keep), negs[keep], redrawn


def rel_err(got, ref, floor=0.0):
    """Max-norm and 2-norm of the difference relative to those of the reference; a reference
    smaller than `floor` per element is measured against the floor instead."""
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    dn = np.abs(got - ref)
    inf = dn.max() / max(np.abs(ref).max(), floor, 1e-300) if ref.size else 0.0
    l2 = np.sqrt((dn ** 2).sum()) / max(np.sqrt((ref ** 2).sum()), floor * np.sqrt(ref.size), 1e-300) if ref.size else 0.0
    return float(inf), float(l2)


def dense_gradient_floor(dense):
    """A gradient tensor that is zero in exact arithmetic holds rounding noise on both sides (u2
    always; u1 when every hidden unit of the attention MLP has the same sign for all inputs of an
    intersection, as happens at very small widths).  Tensors below 1e-4 of the largest MLP gradient
    are therefore measured against that level."""
    return 1e-4 * max(float(np.abs(v).max()) for v in dense.values())


def assert_close(got, ref, name, tol=TOL, floor=0.0):
    assert np.asarray(got).shape == np.asarray(ref).shape, name
    assert np.all(np.isfinite(got)), name
    inf, l2 = rel_err(got, ref, floor)
    assert inf <= tol and l2 <= tol, "%s: max-norm %.3g, 2-norm %.3g (tol %.1g)" % (name, inf, l2, tol)


def assert_zero_gradient(got_u2, ref_dense, tol=TOL):
    """The output bias u2 of the attention MLP shifts the logits of all inputs of an
    intersection alike, and the softmax over inputs ignores such a shift: its
    gradient is zero in exact arithmetic and both sides hold rounding noise only.
    It is therefore compared absolutely, on the scale of the projection's output
    bias gradient."""
    assert np.all(np.isfinite(got_u2))
    assert np.abs(ref_dense["u2"]).max() <= 1e-9 * np.abs(ref_dense["b2"]).max()
    assert np.abs(got_u2).max() <= tol * np.abs(ref_dense["b2"]).max(), "grad u2 not ~0"


def assert_rows_close(got, ref, name, tol=1e-3, scale=None):
    """Row by row, relative to the row's largest entry (or to `scale`, one value per row)."""
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    scale = np.abs(ref).max(axis=1) if scale is None else np.asarray(scale, np.float64)
    err = np.abs(got - ref).max(axis=1)
    big = scale > 1e-30
    worst = (err[big] / scale[big]).max() if big.any() else 0.0
    off = np.abs(got - ref) > tol * scale[:, None]
    assert worst <= tol, "%s: worst row-relative error %.3g; rows (entries beyond the tolerance, the first of them): %s; errors of all rows: %s" % (
        name, worst, [(int(i), int(off[i].sum()), np.flatnonzero(off[i])[:8].tolist()) for i in np.flatnonzero(off.any(axis=1) & big)[:8]],
        ["%.1e" % x for x in err[:64] / np.maximum(scale[:64], 1e-300)])
    assert np.all(err[~big] <= 1e-30), name


def check_forward_backward(case, eng=None, tol=TOL):
    """Plan, index, forward values, loss and every gradient against the oracle."""
    import torch
    eng = eng or case.engine()
    plan = eng.plan(case.qb)
    ref_plan = oplan.build_plan(case.qb, case.schedule, case.b_max)
    got_plan = plan.export()
    for k in ref_plan:
        assert np.array_equal(np.asarray(got_plan[k]), np.asarray(ref_plan[k])), "plan." + k
    f_row, n_rows, step_rows = oplan.forward_rows(ref_plan)
    assert np.array_equal(got_plan["f_row"], f_row) and got_plan["n_f_rows"] == n_rows, "plan.f_row"
    assert np.array_equal(got_plan["f_step_rows"], step_rows), "plan.f_step_rows"

    loss = eng.forward_backward(plan, case.neg_dev())
    torch.cuda.synchronize()
    g = eng.grads()
    M, ref_loss, G, ref_scores = case.oracle_grads()

    # index: bit exact
    u, off, src = oplan.entity_index(ref_plan, case.qb.pos, case.negs)
    assert np.array_equal(g["e_uniq"], u), "e_uniq"
    assert np.array_equal(g["e_seg_off"], off), "e_seg_off"
    assert np.array_equal(g["e_src"], src), "e_src"

    # forward: branch embeddings at the root slots, pair scores
    for q in range(case.B):
        br = om.dnf(case.qb.tree(q))
        slots = ref_plan["root_slot"][ref_plan["root_off"][q]:ref_plan["root_off"][q + 1]]
        for b, s in zip(br, slots):
            assert_close(g["act"][s], om.forward(b, M)[0], "root embedding q%d" % q, tol)
    if case.B:
        assert_close(g["pair_score"].reshape(case.B, case.K + 1), np.stack(ref_scores), "scores", tol)
        got_loss = float(loss.cpu()[0])
        assert abs(got_loss - ref_loss) <= tol * abs(ref_loss), "loss %r vs %r" % (got_loss, ref_loss)

    # gradients
    floor = dense_gradient_floor(G.dense)
    for name in G.dense:
        if name == "u2":
            assert_zero_gradient(g[name], G.dense, tol)
        else:
            assert_close(g[name], G.dense[name], "grad " + name, tol_of(name, tol), floor)
    for tab, uniq, rows in (("E", g["e_uniq"], g["gE"]), ("R", got_plan["r_uniq"], g["gR"])):
        assert sorted(G.rows[tab]) == list(uniq), tab + " touched rows"
        if len(uniq):
            ref_rows = np.stack([G.rows[tab][int(r)] for r in uniq])
            assert_close(rows, ref_rows, "grad " + tab, tol)
            assert_rows_close(rows, ref_rows, "grad rows " + tab)
    plan.free()
    return eng


def _adam_f64(p, m, v, g, t, hp):
    return om.adam_update(np.asarray(p, np.float64), np.asarray(m, np.float64), np.asarray(v, np.float64),
                          np.asarray(g, np.float64), t, lr=hp["lr"], beta1=hp["beta1"], beta2=hp["beta2"],
                          eps=hp["eps"])


def _dense_grads_from_gpu(g, plan_export, shapes):
    out = {n: g[n].astype(np.float64) for n in shapes if n not in ("E", "R")}
    for tab, uniq, rows in (("E", g["e_uniq"], g["gE"]), ("R", plan_export["r_uniq"], g["gR"])):
        full = np.zeros(shapes[tab], np.float64)
        full[uniq] = rows
        out[tab] = full
    return out


def check_update(name, t, hp, lib_before, lib_after, g_own, ref_before, ref_after, gref, delta, tol=TOL,
                 cancels=False, dense_floor=None, exclude=None):
    """One tensor's optimiser step, two ways (see check_train_steps).  All arrays hold the compared
    elements only (tables: the touched rows, in one order on both sides).
    lib_before / lib_after: the library's (p, m, v), fp32; g_own: the library's own gradient;
    ref_before / ref_after: the oracle's (p, m, v), fp64; gref: the oracle's gradient; delta: the
    rounding level of gref per element (or per row, broadcast); exclude: elements (B) must leave
    out for a reason the caller states.  Returns (kept, eligible) of (B)."""
    b_p, b_m, b_v = lib_before
    a_p, a_m, a_v = lib_after
    ulp = np.spacing(np.abs(b_p).astype(np.float32)).astype(np.float64)
    # (A) optimiser alone, all elements
    wp, wm, wv = _adam_f64(b_p, b_m, b_v, g_own, t, hp)
    upd = wp - b_p
    err = np.abs(a_p - wp)
    assert np.all(err <= tol * max(np.abs(upd).max(), 1e-300) + ulp), \
        "%s: Adam on own gradients, worst %.3g" % (name, err.max())
    assert_close(a_m, wm, "m(own g) " + name, tol)
    assert_close(a_v, wv, "v(own g) " + name, tol)
    # (B) end to end
    if name == "u2":     # zero gradient in exact arithmetic: direction is rounding noise
        return None
    if dense_floor is not None and np.abs(gref).max() < dense_floor:
        return None      # the same for a tensor at the noise floor (see dense_gradient_floor)
    tol_b = tol_of(name, tol)
    p0, m0, v0 = ref_before
    hi = _adam_f64(p0, m0, v0, gref + delta, t, hp)[0]
    lo = _adam_f64(p0, m0, v0, gref - delta, t, hp)[0]
    upd_ref = ref_after[0] - p0
    scale = np.abs(upd_ref).max()
    keep = (np.abs(hi - lo) / 2 <= tol_b * scale)
    # dead units (no gradient now, none before): identical input to Adam
    keep |= (gref == 0.0) & (g_own == 0.0) & (m0 == 0.0) & (v0 == 0.0)
    eligible = keep.size
    if exclude is not None:
        keep &= ~np.broadcast_to(exclude, keep.shape)
        eligible -= int(np.broadcast_to(exclude, keep.shape).sum())
    upd_gpu = a_p.astype(np.float64) - b_p.astype(np.float64)
    err = np.abs(upd_gpu - upd_ref)
    bound = tol_b * scale + ulp
    assert np.all(err[keep] <= bound[keep]), \
        "%s update: worst %.3g x bound" % (name, (err[keep] / bound[keep]).max())
    # (a tensor whose terms largely cancel -- u1: the logit gradients of an intersection sum to
    # zero over its inputs -- may keep fewer)
    assert cancels or keep.sum() >= 0.3 * eligible, "%s: only %d of %d elements are well conditioned" % (
        name, keep.sum(), eligible)
    assert_close(a_m, ref_after[1], "m " + name, tol_b)
    assert_close(a_v, ref_after[2], "v " + name, 2 * tol_b)
    return int(keep.sum()), int(eligible)


def gradient_noise(name):
    """Rounding level of a gradient relative to the scale of its terms: bf16 for Wp (every term is
    rounded to bf16, 2^-9 relative; the errors add in quadrature, and over the 4e5 elements of the
    workload's Wp the largest of them is 4-5 standard deviations); else that of dL/ds =
    sigmoid(s)-like, which inherits the absolute error of the fp32 score (sums of d terms of size
    ~gamma: ~1e-5)."""
    return 1e-2 if name == "Wp" else 1e-5


def report_kept(kept, where):
    """Names, per tensor, how much of it check (B) compared end to end."""
    say("%s: update check (B) compared, of each tensor's elements: %s" % (
        where, ", ".join("%s %.1f%%" % (n, 100.0 * k / max(a, 1)) for n, (k, a) in kept.items())))


def check_train_steps(case, steps=3, num_streams=1, tol=TOL):
    """Updates over a few steps with fresh negatives, two ways.

    (A) The optimiser alone, every element: the library's update must equal textbook
        Adam (oracle routine, fp64) applied to the library's own gradients of the
        same step, which ngdb_forward_backward exposes.
    (B) End to end against the oracle's step.  Adam maps a gradient g to about
        lr*g/(|g|+eps): where |g| is comparable with eps the map amplifies rounding
        noise of g without bound relative to the result, so elements whose reference
        update moves by more than the tolerance when the reference gradient is
        perturbed by 1e-5 of the largest gradient entry of the tensor (for the tables: of
        the summed sizes of the row's contributions, which set the fp32 rounding level of
        their sum) are left out of (B) and counted; (A) still covers them.  The share of
        every tensor that (B) compared is printed.
    An fp32 parameter near 0.1 stores an update of 1e-4 only to half an ulp of the
    parameter, so one ulp of the parameter is added to both bounds.
    """
    import torch
    eng = case.engine(num_streams)
    plan = eng.plan(case.qb)
    pexp = plan.export()
    P = om.to_f64(case.params)
    state = om.new_state(P)
    shapes = {k: v.shape for k, v in P.items()}
    for t in range(1, steps + 1):
        negs = case.fresh_negs(7000 + t)
        nd = case.neg_dev(negs)
        eng.forward_backward(plan, nd)
        g_gpu = _dense_grads_from_gpu(eng.grads(), pexp, shapes)
        touched_gpu = {"E": eng.grads()["e_uniq"], "R": pexp["r_uniq"]}
        before_ref = {k: v.copy() for k, v in P.items()}
        state_ref_before = {k: [x.copy() for x in v] for k, v in state.items()}
        b_p, b_m, b_v = eng.params_numpy("p"), eng.params_numpy("m"), eng.params_numpy("v")
        loss = eng.train_step(plan, nd)
        torch.cuda.synchronize()
        ref_loss, G = om.train_step(case.qb, negs, P, state, t, case.hp, case.sem_bits, track_sq=True,
                                    score_bf16=case.score_bf16)
        a_p, a_m, a_v = eng.params_numpy("p"), eng.params_numpy("m"), eng.params_numpy("v")
        if case.B:
            assert abs(float(loss.cpu()[0]) - ref_loss) <= tol * abs(ref_loss)
        assert eng.step_count() == t
        kept = {}
        for name in P:
            rows = slice(None)
            table = name in ("E", "R")
            if table:
                touched = np.zeros(shapes[name][0], bool)
                touched[touched_gpu[name]] = True
                assert sorted(G.rows[name]) == list(np.flatnonzero(touched)), name + " touched rows"
                for bb, aa in ((b_p, a_p), (b_m, a_m), (b_v, a_v)):
                    assert np.array_equal(aa[name][~touched], bb[name][~touched]), name + " untouched rows moved"
                rows = touched
            gref = G.table_dense(name, shapes[name]) if table else G.dense[name]
            if table:     # of a row sum: set by the sizes of its contributions (oracle Grads.mass)
                mass = np.zeros((shapes[name][0], 1))
                for i, v in G.mass[name].items():
                    mass[i, 0] = v
                delta = gradient_noise(name) * mass[rows]
                cancels = False
            else:         # of a dense sum: independent errors of the terms add in quadrature
                rms = np.sqrt(G.dense_sq[name])
                delta = gradient_noise(name) * np.maximum(rms, np.abs(gref).max() * 1e-3)
                cancels = np.abs(gref).max() < 0.05 * rms.max()
            m0, v0 = state_ref_before[name]
            res = check_update(name, t, case.hp, (b_p[name][rows], b_m[name][rows], b_v[name][rows]),
                               (a_p[name][rows], a_m[name][rows], a_v[name][rows]), g_gpu[name][rows],
                               (before_ref[name][rows], m0[rows], v0[rows]),
                               (P[name][rows], state[name][0][rows], state[name][1][rows]), gref[rows], delta,
                               tol=tol, cancels=cancels,
                               dense_floor=None if table else dense_gradient_floor(G.dense))
            if res is not None:
                kept[name] = res
        report_kept(kept, "step %d" % t)
    plan.free()
    return eng


def check_topk(case, k, n_check):
    import torch
    eng = case.engine()
    plan = eng.plan(case.qb)
    ids, dist = eng.rank_all(plan, k)
    torch.cuda.synchronize()
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    M = case.model()
    assert np.all(np.diff(dist, axis=1) >= 0)
    for q in np.random.default_rng(1).choice(case.B, min(n_check, case.B), replace=False):
        full = case.distances_all(case.qb, int(q), M)
        ref_ids, ref_d = orank.topk_all(case.qb, int(q), M, k, case.distances_all)
        assert_close(dist[q], ref_d, "top-k distances q%d" % q)
        # a returned id is right if its true distance is within the k-th best (fp32 may swap near ties)
        assert len(set(ids[q])) == k and ids[q].min() >= 0
        assert np.all(full[ids[q]] <= ref_d[-1] * (1 + 1e-4)), "q%d" % q
        assert_close(dist[q], full[ids[q]], "returned distances belong to returned ids q%d" % q)
    plan.free()


def check_filtered_ranks(case, seed, n_check=None):
    """Answer lists: a few of the truly nearest entities (small ranks, mutual filtering) plus random
    entities; one query without answers; scored prefix n_take shorter than the list for some."""
    import torch
    rng = np.random.default_rng(seed)
    M = case.model()
    B, N = case.B, case.N
    lists, full = [], []
    for q in range(B):
        dist = case.distances_all(case.qb, q, M)
        full.append(dist)
        near = np.argsort(dist, kind="stable")[:12]
        ans = list(rng.choice(near, int(rng.integers(0, 4)), replace=False)) + \
            list(rng.choice(N, int(rng.integers(1, 5)), replace=False))
        ans = list(dict.fromkeys(int(a) for a in ans))
        lists.append([] if q == 1 else ans)
    off = np.concatenate([[0], np.cumsum([len(l) for l in lists])]).astype(np.int32)
    flat = np.asarray([a for l in lists for a in l], np.int32)
    n_take = np.asarray([max(0, len(l) - (q % 3 == 0)) for q, l in enumerate(lists)], np.int32)
    eng = case.engine()
    plan = eng.plan(case.qb)
    dev = lambda x: torch.from_numpy(x).cuda()
    ranks, dist, metrics = eng.rank_answers(plan, dev(off), dev(flat), dev(n_take))
    ranks, dist, metrics = ranks.cpu().numpy(), dist.cpu().numpy(), metrics.cpu().numpy()
    exact = 0
    for q in range(B):
        a = np.asarray(lists[q], np.int64)
        if not len(a):
            continue
        want, d_ref = orank.filtered_ranks(case.qb, q, a, M, case.distances_all)
        got, d_got = ranks[off[q]:off[q + 1]], dist[off[q]:off[q + 1]]
        assert_close(d_got, d_ref, "answer distances q%d" % q)
        other = np.ones(N, bool)
        other[a] = False
        d_other = np.sort(full[q][other])
        # fp32 distances: entities within 1e-5 (relative) of an answer may fall on either side
        lo = 1 + np.searchsorted(d_other, d_ref * (1 - 1e-5), side="left")
        hi = 1 + np.searchsorted(d_other, d_ref * (1 + 1e-5), side="left")
        assert np.all((lo <= got) & (got <= hi)), "q%d: %r vs %r" % (q, got, want)   # exact wherever lo == hi
        exact += int(np.sum(got == want))
    say("filtered ranks: %d of %d equal to the oracle's exactly, the rest inside its fp32 band" % (exact, len(flat)))
    assert exact >= 0.8 * len(flat)      # (in a table of 150 000 rows distances are denser than fp32 resolves)
    # the metric kernel against the oracle's formula on the same ranks, scored prefixes only
    want_m = orank.ranking_metrics([ranks[off[q]:off[q] + n_take[q]] for q in range(B)], ks=(1, 3, 10))
    np.testing.assert_allclose(metrics, want_m, rtol=1e-5, atol=1e-7)
    _, _, m_all = eng.rank_answers(plan, dev(off), dev(flat), None)
    want_all = orank.ranking_metrics([ranks[off[q]:off[q + 1]] for q in range(B)], ks=(1, 3, 10))
    np.testing.assert_allclose(m_all.cpu().numpy(), want_all, rtol=1e-5, atol=1e-7)
    plan.free()
