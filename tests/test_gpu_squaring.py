"""Default path at d >= 32 where the equal factors are composed by squaring on chip: horizons around the rule's edges
(powers of two, all bits set, a terminal cost of its own), each state size, batches below and above one grid, the guard's
way out to the Riccati recursion, breakdown reports, and the rule itself."""
import numpy as np
import pytest
import torch

import bench
from paper_2603_09221_amd import binding, synth
from tests.parity import SOLVE_KEYS, oracle_solve, solve_errors

DEV = "cuda:0"


def solve(b, QT=None, **kw):
    out = binding.ttc_lqr_solve(b.A, b.B, b.Q, b.R, QT, b.x0, b.T, **kw)
    torch.cuda.synchronize()
    return out


def squared(T, bf16, own_QT, d=64, **kw):
    p = binding.Problem(n=1, d=d, m=d, T=T, in_dtype=binding.TTC_BF16 if bf16 else binding.TTC_F32, Q=256,
                        QT=512 if own_QT else None)
    for k, v in kw.items():
        setattr(p, k, v)
    return binding.ttc_lqr_solve_squares(p)


def test_the_rule_takes_long_horizons_and_leaves_short_ones():
    """The library's rule, asked through its query, which bench.py prices the default path with: the horizons up to 40 it
    takes, for either input type, with Q_T = Q (absent, or the very same array) and with a Q_T of its own; every later one;
    none at d = 16, which has its own kernel, none where the caller asks for the product or for the flagged path."""
    for d in (32, 64, 128):
        takes = lambda bf16, own: {T for T in range(1, 41) if squared(T, bf16, own, d=d)}
        assert takes(False, False) == {8} | set(range(12, 41))
        assert takes(True, False) == {12, 14} | set(range(16, 41))
        assert takes(False, True) == {13} | set(range(15, 41))
        assert takes(True, True) == set(range(17, 41))
        for T in (41, 64, 127, 1023, 1024, 1000000):
            assert all(squared(T, b, o, d=d) for b in (False, True) for o in (False, True))
        assert squared(8, False, True, d=d, QT=256) and not squared(8, False, True, d=d, QT=256, sQT=4)
        for kw in (dict(rebase_every=3), dict(flags=binding.TTC_FLAG_PURE_SYMPLECTIC), dict(flags=binding.TTC_FLAG_DOUBLING)):
            assert not squared(64, False, False, d=d, **kw)
        assert bench.default_squares(d, 8, False) and not bench.default_squares(d, 8, False, own_QT=True)
    assert not any(squared(T, False, False, d=16) for T in range(1, 100))
    assert not squared(64, False, False, d=48) and not squared(0, False, False)
    assert bench.alg_flops_default(64, 8, 3, False) != bench.alg_flops(64, 8, 3)
    assert bench.alg_flops_default(64, 9, 3, False) == bench.alg_flops(64, 9, 3)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,own_QT", [("f32", False), ("f32", True), ("bf16", False), ("bf16", True)])
def test_the_rule_is_what_runs(dtype, own_QT):
    """Where the rule does not square, the result is bit for bit that of the product in its default grouping, asked for by
    rebase_every; where it does, it is not.  Horizons on both sides of every edge that a rebase_every can ask for."""
    d, seen = 64, set()
    for T in range(7, 20):
        groups = bench.default_groups(T, dtype)
        ask = [k for k in range(1, T + 1) if -(-T // k) == groups]
        if not ask:
            continue
        b = synth.make_batch(5, d, d, T, seed=T, device=DEV, dtype=dtype)
        QT = (1.5 * b.Q).contiguous() if own_QT else None
        out, seq = solve(b, QT=QT), solve(b, QT=QT, rebase_every=ask[0])
        same = all(torch.equal(out[k], seq[k]) for k in SOLVE_KEYS)
        assert same != squared(T, dtype == "bf16", own_QT, d=d), T
        seen.add(same)
    assert seen == {False, True}


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 5), (32, 2100), (64, 9), (64, 1100), (128, 3), (128, 270)])
@pytest.mark.parametrize("T", [8, 12, 15, 16, 31])
def test_against_the_oracle(d, n, T):
    """1e-4 is the path's tolerance; on ordinary problems the composition keeps 2e-5 per problem (measured 1e-6..5e-6)."""
    b = synth.make_batch(n, d, d, T, seed=d + T, device=DEV)
    out = solve(b)
    assert int(out["info"].abs().max()) == 0
    for k, v in solve_errors(out, oracle_solve(b)).items():
        assert v <= 2e-5, (k, v)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T", [16, 17, 33])
def test_terminal_cost_stage_flag_shared_and_bf16(d, T):
    b = synth.make_batch(11, d, d, T, seed=T, device=DEV)
    QT = (1.5 * b.Q + 0.2 * torch.eye(d, device=DEV)).contiguous()
    for qt, flag in ((QT, False), (QT, True), (None, True)):
        out = solve(b, QT=qt, flags=binding.TTC_FLAG_STAGE_COST_AT_X0 if flag else 0)
        for k, v in solve_errors(out, oracle_solve(b, QT=qt, flag=flag)).items():
            assert v <= 2e-5, (k, v)
    same = solve(b, QT=b.Q)  # Q_T given as the very same array is Q_T = Q
    ref = solve(b)
    for k in SOLVE_KEYS:
        assert torch.equal(same[k], ref[k]), k
    shared = synth.LqrBatch(b.A[:1].expand(11, -1, -1), b.B, b.Q[:1].expand(11, -1, -1), b.R, b.x0, T)
    full = synth.LqrBatch(shared.A.contiguous(), b.B, shared.Q.contiguous(), b.R, b.x0, T)
    got, want = solve(shared), solve(full)
    for k in SOLVE_KEYS:
        assert torch.equal(got[k], want[k]), k
    h = synth.make_batch(7, d, d, T, seed=T + 1, device=DEV, dtype="bf16")
    for k, v in solve_errors(solve(h), oracle_solve(h)).items():  # the oracle consumes the rounded values
        assert v <= 2e-5, (k, v)


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 40), (64, 30), (128, 9)])
def test_cheap_control_takes_the_riccati_recursion_and_growth_stays_accurate(d, n):
    """Cost ratios of 1e2 and more make I + G H large: such problems leave for the printed recursion (mixed here with
    ordinary ones); an unstable open loop with costly control grows it later.  1e-4 as in the guard's own sweep; at a ratio
    of 1e4 four times what the recursion itself (ttc_lqr_solve_tv on repeated matrices) shows."""
    T = 16
    for qs, rs, rho in ((1.0, 1e-2, None), (1e2, 1.0, None), (1e-2, 1e2, 1.2), (1.0, 1.0, 1.2), (1e2, 1e-2, None)):
        b = synth.make_batch(n, d, d, T, seed=d, device=DEV, q_scale=qs, r_scale=rs, rho=rho)
        easy = synth.make_batch(n, d, d, T, seed=d, device=DEV)
        pick = (torch.arange(n, device=DEV) % 3 == 1)[:, None, None]
        mix = synth.LqrBatch(torch.where(pick, b.A, easy.A), easy.B, torch.where(pick, b.Q, easy.Q),
                             torch.where(pick, b.R, easy.R), easy.x0, T)
        for batch in (b, mix):
            out = solve(batch)
            assert int(out["info"].abs().max()) == 0
            ref = oracle_solve(batch)
            tol = 1e-4
            if qs / rs > 1e3:
                rep = lambda t: t.unsqueeze(1).expand(-1, T, -1, -1)
                tv = binding.ttc_lqr_solve_tv(rep(batch.A), rep(batch.B), rep(batch.Q), rep(batch.R), batch.x0)
                tol = max(tol, 4 * max(solve_errors(tv, ref).values()))
            for k, v in solve_errors(out, ref).items():
                assert v <= tol, (qs, rs, rho, k, v)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
def test_breakdowns_are_reported_as_on_the_sequential_path(d):
    """R not positive definite: info = 1; a singular A: info = 2, although composing needs no inverse of A; both NaN, also
    when the problem would have left for the Riccati recursion; the others are what they are alone."""
    n, T = 12, 16
    b = synth.make_batch(n, d, d, T, seed=4, device=DEV)
    A, R, Q = b.A.clone(), b.R.clone(), b.Q.clone()
    R[3] = -R[3]
    A[5] = 0.0
    A[7] = 0.0
    R[7] *= 1e-2  # cheap control beside a singular A
    Q[9] *= 1e2   # cheap control alone
    out = solve(synth.LqrBatch(A, b.B, Q, R, b.x0, T))
    info = out["info"].cpu().numpy()
    assert info[3] == 1 and info[5] == 2 and info[7] == 2 and (np.delete(info, [3, 5, 7]) == 0).all()
    for k in SOLVE_KEYS:
        bad = torch.isnan(out[k].reshape(n, -1)).all(1).cpu().numpy()
        assert bad[[3, 5, 7]].all() and not np.delete(bad, [3, 5, 7]).any(), k
    seq = solve(synth.LqrBatch(A, b.B, Q, R, b.x0, T), rebase_every=3)
    assert (seq["info"].cpu().numpy() == info).all()
    keep = torch.tensor([0, 1, 2, 4, 6, 8, 10, 11], device=DEV)
    alone = solve(synth.LqrBatch(A, b.B, Q, R, b.x0, T).take(keep))
    for k in SOLVE_KEYS:
        assert torch.equal(out[k][keep], alone[k]), k


@pytest.mark.gpu
def test_noalloc_takes_the_same_path():
    for d, T, n in ((64, 16, 1030), (128, 32, 260)):
        b = synth.make_batch(n, d, d, T, seed=6, device=DEV)
        f32 = dict(dtype=torch.float32, device=DEV)
        out = {"P0": torch.empty((n, d, d), **f32), "K0": torch.empty((n, d, d), **f32), "u0": torch.empty((n, d), **f32),
               "value": torch.empty((n,), **f32), "info": torch.empty((n,), dtype=torch.int32, device=DEV)}
        binding.ttc_lqr_solve_noalloc(b.A, b.B, b.Q, b.R, None, b.x0, T, out)
        ref = solve(b)
        for k in SOLVE_KEYS:
            assert torch.equal(out[k], ref[k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 7), (64, 1100), (128, 7)])
@pytest.mark.parametrize("T", [8, 12])
def test_a_small_pivot_starts_the_problem_over_with_pivoting(d, n, T):
    """A stage cost that is not semidefinite: elimination of I + G H in order meets negative pivots, and the sequential
    product, whose solves are pivoted, takes the problem, which
    is well conditioned (float32 on the CPU: errors below 1e-6).  Its neighbours, also those the
    same workgroup takes next, come out as they do alone."""
    b = synth.make_batch(n, d, d, T, seed=d, device=DEV)
    B = 0.1 * b.B + torch.eye(d, device=DEV)
    R = torch.eye(d, device=DEV).repeat(n, 1, 1)
    Q = b.Q.clone()
    Q[1] = torch.diag(torch.where(torch.arange(d, device=DEV) % 3 == 0, -6.0, 1.0))
    out = solve(synth.LqrBatch(b.A, B, Q, R, b.x0, T))
    assert not out["info"].any()
    A1, B1, Q1, R1 = (t[1].double().cpu().numpy() for t in (b.A, B, Q, R))
    P = Q1
    for s in range(T - 1, -1, -1):  # the printed recursion with a general solve
        S, F = R1 + B1.T @ P @ B1, B1.T @ P @ A1
        assert np.linalg.eigvalsh(S).min() < 0 and np.linalg.cond(S) < 10
        K = -np.linalg.solve(S, F)
        P = (Q1 if s else 0) + A1.T @ P @ A1 + F.T @ K
        P = 0.5 * (P + P.T)
    for k, want in (("P0", P), ("K0", K)):
        assert np.linalg.norm(out[k][1].double().cpu().numpy() - want) <= 2e-5 * np.linalg.norm(want), k
    alone = solve(synth.LqrBatch(b.A, B, b.Q, R, b.x0, T))
    keep = torch.arange(n, device=DEV) != 1
    for k in SOLVE_KEYS:
        assert torch.equal(out[k][keep], alone[k][keep]), k


def recursion64(b, QT=None):
    """P_0, K_0 of the printed recursion in float64 with general solves (R + B^T P B need not be positive definite)."""
    A, B, Q, R, _ = b.numpy64()
    t = lambda M: M.swapaxes(-1, -2)
    Q, R = 0.5 * (Q + t(Q)), 0.5 * (R + t(R))
    P = Q if QT is None else 0.5 * (QT + t(QT))
    for s in range(b.T - 1, -1, -1):
        F = t(B) @ P @ A
        K = -np.linalg.solve(R + t(B) @ P @ B, F)
        P = (Q if s else 0) + t(A) @ P @ A + t(F) @ K
        P = 0.5 * (P + t(P))
    return {"P0": P, "K0": K}


def problem_errors(out, ref):
    """The larger of the errors of P_0 and K_0, per problem (NaN where there is no answer)."""
    rel = lambda k: np.linalg.norm(out[k].double().cpu().numpy() - ref[k], axis=(-1, -2)) / np.linalg.norm(ref[k], axis=(-1, -2))
    return np.maximum(rel("P0"), rel("K0"))


def indefinite(n, d, T, seed=None):
    """Stage costs with eigenvalues of about -0.2: R + B^T P B becomes indefinite, and regular, within a few steps."""
    b = synth.make_batch(n, d, d, T, seed=d + T if seed is None else seed, device=DEV)
    b.Q.sub_(0.2 * torch.eye(d, device=DEV))
    return b


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 40), (64, 30), (128, 9)])
@pytest.mark.parametrize("T", [12, 15, 32])
def test_a_stage_cost_that_is_not_semidefinite_is_answered_as_by_the_product(d, n, T):
    """The recursion refuses such problems and squaring loses their digits; the sequential product, whose solves are
    pivoted, answers them.  At these horizons rebase_every = 3 is the product's own grouping.  What it answers is answered,
    and as well: problems near a singular R + B^T P B lose digits on either path (1e-4 and more), and there the errors of
    two float32 evaluations are independent draws, for which 10 is allowed."""
    b = indefinite(n, d, T)
    ref = recursion64(b)
    out, seq = solve(b), solve(b, rebase_every=3)
    answered = (seq["info"] == 0).cpu().numpy()
    assert answered.mean() >= 0.5
    assert not out["info"].cpu().numpy()[answered].any()
    err, err_seq = problem_errors(out, ref)[answered], problem_errors(seq, ref)[answered]
    print(d, T, "median %.1e %.1e, largest %.1e %.1e" % (np.median(err), np.median(err_seq), err.max(), err_seq.max()))
    assert (err <= np.maximum(1e-4, 10 * err_seq)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 7000), (64, 2100), (128, 530)])
def test_problems_handed_on_stay_by_themselves(d, n):
    """Ordinary problems beside ones of each kind that is handed on, more than one pass of the grid, outputs left out and in
    a captured graph: everything is what it is alone."""
    T = 12
    b = synth.make_batch(n, d, d, T, seed=3, device=DEV)
    odd, ind = synth.make_batch(n, d, d, T, seed=3, device=DEV, r_scale=1e-3), indefinite(n, d, T, seed=3)
    kind = torch.arange(n, device=DEV) % 7
    b.R[kind == 2] = odd.R[kind == 2]   # over the limit
    b.Q[kind == 4] = ind.Q[kind == 4]   # not semidefinite
    b.A[n - 3] = 0.0                    # singular
    b.R[n - 5].neg_()                   # not positive definite
    out = solve(b)
    info = out["info"].cpu().numpy()
    assert info[n - 3] == 2 and info[n - 5] == 1
    for which in (kind == 2, kind == 4, (kind != 2) & (kind != 4)):
        pick = which.nonzero()[:, 0]
        alone = solve(b.take(pick))
        for k in SOLVE_KEYS + ("info",):
            assert torch.equal(out[k][pick].nan_to_num(nan=1e30), alone[k].nan_to_num(nan=1e30)
                               if alone[k].is_floating_point() else alone[k]), k
    few = binding.ttc_lqr_solve(b.A, b.B, b.Q, b.R, None, b.x0, T, want_P0=False, want_K0=False)
    assert torch.equal(few["u0"].nan_to_num(nan=1e30), out["u0"].nan_to_num(nan=1e30))
    res = {k: torch.zeros_like(v) for k, v in out.items()}
    graph = torch.cuda.CUDAGraph()
    ws = torch.empty(binding.ttc_lqr_workspace_bytes(binding.make_problem(b.A, b.B, b.Q, b.R, None, b.x0, T)),
                     dtype=torch.uint8, device=DEV)
    with torch.cuda.graph(graph):
        binding.ttc_lqr_solve(b.A, b.B, b.Q, b.R, None, b.x0, T, out=res, workspace=ws)
    for _ in range(3):
        for v in res.values():
            v.zero_()
        graph.replay()
        solve(b.take(slice(0, 5)))
        torch.cuda.synchronize()
        for k in SOLVE_KEYS + ("info",):
            got, want = (res[k].nan_to_num(nan=1e30), out[k].nan_to_num(nan=1e30)) if k != "info" else (res[k], out[k])
            assert torch.equal(got, want), k


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 12), (64, 10), (128, 5)])
@pytest.mark.parametrize("dtype,T,qt,r,rho", [
    ("f32", 16, 30, 1.0, None), ("f32", 31, 30, 1.0, None), ("f32", 32, None, 1e2, 1.2), ("f32", 64, None, 1.0, 1.2),
    ("bf16", 31, 10, 1.0, None), ("bf16", 32, 30, 1.0, None), ("bf16", 31, 100, 1.0, None), ("bf16", 32, 1000, 1.0, None),
    ("bf16", 12, None, 1 / 30, None), ("bf16", 32, None, 1 / 30, None), ("bf16", 64, None, 1.0, 1.2)])
def test_what_the_product_kept_stays_with_squaring(d, n, dtype, T, qt, r, rho):
    """A large terminal cost, an unstable open loop over a long horizon and, with bfloat16 inputs, a ratio of the scales of 30
    make max |I + G H| large without costing the digits that cheap control costs: the grouped product kept these problems,
    and the recursion that a single limit sent them to is up to twice as slow.  They are not what the recursion gives bit
    for bit (a few at the edge of a limit may be), and within 2e-5; with bfloat16 inputs and cheap control within 1e-4, a
    tenth of the product's own error on them."""
    b = synth.make_batch(n, d, d, T, seed=d + T, device=DEV, dtype=dtype, r_scale=r)
    if rho:
        b.A.mul_(rho / 1.1)
    QT = None if qt is None else (qt * b.Q).contiguous()
    out = solve(b, QT=QT)
    assert not out["info"].any()
    err = problem_errors(out, recursion64(b, None if QT is None else QT.double().cpu().numpy()))
    steps = [m[:, None].expand(-1, T, -1, -1).contiguous() for m in (b.A, b.B, b.Q, b.R)]
    if QT is not None:
        steps[2][:, T - 1] = QT
    tv = binding.ttc_lqr_solve_tv(*steps, b.x0)
    torch.cuda.synchronize()
    same = (out["P0"] == tv["P0"]).flatten(1).all(1)
    print(d, dtype, T, qt, r, rho, "%.1e" % err.max(), int(same.sum()))
    assert same.sum() <= n // 4
    assert err.max() <= (1e-4 if r < 1 else 2e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(32, 9), (64, 9), (128, 5)])
def test_dynamics_far_from_diagonal_and_scaled(d, n):
    """Whether A is singular is seen from its distance to a diagonal matrix, or else factored: dense dynamics, a permutation (no diagonal at
    all), columns in units far apart and a diagonal far from one are solved (2e-5 as above), and reported only where singular."""
    T = 16
    b = synth.make_batch(n, d, d, T, seed=3, device=DEV)
    A = b.A.clone()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2)
    A[0] = torch.randn((d, d), device=DEV, generator=gen) / d ** 0.5
    A[1] = torch.eye(d, device=DEV).roll(1, 0)
    A[2] = 0.3 * A[2]
    A[3] = 0.0
    A[4, :, 5] = A[4, :, 4]
    out = solve(synth.LqrBatch(A, b.B, b.Q, b.R, b.x0, T))
    info = out["info"].cpu().numpy()
    assert info[3] == 2 and info[0] == info[1] == info[2] == 0 and (info[5:] == 0).all()
    ref = oracle_solve(synth.LqrBatch(A, b.B, b.Q, b.R, b.x0, T))
    for p in [q for q in range(n) if q not in (3, 4)]:
        for k, v in solve_errors({k: out[k][p:p + 1] for k in SOLVE_KEYS}, {k: ref[k][p:p + 1] for k in SOLVE_KEYS}).items():
            assert v <= 2e-5, (p, k, v)
