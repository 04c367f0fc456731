"""Problems whose states and controls come in units of very different size: x' = D x, u' = E u with powers of two, which float32
carries through exactly.  Products of split operands (ttc_split.hpp) keep 40 binary digits below the largest entry of a column of an
operand; the results have to be those of the same problem in units of one all the same.

Both are held against float64, column by column and in units of one.  The bound is the library's own error on the problem in units of
one: twice that for the tenth-worst percent of the columns, eight times for the worst one, the largest of a few hundred with a long tail
(columns that are small differences; a column that has lost its digits is off by 1e-4 and more), and no less than 1e-6 and 2e-6
(16 and 32 roundings of 6e-8), where the former happens to be small."""
import functools

import numpy as np
import pytest
import torch

from oracle import lqr_grad_oracle, lqr_oracle
from paper_2603_09221_amd import binding, synth

DEV = "cuda:0"
N = 3


def _exponents(kind, d):
    """Binary exponents of the units of the d states."""
    how, k = kind
    e = np.zeros(d)
    if how == "one":
        e[d // 3] = k
    elif how == "alternate":      # both sizes in every 16-wide tile
        e[1::2] = k
    elif how == "graded":
        e = np.round(np.linspace(-k / 2, k / 2, d))[np.random.default_rng(3).permutation(d)]
    return e


KINDS = [("one", 7), ("one", 17), ("one", 30), ("one", -30), ("alternate", 5), ("alternate", 6), ("alternate", 7), ("alternate", 8), ("alternate", 12), ("alternate", 30), ("graded", 24)]
ONE = ("one", 0)


class _Units:
    def __init__(self, kind, d):
        self.D = 2.0 ** _exponents(kind, d)
        self.E = 2.0 ** -_exponents(("alternate", kind[1]), d)

    def problem(self, A, B, Q, R, x0):
        D, E = (torch.tensor(v, dtype=torch.float32, device=A.device) for v in (self.D, self.E))
        out = (D[:, None] * A / D, D[:, None] * B / E, Q / D[:, None] / D, R / E[:, None] / E, D * x0)
        return tuple(t.to(A.dtype).contiguous() for t in out)


def _np(t):
    return t.double().cpu().numpy()


def _columns(got, want, vectors=False):
    """Relative errors of the columns of matrices (vectors: of vectors): the worst but a tenth, and the worst."""
    axis = -1 if vectors else -2
    num, den = np.linalg.norm(got - want, axis=axis), np.linalg.norm(want, axis=axis)
    e = num / np.where(den > 0, den, 1)
    return float(np.quantile(e, 0.9)), float(e.max())


def _first_step_errors(out, ref, un):
    assert int(out["info"].abs().max()) == 0
    return dict(P0=_columns(_np(out["P0"]) * un.D[:, None] * un.D, ref["P0"]),
                K0=_columns(_np(out["K0"]) / un.E[:, None] * un.D, ref["K0"]),
                u0=_columns(_np(out["u0"]) / un.E, ref["u0"], True))


def _rollout_errors(out, U, X, un):
    assert int(out["info"].abs().max()) == 0
    return dict(U=_columns(_np(out["U"]) / un.E, U, True), X=_columns(_np(out["X"]) / un.D, X, True))


def _gradient_errors(out, ref, un):
    assert int(out["info"].abs().max()) == 0
    D, E = un.D, un.E
    return dict(gA=_columns(_np(out["gA"]) * D[:, None] / D, ref["gA"]), gB=_columns(_np(out["gB"]) * D[:, None] / E, ref["gB"]),
                gQ=_columns(_np(out["gQ"]) / D[:, None] / D, ref["gQ"]), gR=_columns(_np(out["gR"]) / E[:, None] / E, ref["gR"]),
                gx0=_columns(_np(out["gx0"]) * D, ref["gx0"], True))


def _hold(case, got, one, floor=(1e-6, 2e-6)):
    print(case, {k: "%.1e %.1e (%.1e %.1e)" % (got[k] + one[k]) for k in got})
    for k in got:
        assert got[k][0] <= max(2 * one[k][0], floor[0]) and got[k][1] <= max(8 * one[k][1], floor[1]), (case, k)


def _tv(d):
    b = synth.make_tv_batch(N, d, d, 5, seed=23, device=DEV)
    g = torch.randn((N, d), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV)
    return (b.A, b.B, b.Q, b.R, b.x0), g


@functools.lru_cache(None)
def _tv_ref(d):
    p, g = _tv(d)
    p64 = tuple(_np(t) for t in p)
    return lqr_oracle.riccati_solve_tv(*p64), lqr_oracle.riccati_rollout_tv(*p64), lqr_grad_oracle.lqr_gradients_tv(*p64, _np(g))


def _tv_errors(d, kind):
    p, g = _tv(d)
    un = _Units(kind, d)
    q = un.problem(*p)
    first, roll, grad = _tv_ref(d)
    errs = _first_step_errors(binding.ttc_lqr_solve_tv(*q), first, un)
    errs.update(_rollout_errors(binding.ttc_lqr_rollout_tv(*q), roll[0], roll[1], un))
    E = torch.tensor(un.E, dtype=torch.float32, device=DEV)
    errs.update(_gradient_errors(binding.ttc_lqr_backward_tv(*q, (g / E).contiguous()), grad, un))
    return errs


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("kind", KINDS, ids=str)
def test_time_heterogeneous(d, kind):
    _hold((d, kind), _tv_errors(d, kind), _tv_errors(d, ONE))


def _dense(d, T, dtype, costs):
    b = synth.make_batch(N, d, d, T, seed=29, device=DEV, dtype=dtype)
    g = torch.randn((N, d), generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    Q, QT = b.Q.clone(), None
    if costs == "half":           # every second state costs nothing by itself
        Q[:, 1::2, :] = 0
        Q[:, :, 1::2] = 0
    elif costs == "terminal":     # and here none but the last does
        QT, Q = Q, torch.zeros_like(Q)
    elif costs == "cheap":        # handed to the recursion
        return (b.A, b.B, Q, (b.R * 2.0 ** -9).to(b.R.dtype), b.x0), QT, g
    elif costs == "light":        # one state in two costs next to nothing by itself
        s = torch.ones(d, device=DEV)
        s[1::2] = 2.0 ** -14
        Q = (Q * s[:, None] * s).to(Q.dtype)
    return (b.A, b.B, Q, b.R, b.x0), QT, g


@functools.lru_cache(None)
def _dense_ref(d, T, dtype, costs):
    p, QT, g = _dense(d, T, dtype, costs)
    A, B, Q, R, x0 = (_np(t) for t in p)
    QT = None if QT is None else _np(QT)
    return (lqr_oracle.riccati_solve(A, B, Q, R, QT, x0, T), lqr_oracle.riccati_rollout(A, B, Q, R, QT, x0, T),
            lqr_grad_oracle.lqr_gradients(A, B, Q, R, QT, x0, T, _np(g)))


def _dense_errors(d, T, dtype, costs, kind, calls):
    p, QT, g = _dense(d, T, dtype, costs)
    un = _Units(kind, d)
    A, B, Q, R, x0 = un.problem(*p)
    if QT is not None:
        QT = un.problem(p[0], p[1], QT, p[3], p[4])[2]
    first, roll, grad = _dense_ref(d, T, dtype, costs)
    errs = {}
    if "solve" in calls:
        errs.update(_first_step_errors(binding.ttc_lqr_solve(A, B, Q, R, QT, x0, T), first, un))
    if "rollout" in calls:
        errs.update(_rollout_errors(binding.ttc_lqr_rollout(A, B, Q, R, QT, x0, T), roll[0], roll[1], un))
    if "backward" in calls:
        E = torch.tensor(un.E, dtype=torch.float32, device=DEV)
        errs.update(_gradient_errors(binding.ttc_lqr_backward(A, B, Q, R, QT, x0, T, (g / E).contiguous()), grad, un))
    return errs


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("kind", KINDS, ids=str)
def test_rollout_and_backward(d, kind):
    args = (d, 4, "f32", "all")
    calls = ("rollout", "backward")
    _hold((d, kind), _dense_errors(*args, kind, calls), _dense_errors(*args, ONE, calls))


# T = 8, 16 and 21 are composed by squaring (8 and 16 never apply a power, 21 does); 21 with a Q_T of its own too
@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T,dtype,costs", [(8, "f32", "all"), (16, "bf16", "all"), (21, "f32", "all"), (16, "f32", "half"),
                                           (21, "f32", "terminal"), (16, "f32", "light"), (16, "f32", "cheap")])
@pytest.mark.parametrize("kind", KINDS, ids=str)
def test_squaring(d, T, dtype, costs, kind):
    args = (d, T, dtype, costs)
    A, B, Q, R, x0 = _dense(*args)[0]
    QT = _dense(*args)[1]
    assert binding.ttc_lqr_solve_squares(binding.make_problem(A, B, Q, R, QT, x0, T))
    _hold((args, kind), _dense_errors(*args, kind, ("solve",)), _dense_errors(*args, ONE, ("solve",)))


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("cond", [1e2, 1e4, 1e6])
def test_ill_conditioned_control_costs(d, cond):
    """R with eigenvalues from 1 to cond along directions of no coordinate: squaring has B R^{-1} B^T, by the inverse of R at d = 128 and a
    solve elsewhere, where the recursion solves with R + B^T P B.  Their errors grow alike, as the condition number."""
    T = 16
    p, _, _ = _dense(d, T, "f32", "all")
    U = torch.linalg.qr(torch.randn((N, d, d), generator=torch.Generator().manual_seed(1), dtype=torch.float64))[0]
    R = (U * torch.logspace(0, float(np.log10(cond)), d, dtype=torch.float64)) @ U.transpose(-1, -2)
    R = (0.5 * (R + R.transpose(-1, -2))).float().to(DEV)
    A, B, Q, _, x0 = p
    assert binding.ttc_lqr_solve_squares(binding.make_problem(A, B, Q, R, None, x0, T))
    ref = lqr_oracle.riccati_solve(*(_np(t) for t in (A, B, Q, R)), None, _np(x0), T)
    steps = [t[:, None].expand(N, T, d, d).contiguous() for t in (A, B, Q, R)]
    un = _Units(ONE, d)
    got = _first_step_errors(binding.ttc_lqr_solve(A, B, Q, R, None, x0, T), ref, un)
    rec = _first_step_errors(binding.ttc_lqr_solve_tv(*steps, x0), ref, un)
    _hold((d, cond), got, rec, (4e-6, 1e-5))  # (the floor: what squaring itself shows here, 1.6e-6, and its worst column)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
def test_states_that_reach_nothing(d):
    """States that neither cost anything nor move one that does (padding), in units of their own."""
    T, live = 16, d - 7
    p, _, _ = _dense(d, T, "f32", "all")
    A, B, Q, R, x0 = (t.clone() for t in p)
    A[:, :live, live:] = 0
    A[:, live:, :live] = 0
    Q[:, live:] = 0
    Q[:, :, live:] = 0
    A[:, live:, :] *= 2.0 ** 20
    A[:, :, live:] *= 2.0 ** -20
    B[:, live:] *= 2.0 ** 20
    out = binding.ttc_lqr_solve(A, B, Q, R, None, x0, T)
    ref = lqr_oracle.riccati_solve(*(_np(t) for t in (A, B, Q, R)), None, _np(x0), T)
    errs = dict(P0=_columns(_np(out["P0"]), ref["P0"]), K0=_columns(_np(out["K0"]), ref["K0"]),
                u0=_columns(_np(out["u0"]), ref["u0"], True))
    print(d, errs)
    assert int(out["info"].abs().max()) == 0
    one = _dense_errors(d, T, "f32", "all", ONE, ("solve",))
    _hold(d, errs, one)


@pytest.mark.gpu
def test_two_subsystems_of_unlike_weight():
    """A decoupled pair in every tile, the costs of one 2^-40 times those of the other: each is solved as if it were alone."""
    d, T = 64, 4
    b = synth.make_tv_batch(N, d, d, T, seed=31, device=DEV)
    own = torch.zeros(d, dtype=torch.bool, device=DEV)
    own[::2] = True
    same = (own[:, None] == own[None, :]).float()
    w = torch.where(own, 1.0, 2.0 ** -20)
    A, B = b.A * same, b.B * same
    Q, R = b.Q * same * w[:, None] * w, b.R * same * w[:, None] * w
    out = binding.ttc_lqr_solve_tv(A, B, Q, R, b.x0)
    ref = lqr_oracle.riccati_solve_tv(*(_np(t) for t in (A, B, b.Q * same, b.R * same, b.x0)))
    assert int(out["info"].abs().max()) == 0
    wn = w.double().cpu().numpy()
    errs = dict(P0=_columns(_np(out["P0"]) / wn[:, None] / wn, ref["P0"]), K0=_columns(_np(out["K0"]), ref["K0"]))
    print(errs)
    assert max(e[1] for e in errs.values()) <= 4e-6   # (columns of 32 terms; errors of a step are 5e-7 here)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
def test_columns_of_a_of_unlike_size(d):
    """States that the next step hardly depends on, some of them less than others: columns of K_0 and P_0 in proportion."""
    p, _ = _tv(d)
    c = 2.0 ** -np.random.default_rng(6).permutation(np.round(np.linspace(0, 24, d)))
    C = torch.tensor(c, dtype=torch.float32, device=DEV)
    A = p[0].clone()
    A[:, 0] *= C
    ref = lqr_oracle.riccati_solve_tv(*(_np(t) for t in (A,) + p[1:]))
    got = _first_step_errors(binding.ttc_lqr_solve_tv(A, *p[1:]), ref, _Units(ONE, d))
    # (all of a column of P_0 is a sum of d products here: 3 and 6 times sqrt(128) roundings)
    _hold(d, got, _tv_errors(d, ONE), (2e-6, 4e-6))
