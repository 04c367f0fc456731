"""Default path of ttc_lqr_solve at d = 16: the equal factors composed by squaring, one problem to a wavefront or four, with its ways out
(cheap control, an unstable open loop, costs that are not semidefinite, breakdowns)."""
import numpy as np
import pytest
import torch

from paper_2603_09221_amd import binding, synth
from tests.parity import SOLVE_KEYS, oracle_solve, solve_errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 16
SMALL, LARGE = (1, 2, 7), (3073, 3075)  # one problem to a wavefront; four, with a ragged last quad


def solve(b, QT=None, **kw):
    out = binding.ttc_lqr_solve(b.A, b.B, b.Q, b.R, QT, b.x0, b.T, **kw)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n", SMALL + LARGE)
@pytest.mark.parametrize("T", [1, 2, 3, 4, 7, 8, 31, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_against_the_oracle(n, T, dtype):
    """2e-5 per problem, a fifth of the path's tolerance: a composition's error is a few float32 roundings times max |I + G H| (below 9 on
    these), over at most six of them; measured 4e-7 (T = 1) to 1.1e-5 (T = 31).  The oracle consumes rounded bfloat16 values.  Spectral radius
    0.98 at T = 64, about 1.1 else."""
    b = synth.make_batch(n, D, D, T, seed=T + n, device=DEV, dtype=dtype, rho=0.98 if T > 32 else None)
    QT = (1.5 * b.Q + 0.2 * torch.eye(D, device=DEV)).to(b.Q.dtype).contiguous()
    for qt, flag in ((None, False), (QT, True)):
        out = solve(b, QT=qt, flags=binding.TTC_FLAG_STAGE_COST_AT_X0 if flag else 0)
        assert int(out["info"].abs().max()) == 0
        for k, v in solve_errors(out, oracle_solve(b, QT=qt, flag=flag)).items():
            assert v <= 2e-5, (k, v)


@pytest.mark.parametrize("n", [5, 3073])
def test_forms_of_the_input(n):
    """Matrices shared by all problems, Q_T given as the very same array, outputs left out: bit for bit what the plain call gives."""
    b = synth.make_batch(n, D, D, 11, seed=2, device=DEV)
    shared = synth.LqrBatch(b.A[:1].expand(n, -1, -1), b.B, b.Q[:1].expand(n, -1, -1), b.R, b.x0, 11)
    full = synth.LqrBatch(shared.A.contiguous(), b.B, shared.Q.contiguous(), b.R, b.x0, 11)
    got, want = solve(shared), solve(full)
    again, less = solve(full, QT=full.Q), solve(full, want_P0=False, want_K0=False)
    for k in SOLVE_KEYS:
        assert torch.equal(got[k], want[k]) and torch.equal(again[k], want[k]), k
    assert torch.equal(less["u0"], want["u0"]) and torch.equal(less["value"], want["value"])


@pytest.mark.parametrize("n", [9, 3074])
@pytest.mark.parametrize("r,rho,qt,T", [(0.1, None, None, 9), (0.01, None, None, 33), (1.0, 1.3, None, 16), (1.0, 1.3, None, 64),
                                        (100.0, 1.2, None, 33), (1.0, None, 30.0, 17), (1.0, None, 1000.0, 17)])
def test_ways_out(n, r, rho, qt, T):
    """Cheap control and a large terminal cost go to the recursion, an unstable open loop applies a power more often and pivots: the path's
    1e-4 (measured 2e-6..5e-5)."""
    b = synth.make_batch(n, D, D, T, seed=T, device=DEV, r_scale=r, rho=rho)
    QT = None if qt is None else (qt * b.Q).contiguous()
    out = solve(b, QT=QT)
    assert int(out["info"].abs().max()) == 0
    for k, v in solve_errors(out, oracle_solve(b, QT=QT)).items():
        assert v <= 1e-4, (k, v)


@pytest.mark.parametrize("n", [13, 3073])
def test_what_squaring_cannot_do_is_what_the_product_gives(n):
    """A singular A, an R or a stage cost that is not (semi)definite, a NaN: reports and outputs of the sequential product (rebase_every asks
    for it in its default grouping), bit for bit; their neighbours are solved."""
    T = 5
    b = synth.make_batch(n, D, D, T, seed=4, device=DEV)
    A, Q, R = b.A.clone(), b.Q.clone(), b.R.clone()
    A[1, :, 3] = 0
    R[4] -= 3 * torch.eye(D, device=DEV)
    Q[8] -= 0.6 * torch.eye(D, device=DEV)
    A[11, 2, 2] = float("nan")
    out = binding.ttc_lqr_solve(A, b.B, Q, R, None, b.x0, T)
    seq = binding.ttc_lqr_solve(A, b.B, Q, R, None, b.x0, T, rebase_every=3)  # ceil(T / 3) groups, as by default
    torch.cuda.synchronize()
    assert torch.equal(out["info"], seq["info"])
    info = out["info"].cpu().numpy()
    assert info[1] == 2 and info[4] == 1 and info[11] != 0
    for k in SOLVE_KEYS:
        for p in (1, 4, 8, 11):
            assert torch.equal(out[k][p].nan_to_num(7.0), seq[k][p].nan_to_num(7.0)), (k, p)
    ref = oracle_solve(synth.LqrBatch(b.A, b.B, b.Q, b.R, b.x0, T))
    fine = np.array([p for p in range(n) if p not in (1, 4, 8, 11)])
    pick = lambda x: x[torch.as_tensor(fine, device=x.device)]
    for k, v in solve_errors({k: pick(out[k]) for k in SOLVE_KEYS}, {k: ref[k][fine] for k in SOLVE_KEYS}).items():
        assert v <= 1e-4, (k, v)


@pytest.mark.parametrize("n", [6, 3073])
def test_dense_dynamics(n):
    """An A nowhere near a diagonal matrix: whether it is singular is asked of a pivoted factorisation."""
    b = synth.make_batch(n, D, D, 12, seed=6, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    b = synth.LqrBatch(torch.randn(b.A.shape, device=DEV, generator=gen) * 0.25, b.B, b.Q, b.R, b.x0, 12)
    out = solve(b)
    assert int(out["info"].abs().max()) == 0
    for k, v in solve_errors(out, oracle_solve(b)).items():
        assert v <= 2e-5, (k, v)


def recursion64(A, B, Q, R, T):
    """P_0 and K_0 of the printed recursion in float64 with general solves (R + B^T P B need not be positive definite)."""
    t = lambda M: M.swapaxes(-1, -2)
    A, B, Q, R = (M.double().cpu().numpy() for M in (A, B, Q, R))
    Q, R = 0.5 * (Q + t(Q)), 0.5 * (R + t(R))
    P = Q
    for s in range(T - 1, -1, -1):
        F = t(B) @ P @ A
        K = -np.linalg.solve(R + t(B) @ P @ B, F)
        P = (Q if s else 0) + t(A) @ P @ A + t(F) @ K
        P = 0.5 * (P + t(P))
    return {"P0": P, "K0": K}


def indefinite(kind, n, T):
    """Stage costs with eigenvalues of about -0.2, or, with B and R near the identity, one of -1 under a positive diagonal."""
    b = synth.make_batch(n, D, D, T, seed=D + T, device=DEV)
    eye = torch.eye(D, device=DEV)
    if kind == "shifted":
        b.Q.sub_(0.2 * eye)
        return b
    gen = torch.Generator().manual_seed(n + T)
    turn = torch.linalg.qr(torch.randn((n, D, D), generator=gen, dtype=torch.float64))[0]
    Q = (torch.eye(D, dtype=torch.float64) - 2 * turn[:, :, :1] @ turn[:, :, :1].transpose(1, 2)).float().to(DEV)
    assert kind == "turned"
    keep = (Q.diagonal(dim1=1, dim2=2) > 0).all(1)
    Q[~keep] = eye
    return synth.LqrBatch(b.A, eye + 0.1 * b.B, Q, eye.repeat(n, 1, 1), b.x0, T)


@pytest.mark.parametrize("n", [400, 3300])
@pytest.mark.parametrize("kind,T", [("shifted", 4), ("shifted", 12), ("shifted", 15), ("shifted", 32), ("turned", 3), ("turned", 4),
                                    ("turned", 8)])
def test_a_stage_cost_that_is_not_semidefinite_is_answered_as_by_the_product(n, kind, T):
    """Squaring loses their digits where I + G H comes near a singular matrix, be it in a late squaring and under a positive diagonal; the
    sequential product, whose solves are pivoted, answers them.  What it answers is answered, and as well: problems near a singular
    R + B^T P B lose digits on either path, and there the errors of two float32 evaluations are independent draws, for which 10 is allowed.
    One problem may be beyond that: of the shifted ones, a float32 recursion with general solves is with 4 to 6 of 400, 14 to 47 of 3300."""
    b = indefinite(kind, n, T)
    out, seq = solve(b), solve(b, rebase_every=3)
    ref = recursion64(b.A, b.B, b.Q, b.R, T)
    answered = (seq["info"] == 0).cpu().numpy()
    assert answered.mean() >= 0.5
    assert not out["info"].cpu().numpy()[answered].any()
    rel = lambda o, k: np.linalg.norm(o[k].double().cpu().numpy() - ref[k], axis=(1, 2)) / np.linalg.norm(ref[k], axis=(1, 2))
    err, err_seq = (np.maximum(rel(o, "P0"), rel(o, "K0"))[answered] for o in (out, seq))
    print(kind, T, "median %.1e %.1e, largest %.1e %.1e" % (np.median(err), np.median(err_seq), err.max(), err_seq.max()))
    assert (err > np.maximum(1e-4, 10 * err_seq)).sum() <= 1


@pytest.mark.parametrize("n", [9, 3074])
@pytest.mark.parametrize("T", [4, 8, 17, 33])
@pytest.mark.parametrize("share", [0.0, 1e-3])
def test_a_terminal_cost_beside_a_small_running_cost_is_squared(n, T, share):
    """The guard is on I + P G, which such a terminal cost passes: 2e-5 as on ordinary problems, and not what the recursion gives bit for
    bit, which takes up to four times as long."""
    b = synth.make_batch(n, D, D, T, seed=T, device=DEV, rho=0.98)
    QT, b.Q = b.Q, share * b.Q
    out = solve(b, QT=QT)
    assert int(out["info"].abs().max()) == 0
    for k, v in solve_errors(out, oracle_solve(b, QT=QT)).items():
        assert v <= 2e-5, (k, v)
    steps = [m[:, None].expand(-1, T, -1, -1).contiguous() for m in (b.A, b.B, b.Q, b.R)]
    steps[2][:, T - 1] = QT
    tv = binding.ttc_lqr_solve_tv(*steps, b.x0)
    torch.cuda.synchronize()
    assert not (out["P0"] == tv["P0"]).flatten(1).all(1).any()


@pytest.mark.parametrize("n", [40, 3300])
@pytest.mark.parametrize("T", [2, 8, 9])
@pytest.mark.parametrize("qt,r", [(3.0, 1.0), (6.0, 1.0), (10.0, 1.0), (0.0, 0.1)])
def test_a_terminal_cost_is_applied_as_accurately_as_by_the_product(n, T, qt, r):
    """Q_T = 3 to 10 Q, and Q_T alone with a control a tenth as dear, where elimination of I + Q_T G in order meets small pivots: 2e-5 as on
    ordinary problems (2e-6..5e-6; without a search for pivots up to 8e-5)."""
    b = synth.make_batch(n, D, D, T, seed=1, device=DEV, r_scale=r)
    if qt:
        QT = (qt * b.Q).contiguous()
    else:
        QT, b.Q = b.Q, torch.zeros_like(b.Q)
    out = solve(b, QT=QT)
    assert int(out["info"].abs().max()) == 0
    t = lambda M: M.swapaxes(-1, -2)
    A, B, Q, R, P = (M.double().cpu().numpy() for M in (b.A, b.B, b.Q, b.R, QT))
    for s in range(T - 1, -1, -1):
        F = t(B) @ P @ A
        K = -np.linalg.solve(R + t(B) @ P @ B, F)
        P = (Q if s else 0) + t(A) @ P @ A + t(F) @ K
    rel = lambda x, y: (np.linalg.norm(x.double().cpu().numpy() - y, axis=(1, 2)) / np.linalg.norm(y, axis=(1, 2))).max()
    assert max(rel(out["P0"], P), rel(out["K0"], K)) <= 2e-5
