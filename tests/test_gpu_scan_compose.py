"""Compositions at d = 16 from register to register, and those that leave for the pivoted solve (max |I + G1 H2| above 24, where
control is cheap), in the same call."""
import numpy as np
import pytest
import torch

from oracle import lqr_oracle
from paper_2603_09221_amd import binding, synth

DEV = "cuda:0"


def _first_round(b, R):
    """max |I + G1 H2| of the compositions of the first round, in float64."""
    A, B, Q, R = (t.double().cpu().numpy() for t in (b.A, b.B, b.Q, R))
    T = A.shape[1]
    G = B @ np.linalg.solve(0.5 * (R + np.swapaxes(R, -1, -2)), np.swapaxes(B, -1, -2))
    # element k is step k + 1: G of that step and the cost on the state it starts from, Q[k]; pairs (0, 1), (2, 3), ..
    first = np.arange(0, T - 1, 2)
    K = np.eye(16) + G[:, first + 1] @ Q[:, first + 1]
    return np.abs(K).reshape(K.shape[0], K.shape[1], -1).max(-1)


def _err(got, want):
    got, want = got.double().cpu().numpy(), want
    n = got.shape[0]
    return np.linalg.norm((got - want).reshape(n, -1), axis=1) / np.linalg.norm(want.reshape(n, -1), axis=1)


@pytest.mark.gpu
@pytest.mark.parametrize("n,T", [(1, 2), (3, 3), (5, 64), (2, 129), (40, 200)])
@pytest.mark.parametrize("cheap", [1.0, 1e-1, 1e-2])
def test_both_solves_of_a_composition(n, T, cheap):
    b = synth.make_tv_batch(n, 16, 16, T, seed=T, device=DEV)
    R = b.R.clone()
    R[::2] *= cheap          # every second problem
    if T > 4:
        R[:, T // 2] *= cheap  # and one step of all
    out = binding.ttc_lqr_solve_tv_scan(b.A, b.B, b.Q, R, b.x0)
    seq = binding.ttc_lqr_solve_tv(b.A, b.B, b.Q, R, b.x0)
    torch.cuda.synchronize()
    if cheap == 1e-2 and n > 1:  # both ways are taken in this call (a composition of the first round is over 24, or well below)
        mu = _first_round(b, R)
        print("max |I + G1 H2|", mu.min(), mu.max())
        assert mu.max() > 48 and mu.min() < 12
    ref = lqr_oracle.riccati_solve_tv(*(t.double().cpu().numpy() for t in (b.A, b.B, b.Q, R, b.x0)))
    assert int(out["info"].abs().max()) == 0
    for k in ("P0", "K0", "u0"):
        # 2e-6 is what ordinary problems show; cheap control costs a composition up to a digit in the pair (G, H), whose size is the
        # cost ratio: a hundred roundings of 6e-8 at a ratio of 100
        bound = max(2e-6 + 6e-8 / cheap * 2, 4 * _err(seq[k], ref[k]).max())
        e = _err(out[k], ref[k]).max()
        print(n, T, cheap, k, e, bound)
        assert e <= bound


@pytest.mark.gpu
def test_an_indefinite_stage_cost_leaves_for_the_pivoted_solve():
    """I + G1 H2 then has pivots below 1/4 or of either sign; elimination in order is not used."""
    n, T = 6, 9
    b = synth.make_tv_batch(n, 16, 16, T, seed=3, device=DEV)
    Q = b.Q.clone()
    Q[1::2, 2:5] -= 0.6 * torch.eye(16, device=DEV)
    out = binding.ttc_lqr_solve_tv_scan(b.A, b.B, Q, b.R, b.x0)
    torch.cuda.synchronize()
    ref = lqr_oracle.riccati_solve_tv(*(t.double().cpu().numpy() for t in (b.A, b.B, Q, b.R, b.x0)))
    assert int(out["info"].abs().max()) == 0
    # the elements are pivoted solves of I + G1 H2, whose condition number the indefinite costs raise: its roundings, 6e-8 each, that often,
    # in every one of the four rounds and both products of the solution
    A, B, Qn, R = (t.double().cpu().numpy() for t in (b.A, b.B, Q, b.R))
    G = B @ np.linalg.solve(0.5 * (R + np.swapaxes(R, -1, -2)), np.swapaxes(B, -1, -2))
    H = 0.5 * (Qn + np.swapaxes(Qn, -1, -2))
    cond = max(np.linalg.cond(np.eye(16) + G[:, s] @ H[:, s]).max() for s in range(T))
    e = _err(out["P0"], ref["P0"]).max()
    print("indefinite", cond, e)
    assert e <= max(2e-6, 8 * 6e-8 * cond)
