"""The register-to-register recursion at d = 16 (one problem per wavefront, or four) and the backward kernel built on it, at
the sizes where they can go wrong: horizons of one to five steps (the steps are taken in pairs and their reads run two
steps ahead), batches on both sides of the crossover and beyond one pass of the persistent grid, bfloat16 inputs, shared
and strided matrices."""
import pytest
import torch

from oracle import lqr_grad_oracle as go
from oracle import lqr_oracle
from paper_2603_09221_amd import binding, synth
from tests.parity import SOLVE_KEYS, max_errors, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_and_four_problems_per_wavefront_agree_bit_for_bit(T, dtype):
    """Both shapes apply the same operations to every entry.  12301 problems go four to a wavefront with a ragged last
    quad, their first 77 one to a wavefront; those also against the oracle on the stored values (float32 recursion: 2e-5)."""
    b = synth.make_tv_batch(12301, 16, 16, T, seed=T, device=DEV, dtype=dtype)
    few = b.take(slice(0, 77))
    four = binding.ttc_lqr_solve_tv(b.A, b.B, b.Q, b.R, b.x0)
    one = binding.ttc_lqr_solve_tv(few.A, few.B, few.Q, few.R, few.x0)
    torch.cuda.synchronize()
    assert int(four["info"].abs().max()) == 0
    for k in SOLVE_KEYS:
        assert torch.equal(four[k][:77], one[k]), k
    A, B, Q, R, x0 = few.numpy64()
    for k, v in max_errors(one, lqr_oracle.riccati_solve_tv(A, B, Q, R, x0)).items():
        assert v <= 2e-5, (k, v)


@pytest.mark.parametrize("T", [1, 3, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_over_several_passes_of_the_grid(T, dtype):
    """5003 problems: more than the resident workgroups, so that workspace slots are used again; a sample against the
    oracle on the stored values.  Tolerance as for the other sizes (2e-5: two float32 trajectories)."""
    n = 5003
    b = synth.make_tv_batch(n, 16, 16, T, seed=10 + T, device=DEV, dtype=dtype)
    g = torch.randn((n, 16), generator=torch.Generator().manual_seed(T)).to(DEV)
    out = binding.ttc_lqr_backward_tv(b.A, b.B, b.Q, b.R, b.x0, g)
    torch.cuda.synchronize()
    assert int(out["info"].abs().max()) == 0
    pick = torch.tensor([0, 1, 2047, 4095, 4096, 5002], device=DEV)
    ref = go.lqr_gradients_tv(*b.take(pick).numpy64(), g[pick].cpu().double().numpy())
    for k in ("gA", "gB", "gQ", "gR", "gx0"):
        got = out[k][pick].cpu().numpy().reshape(len(pick), -1)
        assert float(rel_err(got, ref[k].reshape(len(pick), -1)).max()) <= 2e-5, k


def test_backward_with_shared_matrices_and_a_terminal_cost_of_its_own():
    n, T = 33, 5
    b = synth.make_batch(n, 16, 16, T, seed=3, device=DEV)
    QT = (1.5 * b.Q + 0.2 * torch.eye(16, device=DEV)).contiguous()
    g = torch.randn((n, 16), generator=torch.Generator().manual_seed(8)).to(DEV)
    A0 = b.A[:1].expand(n, -1, -1)
    out = binding.ttc_lqr_backward(A0, b.B, b.Q, b.R, QT, b.x0, T, g)
    torch.cuda.synchronize()
    assert int(out["info"].abs().max()) == 0
    _, B, Q, R, x0 = b.numpy64()
    ref = go.lqr_gradients(A0.cpu().double().numpy(), B, Q, R, QT.cpu().double().numpy(), x0, T, g.cpu().double().numpy())
    for k in ("gA", "gB", "gQ", "gR", "gQT", "gx0"):
        assert float(rel_err(out[k].cpu().numpy().reshape(n, -1), ref[k].reshape(n, -1)).max()) <= 2e-5, k


def test_a_breakdown_stays_with_its_problem():
    """R of one step not positive definite: that problem reports the step and is NaN, its neighbours in the wavefront not."""
    n, T = 6200, 4
    b = synth.make_tv_batch(n, 16, 16, T, seed=5, device=DEV)
    R = b.R.clone()
    R[1234, 2] = -R[1234, 2] * 1e3
    for m in (n, 1300):
        out = binding.ttc_lqr_solve_tv(b.A[:m], b.B[:m], b.Q[:m], R[:m], b.x0[:m])
        bw = binding.ttc_lqr_backward_tv(b.A[:m], b.B[:m], b.Q[:m], R[:m], b.x0[:m], torch.ones((m, 16), device=DEV))
        torch.cuda.synchronize()
        for o, key in ((out, "u0"), (bw, "gA")):
            assert int(o["info"][1234]) == T - 2 and int((o["info"] != 0).sum()) == 1
            bad = torch.isnan(o[key].reshape(m, -1)).any(1)
            assert bool(bad[1234]) and int(bad.sum()) == 1
