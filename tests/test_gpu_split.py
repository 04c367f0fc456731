"""Products on the float16 matrix cores from operands split into two terms (ttc_split.hpp): the recursion that runs on them, with
dynamics on either side of the identity that is taken out of A, entries of very different size and costs far from one."""
import numpy as np
import pytest
import torch

from oracle import lqr_oracle
from paper_2603_09221_amd import binding, synth

DEV = "cuda:0"

# A dot product of d terms in float32 is off by about sqrt(d) * 2^-24 = 7e-7 at d = 128; a step chains a handful of them and one
# solve, whose condition number is below ten on these inputs.
TOL = 5e-6


def _dynamics(kind, A, gen):
    n, d = A.shape[0], A.shape[-1]
    N = torch.randn((n, 1, d, d), generator=gen, device=DEV) / d ** 0.5
    if kind == "minus":      # near -I
        return -A
    if kind == "mixed":      # diagonal entries of either sign
        s = torch.ones(d, device=DEV)
        s[1::2] = -1.0
        return A * s[None, None, None, :]
    if kind == "dense":      # no diagonal to speak of
        return (0.9 * N).expand_as(A).contiguous()
    if kind == "graded":     # columns from 1 down to 2^-20: most of a column far below the largest entry
        return A * torch.exp2(-torch.linspace(0, 20, d, device=DEV))[None, None, None, :]
    return A


@pytest.mark.gpu
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("kind,scale", [("plain", 0), ("minus", 0), ("mixed", 0), ("dense", 0), ("graded", 0), ("plain", 40),
                                        ("plain", -40)])
def test_recursion_on_split_products(d, kind, scale):
    n, T = 5, 4
    b = synth.make_tv_batch(n, d, d, T, seed=17, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(5)
    A = _dynamics(kind, b.A, gen)
    Q, R = b.Q * 2.0 ** scale, b.R * 2.0 ** scale
    out = binding.ttc_lqr_solve_tv(A, b.B, Q, R, b.x0)
    torch.cuda.synchronize()
    ref = lqr_oracle.riccati_solve_tv(*(t.double().cpu().numpy() for t in (A, b.B, Q, R, b.x0)))
    assert int(out["info"].abs().max()) == 0
    for k in ("P0", "K0", "u0", "value"):
        got, want = out[k].double().cpu().numpy().reshape(n, -1), ref[k].reshape(n, -1)
        err = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
        print(d, kind, scale, k, err.max())
        assert err.max() <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_what_is_not_finite_stays_so(bad):
    n, d, T = 3, 64, 3
    b = synth.make_tv_batch(n, d, d, T, seed=18, device=DEV)
    good = binding.ttc_lqr_solve_tv(b.A, b.B, b.Q, b.R, b.x0)
    A = b.A.clone()
    A[1, 1, 3, 5] = bad
    out = binding.ttc_lqr_solve_tv(A, b.B, b.Q, b.R, b.x0)
    torch.cuda.synchronize()
    assert not torch.isfinite(out["u0"][1]).any()
    for q in (0, 2):
        assert torch.equal(out["u0"][q], good["u0"][q]) and int(out["info"][q]) == 0
