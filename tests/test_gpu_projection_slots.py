"""GAP / ADMM projection at the edges of its frame slots (even slot counts up to
32, the loop over frames beyond) and of its 64-pixel workgroups, with binary
(packed) and graded masks, against the formula in float64.

lambda = 0 makes the denoiser the identity, so two GAP iterations are two
projections. Tolerance: every value passes through two sums of at most B terms
of magnitude <= 1 in float32, a division by S >= 0.25 and two fused
multiply-adds, each exact to 2^-24 of its operands' sum.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver", ["gap", "admm"])
@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("nx,ny", [(1, 1), (7, 9), (8, 8), (5, 13), (33, 31)])
@pytest.mark.parametrize("B", [1, 2, 3, 9, 10, 31, 32, 33])
def test_projection_slots(B, nx, ny, graded, solver):
    from paper_2005_08028_amd import scitv

    rng = np.random.default_rng(1000 * B + nx)
    C = rng.uniform(0.5, 1.0, (B, nx, ny)) if graded else (rng.uniform(size=(B, nx, ny)) < 0.6).astype(float)
    C = C.astype(np.float32)
    Y = (C * rng.uniform(size=(B, nx, ny))).sum(0).astype(np.float32)
    rho = 0.25
    c, y = C.astype(np.float64), Y.astype(np.float64)
    S = (c * c).sum(0) + (rho if solver == "admm" else 0.0)
    W = np.where(S > 0, 1.0 / np.where(S > 0, S, 1.0), 0.0)
    x = c * y
    for _ in range(2):  # u stays 0: theta = s = u + x
        x = x + c * ((y - (c * x).sum(0)) * W)
    ctx = scitv.Context(0)
    fn = scitv.sci_gap_tv if solver == "gap" else scitv.sci_admm_tv
    prm = scitv.solver_params(outer_iters=2, rho=rho if solver == "admm" else 0.0, lam=0.0, n_inner=1)
    got, _ = fn(ctx.handle, torch.from_numpy(Y).cuda(), torch.from_numpy(C).cuda(), prm)
    got = got.cpu().numpy().astype(np.float64)
    ctx.close()
    scale = max(1.0, np.abs(c * y).max()) * max(1.0, W.max()) * B
    assert np.abs(got - x).max() <= 4 * (B + 4) * 2.0 ** -24 * scale
