"""The solvers' setup: masks that are 0 / 1 in some 64-pixel blocks only (one
graded entry at a block's edge), with theta^(0) from the measurement or from
X_init, in a context that solved with other masks before; against the formula
in float64.

lambda = 0 makes the denoiser the identity, so two GAP or ADMM iterations are
two projections. Tolerance: every value passes through two sums of at most B
terms of magnitude <= 1 in float32, a division by S >= 0.25 and two fused
multiply-adds, each exact to 2^-24 of its operands' sum.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("init", [False, True])
@pytest.mark.parametrize("solver", ["gap", "admm", "noalloc"])
@pytest.mark.parametrize("pixel", [0, 63, 64, 127, 128, -1])
@pytest.mark.parametrize("B", [1, 8, 31, 32, 33])
def test_setup_blocks(B, pixel, solver, init):
    from paper_2005_08028_amd import scitv

    nx, ny = 13, 15  # 195 pixels: three blocks and three pixels
    rng = np.random.default_rng(100 * B + pixel)
    plain = (rng.uniform(size=(B, nx, ny)) < 0.6).astype(np.float32)
    C = plain.copy()
    C.reshape(B, -1)[rng.integers(B), pixel] = 0.75
    Y = (C * rng.uniform(size=(B, nx, ny))).sum(0).astype(np.float32)
    X0 = rng.uniform(size=(B, nx, ny)).astype(np.float32) if init else None
    rho = 0.25 if solver == "admm" else 0.0
    c, y = C.astype(np.float64), Y.astype(np.float64)
    S = (c * c).sum(0) + rho
    W = np.where(S > 0, 1.0 / np.where(S > 0, S, 1.0), 0.0)
    x = X0.astype(np.float64) if init else c * y
    for _ in range(2):  # u stays 0: theta = s = u + x
        x = x + c * ((y - (c * x).sum(0)) * W)

    ctx = scitv.Context(0)
    fn = {"gap": scitv.sci_gap_tv, "admm": scitv.sci_admm_tv, "noalloc": scitv.sci_gap_tv_noalloc}[solver]
    prm = scitv.solver_params(outer_iters=2, rho=rho, lam=0.0, n_inner=1)
    y_t = torch.from_numpy(Y).cuda()
    out = [torch.empty(B, nx, ny, device="cuda") for _ in range(2)]
    for masks in (plain, C):
        fn(ctx.handle, y_t, torch.from_numpy(masks).cuda(), prm, *out,
           X_init=None if X0 is None else torch.from_numpy(X0).cuda())
    got = out[0].cpu().numpy().astype(np.float64)
    ctx.close()
    scale = max(1.0, np.abs(c * y).max()) * max(1.0, W.max()) * B
    assert np.abs(got - x).max() <= 4 * (B + 4) * 2.0 ** -24 * scale
