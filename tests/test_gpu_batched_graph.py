"""Replayed batched graphs hold the weight and the iteration counts they were
captured with: calls on the same buffers that differ in these alone each give
the bits of their own lone solves."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lams", [(1e-7, 4e-7), (0.1234561, 0.1234564)])
def test_graph_per_weight(lams):
    from paper_2005_08028_amd import scitv

    g = torch.Generator(device="cuda").manual_seed(3)
    C = (torch.rand((4, 40, 70), device="cuda", generator=g) > 0.5).float()
    Y = 2 * torch.rand((40, 70), device="cuda", generator=g)
    X = torch.empty_like(C)
    ctx = scitv.Context(0)
    lone = []
    for lam in lams * 2:
        prm = scitv.solver_params(outer_iters=4, tv="itv2d", lam=lam, n_inner=5, use_graph=True)
        scitv.sci_gap_tv_batched(ctx.handle, [dict(Y=Y, C=C, X_out=X)], prm)
        one = scitv.solver_params(outer_iters=4, tv="itv2d", lam=lam, n_inner=5, schedule="fused")
        lone.append(scitv.sci_gap_tv(ctx.handle, Y, C, one)[0])
        assert torch.equal(X, lone[-1]), lam
    assert not torch.equal(lone[0], lone[1])
    ctx.close()


def test_graph_per_iteration_count():
    from paper_2005_08028_amd import scitv

    g = torch.Generator(device="cuda").manual_seed(4)
    C = (torch.rand((3, 30, 50), device="cuda", generator=g) > 0.5).float()
    Y = 2 * torch.rand((30, 50), device="cuda", generator=g)
    X, T = torch.empty_like(C), torch.empty_like(C)
    ctx = scitv.Context(0)
    lone = []
    for its in (100, 101, 109, 100):
        prm = scitv.solver_params(outer_iters=5, tv="atv", lam=0.1, n_inner=3, use_graph=True)
        scitv.sci_gap_tv_batched(ctx.handle, [dict(Y=Y, C=C, X_out=X, Theta_out=T, outer_iters=its)], prm)
        one = scitv.solver_params(outer_iters=its, tv="atv", lam=0.1, n_inner=3, schedule="fused")
        lone.append(scitv.sci_gap_tv(ctx.handle, Y, C, one)[0])
        assert torch.equal(X, lone[-1]), its
    assert not torch.equal(lone[0], lone[1])
    ctx.close()
