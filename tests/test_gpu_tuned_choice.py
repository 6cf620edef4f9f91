"""A choice that the context kept from an untuned call gives way to the one that
sci_autotune finds for the same parameters: the call then launches what an
explicit request for the tuned shape and pass count launches."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_cold_16bit_shape import launches  # noqa: E402


@pytest.mark.parametrize("dual", ["f32", "bf16"])
@pytest.mark.parametrize("B,nx,ny,n", [(3, 70, 130, 7), (2, 200, 90, 12), (8, 256, 256, 7), (12, 300, 520, 12)])
def test_tuned_choice_replaces_a_kept_one(B, nx, ny, n, dual):
    from paper_2005_08028_amd import scitv

    X = torch.rand((B, nx, ny), device="cuda")
    T = torch.empty_like(X)
    ctx = scitv.Context(0)

    def runs(**kw):
        prm = scitv.tv_params(tv="itv2d", lam=0.1, n_inner=n, dual_dtype=dual, **kw)
        call = lambda s=None: scitv.sci_tv_denoise(ctx.handle, X, prm, Theta_out=T, stream=s)  # noqa: E731
        call()
        return launches(scitv.lib, call)

    runs()  # kept
    shape, passes, _ = scitv.sci_autotune(ctx.handle, X, scitv.tv_params(tv="itv2d", lam=0.1, n_inner=n, dual_dtype=dual))
    assert runs() == runs(tile_shape=shape, tile_passes=passes)
    ctx.close()
