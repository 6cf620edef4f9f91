"""Row-pipelined denoiser passes at the edges of their strips, segments and
frame groups, against one streaming pass per iteration: the two evaluate the
same expressions in the same order, so with float32 duals every output agrees
bit for bit. Starting duals carry values in the entries that hold no
difference, which a pass must ignore (and return as 0)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def both(tv, nx, ny, B, n, warm, shape, accel=True):
    from paper_2005_08028_amd import scitv

    g = torch.Generator(device="cuda").manual_seed(7 * nx + ny + 1000 * B)
    X = torch.rand((B, nx, ny), device="cuda", generator=g)
    P = 0.4 * torch.randn((2, B, nx, ny), device="cuda", generator=g) if warm else None
    ctx = scitv.Context(0)
    out = []
    for schedule in ("stream", "fused"):
        kw = dict(tile_shape=shape, tile_passes=1) if schedule == "fused" else {}
        prm = scitv.tv_params(tv=tv, lam=0.07, n_inner=n, accel=accel, schedule=schedule, **kw)
        D = torch.full((2, B, nx, ny), 9.0, device="cuda")
        th, _, _, _ = scitv.sci_tv_denoise(ctx.handle, X, prm, dual_init=P, dual_out=D)
        out += [th, D]
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(out[0], out[2])
    assert torch.equal(out[1], out[3])
    assert not out[3][0, :, :, -1].any() and not out[3][1, :, -1, :].any()


@pytest.mark.parametrize("tv", ["atv", "itv2d"])
@pytest.mark.parametrize("n", [1, 2, 5, 10])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 107), (33, 108), (31, 117), (32, 128), (40, 129), (65, 215), (70, 3)])
@pytest.mark.parametrize("warm", [False, True])
def test_rows_edges(tv, n, nx, ny, warm):
    from paper_2005_08028_amd import scitv

    shape = next(k for k in range(1, scitv.sci_tile_shape_count() + 1) if scitv.sci_tile_shape_pipelined(k))
    both(tv, nx, ny, 2, n, warm, shape)


@pytest.mark.parametrize("B", [1, 8, 9, 10, 11, 17, 23, 25])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 53), (9, 54), (30, 64), (25, 65), (64, 3)])
@pytest.mark.parametrize("warm", [False, True])
def test_vtv_edges(B, nx, ny, warm):
    both("vtv", nx, ny, B, 4, warm, 0)
    both("vtv", nx, ny, B, 6, warm, 0, accel=False)
