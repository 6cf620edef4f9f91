"""The untuned choice of tile shape and pass count: whatever it picks, float32
calls return the bits of one streaming pass per iteration; 16-bit calls keep
the split of passes their rounding depends on (about five iterations each); a
batch that changes shape as its problems finish returns the bits of lone
solves."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2005_08028_amd import scitv
    c = scitv.Context(0)
    yield c.handle
    c.close()


def call(ctx, X, P, **kw):
    from paper_2005_08028_amd import scitv
    prm = scitv.tv_params(lam=0.09, **kw)
    D = torch.full((2,) + tuple(X.shape), 9.0, device="cuda", dtype=scitv.DUAL_TORCH[prm.dual_dtype])
    th, _, _, _ = scitv.sci_tv_denoise(ctx, X, prm, dual_init=P, dual_out=D)
    cold, _, _, _ = scitv.sci_tv_denoise(ctx, X, prm)
    return th, D, cold


def inputs(nx, ny, B, warm, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(nx + 7 * ny + 31 * B)
    X = torch.rand((B, nx, ny), device="cuda", generator=g)
    P = (0.4 * torch.randn((2, B, nx, ny), device="cuda", generator=g)).to(dtype) if warm else None
    return X, P


# one size for each region of the rule: few tiles, one to several rounds of
# each kind of tile, row segments that fill the chip once and several times
@pytest.mark.parametrize("nx,ny,B", [(1, 1, 1), (40, 33, 2), (128, 130, 8), (256, 256, 8), (300, 277, 16),
                                     (517, 389, 10), (700, 300, 24), (1024, 500, 16)])
@pytest.mark.parametrize("tv,n,accel", [("itv2d", 1, True), ("atv", 5, True), ("itv2d", 10, True), ("atv", 14, False),
                                        ("itv2d", 23, True)])
@pytest.mark.parametrize("warm", [False, True])
def test_float32_default_equals_streaming(ctx, nx, ny, B, tv, n, accel, warm):
    X, P = inputs(nx, ny, B, warm)
    a = call(ctx, X, P, tv=tv, n_inner=n, accel=accel)
    b = call(ctx, X, P, tv=tv, n_inner=n, accel=accel, schedule="stream")
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("nx,ny,B", [(40, 33, 2), (300, 277, 16)])
@pytest.mark.parametrize("n", [3, 10, 14])
def test_16bit_default_keeps_its_passes(ctx, dtype, nx, ny, B, n):
    X, P = inputs(nx, ny, B, True, torch.bfloat16 if dtype == "bf16" else torch.float16)
    a = call(ctx, X, P, tv="itv2d", n_inner=n, dual_dtype=dtype)
    b = call(ctx, X, P, tv="itv2d", n_inner=n, dual_dtype=dtype, schedule="fused", tile_shape=1, tile_passes=(n + 4) // 5)
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("tv,n", [("atv", 5), ("itv2d", 8)])
def test_uneven_batch_equals_lone_solves(ctx, tv, n, graph):
    from paper_2005_08028_amd import scitv

    g = torch.Generator(device="cuda").manual_seed(5)
    items, lone = [], []
    for nx, ny, B, T in [(900, 700, 8, 2), (64, 70, 8, 9), (256, 200, 3, 5), (512, 512, 10, 3), (31, 300, 1, 7)]:
        C = (torch.rand((B, nx, ny), device="cuda", generator=g) < 0.5).float()
        Y = (C * torch.rand((B, nx, ny), device="cuda", generator=g)).sum(0)
        items.append(dict(Y=Y, C=C, X_out=torch.empty_like(C), outer_iters=T))
        prm = scitv.solver_params(outer_iters=T, tv=tv, lam=0.1, n_inner=n)
        lone.append(scitv.sci_gap_tv(ctx, Y, C, prm)[0])
    prm = scitv.solver_params(outer_iters=4, tv=tv, lam=0.1, n_inner=n, use_graph=graph)
    for _ in range(2):
        for it in items:
            it["X_out"].fill_(-1.0)
        scitv.sci_gap_tv_batched(ctx, items, prm)
        for it, x in zip(items, lone):
            assert torch.equal(it["X_out"], x)
