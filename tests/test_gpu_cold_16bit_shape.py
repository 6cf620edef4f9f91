"""A cold one-pass call that keeps no dual stores none, so with 16-bit storage
it launches what the float32 call launches, the chosen shape included: the
captured kernel nodes of the two calls are the same, and so are the bits."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class NodeParams(ctypes.Structure):
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def launches(lib, call):
    """(kernel, grid, block) of everything call(stream) launches."""
    s = torch.cuda.Stream()
    handle, graph, n = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
    torch.cuda.synchronize()
    assert lib.hipStreamBeginCapture(handle, ctypes.c_int(1)) == 0  # thread-local
    try:
        call(s)
    finally:
        assert lib.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert lib.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for k in range(n.value):
        p = NodeParams()
        assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(nodes[k]), ctypes.byref(p)) == 0
        out.append((p.func, p.grid.x, p.block.x))
    assert lib.hipGraphDestroy(graph) == 0
    return out


@pytest.mark.parametrize("dual", ["bf16", "f16"])
@pytest.mark.parametrize("tv", ["atv", "itv2d"])
@pytest.mark.parametrize("nx,ny,B,n,shape", [(640, 480, 4, 5, 0), (740, 1041, 10, 10, 0), (33, 70, 2, 5, 0),
                                             (200, 130, 3, 4, 8), (200, 130, 3, 10, 16)])
def test_cold_call_runs_the_float32_kernel(tv, dual, nx, ny, B, n, shape):
    from paper_2005_08028_amd import scitv

    X = torch.rand((B, nx, ny), device="cuda")
    got = {}
    ctx = scitv.Context(0)
    for dt in ("f32", dual):
        prm = scitv.tv_params(tv=tv, lam=0.07, n_inner=n, dual_dtype=dt, schedule="fused", tile_shape=shape,
                              tile_passes=1)
        T = torch.empty_like(X)
        run = lambda s=None: scitv.sci_tv_denoise(ctx.handle, X, prm, Theta_out=T, stream=s)  # noqa: B023
        run()
        torch.cuda.synchronize()
        bits = T.clone()
        got[dt] = (launches(scitv.lib, run), bits)
    ctx.close()
    assert len(got["f32"][0]) == 1
    assert got[dual][0] == got["f32"][0]
    assert torch.equal(got[dual][1], got["f32"][1])
