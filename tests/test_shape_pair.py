"""The pair of tile shapes of an uneven batch, weighed on the host: the smallest
total over all pairs, and a second shape only where it lowers the total (every
active count alike: one shape)."""
import ctypes
import itertools

import numpy as np
import pytest

torch = pytest.importorskip("torch")


def _pick(cost, launches):
    from paper_2005_08028_amd import scitv

    f = scitv.lib["_ZN3sci15pick_shape_pairEiiPKdS1_Pi"]
    D = ctypes.POINTER(ctypes.c_double)
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int, D, D, ctypes.POINTER(ctypes.c_int)]
    cost, launches = np.ascontiguousarray(cost, float), np.ascontiguousarray(launches, float)
    shape = (ctypes.c_int * 2)()
    n = f(*cost.shape, cost.ctypes.data_as(D), launches.ctypes.data_as(D), shape)
    return n, tuple(shape)


@pytest.mark.parametrize("ns,nc", [(1, 1), (2, 3), (16, 1), (16, 12), (5, 40)])
def test_smallest_total(ns, nc):
    rng = np.random.default_rng(ns * 100 + nc)
    for _ in range(20):
        cost, launches = rng.integers(1, 12, (ns, nc)).astype(float), rng.integers(1, 9, nc).astype(float)
        n, (a, b) = _pick(cost, launches)
        total = lambda a, b: float((launches * np.minimum(cost[a], cost[b])).sum())  # noqa: E731
        assert total(a, b) == min(total(i, j) for i, j in itertools.product(range(ns), repeat=2))
        single = min(total(i, i) for i in range(ns))
        assert n == (2 if total(a, b) < single else 1) and (a == b) == (n == 1)


def test_one_best_shape_needs_no_second():
    cost = np.array([[3.0, 5.0], [2.0, 4.0], [1.0, 3.0], [2.0, 9.0]])
    assert _pick(cost, [7, 1]) == (1, (2, 2))
    assert _pick(np.array([[4.0], [2.0], [2.0]]), [3]) == (1, (1, 1))
    assert _pick(np.array([[1.0, 9.0], [9.0, 1.0], [4.0, 4.0]]), [1, 1]) == (2, (0, 1))
