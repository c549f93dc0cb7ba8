"""GPU parity of narrow rotations (pv_block_rotate with few columns) on both
sides of the rule that chooses one thread per entry, against numpy in FP64.

Tolerance, elementwise with |X|, |Q| the absolute values: a complex entry sums
2 nx products per part, each sum off by at most (2 nx + 2) eps times the sum of
the products' absolute values, and the joins add three roundings (factor 2 for
the two parts); a complex64 result adds its own rounding."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402

from gpu_common import dev, host  # noqa: E402

EPS = np.finfo(np.float64).eps


def block(rows, n, dtype, seed):
    g = np.random.default_rng(seed)
    return (g.standard_normal((rows, n)) + 1j * g.standard_normal((rows, n))).astype(dtype)


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("rows,nx,ny", [(1, 2, 1), (255, 1, 1), (257, 1, 64), (3001, 7, 5), (18750, 8, 8), (18751, 8, 8),
                                        (62500, 24, 2), (62501, 24, 2), (40001, 20, 4), (150001, 8, 1), (2100001, 1, 1),
                                        (700001, 4, 4)])
def test_narrow_rotation(rows, nx, ny, dtype, accumulate):
    X, Y0 = block(rows, nx, dtype, 13), block(rows, ny, dtype, 14)
    Q = block(nx, ny, np.complex128, 15)
    Y = dev(Y0)
    pv.pv_block_rotate(dev(X), dev(Q), Y, accumulate=accumulate)
    X, Y0 = X.astype(np.complex128), Y0.astype(np.complex128)
    ref, size = X @ Q, np.abs(X) @ np.abs(Q)
    if accumulate:
        ref, size = ref + Y0, size + np.abs(Y0)
    bound = 2 * (2 * nx + 5) * EPS * size
    if dtype == np.complex64:
        bound = bound + np.finfo(np.float32).eps * size
    assert (np.abs(host(Y) - ref) <= bound).all()
