"""GPU parity of the tall-skinny products (pv_gram, pv_block_rotate) at the
edges of their tiles: 16-column instructions, 32-column waves, 64-column
workgroups, 8-row and 32-row steps, and every remainder beside them.

Tolerances, elementwise against numpy in FP64 with |X|, |Y|, |Q| the absolute
values: a sum of n products, in any order and with fused or rounded products,
is off by at most (n + 2) eps times the sum of the products' absolute values;
a complex entry sums 2 n of them per part (factor 2 for the two parts), and a
complex64 result adds its own rounding."""

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


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("rows,nx,ny", [(1, 1, 1), (3, 2, 5), (7, 16, 16), (8, 17, 1), (9, 1, 33), (31, 15, 32),
                                        (33, 32, 16), (257, 33, 31), (1000, 48, 64), (4099, 64, 64),
                                        (70001, 32, 32), (70003, 8, 64), (70004, 64, 3)])
def test_gram_edges(rows, nx, ny, dtype):
    X, Y = block(rows, nx, dtype, 1), block(rows, ny, dtype, 2)
    G = host(pv.pv_gram(dev(X), dev(Y)))
    X, Y = X.astype(np.complex128), Y.astype(np.complex128)
    bound = 2 * (2 * rows + 2) * EPS * (np.abs(X).T @ np.abs(Y))
    assert (np.abs(G - X.conj().T @ Y) <= bound).all()


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("rows,nx,ny", [(1, 1, 1), (5, 3, 2), (15, 16, 16), (17, 17, 33), (64, 4, 64), (65, 31, 15),
                                        (127, 64, 17), (1000, 32, 32), (4099, 33, 48), (70001, 32, 32),
                                        (70003, 64, 64), (70005, 20, 8)])
def test_rotate_edges(rows, nx, ny, dtype, accumulate):
    X, Y0 = block(rows, nx, dtype, 3), block(rows, ny, dtype, 4)
    Q = block(nx, ny, np.complex128, 5)
    Y = dev(Y0)
    pv.pv_block_rotate(dev(X), dev(Q), Y, accumulate=accumulate)
    X, Y0 = X.astype(np.complex128), Y0.astype(np.complex128)
    ref, size = X @ Q, np.abs(X) @ np.abs(Q)
    if accumulate:
        ref, size = ref + Y0, size + np.abs(Y0)
    bound = 2 * (2 * nx + 3) * EPS * size
    if dtype == np.complex64:
        bound = bound + np.finfo(np.float32).eps * size
    assert (np.abs(host(Y) - ref) <= bound).all()
