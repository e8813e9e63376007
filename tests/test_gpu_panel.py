"""The diagonal tile's POTRF and the panel TRSM at every number of 64-blocks a
tile can have at its ends (2 and 32 per tile, and odd counts of 128), and for
pivots outside the range of the in-kernel square root."""
import numpy as np
import pytest

import synth
from _gpu import M, factor_dense, log, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,n,exp2", [
    (128, 128, 0), (128, 129, 0), (384, 1000, 0), (640, 640, 0), (2048, 2048, 0), (1152, 2400, 0),
    (128, 300, -910), (256, 600, 920), (384, 500, -901), (128, 300, -899), (128, 300, 899)])
def test_factor_of_scaled_integers_is_exact(tile, n, exp2):
    """A = S S^T, S = 2^(exp2 // 2) L0 with a small integer L0: the factor is S
    bit for bit, whichever way a pivot is taken."""
    mod = M()
    L0 = synth.int_lower(n, 5) * 2.0 ** (exp2 // 2)
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, L0 @ L0.T)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        assert np.array_equal(factor_dense(h, n), L0)
    finally:
        mod.mpchol_destroy(h)


@pytest.mark.parametrize("tile,n,col,val", [(256, 600, 70, -1.0), (256, 600, 255, 0.0), (512, 512, 511, -2.0),
                                            (128, 300, 299, float("nan"))])
def test_bad_pivot_column(tile, n, col, val):
    """A diagonal entry lowered so that exactly its pivot fails: info is its 1-based column."""
    mod = M()
    L0 = synth.int_lower(n, 6)
    A = L0 @ L0.T
    A[col, col] = A[col, col] - L0[col, col] ** 2 + val
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, A)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == col + 1
    finally:
        mod.mpchol_destroy(h)


@pytest.mark.parametrize("tile,n", [(128, 256), (128, 384), (128, 1500), (256, 2048), (384, 3000), (512, 2100),
                                    (1024, 3072)])
def test_update_block_shapes(tile, n):
    """Trailing updates whose grids fall on either side of the block-shape rules,
    one panel column and pairs: integer products are exact in any order."""
    mod = M()
    L0 = synth.int_lower(n, 8)
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, L0 @ L0.T)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        assert np.array_equal(factor_dense(h, n), L0)
    finally:
        mod.mpchol_destroy(h)


@pytest.mark.parametrize("n,tile,pad,shift", [(1, 128, 0, 0), (127, 128, 1, 0), (129, 128, 0, 0), (300, 128, 1, 1),
                                              (300, 128, 0, 1), (1030, 512, 2, 0)])
def test_get_factor_layouts(n, tile, pad, shift):
    """The dense copy in every class at odd sizes, leading dimensions and bases: the
    same values through each layout, zero above the diagonal, nothing else touched."""
    torch = torch_cuda()
    mod = M()
    nt = -(-n // tile)
    um = np.asfortranarray(np.tril((np.arange(nt * nt).reshape(nt, nt) % 4).astype(np.uint8), -1))
    L0 = synth.int_lower(n, 9)
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, L0 @ L0.T)
        mod.mpchol_precision_map(h, mod.RULE_USER, 1e-9, um)
        assert mod.mpchol_factor(h) == 0
        buf = torch.full((shift + n * (n + pad),), 7.0, dtype=torch.float64, device="cuda")
        Lt = buf[shift:].view(n, n + pad)
        mod.mpchol_get_factor(h, Lt.T, n)
        torch.cuda.synchronize()
    finally:
        mod.mpchol_destroy(h)
    assert np.array_equal(Lt[:, :n].cpu().numpy().T, L0)
    assert torch.all(Lt[:, n:] == 7.0) and torch.all(buf[:shift] == 7.0)


@pytest.mark.parametrize("tile,n", [(256, 1024), (512, 1024), (1024, 1024), (2048, 2048), (1024, 2048)])
def test_factor_error_does_not_grow_with_the_tile(tile, n):
    """A - L L^T in long double on entries that stay large under elimination: the
    last 256 of the diagonal, and (i + n/2, i), whose rows are 0.9 alike.  A value
    of size A is to be rounded once per 64 columns and at most 24 times within its
    own block of 64, each with a standard deviation of at most u A / sqrt(3); the
    sums of 64 products, about A 32 / n each, add less than (u A)^2 to the
    variance.  (Rounded at every product: 2 to 5 times this bound.)"""
    rng = np.random.default_rng(17)
    X = rng.standard_normal((n, 2 * n))
    X[n // 2:] = 0.9 * X[:n // 2] + np.sqrt(0.19) * X[n // 2:]
    A = X @ X.T / (2 * n)
    A = (A + A.T) / 2
    mod = M()
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, A)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        L = factor_dense(h, n).astype(np.longdouble)
    finally:
        mod.mpchol_destroy(h)
    last, half = np.arange(n - 256, n), np.arange(n // 2 - 128, n // 2)
    for rows, cols in ((last, last), (half + n // 2, half)):
        res = A[rows, cols] - (L[rows] * L[cols]).sum(axis=1)
        size = np.sqrt(A[rows, rows] * A[cols, cols])
        rms = float(np.sqrt(np.mean((res / size) ** 2))) * 2.0 ** 53
        bound = np.sqrt((cols.max() / 64 + 24) / 3 + 1)
        log(f"  n={n} tile={tile}: {rms:.2f} u, bound {bound:.2f} u")
        assert rms <= bound


@pytest.mark.parametrize("tile,n,col", [(128, 300, 5), (128, 300, 100), (256, 600, 70), (256, 600, 599), (512, 1100, 511)])
def test_infinite_diagonal_entry(tile, n, col):
    """A quotient by an infinite pivot is 0, in the pivot's own block of 64, in the
    tile's other blocks and in the panel below: the other rows and columns are
    the factor of the matrix without that one."""
    mod = M()
    L0 = synth.int_lower(n, 6)
    A = L0 @ L0.T + n * np.eye(n)
    others = np.delete(np.arange(n), col)
    want = np.zeros((n, n))
    want[np.ix_(others, others)] = np.linalg.cholesky(A[np.ix_(others, others)])
    want[col, :col] = np.linalg.solve(want[:col, :col], A[:col, col]) if col else 0.0
    A[col, col] = np.inf
    h = mod.mpchol_create(n, tile)
    try:
        mod.mpchol_set_matrix(h, A)
        mod.mpchol_precision_map(h, mod.RULE_FP64)
        assert mod.mpchol_factor(h) == 0
        assert mod.mpchol_logdet(h) == np.inf
        got = factor_dense(h, n)
    finally:
        mod.mpchol_destroy(h)
    assert got[col, col] == np.inf and np.all(got[col + 1:, col] == 0.0)
    got[col, col] = 0.0
    assert np.abs(got - want).max() <= n * 2.0 ** -53 * np.sqrt(np.diagonal(A)[others].max())
