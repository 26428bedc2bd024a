"""Float32 products as products of three bfloat16 parts: the split on the CPU (its
exactness and what the products that are left out amount to), and on the GPU the
product by itself at the edges of both row tiles and with operands whose parts
leave bfloat16's range."""
import numpy as np
import pytest

from oracle.bf16 import round_bf16
from tests.gpu_util import announce, to_dev

U = 2.0 ** -24  # unit roundoff of float32


def _parts(x):
    """The three bfloat16 parts of float32 values (as float64)."""
    x = x.astype(np.float64)
    h = round_bf16(x.astype(np.float32)).astype(np.float64)
    m = round_bf16((x - h).astype(np.float32)).astype(np.float64)
    low = round_bf16((x - h - m).astype(np.float32)).astype(np.float64)
    return h, m, low


def test_three_parts_are_exact():
    """h + m + l is the value itself for every float32 value below 2^111 times 2^16;
    the three products of parts left out are within 2^-24 of a product (the rounding
    that float32 gives it)."""
    rng = np.random.default_rng(4)
    x = (rng.uniform(1, 2, 200000) * 2.0 ** rng.integers(-149, 111, 200000)).astype(np.float32)
    lifted = (x.astype(np.float64) * 2.0 ** 16).astype(np.float32)
    assert np.array_equal(sum(_parts(lifted)), lifted.astype(np.float64))
    a, b = (rng.uniform(1, 2, 200000).astype(np.float32) for _ in range(2))
    (_, am, al), (_, bm, bl) = _parts(a), _parts(b)
    left = np.abs(am * bl + al * bm + al * bl)
    assert np.max(left / (a.astype(np.float64) * b)) <= 2.0 ** -24


def _gemm(gpu_lib, A, X, trans):
    import torch
    Y = gpu_lib.gemm(to_dev(A), to_dev(X), trans=trans)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


def _ref(A, X, trans):
    A64, X64 = (A.T if trans else A).astype(np.float64), X.astype(np.float64)
    return A64 @ X64, np.abs(A64) @ np.abs(X64)


# the 256-row tile in both directions: remainders of rows, reduction steps and
# column blocks, one column pass and two; the 128-row tile next to its limits
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,d", [(6401, 1103, 97), (6401, 1103, 280), (6401, 1103, 289), (6145, 1024, 32),
                                   (6144, 1024, 33), (6401, 1023, 64)])
@pytest.mark.parametrize("trans", [False, True])
def test_gemm_row_tiles(gpu_lib, m, n, d, trans):
    announce("float32 gemm tiles", m, n, d, trans)
    rng = np.random.default_rng(m + n + d)
    A = rng.standard_normal((n, m) if trans else (m, n)).astype(np.float32)
    X = rng.standard_normal((n, d)).astype(np.float32)
    ref, bound = _ref(A, X, trans)
    assert np.all(np.abs(_gemm(gpu_lib, A, X, trans) - ref) <= 2 * n * U * bound)


@pytest.mark.gpu
@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("ea,ex", [(-118, 98), (-125, 100), (98, -118), (100, -125), (-118, 0), (0, -118),
                                   (-125, 127), (127, -126)])
@pytest.mark.parametrize("where", ["all", "some"])
def test_gemm_small_operands(gpu_lib, trans, ea, ex, where):
    """Operands whose parts would fall under bfloat16's smallest denormal, against
    large ones: every result an ordinary float32, as accurate as any.  "some": only
    every fifth reduction index holds them, beside operands near 1."""
    announce("float32 gemm small operands", trans, ea, ex, where)
    rng = np.random.default_rng(ea + 200)
    m, k, d = 75, 83, 40
    A, X = rng.uniform(1, 1.9, (m, k)), rng.uniform(1, 1.9, (k, d)) * rng.choice([-1, 1], (k, d))
    if where == "all":
        X = np.abs(X)  # (no cancellation)
        A, X = A * 2.0 ** (ea - 7 * (ea > ex)), X * 2.0 ** (ex - 7 * (ex > ea))  # (sums within range)
    else:
        A[:, ::5] *= 2.0 ** ea
        X[::5] *= 2.0 ** ex
    A, X = A.astype(np.float32), X.astype(np.float32)
    A = np.ascontiguousarray(A.T) if trans else A
    ref, bound = _ref(A, X, trans)
    assert np.all(np.abs(_gemm(gpu_lib, A, X, trans) - ref) <= 2 * k * U * bound)


@pytest.mark.gpu
@pytest.mark.parametrize("trans", [False, True])
def test_gemm_range_ends(gpu_lib, trans):
    """Values that round up to an infinity in bfloat16, and infinities and values
    that are no number, which reach their own rows and columns only."""
    announce("float32 gemm range ends", trans)
    rng = np.random.default_rng(8)
    m, k, d = 75, 83, 40
    top = np.float32(np.finfo(np.float32).max)
    A, X = rng.standard_normal((m, k)).astype(np.float32), (rng.standard_normal((k, d)) / 64).astype(np.float32)
    A[5, 7] = top
    ref, bound = _ref(A, X, False)
    At = np.ascontiguousarray(A.T) if trans else A
    assert np.all(np.abs(_gemm(gpu_lib, At, X, trans) - ref) <= 2 * k * U * bound)
    A[9, 80], A[40, 3], X[50, 6] = np.inf, np.nan, -np.inf
    At = np.ascontiguousarray(A.T) if trans else A
    Y = _gemm(gpu_lib, At, X, trans)
    with np.errstate(invalid="ignore"):
        ref = A.astype(np.float64) @ X.astype(np.float64)
    fine = np.ones((m, d), bool)
    fine[[9, 40]] = False
    fine[:, 6] = False
    assert np.array_equal(np.isnan(Y), np.isnan(ref)) and np.array_equal(np.isinf(Y), np.isinf(ref))
    assert np.array_equal(np.sign(Y[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    assert np.all(np.abs(Y[fine] - ref[fine]) <= 2 * k * U * bound[fine])


def _jump(rng, k, n):
    """Columns of k = 64 values whose second-last 16 are a hundred times and whose
    last 16 hold one value 2^25 times the first: every fourth one; the others
    Gaussian and as large."""
    A = rng.standard_normal((k, n)) * 2.0 ** 25
    for j in range(0, n, 4):
        sign = rng.choice([-1.0, 1.0], k)
        A[:, j] = rng.uniform(1.0, 1.9, k) * sign
        A[32:48, j] = rng.uniform(200.0, 250.0, 16) * sign[32:48]
        A[48 + rng.integers(16), j] = 2.0 ** 25
    return A


def _large_row(rng, k, n):
    """One row 2^19 times the others: the bases' other columns are as small there."""
    A = rng.standard_normal((k, n))
    A[37] *= 2.0 ** 19
    return A


@pytest.mark.gpu
@pytest.mark.parametrize("form", [_jump, _large_row])
@pytest.mark.parametrize("trans", [False, True])
def test_gemm_uneven_values(gpu_lib, form, trans):
    """Every output is as accurate as a float32 dot product, whatever the size of
    the other values of its row and column: within 64 roundings of sum |a x|, for X
    Gaussian and as uneven as A."""
    announce("float32 gemm uneven", form.__name__, trans)
    rng = np.random.default_rng(11)
    A = form(rng, 64, 200).T.astype(np.float32)
    for X in (rng.standard_normal((64, 48)), 1.0 / form(rng, 64, 48)):
        X = X.astype(np.float32)
        ref, bound = _ref(A, X, False)
        Y = _gemm(gpu_lib, np.ascontiguousarray(A.T) if trans else np.ascontiguousarray(A), X, trans)
        assert np.all(np.abs(Y - ref) <= 64 * U * bound)


@pytest.mark.gpu
@pytest.mark.parametrize("form", [_jump, _large_row])
def test_decompose_uneven_values(gpu_lib, form):
    """The last product of a decomposition, L V^T = Q^T A, entry by entry: within
    64 + 4 roundings of sum |q a| (the product and Q's own) and 8 of sum |l v|."""
    import torch
    announce("float32 decompose uneven", form.__name__)
    A = form(np.random.default_rng(12), 64, 200).astype(np.float32)
    out = gpu_lib.decompose(to_dev(A), 40, 8 if form is _jump else 0, 0, seed=3)
    torch.cuda.synchronize()
    Q, L, V = (x.cpu().numpy().astype(np.float64) for x in out)
    A64 = A.astype(np.float64)
    err = np.abs(L @ V.T - Q.T @ A64)
    assert np.all(err <= U * (68 * np.abs(Q).T @ np.abs(A64) + 8 * np.abs(L) @ np.abs(V).T))


def _decompose(gpu_lib, A, d, q, seed):
    import torch
    out = gpu_lib.decompose(to_dev(A), d, 0, q, seed=seed)
    torch.cuda.synchronize()
    return (x.cpu().numpy().astype(np.float64) for x in out)


def _check_products(A, Q, L, V, seed):
    """Both products of a decomposition at q = 0 against 64 bits, each row relative to
    its own size: Y = A Omega = Q R row by row (a rounding error dY reaches row i as
    dY_i and as Q_i Q^T dY; Q's own rounding as Q_i R), L V^T = Q^T A entry by entry
    (see test_decompose_uneven_values)."""
    from oracle import philox
    m, n = A.shape
    A64 = A.astype(np.float64)
    om = philox.gaussian_matrix(seed, n, L.shape[0]).astype(np.float32).astype(np.float64)
    Y, bound = A64 @ om, np.abs(A64) @ np.abs(om)
    err = np.linalg.norm(Y - Q @ (Q.T @ Y), axis=1)
    own, all_rows = np.linalg.norm(bound, axis=1), np.linalg.norm(bound)
    assert np.all(err <= U * ((n + 4) * own + np.linalg.norm(Q, axis=1) * ((n + 4) * all_rows + 8 * np.linalg.norm(Y))))
    err = np.abs(L @ V.T - Q.T @ A64)
    assert np.all(err <= U * ((m + 4) * np.abs(Q).T @ np.abs(A64) + 8 * np.abs(L) @ np.abs(V).T))


# the decompositions' form at the 256-row tile in both directions, with ragged
# reductions: one column pass and two; nine column blocks at the 128-row tile
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,d", [(6401, 1111, 40), (1111, 6401, 40), (6401, 1111, 224), (1111, 6401, 225),
                                   (1300, 700, 280), (6145, 1024, 1), (4374, 5904, 22)])
def test_decompose_row_tiles(gpu_lib, m, n, d):
    announce("float32 decompose tiles", m, n, d)
    A = np.random.default_rng(m + d).standard_normal((m, n)).astype(np.float32)
    _check_products(A, *_decompose(gpu_lib, A, d, 0, 5), 5)


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [-60, -30, -18])
@pytest.mark.parametrize("side", ["rows", "columns"])
def test_decompose_small_rows(gpu_lib, side, shift):
    """Rows or columns far smaller than the others, graded ones among them, are as
    accurate relative to themselves."""
    announce("float32 decompose small rows", side, shift)
    A = np.random.default_rng(21).standard_normal((300, 260))
    scale = np.ones(300 if side == "rows" else 260)
    scale[:96] = 2.0 ** shift
    scale[96:144] = 2.0 ** (shift * np.arange(48) / 48)
    A = (A * scale[:, None] if side == "rows" else A * scale).astype(np.float32)
    _check_products(A, *_decompose(gpu_lib, A, 40, 0, 6), 6)
