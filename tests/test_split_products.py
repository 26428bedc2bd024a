"""The float32 products on the 16-bit matrix cores: the two-part float16
split on the CPU (its error bound), and on the GPU whole decompositions whose
products take it, at tile edges, ragged reductions and extreme scales."""
import numpy as np
import pytest

import oracle
from oracle.metrics import recon_diff
from tests.gpu_util import announce


def _split(x, s):
    with np.errstate(over="ignore"):
        t = x.astype(np.float64) * s  # exact: s is a power of two
        h = t.astype(np.float16)
        low = (t - h.astype(np.float64)).astype(np.float16)
    return h.astype(np.float64), low.astype(np.float64)


def test_split_error_bounds():
    """h + l is within half a unit of float32's last place (2^-23 of the
    leading bit) for scaled values in [2^-2, 2^15), and within 2^-25 (half of
    float16's smallest step) below; three partial products are within
    2^-21 + 2^-22 of the exact product."""
    rng = np.random.default_rng(3)
    x = (rng.uniform(1, 2, 200000) * 2.0 ** rng.integers(-20, 15, 200000) * rng.choice([-1, 1], 200000)).astype(np.float32)
    h, low = _split(x, 1.0)
    err = np.abs(x.astype(np.float64) - h - low)
    lead = 2.0 ** np.floor(np.log2(np.abs(x.astype(np.float64))))
    assert np.all(err <= np.maximum(2.0 ** -23 * lead, 2.0 ** -25))
    a, b = rng.standard_normal(100000).astype(np.float32), rng.standard_normal(100000).astype(np.float32)
    ah, al = _split(a, 2.0 ** 7)
    bh, bl = _split(b, 2.0 ** 12)
    got = (al * bh + ah * bl + ah * bh) * 2.0 ** -19
    ref = a.astype(np.float64) * b.astype(np.float64)
    big = (np.abs(a) > 2.0 ** -8) & (np.abs(b) > 2.0 ** -8)
    assert np.max(np.abs(got - ref)[big] / np.abs(ref)[big]) <= 2.0 ** -21 + 2.0 ** -22


# one and several column blocks and passes; rows and reductions at and around
# the tile (128 and 256 rows) and step (32) sizes; a short step alone
SHAPES = [(32, 32, 5), (33, 31, 31), (40, 7, 3), (127, 65, 33), (129, 97, 64), (257, 449, 225), (6200, 1100, 40),
          (700, 640, 289), (1030, 2050, 100)]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,d", SHAPES)
def test_decompose_tile_edges(gpu_lib, m, n, d):
    """A Gaussian A has a well-conditioned sketch, so the approximation must
    match the oracle's within the float32 gate (1e-5)."""
    _check(gpu_lib, np.random.default_rng(m + n).standard_normal((m, n)), d)


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["late rows", "late columns", "graded rows", "graded columns", "tiny", "huge",
                                  "zero rows", "spike"])
def test_decompose_scales(gpu_lib, case):
    """Values that grow after the first reduction step (a row's scale is taken
    there), rows and columns of very different size, and magnitudes outside
    float16's and near float32's limits: relative accuracy as ever."""
    m, n = 300, 260
    A = np.random.default_rng(5).standard_normal((m, n))
    if case == "late rows":
        A[:96] *= 2.0 ** -30
    elif case == "late columns":
        A[:, :96] *= 2.0 ** -30
    elif case == "graded rows":
        A *= 2.0 ** -(np.arange(m) % 24)[:, None]
    elif case == "graded columns":
        A *= 2.0 ** -(np.arange(n) % 24)[None, :]
    elif case == "tiny":
        A *= 2.0 ** -118
    elif case == "huge":
        A *= 2.0 ** 100
    elif case == "zero rows":
        A[:40] = 0.0
        A[100] = 0.0
        A[:, 3] = 0.0
    elif case == "spike":
        A[200, 100] = 3.0e4
        A[7, 259] = -2.0e4
    _check(gpu_lib, A, 40, case)


@pytest.mark.gpu
def test_decompose_infinity_is_reported(gpu_lib):
    A = np.random.default_rng(6).standard_normal((200, 180)).astype(np.float32)
    A[50, 170] = np.inf
    import torch
    ctx = gpu_lib.Context(0)
    gpu_lib.decompose(torch.from_numpy(A).cuda(), 20, 5, 0, seed=2, ctx=ctx)
    torch.cuda.synchronize()
    assert ctx.info()["nonfinite"] == 1


def _check(gpu_lib, A, d, what=""):
    import torch
    announce("split products", A.shape, d, what)
    A32 = A.astype(np.float32)
    out = gpu_lib.decompose(torch.from_numpy(A32).cuda(), d, 0, 1, seed=9, ctx=gpu_lib.Context(0))
    torch.cuda.synchronize()
    Q, L, V = (x.cpu().numpy().astype(np.float64) for x in out)
    A64 = A32.astype(np.float64)
    ref = oracle.ruqlp(A64, d, 0, 1, 9, omega_dtype="f32")
    assert recon_diff(Q, L, V, *ref) <= 1e-5 * np.linalg.norm(A64)
    gate = 16 * np.sqrt(d) * 2.0 ** -24  # float32 orthogonality gate
    assert np.linalg.norm(Q.T @ Q - np.eye(d)) <= gate and np.linalg.norm(V.T @ V - np.eye(d)) <= gate
