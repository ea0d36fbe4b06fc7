"""FP32 products are FP32: on operands whose large entries lie off the diagonal,
of one sign, and at both ends of the FP32 range.  One layer X^2 against FP64,
at orders of every tile size (257 and 258: 32 rows, 1026: 64, 2046: 96, 2050: the
256 x 256 kernel)."""

import numpy as np
import pytest

from gpu_util import banner, to_dev

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
ORDERS = [258, 1026, 2046, 2050]


@pytest.fixture(scope="module")
def pk():
    import paper_2107_02737_amd as pk
    pk.load_library()
    return pk


def _square(pk, x32):
    import torch
    X = to_dev(x32)
    Y = torch.empty_like(X)
    pk.sp2_layer(X, "fp32", 1, Y, pk.allocate_workspace(len(x32)))
    return Y.cpu().numpy().astype(np.float64)


def _symmetric(a):
    return np.triu(a) + np.triu(a, 1).T


def _dimers(n, seed):
    """Sublattice-ordered dimers: row i's largest entry, 1/2 to 0.7, is in column
    i + n/2, far from the diagonal, which is zero."""
    rng = np.random.default_rng(seed)
    x = _symmetric(0.1 / np.sqrt(n) * rng.standard_normal((n, n), dtype=np.float32))
    np.fill_diagonal(x, 0.0)
    i = np.arange(n // 2)
    x[i, i + n // 2] = x[i + n // 2, i] = rng.uniform(0.5, 0.7, n // 2)
    return x.astype(np.float32)


def _one_sign(n, seed):
    rng = np.random.default_rng(seed)
    return _symmetric(rng.uniform(0.5, 1.0, (n, n)) / n).astype(np.float32)


def _nearest(x):
    """Sums of the squares of each row in FP32, every addition rounded to nearest,
    over pieces of 128 values and then over the pieces."""
    def add(s, t):
        return (s.astype(np.float64) + t).astype(np.float32)
    total = np.zeros(len(x), np.float32)
    for k in range(0, x.shape[1], 128):
        s = np.zeros(len(x), np.float32)
        for c in x[:, k:k + 128].T:
            s = add(s, c * c)
        total = add(total, s.astype(np.float64))
    return total


@pytest.mark.parametrize("operand", [_dimers, _one_sign])
@pytest.mark.parametrize("n", ORDERS[:-1])
def test_no_bias_beyond_rounding(pk, operand, n):
    """The diagonal of X^2 is a sum of squares; its mean signed error is that of
    FP32 sums rounded to nearest.  (That one is not zero: addends of the size of
    the last bit, the smaller the more frequent, are rounded down more often than
    up.)  An addition errs by at most u times the sum, u / sqrt(3) in the mean square,
    and an entry meets no more than 152 of them (pieces of 128 at the most, then at
    most 24 pieces): the means over n entries of 8 matrices, two of them, differ
    by at most 5 sqrt(2 * 152 / 3 / 8n) u."""
    mean = np.zeros(2)
    for seed in range(8):
        banner(f"fp32 bias {operand.__name__} N={n} seed={seed}")
        x32 = operand(n, seed)
        x = x32.astype(np.float64)
        r = (x * x).sum(1)
        for k, s in enumerate((np.diag(_square(pk, x32)), _nearest(x))):
            mean[k] += ((s - r) / (U32 * r)).mean() / 8
    print(f"  mean {mean[0]:+.3f} u, rounded to nearest {mean[1]:+.3f} u", flush=True)
    assert abs(mean[0] - mean[1]) <= 5 * np.sqrt(2 * 152 / 3 / (8 * n))


@pytest.mark.parametrize("n", [33, 257] + ORDERS)
def test_smallest_magnitudes(pk, n):
    """[A, tB; tB^T, A] with entries of A in [1/2, 1), B = 1 + 2^-11 and t = 2^-124: the
    products that matter are normal numbers, and their sums keep FP32's bound."""
    banner(f"fp32 tiny N={n}")
    rng = np.random.default_rng(n)
    x = rng.uniform(0.5, 1.0, (n, n))
    k = n // 2
    x[:k, k:] = (1 + 2.0 ** -11) * 2.0 ** -124
    x32 = _symmetric(x).astype(np.float32)
    x = x32.astype(np.float64)
    y, r = _square(pk, x32), x @ x
    assert np.all(np.abs(y - r) <= (n + 4) * U32 * r)


@pytest.mark.parametrize("n", [33, 257] + ORDERS)
def test_largest_magnitudes(pk, n):
    """The largest finite values stay finite: only the sums that pass FP32's
    range, two of the diagonal, are infinite."""
    banner(f"fp32 huge N={n}")
    rng = np.random.default_rng(n)
    x32 = _symmetric(rng.uniform(0.5, 1.0, (n, n)) / n).astype(np.float32)
    i, j = 1, n - 2
    x32[i, j] = x32[j, i] = np.float32(float.fromhex("0x1.fffffep127"))
    x = x32.astype(np.float64)
    y, r = _square(pk, x32), x @ x
    big = np.zeros((n, n), bool)
    big[i, i] = big[j, j] = True
    assert np.all(np.isposinf(y[big]))
    assert np.all(np.abs(y - r)[~big] <= ((n + 4) * U32 * r)[~big])


@pytest.mark.parametrize("n", [258, 1026])
def test_solve_of_a_dimer_chain(pk, n):
    """Recorded traces of an FP32 solve against the same layers in FP64: a layer
    rounds each diagonal entry (at most 1) by sqrt(152 / 3) u in the mean square,
    independent over n entries and the layers; later layers amplify by no more
    than the inverse of the mapped gap (4); 5 standard deviations, twice that
    for the second trace, whose derivative is 2 S."""
    import torch
    banner(f"fp32 dimer chain N={n}")
    h = to_dev(-_dimers(n, 99))
    _, info = pk.density(h, n // 2, precision="fp32", refine="none", return_info=True)
    hist = pk.sp2_history(info["workspace"])
    lo, hi = info["eps_min"], info["eps_max"]
    s = (hi * torch.eye(n, device="cuda", dtype=torch.float64) - h.double()) / (hi - lo)
    assert info["converged"]
    for k, (a, b, _) in enumerate(hist["coef"]):
        tol = 5 * 4 * np.sqrt((k + 1) * n * 152 / 3) * U32
        assert abs(hist["t1"][k] - s.trace().item()) <= tol
        assert abs(hist["t2"][k] - (s * s).sum().item()) <= 2 * tol
        s = a * (s @ s) + b * s
