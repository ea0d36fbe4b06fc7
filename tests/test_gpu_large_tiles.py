"""The 256 x 256 kernels (k_sym_split, k_sym_f32, k_split_tail) at orders that
smaller tiles do not serve: layers of n = 2049 with the last round of tiles split
along K and without, and the two- and four-segment products of the derivatives
with pieces (n = 2049) and in whole tiles (n = 4097)."""

import numpy as np
import pytest

import oracle
from gpu_util import banner, to_dev

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def pk():
    import paper_2107_02737_amd as pk
    pk.load_library()
    return pk


def _operand(n, seed):
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((n, n), dtype=np.float32) * np.float32(0.3 / np.sqrt(n))
    x = np.triu(a) + np.triu(a, 1).T
    x[np.diag_indices(n)] = rng.uniform(0.0, 1.0, n).astype(np.float32)
    return x


def _reference(x32, precision, sign):
    """The layer's FP64 value from the operands it multiplies, and the bound of its
    FP32 sums (as for the layers of n <= 1000 in test_gpu_kernels.py)."""
    import torch
    n = len(x32)
    x = to_dev(x32).double()
    a, b = (1.0, 0.0) if sign > 0 else (-1.0, 2.0)
    if precision == "fp32":
        r, acc = x @ x, x.abs() @ x.abs()
        y = a * r + b * x
        return y, (n + 4) * U32 * acc + 2 * U32 * r.abs() + 4 * U32 * x.abs() + 2 * U32 * y.abs()
    t = x32.copy()
    t[np.diag_indices(n)] -= np.float32(0.5)
    hi, lo = oracle.split_fp16_scaled(t) if precision == "fp16x3" else oracle.split_bf16(t)
    s = 2.0 ** (-2 * oracle.FP16_SPLIT_SCALE_LOG2) if precision == "fp16x3" else 1.0
    hi, lo = (torch.from_numpy(v.astype(np.float64)).cuda() for v in (hi, lo))
    if precision == "bf16x1":
        lo.zero_()
    r = (hi @ hi + hi @ lo + lo @ hi) * s
    hi.abs_(), lo.abs_()
    acc = (hi @ hi + hi @ lo + lo @ hi) * s
    y = a * r + (a + b) * x - 0.25 * a * torch.eye(n, device="cuda", dtype=torch.float64)
    return y, ((3 * n + 4) * U32 * acc + 2 * U32 * r.abs() + 4 * U32 * x.abs() + 4 * U32 * y.abs()
               + U32)


@pytest.mark.parametrize("pieces", [True, False])
@pytest.mark.parametrize("precision", ["fp32", "bf16x1", "bf16x3", "fp16x3"])
def test_layer_in_pieces_and_whole(pk, precision, pieces, monkeypatch):
    import torch
    n, ld = 2049, 2055
    if not pieces:
        monkeypatch.setenv("SP2_NO_SPLITK", "1")
    x32 = _operand(n, 1)
    for sign in (1, -1):
        banner(f"large tiles layer {precision} pieces={pieces} sign={sign}")
        X = to_dev(x32, ld)
        Y = torch.full((n, ld), 7.0, device="cuda")
        pk.sp2_layer(X, precision, sign, Y[:, :n], pk.allocate_workspace(n))
        ref, bound = _reference(x32, precision, sign)
        y = Y[:, :n]
        assert torch.equal(y, y.T)
        assert bool((Y[:, n:] == 7.0).all())
        assert bool(((y.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("n,precision,unit", [(2049, "bf16x3", 2.0 ** -17), (2049, "fp32", U32),
                                              (4097, "bf16x3", 2.0 ** -17)])
def test_derivatives(pk, n, precision, unit):
    """Forward and adjoint derivative against first-order perturbation theory:
    25 layers, each off by the unit of its products, amplified by the mapped gap
    (1 in about 30)."""
    import torch
    banner(f"large tiles derivatives {precision} N={n}")
    g = torch.Generator(device="cuda").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))
    occ = n // 2
    e = 0.5 + 1.5 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    e[:occ] *= -1
    h = ((q * e) @ q.T.contiguous()).float()
    h = torch.triu(h) + torch.triu(h, 1).T
    o, w = q[:, :occ].contiguous(), q[:, occ:].contiguous()
    _, info = pk.density(h, occ, precision=precision, checkpoint_every=4, return_info=True,
                         split_derivatives=precision == "bf16x3")
    for call in (pk.sp2_jvp, pk.sp2_vjp):
        a = torch.randn(n, n, generator=g, device="cuda")
        a = torch.triu(a) + torch.triu(a, 1).T
        got = torch.empty_like(a)
        call(info["workspace"], a, got)
        c = (o.T.contiguous() @ a.double() @ w) / (e[:occ, None] - e[None, occ:])
        ref = o @ c @ w.T.contiguous()
        ref = ref + ref.T
        assert ((got.double() - ref).norm() / ref.norm()).item() <= 25 * 30 * unit
