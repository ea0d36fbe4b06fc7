"""k_sym_wave, k_wave_f32 and k_sym_mid (the products of small orders) at the
edges of their tile sizes: one layer against the FP64 product of the operands it
multiplies, two layers inside a solve, whose recorded traces must be those
of the returned iterate, and the two- and four-segment FP32 products of the
derivatives."""

import numpy as np
import pytest

import oracle
from gpu_util import banner, to_dev

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
# one and two tiles; the last and first order of each tile size (32 rows: n <= 704,
# 64: <= 1984) and of some numbers of K pieces
ORDERS = [1, 31, 32, 33, 64, 65, 97, 255, 257, 449, 703, 705, 1001, 1281, 1537, 1983, 1985]


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


def _planes(x32, precision):
    t = x32.copy()
    t[np.diag_indices(t.shape[0])] -= np.float32(0.5)
    if precision == "fp16x3":
        hi, lo = oracle.split_fp16_scaled(t)
        scale = 2.0 ** (-2 * oracle.FP16_SPLIT_SCALE_LOG2)
    else:
        hi, lo = oracle.split_bf16(t)
        scale = 1.0
    if precision == "bf16x1":
        lo = np.zeros_like(lo)
    return hi.astype(np.float64), lo.astype(np.float64), scale


@pytest.mark.parametrize("n", ORDERS)
def test_layer_at_tile_edges(pk, n):
    import torch
    x32 = _operand(n, n)
    for k, precision in enumerate(("bf16x3", "fp16x3", "bf16x1")):
        hi, lo, s = (torch.from_numpy(v).to("cuda") if isinstance(v, np.ndarray) else v
                     for v in _planes(x32, precision))
        r = (hi @ hi + hi @ lo + lo @ hi) * s
        bound = (3 * n + 4) * U32 * (hi.abs() @ hi.abs() + hi.abs() @ lo.abs()
                                     + lo.abs() @ hi.abs()) * s
        x = to_dev(x32).double()
        ld = n + (0, 3, 64)[k]
        X = torch.zeros(n, ld, device="cuda")[:, :n]
        X.copy_(to_dev(x32))
        for sign in (1, -1):
            banner(f"wave layer {precision} N={n} ld={ld} sign={sign}")
            Y = torch.full((n, ld), 7.0, device="cuda")
            pk.sp2_layer(X, precision, sign, Y[:, :n], pk.allocate_workspace(n))
            a, b = (1.0, 0.0) if sign > 0 else (-1.0, 2.0)
            ref = a * r + (a + b) * x - 0.25 * a * torch.eye(n, device="cuda", dtype=torch.float64)
            tol = bound + 2 * U32 * r.abs() + 4 * U32 * x.abs() + 4 * U32 * ref.abs() + U32
            y = Y[:, :n].double()
            assert torch.equal(Y[:, :n], Y[:, :n].T)
            assert bool((Y[:, n:] == 7.0).all())
            assert bool(((y - ref).abs() <= tol).all())


@pytest.mark.parametrize("n", ORDERS[1:])
def test_traces_are_those_of_the_iterate(pk, n):
    import torch
    h = to_dev(_operand(n, 7 * n))
    for precision in ("bf16x3", "fp16x3", "bf16x1"):
        banner(f"wave traces {precision} N={n}")
        P, info = pk.density(h, n // 2, precision=precision, refine="none", max_iter=2, tol=0.0,
                             stop_rule=0, allow_unconverged=True, return_info=True)
        hist = pk.sp2_history(info["workspace"])
        p = P.double()
        t1, t2 = p.trace().item(), (p * p).sum().item()
        # FP64 sums of the same FP32 entries in another order
        assert abs(hist["t1"][2] - t1) <= 1e-12 * n * max(1.0, abs(t1))
        assert abs(hist["t2"][2] - t2) <= 1e-12 * n * max(1.0, t2)
        # the two recorded layers in FP64 from the same bounds
        lo, hi = info["eps_min"], info["eps_max"]
        s = (hi * torch.eye(n, device="cuda", dtype=torch.float64) - h.double()) / (hi - lo)
        for a, b, _ in hist["coef"]:
            s = a * (s @ s) + b * s
        # operand roundings 2^-8, 2^-16 or 2^-22 of entries whose rows have norm <= 1, twice over
        u = {"bf16x1": 2.0 ** -8, "bf16x3": 2.0 ** -16, "fp16x3": 2.0 ** -22}[precision]
        assert (p - s).abs().max().item() <= 8 * (u + 3 * n * U32)


@pytest.mark.parametrize("n", ORDERS)
def test_fp32_layer_at_tile_edges(pk, n):
    """The bound of a plain FP32 product (n u sum |a||b|) holds for the product
    in BF16 triples: what it leaves out is below u / 4 per product."""
    import torch
    x32 = _operand(n, 3 * n)
    x = to_dev(x32).double()
    r, bound = x @ x, (n + 4) * U32 * (x.abs() @ x.abs())
    X = torch.zeros(n, n + 5, device="cuda")[:, :n]
    X.copy_(to_dev(x32))
    for sign in (1, -1):
        banner(f"wave layer fp32 N={n} sign={sign}")
        Y = torch.full((n, n + 5), 7.0, device="cuda")
        pk.sp2_layer(X, "fp32", sign, Y[:, :n], pk.allocate_workspace(n))
        ref = r if sign > 0 else 2 * x - r
        y = Y[:, :n].double()
        assert torch.equal(Y[:, :n], Y[:, :n].T)
        assert bool((Y[:, n:] == 7.0).all())
        assert bool(((y - ref).abs() <= bound + 2 * U32 * (x.abs() + ref.abs())).all())


def test_fp32_layer_with_infinities(pk):
    """An infinite entry spoils its own row and column and nothing else."""
    import torch
    n = 130
    x32 = np.abs(_operand(n, 5)) + np.float32(0.1)
    x32[7, 90] = x32[90, 7] = np.inf
    Y = torch.empty(n, n, device="cuda")
    pk.sp2_layer(to_dev(x32), "fp32", 1, Y, pk.allocate_workspace(n))
    y = Y.cpu().numpy()
    hit = np.zeros((n, n), bool)
    hit[[7, 90]] = hit[:, [7, 90]] = True
    assert np.all(np.isposinf(y[hit]))
    assert np.all(np.isfinite(y[~hit]))


@pytest.mark.parametrize("n", [33, 257, 703, 1001, 1537])
def test_fp32_pair_products(pk, n):
    """Forward derivative with FP32 products (two K segments per layer, four in
    the refinement) against first-order perturbation theory."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))
    occ = n // 2
    e = 0.5 + 1.5 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    e[:occ] *= -1
    h = ((q * e) @ q.T.contiguous()).float()
    h = torch.triu(h) + torch.triu(h, 1).T
    a = torch.randn(n, n, generator=g, device="cuda")
    a = torch.triu(a) + torch.triu(a, 1).T
    banner(f"wave fp32 pairs N={n}")
    _, p1 = pk.jvp(h, occ, a, precision="fp32")
    e, v = torch.linalg.eigh(h.double())
    o, w = v[:, :occ].contiguous(), v[:, occ:].contiguous()
    c = (o.T.contiguous() @ a.double() @ w) / (e[:occ, None] - e[None, occ:])
    ref = o @ c @ w.T.contiguous()
    ref = ref + ref.T
    rel = ((p1.double() - ref).norm() / ref.norm()).item()
    # FP32 rounding of some 25 layers, amplified by the mapped gap (1 in about 30)
    assert rel <= 25 * 30 * U32


@pytest.mark.parametrize("n", [1793, 2017, 2047, 2048, 2049])
def test_96_row_tiles(pk, n):
    """The first and last orders of the 96-row tiles, whose last row of tiles
    ends past the padded order, and the order after them."""
    test_layer_at_tile_edges(pk, n)
    test_traces_are_those_of_the_iterate(pk, n)


@pytest.mark.parametrize("n", [1793, 2047])
def test_split_pair_of_96_row_tiles(pk, n):
    """Forward derivative with BF16X3 pair products against first-order
    perturbation theory; such a product leaves out 2^-17 of its terms (25
    layers, a mapped gap of 1 in about 30)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    q, _ = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))
    occ = n // 2
    e = 0.5 + 1.5 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    e[:occ] *= -1
    h = ((q * e) @ q.T.contiguous()).float()
    h = torch.triu(h) + torch.triu(h, 1).T
    a = torch.randn(n, n, generator=g, device="cuda")
    a = torch.triu(a) + torch.triu(a, 1).T
    banner(f"wave split pairs N={n}")
    _, p1 = pk.jvp(h, occ, a, precision="bf16x3", split_derivatives=True)
    o, w = q[:, :occ].contiguous(), q[:, occ:].contiguous()
    c = (o.T.contiguous() @ a.double() @ w) / (e[:occ, None] - e[None, occ:])
    ref = o @ c @ w.T.contiguous()
    ref = ref + ref.T
    assert ((p1.double() - ref).norm() / ref.norm()).item() <= 25 * 30 * 2.0 ** -17


@pytest.mark.parametrize("n", [3841, 4033, 4095, 4096, 4097])
def test_192_row_tiles(pk, n):
    """The first and last orders of the 192-row tiles (k_sym_mid), whose last
    row of tiles ends past the padded order, and the order after them."""
    test_layer_at_tile_edges(pk, n)
    test_traces_are_those_of_the_iterate(pk, n)


def test_split_pair_of_192_row_tiles(pk):
    test_split_pair_of_96_row_tiles(pk, 4095)


@pytest.mark.parametrize("n", [1728, 1729, 1793, 2047, 2048, 2049])
def test_fp32_96_row_tiles(pk, n):
    """FP32 layers from the last order of 64-row tiles to the first past the
    96-row ones, and the pair products of one."""
    test_fp32_layer_at_tile_edges(pk, n)
    if n == 2047:
        test_fp32_pair_products(pk, n)


@pytest.mark.parametrize("n", [1791, 1792])
def test_last_orders_of_64_row_tiles(pk, n):
    """Both kinds of 64-row tiles, split and FP32, serve n <= 1792."""
    test_layer_at_tile_edges(pk, n)
    test_traces_are_those_of_the_iterate(pk, n)
    test_fp32_layer_at_tile_edges(pk, n)
