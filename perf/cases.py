"""Timed cases of the density-matrix library, through its Python entry points.

listed() names the cases, draw(rng) gives more of the same ranges; a case is a
dict of plain values.  prepare() makes what a program holds before the call (the
Hamiltonian on the GPU, a kept workspace, a derivative tape), run() is one pass
and returns its outputs, exact() the same in FP64 with plain torch, work() the
bytes and operations that one pass cannot do without.

Kinds of case:
  solve     one density matrix (the call of every molecular-dynamics step)
  mdstep    HOMO/LUMO estimates from the previous step, then the accelerated solve
  layer     one expansion layer X^2 or 2X - X^2
  gradient  solve with a derivative tape and the adjoint of Tr(W P) (autograd)
  response  forward derivative on a kept tape (one per Krylov vector of XL-BOMD)
  nvt       both halves of one canonical integration step
"""

import math

import torch

import paper_2107_02737_amd as pk

DEV = "cuda"

# The solver options in use.  "default": the library's own (BF16 pair, FP32
# refinement, Gershgorin bounds); "fp32eq": the FP32-equivalent mode of the
# benchmark (FP16 pair throughout, 8 Lanczos bound steps, tol 2e-3 before the
# refinement); "fp32": plain FP32 layers.
MODES = {
    "default": dict(precision="bf16x3", refine="fp32"),
    "fp32eq": dict(precision="fp16x3", refine="split", bound_steps=8, tol=2e-3),
    "fp32": dict(precision="fp32", refine="fp32", bound_steps=8),
}
# Layers of one solve (measured: Gershgorin or Lanczos bounds, accelerated).
LAYERS = {"default": 26, "fp32eq": 20, "fp32": 20, "accelerated": 13}
PRODUCTS = {"bf16x1": 1, "bf16x3": 3, "fp16x3": 3, "fp32": 1}


def listed():
    return [
        # The small random-spectrum matrix of the tests and the smoke check:
        # latency of the whole call.
        dict(name="solve_gapped_256", kind="solve", matrix="gapped", n=256, mode="default"),
        # A water box of 67 molecules (the paper's dynamics use some tens to a
        # hundred): one solve per time step, an order that is no multiple of 256.
        dict(name="solve_water_402", kind="solve", matrix="water", n=402, mode="fp32eq"),
        # A mid-sized box with the library's defaults.
        dict(name="solve_water_2046", kind="solve", matrix="water", n=2046, mode="default"),
        # The headline benchmark: 1024 molecules.
        dict(name="solve_water_6144", kind="solve", matrix="water", n=6144, mode="fp32eq"),
        # The trajectory benchmark's order (2730 molecules), the largest call.
        dict(name="solve_water_16380", kind="solve", matrix="water", n=16380, mode="default"),
        # One accelerated molecular-dynamics step at the order of the
        # derivative tests (682 molecules).
        dict(name="mdstep_water_4092", kind="mdstep", matrix="water", n=4092, mode="fp32eq"),
        # Single layers: the FP16 pair at a ragged order, the single BF16
        # product, and plain FP32.
        dict(name="layer_fp16x3_1000", kind="layer", n=1000, precision="fp16x3", sign=-1, pad=0),
        dict(name="layer_bf16x1_3072", kind="layer", n=3072, precision="bf16x1", sign=1, pad=0),
        dict(name="layer_fp32_1536", kind="layer", n=1536, precision="fp32", sign=1, pad=64),
        # A training or force step: forward with a tape, backward through it.
        dict(name="gradient_gapped_1026", kind="gradient", matrix="gapped", n=1026, mode="default",
             split=False),
        # One response of the XL-BOMD kernel on a kept tape.
        dict(name="response_gapped_2046", kind="response", matrix="gapped", n=2046, mode="default",
             split=True),
        # The integration step of the 1024-molecule box (9216 coordinates).
        dict(name="nvt_9216", kind="nvt", n=9216, scheme=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "mdstep", "layer", "layer", "gradient",
                       "response", "nvt"])
    if kind == "solve":
        if rng.random() < 0.3:
            return dict(kind=kind, matrix="gapped", n=_log_int(rng, 200, 2048),
                        mode=rng.choice(["default", "fp32eq", "fp32"]))
        return dict(kind=kind, matrix="water", n=6 * _log_int(rng, 40, 1600),
                    mode=rng.choice(["default", "fp32eq", "fp32eq"]))
    if kind == "mdstep":
        return dict(kind=kind, matrix="water", n=6 * _log_int(rng, 64, 1024), mode="fp32eq")
    if kind == "layer":
        return dict(kind=kind, n=_log_int(rng, 200, 8192),
                    precision=rng.choice(["bf16x1", "bf16x3", "fp16x3", "fp32"]),
                    sign=rng.choice([1, -1]), pad=rng.choice([0, 0, 1, 64]))
    if kind in ("gradient", "response"):
        return dict(kind=kind, matrix="gapped", n=_log_int(rng, 200, 2048), mode="default",
                    split=rng.choice([False, True]))
    return dict(kind=kind, n=3 * _log_int(rng, 200, 1 << 21), scheme=rng.choice([0, 1]))


# ---- inputs ---------------------------------------------------------------

def _gen(seed, stream=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + stream)


def _cells(m):
    """Near-cubic grid with at least m cells."""
    c = round(m ** (1.0 / 3.0))
    dims = [(a, b, k) for a in range(max(1, c - 1), c + 2) for b in range(a, c + 2)
            for k in range(b, c + 2) if a * b * k >= m]
    return min(dims, key=lambda d: (d[2], d[0] * d[1] * d[2]))


def _water(n, seed, wobble=0.0):
    """Tight-binding Hamiltonian of n/6 water molecules at 1 g/cm^3 (six
    orbitals each), centres on a jittered grid, random orientations; wobble
    displaces every molecule (the previous step of a trajectory)."""
    m = n // 6
    g = _gen(seed)
    f64 = dict(device=DEV, dtype=torch.float64)
    edge = (m * 29.915) ** (1.0 / 3.0)
    dims = _cells(m)
    spacing = torch.tensor([edge / d for d in dims], **f64)
    cell = torch.randperm(dims[0] * dims[1] * dims[2], generator=g, device=DEV)[:m]
    idx = torch.stack([cell // (dims[1] * dims[2]), (cell // dims[2]) % dims[1], cell % dims[2]], 1)
    jitter = torch.clamp((spacing - 2.5) / 2, min=0.05)
    centre = (idx.to(torch.float64) + 0.5) * spacing
    centre = centre + (torch.rand(m, 3, generator=g, **f64) * 2 - 1) * jitter
    q = torch.randn(m, 4, generator=g, **f64)
    centre = centre + wobble * torch.randn(m, 3, generator=g, **f64)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1)
    half = math.radians(104.5) / 2
    local = torch.tensor([[0, 0, 0], [0.96 * math.sin(half), 0, 0.96 * math.cos(half)],
                          [-0.96 * math.sin(half), 0, 0.96 * math.cos(half)]], **f64)
    atoms = centre[:, None, :] + (rot.view(m, 1, 3, 3) * local[None, :, None, :]).sum(-1)
    atoms = atoms.reshape(3 * m, 3)
    atom_of = (3 * torch.arange(m, device=DEV)[:, None]
               + torch.tensor([0, 0, 0, 0, 1, 2], device=DEV)).reshape(-1)
    h = torch.empty(n, n, device=DEV)
    for a in range(0, n, 1536):   # rows in blocks keep the distance matrix small
        rows = atom_of[a:a + 1536]
        r2 = torch.zeros(len(rows), 3 * m, **f64)
        for k in range(3):
            d = atoms[rows, k][:, None] - atoms[None, :, k]
            r2 += (d - edge * torch.round(d / edge)) ** 2
        r = r2.sqrt()
        hop = torch.where((r < 6.0) & (r > 0.0), -torch.exp(-r), 0.0)
        h[a:a + 1536] = hop[:, atom_of].float()
    h = torch.triu(h, 1)
    h = h + h.T
    h.diagonal().copy_(torch.tensor([-1.0, -0.5, -0.5, -0.5, -0.3, -0.3], device=DEV).repeat(m))
    return h, 4 * m


def _gapped(n, seed):
    """Q diag(e) Q^T, half the levels in [-2, -0.5], half in [0.5, 2]."""
    g = _gen(seed)
    a = torch.randn(n, n, generator=g, device=DEV, dtype=torch.float64)
    q, _ = torch.linalg.qr(a)
    occ = n // 2
    e = 0.5 + 1.5 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    e[:occ] *= -1
    h = ((q * e) @ q.T.contiguous()).float()
    return torch.triu(h) + torch.triu(h, 1).T, occ


def _hamiltonian(case, seed):
    if case["matrix"] == "water":
        return _water(case["n"], seed)
    return _gapped(case["n"], seed)


def _symmetric(n, seed, std):
    a = std * torch.randn(n, n, generator=_gen(seed, 1), device=DEV)
    return torch.triu(a) + torch.triu(a, 1).T


def _iterate(n, seed):
    """A symmetric matrix with eigenvalues in [0, 1] as the layers meet it:
    random off-diagonal part, diagonal entries between 0 and 1."""
    x = _symmetric(n, seed, 0.08 / math.sqrt(n))
    x.diagonal().copy_(0.2 + 0.6 * torch.rand(n, generator=_gen(seed, 2), device=DEV))
    return x


def _options(case):
    o = dict(MODES[case["mode"]])
    if case["kind"] in ("gradient", "response"):
        o.update(checkpoint_every=4, split_derivatives=bool(case["split"]))
    return o


def _workspace(n, o):
    return pk.allocate_workspace(n, pk.make_options(**o), DEV)


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    s = dict(case=case)
    if kind == "solve":
        s["H"], s["n_occ"] = _hamiltonian(case, seed)
        s["opts"] = _options(case)
        s["ws"] = _workspace(n, s["opts"])
    elif kind == "mdstep":
        s["H"], s["n_occ"] = _water(n, seed)
        s["H_old"], _ = _water(n, seed, wobble=0.004)
        s["opts"] = _options(case)
        s["ws"] = _workspace(n, s["opts"])
        s["P_old"] = pk.density(s["H_old"], s["n_occ"], workspace=s["ws"], **s["opts"])
    elif kind == "layer":
        ld = n + case["pad"]
        s["X"] = torch.zeros(n, ld, device=DEV)[:, :n]
        s["X"].copy_(_iterate(n, seed))
        s["Y"] = torch.zeros(n, ld, device=DEV)[:, :n]
        s["ws"] = _workspace(n, dict(precision=case["precision"], refine="none"))
    elif kind == "gradient":
        s["H"], s["n_occ"] = _hamiltonian(case, seed)
        s["H"].requires_grad_(True)
        s["W"] = _symmetric(n, seed, 1.0)
        s["opts"] = _options(case)
        s["ws"] = _workspace(n, s["opts"])
    elif kind == "response":
        s["H"], s["n_occ"] = _hamiltonian(case, seed)
        s["H1"] = _symmetric(n, seed, 1e-3)
        s["P1"] = torch.empty_like(s["H1"])
        s["opts"] = _options(case)
        s["ws"] = _workspace(n, s["opts"])
        pk.density(s["H"], s["n_occ"], workspace=s["ws"], **s["opts"])
    else:
        g = _gen(seed)
        f64 = dict(device=DEV, dtype=torch.float64, generator=g)
        s["R"], s["V"] = torch.randn(n, **f64), 0.005 * torch.randn(n, **f64)
        s["F"], s["F_new"] = torch.randn(n, **f64), torch.randn(n, **f64)
        s["eta"] = torch.randn(n, **f64)
        mass = 103.642 * torch.tensor([15.999, 1.008, 1.008], device=DEV, dtype=torch.float64)
        s["mass"] = mass.repeat_interleave(3).repeat(-(-n // 9))[:n].contiguous()
        s["params"] = pk.nvt_params(**_nvt(case))
    return s


def _nvt(case):
    return dict(dt=0.5, kt=0.0431, gamma_tc=0.02, gamma_l=0.01, scheme=case["scheme"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "solve":
        return {"P": pk.density(s["H"], s["n_occ"], workspace=s["ws"], **s["opts"])}
    if kind == "mdstep":
        homo, lumo = pk.homo_lumo(s["H_old"], s["P_old"], steps=12, workspace=s["ws"])
        P = pk.density(s["H"], s["n_occ"], workspace=s["ws"], homo=homo, lumo=lumo, **s["opts"])
        return {"P": P, "homo": homo, "lumo": lumo}
    if kind == "layer":
        return {"Y": pk.sp2_layer(s["X"], case["precision"], case["sign"], s["Y"], s["ws"])}
    if kind == "gradient":
        P = pk.SP2Density.apply(s["H"], s["n_occ"], dict(s["opts"], workspace=s["ws"]))
        (G,) = torch.autograd.grad(P, s["H"], s["W"])
        return {"P": P.detach(), "G": G}
    if kind == "response":
        return {"P1": pk.sp2_jvp(s["ws"], s["H1"], s["P1"])}
    pk.sp2_nvt_first_half(s["R"], s["V"], s["F"], s["eta"], s["mass"], s["params"])
    pk.sp2_nvt_second_half(s["V"], s["F_new"], s["mass"], s["params"])
    return {"R": s["R"], "V": s["V"]}


# ---- the same in FP64 -------------------------------------------------------

def _eigh(H, n_occ):
    e, v = torch.linalg.eigh(H.detach().double())
    return e, v[:, :n_occ].contiguous(), v[:, n_occ:].contiguous()


def _projector(occ):
    return occ @ occ.T.contiguous()


def _first_order(e, occ, virt, A):
    """First-order change of the projector on occ under A (its own adjoint)."""
    n_occ = occ.shape[1]
    a = A.double()
    c = (occ.T.contiguous() @ a @ virt) / (e[:n_occ, None] - e[None, n_occ:])
    d = occ @ c @ virt.T.contiguous()
    return d + d.T


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "solve":
        if n > 12288:
            return None   # the diagonalisation takes too long
        H, n_occ = _hamiltonian(case, seed)
        return {"P": _projector(_eigh(H, n_occ)[1])}
    if kind == "mdstep":
        H, n_occ = _water(n, seed)
        return {"P": _projector(_eigh(H, n_occ)[1]), "homo": None, "lumo": None}
    if kind == "layer":
        x = _iterate(n, seed).double()
        y = x @ x
        return {"Y": y if case["sign"] > 0 else 2 * x - y}
    if kind in ("gradient", "response"):
        H, n_occ = _hamiltonian(case, seed)
        e, occ, virt = _eigh(H, n_occ)
        if kind == "response":
            return {"P1": _first_order(e, occ, virt, _symmetric(n, seed, 1e-3))}
        return {"P": _projector(occ), "G": _first_order(e, occ, virt, _symmetric(n, seed, 1.0))}
    s = prepare(case, seed)
    p = _nvt(case)
    R, V, F, m, dt, g = s["R"], s["V"], s["F"], s["mass"], p["dt"], p["gamma_tc"]
    c_l = (1 - p["gamma_l"] * dt / 2) / (1 + p["gamma_l"] * dt / 2)
    h = dt / (2 * m)
    noise = torch.sqrt(p["kt"] * (1 - c_l * c_l) / m) * s["eta"]
    if case["scheme"] == 0:
        v1 = V + h * (F - g * V)
        w = c_l * v1 + noise
        v = (w + h * s["F_new"]) / (1 + g * h)
    else:
        f = torch.sqrt((1 - g * h) / (1 + g * h))
        v1 = V + h * F
        w = f * (c_l * (f * v1) + noise)
        v = w + h * s["F_new"]
    return {"R": R + dt / 2 * v1 + dt / 2 * w, "V": v}


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "nvt":
        # R, V read and written, F, eta, mass read, then V, F, mass, V
        return {"bytes": 8.0 * 8 * n, "flops": 30.0 * n}
    cube, square = float(n) ** 3, 4.0 * n * n
    if kind == "layer":
        # a symmetric result: half of a full product's 2 n^3
        return {"bytes": 2 * square, "flops": PRODUCTS[case["precision"]] * cube}
    o = MODES[case["mode"]]
    layers = LAYERS["accelerated" if kind == "mdstep" else case["mode"]]
    products = PRODUCTS[o["precision"]]
    flops = layers * products * cube + 2 * (3 if o["refine"] == "split" else 1) * cube
    if kind == "solve":
        return {"bytes": 2 * square, "flops": flops}
    if kind == "mdstep":
        return {"bytes": 4 * square, "flops": flops + 12 * 4 * 4.0 * n * n}
    # derivative layers: S D + D S each, and the refinement's derivative (7 half products)
    each = 3 if case["split"] else 1
    deriv = (2 * layers + 7) * each * cube
    if kind == "gradient":
        return {"bytes": 4 * square, "flops": flops + deriv}
    # the response recomputes the forward layers from the tape
    return {"bytes": 2 * square, "flops": layers * products * cube + deriv}
