"""Workloads of the library as its users call it, for timing and for comparing results.

Every case goes through the package's public functions: ``fuse_stack`` (FP32,
FP64 and mixed precision, plain and robust averaging, both boundary
conditions), ``solve_slices`` (uneven batches, eager and captured),
``ScreenedPoissonSolve`` (forward and backward), ``fuse_stack_backward`` and
``fuse_color``.  Inputs are EM-like: a band-limited noise texture with Gaussian
blobs, per-slice gain and offset and, for stacks, a linear illumination ramp,
clipped to uint8.

``fuse_stack_streamed`` is the same ``fuse_stack`` call per chunk between two
PCIe copies that bound it, so it has no case of its own.  The per-slice reports
(cycle counts, residuals) describe the iteration and are not outputs here.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1506_02079_amd as gdf

DEV = "cuda"
SIGMA_XY, SIGMA_Z = 1.0, 3.0          # the paper's widths, the library's defaults
R_XY, R_Z = 3, 9                      # floor(3 sigma) taps on either side
TAPS = 2 * (2 * R_XY + 1) + (2 * R_Z + 1)


# ------------------------------------------------------------------ the cases

def _fuse(name, S, H, W, alpha, precision="fp32", tol=1e-6, bc="neumann", robust=False, smooth=False,
          fine_sweeps=0, sor=False):
    return {"name": name, "kind": "fuse", "S": S, "H": H, "W": W, "alpha": alpha, "precision": precision,
            "tol": tol, "bc": bc, "robust": robust, "smooth": smooth, "fine_sweeps": fine_sweeps, "sor": sor}


def listed():
    return [
        # a thumbnail or a unit test's stack: nothing but latency and launches
        _fuse("fuse_tiny", 6, 96, 80, 0.01),
        # the plain method in double precision on a small stack (a reference run)
        _fuse("fuse_small_fp64", 8, 256, 256, 0.01, precision="fp64"),
        # a cut-out with odd sides, the paper's weak screening, the smoothed stack kept as well
        _fuse("fuse_ragged_smooth", 33, 1021, 1531, 0.001, smooth=True),
        # the benchmark's stack and settings: a block of an EM volume
        _fuse("fuse_block", 64, 2048, 2048, 0.01, fine_sweeps=4, sor=True),
        # damaged slices in the stack: robust cross-slice averaging
        _fuse("fuse_robust", 40, 1536, 1280, 0.01, robust=True),
        # the paper's Fourier basis: wrap-around slices
        _fuse("fuse_periodic", 12, 1024, 1200, 0.01, bc="periodic"),
        # whole sections at the paper's slice size and weight, refined in double precision
        _fuse("fuse_sections_mixed", 2, 21504, 26624, 0.001, precision="mixed", tol=1e-9),
        # sections of many sizes and weights, captured once and replayed
        {"name": "batch_uneven_graph", "kind": "batch", "n": 96, "lo": 512, "hi": 4096, "step": 256,
         "sizes": 1002, "alpha_lo": 0.001, "alpha_hi": 0.1, "graph": True},
        # many patches of odd sizes in one eager call
        {"name": "batch_patches", "kind": "batch", "n": 200, "lo": 17, "hi": 300, "step": 1,
         "sizes": 7, "alpha_lo": 0.001, "alpha_hi": 0.1, "graph": False},
        # a training step through the solve: forward, loss, gradients of both images and of alpha
        {"name": "train_step", "kind": "train", "S": 16, "H": 1024, "W": 1024, "alpha": 0.01},
        # the gradient of a loss with respect to the raw stack: adjoint solve and transposed smoothing
        {"name": "stack_gradient", "kind": "stackgrad", "S": 24, "H": 901, "W": 1100, "alpha": 0.01},
        # a low-frequency colour image with a grey image's gradients
        {"name": "color", "kind": "color", "C": 3, "H": 4096, "W": 4096, "alpha": 0.01},
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _side(rng, lo, hi):
    """A side, log-uniform; half of them multiples of 4, the others as they come."""
    v = _logint(rng, lo, hi)
    return v if rng.random() < 0.5 else max(4, v // 4 * 4)


def draw(rng):
    alpha = round(math.exp(rng.uniform(math.log(0.001), math.log(0.1))), 5)
    kind = rng.choice(["fuse"] * 6 + ["batch"] * 2 + ["train", "stackgrad", "color"])
    if kind == "fuse":
        precision = rng.choice(["fp32"] * 4 + ["mixed", "fp64"])
        H, W = _side(rng, 60, 2400), _side(rng, 60, 2400)
        robust = precision != "fp64" and rng.random() < 0.2
        bc = "periodic" if rng.random() < 0.15 else "neumann"
        cap = {"fp32": 2.6e8, "mixed": 6e7, "fp64": 1.6e7}[precision] * (0.2 if bc == "periodic" else 1.0)
        S = _logint(rng, 2, max(3, min(64, int(cap / (H * W)))))
        sor = precision == "fp32" and bc == "neumann" and rng.random() < 0.3
        c = _fuse("", S, H, W, alpha, precision, 1e-9 if precision == "mixed" else 1e-6, bc, robust,
                  rng.random() < 0.3, 4 if sor else 0, sor)
        del c["name"]
        return c
    if kind == "batch":
        hi = _logint(rng, 64, 3000)
        lo = max(9, hi // rng.randint(2, 12))
        n = _logint(rng, 3, max(4, min(300, int(1.5e8 / (0.4 * hi * hi)))))
        return {"kind": "batch", "n": n, "lo": lo, "hi": hi, "step": rng.choice([1, 1, 4, 32]),
                "sizes": rng.randrange(1 << 20), "alpha_lo": 0.001, "alpha_hi": 0.1, "graph": rng.random() < 0.5}
    if kind == "color":
        return {"kind": "color", "C": rng.choice([3, 4]), "H": _side(rng, 200, 4000), "W": _side(rng, 200, 4000),
                "alpha": alpha}
    H, W = _side(rng, 100, 1600), _side(rng, 100, 1600)
    return {"kind": kind, "S": _logint(rng, 2, max(3, min(48, int(4e7 / (H * W))))), "H": H, "W": W, "alpha": alpha}


# ----------------------------------------------------------------- the inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _taps(sigma, radius):
    return [math.exp(-d * d / (2.0 * sigma * sigma)) for d in range(-radius, radius + 1)]


def _blur(v, taps):
    """Separable blur of the last two axes, edges replicated, weights normalised."""
    r = len(taps) // 2
    total = sum(taps)
    for dim in (-1, -2):
        n = v.shape[dim]
        out = torch.zeros_like(v)
        for k, t in enumerate(taps):
            d = k - r
            if abs(d) >= n:
                idx = torch.full((n,), 0 if d < 0 else n - 1, device=v.device)
                out.add_(v.index_select(dim, idx), alpha=t / total)
                continue
            if d == 0:
                out.add_(v, alpha=t / total)
            elif d > 0:
                out.narrow(dim, 0, n - d).add_(v.narrow(dim, d, n - d), alpha=t / total)
                out.narrow(dim, n - d, d).add_(v.narrow(dim, n - 1, 1), alpha=t / total)
            else:
                out.narrow(dim, -d, n + d).add_(v.narrow(dim, 0, n + d), alpha=t / total)
                out.narrow(dim, 0, -d).add_(v.narrow(dim, 0, 1), alpha=t / total)
        v = out
    return v


def _texture(seed, H, W):
    """Band-limited noise (std about 8, width 1.5 px) and up to 40 Gaussian blobs."""
    g = _gen(seed)
    base = _blur(torch.randn((H, W), generator=g, device=DEV), _taps(1.5, 5)).mul_(8.0 * 2.0 * math.sqrt(math.pi) * 1.5)
    p = torch.rand((4, max(2, min(40, H * W // 1500))), generator=g, device=DEV)
    cy, cx, sb, amp = p[0] * H, p[1] * W, 3.0 + 17.0 * p[2], 20.0 + 100.0 * p[3]
    gy = torch.exp(-((torch.arange(H, device=DEV)[:, None] - cy) / sb) ** 2 / 2) * amp
    gx = torch.exp(-((torch.arange(W, device=DEV)[:, None] - cx) / sb) ** 2 / 2)
    return base.add_(gy @ gx.t()).add_(60.0)


def _slice_u8(base, r, ramp=False):
    v = base * r.uniform(0.8, 1.2) + r.uniform(-20.0, 20.0)
    if ramp:
        H, W = base.shape
        v += r.uniform(-0.01, 0.01) * (torch.arange(W, device=DEV) - W / 2)
        v += r.uniform(-0.01, 0.01) * (torch.arange(H, device=DEV) - H / 2)[:, None]
    return v.round_().clamp_(0, 255).to(torch.uint8)


def _stack(seed, S, H, W, damage=False):
    base, r = _texture(seed, H, W), random.Random(seed)
    out = torch.empty((S, H, W), dtype=torch.uint8, device=DEV)
    for z in range(S):
        out[z] = _slice_u8(base, r, ramp=H * W < 1 << 26)
        if damage and z % 7 == 3:     # a lost tile in some slices
            y0, x0 = r.randrange(max(1, H // 2)), r.randrange(max(1, W // 2))
            out[z, y0:y0 + H // 3, x0:x0 + W // 3] = 255 * r.randrange(2)
    return out


def _batch_shapes(case):
    r = random.Random(case["sizes"])
    steps = (case["hi"] - case["lo"]) // case["step"]
    return [(case["lo"] + case["step"] * r.randint(0, steps), case["lo"] + case["step"] * r.randint(0, steps),
             r.uniform(case["alpha_lo"], case["alpha_hi"])) for _ in range(case["n"])]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "fuse":
        return {"case": case, "stack": _stack(seed, case["S"], case["H"], case["W"], case["robust"])}
    if kind == "batch":
        go, gs, alpha = [], [], []
        r = random.Random(seed)
        for i, (H, W, a) in enumerate(_batch_shapes(case)):
            base = _texture(seed * 4099 + i, H, W)
            go.append(_slice_u8(base, r))
            gs.append(_blur(base, _taps(1.0, 3)))
            alpha.append(a)
        return {"case": case, "go": go, "gs": gs, "alpha": alpha}
    if kind == "color":
        grey = _slice_u8(_texture(seed, case["H"], case["W"]), random.Random(seed)).float()
        low = _blur(_blur(grey, _taps(4.0, 12)), _taps(4.0, 12))
        color = torch.stack([low * (0.5 + 0.2 * k) + 10.0 * k for k in range(case["C"])])
        return {"case": case, "grey": grey, "color": color}
    S, H, W = case["S"], case["H"], case["W"]
    stack = _stack(seed, S, H, W)
    if kind == "train":
        gs = _blur(stack.float().mean(0, keepdim=True) * 0.5 + stack.float() * 0.5, _taps(1.0, 3))
        target = torch.rand((S, H, W), generator=_gen(seed + 1), device=DEV) * 255.0
        return {"case": case, "gs": gs.requires_grad_(), "go": stack.float().requires_grad_(), "target": target,
                "alpha": torch.tensor(case["alpha"], device=DEV, requires_grad=True)}
    f = stack.float() + torch.randn((S, H, W), generator=_gen(seed + 1), device=DEV)
    grad = 2.0 * (f - _blur(stack.float(), _taps(1.0, 3)))
    return {"case": case, "stack": stack, "f": f, "grad": grad}


# ------------------------------------------------------------------- the call

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "fuse":
        out = gdf.fuse_stack(state["stack"], case["alpha"], bc=case["bc"], tol=case["tol"],
                             precision=case["precision"], robust=case["robust"], return_smooth=case["smooth"],
                             fine_sweeps=case["fine_sweeps"], sor=case["sor"])
        return [out[0], out[2]] if case["smooth"] else [out[0]]
    if kind == "batch":
        # (the slices of the answer lie one after the other in one buffer)
        f, _ = gdf.solve_slices(state["gs"], state["go"], state["alpha"], use_graph=case["graph"])
        return [f[0]._base if f[0]._base is not None else f[0]]
    if kind == "color":
        return [gdf.fuse_color(state["color"], state["grey"], case["alpha"])[0]]
    if kind == "train":
        gs, go, alpha = state["gs"], state["go"], state["alpha"]
        gs.grad = go.grad = alpha.grad = None
        f = gdf.ScreenedPoissonSolve.apply(gs, go, alpha)
        ((f - state["target"]) ** 2).sum().backward()
        return [f.detach(), gs.grad, go.grad, alpha.grad]
    return [gdf.fuse_stack_backward(state["grad"], state["f"], state["stack"], case["alpha"])[0]]


def work(case):
    """Inputs read once, outputs written once; the smoothing's taps (a multiply
    and an add each) and one application of the five-point operator per pixel."""
    kind = case["kind"]
    if kind == "fuse":
        px = case["S"] * case["H"] * case["W"]
        e = {"fp32": 4, "fp64": 8, "mixed": 8}[case["precision"]]
        g = (8 if case["precision"] == "fp64" else 4) if case["smooth"] else 0
        return {"bytes": px * (1 + e + g), "flops": px * (2 * TAPS + 10)}
    if kind == "batch":
        px = sum(H * W for H, W, _ in _batch_shapes(case))
        return {"bytes": px * (1 + 4 + 4), "flops": px * 10}
    if kind == "color":
        px = case["H"] * case["W"]
        return {"bytes": px * (4 + 8 * case["C"]), "flops": px * case["C"] * 10}
    px = case["S"] * case["H"] * case["W"]
    if kind == "train":   # both images and the target in, f and two gradients out
        return {"bytes": px * 6 * 4, "flops": px * 30}
    return {"bytes": px * 2 * 4, "flops": px * (2 * TAPS + 20)}


# -------------------------------------------- the same in 64 bits, plain torch

def _basis(n, bc):
    """Orthonormal eigenvectors (rows) and eigenvalues of the 1D pixel-graph Laplacian."""
    j = torch.arange(n, device=DEV)
    k = j[:, None]
    if bc == "neumann":
        m = torch.cos(((k * (2 * j + 1)) % (4 * n)).double() * (math.pi / (2 * n))) * math.sqrt(2.0 / n)
        m[0] = math.sqrt(1.0 / n)
        lam = 2.0 - 2.0 * torch.cos(j.double() * (math.pi / n))
        return m, lam
    ang = ((k * j) % n).double() * (2.0 * math.pi / n)
    m = torch.where(2 * k <= n, torch.cos(ang), torch.sin(ang)) * math.sqrt(2.0 / n)
    m[0] = math.sqrt(1.0 / n)
    if n % 2 == 0:
        m[n // 2] *= math.sqrt(0.5)
    return m, 2.0 - 2.0 * torch.cos(j.double() * (2.0 * math.pi / n))


def _lap(v, bc):
    if bc == "periodic":
        return sum(v - v.roll(d, dim) for dim in (-1, -2) for d in (1, -1))
    out = torch.zeros_like(v)
    d = v[..., 1:] - v[..., :-1]
    out[..., 1:] += d
    out[..., :-1] -= d
    d = v[..., 1:, :] - v[..., :-1, :]
    out[..., 1:, :] += d
    out[..., :-1, :] -= d
    return out


class _Solver:
    """(alpha I + L)^-1 of one slice by its eigenbasis."""

    def __init__(self, H, W, alpha, bc="neumann"):
        self.ch, lh = _basis(H, bc)
        self.cw, lw = (self.ch, lh) if H == W else _basis(W, bc)
        self.den = None if H * W > 1 << 27 else lh[:, None] + lw + alpha
        self.parts = lh, lw, alpha

    def __call__(self, b):
        t = (self.ch @ b) @ self.cw.t()
        lh, lw, alpha = self.parts
        t /= self.den if self.den is not None else lh[:, None] + lw + alpha
        return (self.ch.t() @ t) @ self.cw


def _smooth64(stack, transpose=False):
    """The renormalised truncated Gaussian of a stack (or the transpose of that map)."""
    v = stack.double()
    for dim, sigma, r in ((2, SIGMA_XY, R_XY), (1, SIGMA_XY, R_XY), (0, SIGMA_Z, R_Z)):
        taps, n = _taps(sigma, r), v.shape[dim]
        w = torch.zeros(n, dtype=torch.float64, device=v.device)
        for k, t in enumerate(taps):
            d = k - r
            if abs(d) < n:
                w[max(0, -d):n - max(0, d)] += t
        shape = [1, 1, 1]
        shape[dim] = n
        w = w.view(shape)
        src = v / w if transpose else v
        out = torch.zeros_like(v)
        for k, t in enumerate(taps):
            d = k - r
            if abs(d) < n:
                out.narrow(dim, max(0, -d), n - abs(d)).add_(src.narrow(dim, max(0, d), n - abs(d)), alpha=t)
        v = out if transpose else out / w
    return v


def exact(case, seed):
    kind = case["kind"]
    if kind == "fuse" and case["robust"]:
        return None   # which values an average leaves out is decided by rounding where they tie
    s = prepare(case, seed)
    if kind == "fuse":
        st, alpha, bc = s["stack"], case["alpha"], case["bc"]
        big = case["H"] * case["W"] > 1 << 26   # (few slices: rows in blocks, to bound the memory)
        if big:
            gs = torch.empty(st.shape, dtype=torch.float64, device=DEV)
            for y in range(0, case["H"], 2048):
                a, b = max(0, y - R_XY), min(case["H"], y + 2048 + R_XY)
                # (the block's own edges are further in than the rows kept, or the slice's)
                gs[:, y:y + 2048] = _smooth64(st[:, a:b])[:, y - a:y - a + 2048]
        else:
            gs = _smooth64(st)
        solve = _Solver(case["H"], case["W"], alpha, bc)
        f = torch.empty_like(gs)
        for z in range(case["S"]):
            go = st[z].double()
            f[z] = go + solve(alpha * (gs[z] - go))
        return [f, gs] if case["smooth"] else [f]
    if kind == "batch":
        out = []
        for gs, go, a in zip(s["gs"], s["go"], s["alpha"]):
            go = go.double()
            out.append((go + _Solver(*go.shape, a)(a * (gs.double() - go))).reshape(-1))
        return [torch.cat(out)]
    alpha = float(torch.tensor(case["alpha"], dtype=torch.float32)) if kind == "train" else case["alpha"]
    solve = _Solver(case["H"], case["W"], alpha)
    if kind == "color":
        go = s["grey"].double()
        return [[go + solve(alpha * (c.double() - go)) for c in s["color"]]]
    if kind == "train":
        gs, go, t = s["gs"].detach(), s["go"].detach(), s["target"]
        f, ggs, ggo = (torch.empty(gs.shape, dtype=torch.float64, device=DEV) for _ in range(3))
        ga = 0.0
        for z in range(case["S"]):
            f[z] = go[z].double() + solve(alpha * (gs[z].double() - go[z].double()))
            lam = solve(2.0 * (f[z] - t[z].double()))
            ggs[z], ggo[z] = alpha * lam, _lap(lam, "neumann")
            ga += float((lam * (gs[z].double() - f[z])).sum())
        return [f, ggs, ggo, torch.tensor(ga, dtype=torch.float64)]
    lam = torch.stack([solve(g.double()) for g in s["grad"]])
    return [_smooth64(alpha * lam, transpose=True) + _lap(lam, "neumann")]
