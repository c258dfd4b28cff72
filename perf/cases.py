"""The work this library does for its users, as cases that can be timed.

Every case goes through the public entry points of paper_2603_23343_amd. What
a program keeps between calls (contexts, coefficient fields, networks,
batches, stored matrices) is made in prepare(); run() is one pass.

Kinds:
  kernels  stencil_apply, axpy and dot on one grid (the solver's building
           blocks, called one by one)
  solve    pcg_solve: Jacobi-PCG, constant or cell coefficients
  refined  pcg_solve_refined: FP64 refinement around 16-bit inner solves
  mg       pcg_solve_mg: PCG with the multigrid V-cycle
  batch    pcg_batch_solve: many uneven problems in one launch
  forward  cnn_forward: the network preconditioner's inference
  train    cnn_loss_grad and cnn_adam_step: one training step
  sell     pcg_sell_solve: Jacobi-PCG on a stored sparse matrix

Solves of FP32 right-hand sides run to 1e-8 with an FP64 x (an FP32 x cannot
hold a residual of 1e-6 on the larger grids), and the program takes the
solution back to its own FP32: an error of the solution is up to some twenty
times the residual's, so that is what an FP32-accurate field needs. Solves in
FP64 run to 1e-12, refinement to its default 1e-10.
"""
import math

import numpy as np
import torch

import paper_2603_23343_amd as P
from paper_2603_23343_amd.learned import he_init
from synthetic import batch_sizes, poisson7_csr

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}
BYTES = {"f32": 4, "f64": 8, "bf16": 2, "f16": 2}
CNN_CHANNELS = (2, 16, 16, 16, 1)
RTOL = 1e-8


def listed():
    return [
        # The three building blocks called on their own at the size their
        # bandwidth is quoted on.
        {"name": "kernels-512", "kind": "kernels", "nx": 512, "ny": 512, "nz": 512, "dtype": "f32"},
        # The smallest solve of the benchmark: latency and launches count.
        {"name": "solve-32", "kind": "solve", "nx": 32, "ny": 32, "nz": 32, "dtype": "f32", "coef": False},
        # An ordinary grid with odd edges (scalar rows, ragged tiles).
        {"name": "solve-odd", "kind": "solve", "nx": 101, "ny": 77, "nz": 59, "dtype": "f32", "coef": False},
        # The paper's comparison grid.
        {"name": "solve-paper-grid", "kind": "solve", "nx": 512, "ny": 112, "nz": 64, "dtype": "f32", "coef": False},
        # The benchmark's headline solve.
        {"name": "solve-256", "kind": "solve", "nx": 256, "ny": 256, "nz": 256, "dtype": "f32", "coef": False},
        # The learned workload's operator under plain Jacobi-PCG.
        {"name": "solve-coef-128", "kind": "solve", "nx": 128, "ny": 128, "nz": 128, "dtype": "f32", "coef": True},
        # Mixed precision: BF16 inner solves, FP64 solution.
        {"name": "refined-bf16-256", "kind": "refined", "n": 256, "dtype": "bf16"},
        # The strongest preconditioner on the benchmark's grid.
        {"name": "mg-256", "kind": "mg", "nx": 256, "ny": 256, "nz": 256, "coef": False},
        # The benchmark's batch of 64 cubes, edges log-uniform in [16, 128].
        {"name": "batch-64", "kind": "batch", "count": 64, "sizes": 5, "lo": 16, "hi": 128},
        # One application of the network at the learned workload's size.
        {"name": "forward-128", "kind": "forward", "n": 128},
        # One training step at that size and the workflow's batch.
        {"name": "train-128", "kind": "train", "n": 128, "batch": 8},
        # A matrix without a stencil structure the library could use.
        {"name": "sell-96", "kind": "sell", "nx": 96, "ny": 96, "nz": 96},
    ]


def _edge(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(v, m, lo):
    return max(lo, (v // m) * m)


def draw(rng):
    kind = rng.choice(["kernels", "solve", "solve", "solve", "refined", "mg", "batch", "forward", "train", "sell"])
    if kind == "kernels":
        nx, ny, nz = (_edge(rng, 24, 512) for _ in range(3))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "dtype": rng.choice(["f32", "bf16", "f16", "f64"])}
    if kind == "solve":
        coef = rng.random() < 0.3
        dtype = "f64" if rng.random() < 0.2 else "f32"
        hi = 128 if coef or dtype == "f64" else 256
        nx, ny, nz = (_edge(rng, 16, hi) for _ in range(3))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "dtype": dtype, "coef": coef}
    if kind == "refined":
        return {"kind": kind, "n": _edge(rng, 40, 224), "dtype": rng.choice(["bf16", "f16"])}
    if kind == "mg":
        nx, ny, nz = (_mult(_edge(rng, 48, 224), 32, 32) for _ in range(3))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "coef": rng.random() < 0.4}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(8, 60), "sizes": rng.randint(100, 10 ** 6), "lo": 16,
                "hi": rng.choice([64, 96, 120])}
    if kind == "forward":
        return {"kind": kind, "n": _edge(rng, 24, 120)}
    if kind == "train":
        return {"kind": kind, "n": _edge(rng, 24, 112), "batch": rng.randint(2, 8)}
    nx, ny, nz = (_edge(rng, 24, 88) for _ in range(3))
    return {"kind": kind, "nx": nx, "ny": ny, "nz": nz}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(seed, n, dtype):
    """U[-1, 1) drawn in FP64, rounded to FP32 and then to the storage type."""
    u = torch.rand(n, generator=_gen(seed), dtype=torch.float64, device=DEV) * 2 - 1
    return u if dtype == torch.float64 else u.float().to(dtype)


def _field(seed, nx, ny, nz, corr=8.0):
    """A smooth random field (white noise under a Gaussian of the workload's
    correlation length), mean 0 and standard deviation 1, FP64 [nz, ny, nx]."""
    f = torch.randn(nz, ny, nx, generator=_gen(seed + 7919), dtype=torch.float64, device=DEV)
    for axis, n in ((2, nx), (1, ny), (0, nz)):
        i = torch.arange(n, dtype=torch.float64, device=DEV)
        w = torch.exp(-((i[:, None] - i[None, :]) ** 2) / corr ** 2)
        f = _along(f, w, axis)
    return (f - f.mean()) / f.std()


def _along(f, w, axis):
    """w (symmetric) applied along one axis of f."""
    g = f.movedim(axis, -1).contiguous()
    return (g.reshape(-1, g.shape[-1]) @ w).reshape(g.shape).movedim(-1, axis).contiguous()


def _shift(u, axis, step):
    """u moved by one point along axis, zeros coming in (the ghost points)."""
    v = torch.zeros_like(u)
    n = u.shape[axis]
    if step > 0:
        v.narrow(axis, 1, n - 1).copy_(u.narrow(axis, 0, n - 1))
    else:
        v.narrow(axis, 0, n - 1).copy_(u.narrow(axis, 1, n - 1))
    return v


def _apply64(u, k=None):
    """The seven-point operator in FP64 on [nz, ny, nx] (k: cell values)."""
    if k is None:
        out = 6 * u
        for axis in range(3):
            out -= _shift(u, axis, 1)
            out -= _shift(u, axis, -1)
        return out
    out = torch.zeros_like(u)
    for axis in range(3):
        for step in (1, -1):
            kn = _shift(k, axis, step)
            kf = torch.where(kn == 0, k, 2 * k * kn / (k + kn))
            out += kf * (u - _shift(u, axis, step))
    return out


def _diag64(k):
    d = torch.zeros_like(k)
    for axis in range(3):
        for step in (1, -1):
            kn = _shift(k, axis, step)
            d += torch.where(kn == 0, k, 2 * k * kn / (k + kn))
    return d


def _poisson64(b):
    """A^-1 b for constant coefficients: sine transforms along each axis."""
    shape, lam = b.shape, 0
    for axis, n in enumerate(shape):
        i = torch.arange(1, n + 1, dtype=torch.float64, device=DEV)
        s = math.sqrt(2 / (n + 1)) * torch.sin(math.pi / (n + 1) * (i[:, None] * i[None, :]))
        b = _along(b, s, axis)
        view = [1, 1, 1]
        view[axis] = n
        lam = lam + (2 - 2 * torch.cos(math.pi * i / (n + 1))).reshape(view)
    b = b / lam
    for axis, n in enumerate(shape):
        i = torch.arange(1, n + 1, dtype=torch.float64, device=DEV)
        s = math.sqrt(2 / (n + 1)) * torch.sin(math.pi / (n + 1) * (i[:, None] * i[None, :]))
        b = _along(b, s, axis)
    return b


def _cg64(b, k):
    """A_k^-1 b in FP64 by Jacobi-CG to a residual of 1e-14."""
    dinv = 1 / _diag64(k)
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rho, stop = z.clone(), torch.sum(r * z), 1e-14 * torch.linalg.vector_norm(b)
    for it in range(4000):
        q = _apply64(p, k)
        a = rho / torch.sum(p * q)
        x += a * p
        r -= a * q
        if it % 16 == 0 and torch.linalg.vector_norm(r) <= stop:
            break
        z = dinv * r
        new = torch.sum(r * z)
        p, rho = z + (new / rho) * p, new
    return x


def _shape(case):
    return (case["nx"], case["ny"], case["nz"]) if "nx" in case else (case["n"],) * 3


def _coef(seed, nx, ny, nz):
    g = _field(seed, nx, ny, nz)
    return torch.exp(g).float().reshape(-1), g.float().reshape(-1)


def _refined_b(seed, n):
    """b = A x*, x* the lowest sine mode plus 1e-3 U[-1, 1) noise."""
    s = torch.sin(math.pi * torch.arange(1, n + 1, dtype=torch.float64, device=DEV) / (n + 1))
    x = s[:, None, None] * s[None, :, None] * s[None, None, :]
    x = x + 1e-3 * _uniform(seed, n ** 3, torch.float64).reshape(n, n, n)
    return _apply64(x).reshape(-1), x.reshape(-1)


def _edges(case):
    return batch_sizes(case["count"], case["sizes"], case["lo"], case["hi"])


def _weights(seed):
    return torch.from_numpy(he_init(seed)).to(DEV)


def _pairs(seed, n, batch, k, g):
    """(residual, error) pairs as a solve leaves them: smooth errors e with
    some roughness, r = A e, both scaled by rms(r), in BF16."""
    k64 = k.double().reshape(n, n, n)
    out = torch.empty(batch, 2, n ** 3, dtype=torch.bfloat16, device=DEV)
    for j in range(batch):
        e = _field(seed + 31 * j, n, n, n, corr=4.0)
        e = e + 0.1 * _uniform(seed + 31 * j + 1, n ** 3, torch.float64).reshape(n, n, n)
        r = _apply64(e, k64)
        rho = torch.sqrt(torch.mean(r * r))
        out[j, 0] = (r / rho).reshape(-1).float().to(torch.bfloat16)
        out[j, 1] = (e / rho).reshape(-1).float().to(torch.bfloat16)
    return out.reshape(-1)


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "batch":
        dims = [(e, e, e) for e in _edges(case)]
        s["h"] = P.pcg_batch_create(dims)
        s["b"] = torch.zeros(s["h"].total, dtype=torch.float32, device=DEV)
        for i in range(len(dims)):
            v = s["h"].view(s["b"], i)
            v.copy_(_uniform(seed * 1000 + i, v.numel(), torch.float32))
        s["x"] = torch.zeros(s["h"].total, dtype=torch.float64, device=DEV)
        return s
    nx, ny, nz = _shape(case)
    n = nx * ny * nz
    if kind == "kernels":
        dt = DTYPES[case["dtype"]]
        s["ctx"] = P.pcg_create(nx, ny, nz, dt)
        s["x"], s["y"] = _uniform(seed, n, dt), _uniform(seed + 1, n, dt)
        s["ax"], s["z"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        s["d"] = torch.empty(1, dtype=torch.float32, device=DEV)
        s["n"] = n
    elif kind == "solve":
        dt = DTYPES[case["dtype"]]
        s["ctx"] = P.pcg_create(nx, ny, nz, dt, x_dtype=torch.float64)
        if case["coef"]:
            s["k"], _ = _coef(seed, nx, ny, nz)
            P.pcg_set_coefficients(s["ctx"], s["k"])
        s["b"] = _uniform(seed, n, dt)
        s["x"] = torch.empty(n, dtype=torch.float64, device=DEV)
        s["f64"] = case["dtype"] == "f64"
    elif kind == "refined":
        s["ctx"] = P.pcg_create(nx, ny, nz, DTYPES[case["dtype"]], x_accum=torch.float32)
        s["b"], _ = _refined_b(seed, nx)
        s["x"] = torch.empty(n, dtype=torch.float64, device=DEV)
    elif kind == "mg":
        s["ctx"] = P.pcg_create(nx, ny, nz, torch.float32, x_dtype=torch.float64)
        if case["coef"]:
            s["k"], _ = _coef(seed, nx, ny, nz)
            P.pcg_set_coefficients(s["ctx"], s["k"])
        P.pcg_set_multigrid(s["ctx"])
        s["b"] = _uniform(seed, n, torch.float32)
        s["x"] = torch.empty(n, dtype=torch.float64, device=DEV)
    elif kind in ("forward", "train"):
        s["net"] = P.cnn_create()
        s["shape"] = (nz, ny, nx)
        P.cnn_set_weights(s["net"], _weights(seed))
        s["k"], s["g"] = _coef(seed, nx, ny, nz)
        if kind == "forward":
            s["r"] = _uniform(seed, n, torch.float32)
            s["rr"] = torch.sum(s["r"].double() ** 2).reshape(1)
            s["z"] = torch.empty(n, dtype=torch.float32, device=DEV)
        else:
            s["ctx"] = P.pcg_create(nx, ny, nz, torch.float32)
            P.pcg_set_coefficients(s["ctx"], s["k"])
            P.cnn_set_operator(s["net"], s["ctx"])
            s["batch"] = case["batch"]
            s["pairs"] = _pairs(seed, nx, case["batch"], s["k"], s["g"])
            s["grad"] = torch.empty(P.cnn_num_weights(), dtype=torch.float32, device=DEV)
            s["w"] = torch.empty_like(s["grad"])
            s["loss"] = torch.empty(1, dtype=torch.float64, device=DEV)
    elif kind == "sell":
        rowptr, col, val = poisson7_csr(nx, ny, nz)
        s["A"] = P.pcg_sell_create(rowptr, col, val, n)
        s["b"] = _uniform(seed, n, torch.float32)
        s["x"] = torch.empty(n, dtype=torch.float64, device=DEV)
    return s


def run(s):
    kind = s["kind"]
    if kind == "kernels":
        P.stencil_apply(s["ctx"], s["x"], s["ax"])
        P.axpy(s["ctx"], s["n"], 0.5, s["x"], s["y"], s["z"])
        P.dot(s["ctx"], s["n"], s["x"], s["x"], s["d"])  # a squared norm
        return {"ax": s["ax"], "z": s["z"], "d": s["d"]}
    if kind == "solve":
        P.pcg_solve(s["ctx"], s["b"], s["x"], 1e-12 if s["f64"] else RTOL, 4000)
        return s["x"] if s["f64"] else s["x"].float()
    if kind == "refined":
        P.pcg_solve_refined(s["ctx"], s["b"], s["x"], 1e-10)
        return s["x"]
    if kind == "mg":
        P.pcg_solve_mg(s["ctx"], s["b"], s["x"], RTOL)
        return s["x"].float()
    if kind == "batch":
        P.pcg_batch_solve(s["h"], s["b"], s["x"], RTOL, 2000)
        x = s["x"].float()
        return [s["h"].view(x, i) for i in range(len(s["h"]))]
    if kind == "forward":
        P.cnn_forward(s["net"], s["shape"], s["r"], s["g"], s["z"], s["rr"])
        return s["z"]
    if kind == "train":
        P.cnn_loss_grad(s["net"], s["shape"], s["pairs"], s["g"], s["batch"], s["grad"], s["loss"])
        P.cnn_adam_step(s["net"], s["grad"], 1e-3)
        P.cnn_get_weights(s["net"], s["w"])
        return {"grad": s["grad"], "w": s["w"], "loss": s["loss"]}
    P.pcg_sell_solve(s["A"], s["b"], s["x"], RTOL, 2000)
    return s["x"].float()


# ------------------------------------------------------------------ accounting


def _conv_flops(n):
    return n * sum(2 * 27 * a * b for a, b in zip(CNN_CHANNELS, CNN_CHANNELS[1:]))


def work(case):
    """Inputs read once and outputs written once (a solution in FP32, or FP64
    where that is returned). Flops of a solve: about 20 per point and
    iteration, with the iterations Jacobi-PCG takes on a uniform right-hand
    side (about 1.5 per point of the longest edge at 1e-8, 2 at 1e-12, several
    times that with cell coefficients), 20 V-cycles of about 60 flops for
    multigrid."""
    kind = case["kind"]
    if kind == "batch":
        e = _edges(case)
        return {"bytes": sum(8 * v ** 3 for v in e), "flops": sum(20 * 1.5 * v * v ** 3 for v in e)}
    nx, ny, nz = _shape(case)
    n, longest = nx * ny * nz, max(nx, ny, nz)
    if kind == "kernels":
        es = BYTES[case["dtype"]]
        return {"bytes": 4 * es * n + 4, "flops": 12 * n}
    if kind == "solve":
        es = BYTES[case["dtype"]]
        its = longest * (2.0 if case["dtype"] == "f64" else 1.5) * (4.0 if case["coef"] else 1.0)
        return {"bytes": n * (2 * es + (4 if case["coef"] else 0)), "flops": 20 * n * its}
    if kind == "refined":
        return {"bytes": 16 * n, "flops": 20 * n * 5.0 * longest}
    if kind == "mg":
        return {"bytes": n * (8 + (4 if case["coef"] else 0)), "flops": 20 * 60 * n}
    if kind == "forward":
        return {"bytes": 12 * n + 4 * 15120, "flops": _conv_flops(n)}
    if kind == "train":
        first = 2 * 27 * CNN_CHANNELS[0] * CNN_CHANNELS[1]  # no input gradient for the first layer
        return {"bytes": case["batch"] * 4 * n + 8 * n + 8 * 4 * 15120,
                "flops": case["batch"] * (3 * _conv_flops(n) - first * n)}
    return {"bytes": 8 * n + 8 * 7 * n, "flops": 30 * n * 1.5 * longest}


# ------------------------------------------------------------------ 64 bits


def _net64(r, g, w):
    """The network in FP64: r, g [nz, ny, nx]; w a list of [27, cin, cout]."""
    a = torch.stack([r, g]).reshape(2, -1)
    shape = r.shape
    for layer, wl in enumerate(w):
        cin, cout = wl.shape[1:]
        grid = torch.nn.functional.pad(a.reshape(cin, *shape), (1, 1, 1, 1, 1, 1))
        out = 0
        for t in range(27):
            dz, dy, dx = t // 9, (t // 3) % 3, t % 3
            part = grid[:, dz:dz + shape[0], dy:dy + shape[1], dx:dx + shape[2]].reshape(cin, -1)
            out = out + wl[t].t().contiguous() @ part
        a = torch.relu(out) if layer < 3 else out
    return a.reshape(shape)


def _split(w):
    out, at = [], 0
    for a, b in zip(CNN_CHANNELS, CNN_CHANNELS[1:]):
        out.append(w[at:at + 27 * a * b].reshape(27, a, b))
        at += 27 * a * b
    return out


class _Operator(torch.autograd.Function):
    """A_k u (symmetric, so its own transpose)."""

    @staticmethod
    def forward(ctx, u, k):
        ctx.save_for_backward(k)
        return _apply64(u, k)

    @staticmethod
    def backward(ctx, v):
        return _apply64(v, ctx.saved_tensors[0]), None


def _exact_train(case, seed):
    n, batch = case["n"], case["batch"]
    k, g = _coef(seed, n, n, n)
    pairs = _pairs(seed, n, batch, k, g).double().reshape(batch, 2, n, n, n)
    k64 = k.double().reshape(n, n, n)
    dinv = 1 / _diag64(k64)
    w = _weights(seed).double().requires_grad_()
    loss = torch.zeros((), dtype=torch.float64, device=DEV)
    for j in range(batch):
        rh, eh = pairs[j, 0], pairs[j, 1]
        u = _net64(rh, g.double().reshape(n, n, n), _split(w)) + dinv * rh - eh
        part = torch.sum(u * _Operator.apply(u, k64)) / torch.sum(rh * dinv * rh) / batch
        part.backward()
        loss += part.detach()
    grad = w.grad
    # Adam's first step: the bias-corrected moments are g and g^2
    new = w.detach() - 1e-3 * grad / (grad.abs() + 1e-8)
    return {"grad": grad, "w": new, "loss": loss.reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, e in enumerate(_edges(case)):
            b = _uniform(seed * 1000 + i, e ** 3, torch.float32).double().reshape(e, e, e)
            out.append(_poisson64(b).reshape(-1))
        return out
    nx, ny, nz = _shape(case)
    n, grid = nx * ny * nz, (nz, ny, nx)
    if kind == "kernels":
        dt = DTYPES[case["dtype"]]
        x, y = _uniform(seed, n, dt).double(), _uniform(seed + 1, n, dt).double()
        return {"ax": _apply64(x.reshape(grid)).reshape(-1), "z": 0.5 * x + y, "d": torch.sum(x * x).reshape(1)}
    if kind == "refined":
        return _refined_b(seed, nx)[1]
    if kind == "solve":
        b = _uniform(seed, n, DTYPES[case["dtype"]]).double().reshape(grid)
        if case["coef"]:
            return _cg64(b, _coef(seed, nx, ny, nz)[0].double().reshape(grid)).reshape(-1)
        return _poisson64(b).reshape(-1)
    if kind in ("mg", "sell"):
        b = _uniform(seed, n, torch.float32).double().reshape(grid)
        if case.get("coef"):
            return _cg64(b, _coef(seed, nx, ny, nz)[0].double().reshape(grid)).reshape(-1)
        return _poisson64(b).reshape(-1)
    if kind == "forward":
        g = _coef(seed, nx, ny, nz)[1].double().reshape(grid)
        r = _uniform(seed, n, torch.float32).double().reshape(grid)
        rms = torch.sqrt(torch.mean(r * r))
        return (rms * _net64(r / rms, g, _split(_weights(seed).double()))).reshape(-1)
    return _exact_train(case, seed)
