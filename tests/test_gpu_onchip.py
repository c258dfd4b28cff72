"""Jacobi-PCG with the grid held on the chip (the default form of pcg_solve on
grids that fit) against the FP64 oracle, at the sizes where its boxes can go
wrong: one box, remainders in each dimension, rows longer than a box, planes
that split unevenly, the most points per thread.

Tolerance: FP32 vectors carry a relative rounding error of 2^-24 per operation
and an iteration applies a few; k iterations of well-conditioned early CG keep
the iterate and the residual norm within k * 32 * 2^-24 of the FP64 ones
(k = 20: 4e-5), FP64 storage within k * 32 * 2^-53 (7e-14).
"""
import threading

import numpy as np
import pytest
import torch

import synthetic
from gpu_helpers import dev, host64, make_vec

pytestmark = pytest.mark.gpu
ITERS = 20


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _tol(dtype):
    return ITERS * 32 * (2.0 ** -53 if dtype == torch.float64 else 2.0 ** -24)


def _coef(seed, n):
    return np.exp(synthetic.uniform(seed, n)).astype(np.float32)


# (nz, ny, nx): points per thread 2, 2, 4, 8 and ragged, 10, 32 with long rows, 20, 2 with thin boxes
CONST = [(2, 3, 5), (8, 16, 32), (17, 17, 33), (59, 77, 101), (61, 100, 40), (64, 112, 512), (130, 61, 250), (3, 200, 9)]
VAR = [(2, 3, 5), (16, 16, 32), (29, 37, 48), (59, 77, 101), (128, 128, 128), (7, 130, 70)]


@pytest.mark.parametrize("coef,shape", [(False, s) for s in CONST] + [(True, s) for s in VAR])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_iterates(P, orc, shape, coef, dtype):
    nz, ny, nx = shape
    n = nx * ny * nz
    print("grid", shape, coef, dtype, flush=True)
    b, b64 = make_vec(31, n, dtype)
    k = _coef(32, n) if coef else None
    ref = orc.pcg(shape, b64, rtol=0.0, maxit=ITERS, history=True, kcell=None if k is None else k.astype(np.float64))
    ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64)
    if coef:
        kd = dev(k)
        P.pcg_set_coefficients(ctx, kd)
    x = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    outs = []
    for _ in range(2):  # a second solve on the same context, other work between
        info = P.pcg_solve(ctx, b, x, 0.0, ITERS, raise_on_error=False)
        outs.append(host64(x).copy())
        P.axpy(ctx, n, 1.0, b, b, torch.empty_like(b))
    its = ref["iters"]
    hist = P.pcg_get_history(ctx)
    assert np.array_equal(outs[0], outs[1])
    if its < ITERS:  # CG ended on a tiny grid: only the solution is comparable
        assert np.linalg.norm(outs[0] - ref["x"]) <= 10 * _tol(dtype) * np.linalg.norm(ref["x"])
        return
    tol = _tol(dtype)
    if ref["hist"][-1] < 1e3 * tol:
        return  # converged to rounding: the recursion's last steps are noise
    assert info["iters"] == ITERS
    assert np.linalg.norm(outs[0] - ref["x"]) <= tol * np.linalg.norm(ref["x"])
    assert np.all(np.abs(hist - ref["hist"]) <= tol * ref["hist"][0])


def test_streams_and_threads(P):
    """Contexts on their own streams, solved from several threads together with
    a batched solve: every result is the one of a lone solve, bit for bit."""
    shapes = [(32, 32, 32), (40, 50, 60), (100, 96, 90), (64, 64, 64)]
    jobs = []
    for i, (nz, ny, nx) in enumerate(shapes):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctx = P.pcg_create(nx, ny, nz, torch.float32, stream=s, x_dtype=torch.float64)
            b, _ = make_vec(50 + i, nx * ny * nz, torch.float32)
            x = torch.empty(b.numel(), dtype=torch.float64, device="cuda")
        s.synchronize()
        P.pcg_solve(ctx, b, x, 1e-6, 1000)
        jobs.append((s, ctx, b, x, host64(x).copy()))
    dims = [(24, 24, 24), (40, 30, 20)]
    bs = torch.cuda.Stream()
    bt = P.pcg_batch_create(dims, cfgs=[0, 0], stream=bs)
    bb = dev(synthetic.uniform_f32(60, bt.total))
    bx = torch.zeros(bt.total, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    P.pcg_batch_solve(bt, bb, bx, 1e-6, 1000)
    bwant = host64(bx).copy()
    failed = []

    def work(job):
        try:
            _, ctx, b, x, want = job
            for _ in range(5):
                P.pcg_solve(ctx, b, x, 1e-6, 1000)
                if not np.array_equal(host64(x), want):
                    failed.append("solve")
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    def batch():
        try:
            for _ in range(5):
                P.pcg_batch_solve(bt, bb, bx, 1e-6, 1000)
                if not np.array_equal(host64(bx), bwant):
                    failed.append("batch")
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    ts = [threading.Thread(target=work, args=(j,)) for j in jobs] + [threading.Thread(target=batch)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not failed, failed
