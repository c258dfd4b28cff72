"""Iterates and residual histories of the on-chip form against the FP64 oracle,
for every thread shape and number of points per thread that a plan takes on
grids of up to 4 M points, and for batches.

Tolerance: FP32 vectors carry a relative rounding error of 2^-24 per operation
and an iteration applies a few; k iterations of well-conditioned early CG keep
the iterate and the residual norm within k * 32 * 2^-24 of the FP64 ones
(k = 20: 4e-5), FP64 storage within k * 32 * 2^-53 (7e-14). After 20 iterations
every grid's residual still stands above that (thin grids at 7e-5 of the start,
the others at a hundredth), so every case is compared.
"""
import ctypes
import threading

import numpy as np
import pytest
import torch

import synthetic
from gpu_helpers import dev, host64, make_vec
from test_onchip_plan import Plan

pytestmark = pytest.mark.gpu
ITERS = 20


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _tol(dtype):
    return ITERS * 32 * (2.0 ** -53 if dtype == torch.float64 else 2.0 ** -24)


def _plan(P, shape, dtype, coef):
    fn = P.lib._ZN5pcgmi13resident_planEiiiibiPNS_7ResPlanE
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_bool, ctypes.c_int, ctypes.POINTER(Plan)]
    fn.restype = ctypes.c_bool
    p = Plan()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert fn(shape[2], shape[1], shape[0], P.dtype_code(dtype), coef, cus, ctypes.byref(p))
    return p


F32, F64 = torch.float32, torch.float64
# (nz, ny, nx), threads along x (log2), points per thread
CASES = [(F32, False, s, lx, V) for s, lx, V in [
    ((17, 17, 33), 4, 2), ((8, 16, 32), 5, 2), ((201, 6, 4), 3, 4), ((101, 5, 10), 4, 4), ((7, 4, 250), 5, 4),
    ((17, 236, 4), 3, 6), ((36, 5, 105), 4, 6), ((17, 4, 251), 5, 6), ((61, 100, 40), 3, 8), ((32, 5, 239), 4, 8),
    ((70, 4, 153), 5, 8), ((98, 4, 136), 4, 10), ((183, 4, 98), 3, 12), ((106, 5, 214), 5, 12), ((59, 77, 101), 3, 16),
    ((156, 6, 270), 4, 16), ((236, 5, 230), 3, 20), ((260, 7, 193), 5, 20), ((129, 137, 45), 4, 24),
    ((101, 102, 100), 3, 28), ((130, 61, 250), 5, 28), ((64, 112, 512), 5, 32)]]
CASES += [(F32, True, s, lx, V) for s, lx, V in [
    ((16, 16, 32), 5, 2), ((29, 37, 48), 4, 4), ((261, 6, 35), 3, 6), ((59, 77, 101), 3, 8), ((178, 4, 260), 4, 10),
    ((242, 5, 245), 5, 12), ((121, 149, 46), 4, 16), ((128, 128, 128), 5, 16)]]
CASES += [(F64, False, s, lx, V) for s, lx, V in [
    ((17, 17, 33), 4, 2), ((61, 100, 40), 3, 4), ((67, 4, 235), 4, 6), ((59, 77, 101), 3, 8), ((180, 4, 284), 5, 10),
    ((144, 35, 100), 3, 12), ((269, 17, 177), 5, 16)]]
CASES += [(F64, True, s, lx, V) for s, lx, V in [
    ((16, 16, 32), 5, 2), ((57, 4, 133), 3, 4), ((59, 77, 101), 4, 6), ((134, 17, 170), 4, 8)]]


@pytest.mark.parametrize("dtype,coef,shape,lx,V", CASES)
def test_iterates_and_history(P, orc, dtype, coef, shape, lx, V):
    nz, ny, nx = shape
    n = nx * ny * nz
    p = _plan(P, shape, dtype, coef)
    assert (p.lx, p.V) == (lx, V), (p.lx, p.V, p.G)
    b, b64 = make_vec(31, n, dtype)
    k = np.exp(synthetic.uniform(32, n)).astype(np.float32) if coef else None
    ref = orc.pcg(shape, b64, rtol=0.0, maxit=ITERS, history=True, kcell=None if k is None else k.astype(np.float64))
    assert ref["iters"] == ITERS and ref["hist"][-1] > _tol(dtype), "nothing left to compare"
    tol = _tol(dtype)
    for opts in ({}, {"use_x0": 1}):  # started and judged on the chip; by other kernels
        ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64, **opts)
        if coef:
            kd = dev(k)
            P.pcg_set_coefficients(ctx, kd)
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        info = P.pcg_solve(ctx, b, x, 0.0, ITERS, raise_on_error=False)
        assert P.pcg_get_form(ctx) == P.PCG_FORM_ON_CHIP
        assert info["iters"] == ITERS and info["status"] == P.PCG_E_NOCONV
        xh, hist = host64(x), P.pcg_get_history(ctx)
        print(shape, opts, np.linalg.norm(xh - ref["x"]) / np.linalg.norm(ref["x"]), np.max(np.abs(hist - ref["hist"])), flush=True)
        assert np.linalg.norm(xh - ref["x"]) <= tol * np.linalg.norm(ref["x"])
        assert hist.shape == ref["hist"].shape and np.all(np.abs(hist - ref["hist"]) <= tol * ref["hist"][0])


DIMS = [(16, 16, 16), (17, 23, 9), (128, 128, 128), (33, 33, 33), (64, 8, 140), (250, 60, 31), (5, 200, 77),
        (100, 100, 100), (41, 41, 41), (90, 90, 90)]


def _batch(P, dims, seed, **kw):
    bt = P.pcg_batch_create(dims, **kw)
    return bt, dev(synthetic.uniform_f32(seed, bt.total)), torch.full((bt.total,), np.nan, dtype=torch.float64, device="cuda")


def test_batch_iterates(P, orc):
    bt, b, x = _batch(P, DIMS, 33)
    P.pcg_batch_set_restarts(bt, 0)
    r = P.pcg_batch_solve(bt, b, x, 0.0, ITERS, raise_on_error=False)
    assert P.pcg_batch_get_form(bt) == P.PCG_FORM_ON_CHIP
    assert r["status"] == P.PCG_E_NOCONV and r["iters"] == [ITERS] * len(DIMS)
    for i, (nx, ny, nz) in enumerate(DIMS):
        b64 = host64(bt.view(b, i))
        ref = orc.pcg((nz, ny, nx), b64, rtol=0.0, maxit=ITERS)
        xi = host64(bt.view(x, i))
        assert np.linalg.norm(xi - ref["x"]) <= _tol(F32) * np.linalg.norm(ref["x"]), DIMS[i]
        tr = orc.true_relres((nz, ny, nx), b64, xi)
        assert abs(r["relres"][i] - tr) <= 1e-9 * tr + 1e-13


def test_batch_edges(P, orc):
    """On the chip: a zero right-hand side, one with a NaN, one that converges
    and one that does not within maxit, side by side; then maxit = 0, which takes
    one step, and the batch as it was."""
    dims = [(24, 24, 24), (33, 20, 40), (20, 20, 20), (60, 60, 60)]
    bt, b, x = _batch(P, dims, 34)
    bt.view(b, 0).zero_()
    bt.view(b, 1)[77] = float("nan")
    r = P.pcg_batch_solve(bt, b, x, 1e-3, 60, raise_on_error=False)
    print(r, flush=True)
    assert P.pcg_batch_get_form(bt) == P.PCG_FORM_ON_CHIP
    assert r["status"] == P.PCG_E_BREAKDOWN  # the worst of the four
    assert r["iters"][0] == 0 and r["relres"][0] == 0 and torch.count_nonzero(bt.view(x, 0)).item() == 0
    refs = [orc.pcg((d[2], d[1], d[0]), host64(bt.view(b, i)), rtol=1e-3, maxit=60) if i > 1 else None
            for i, d in enumerate(dims)]
    assert refs[2]["iters"] < 60 and refs[3]["iters"] == 60
    assert abs(r["iters"][2] - refs[2]["iters"]) <= 2 and r["relres"][2] <= 1e-3
    assert r["iters"][3] == 60 and r["relres"][3] > 1e-3
    bt.view(b, 1)[77] = 0.0
    r0 = P.pcg_batch_solve(bt, b, x, 1e-6, 0, raise_on_error=False)
    assert r0["status"] == P.PCG_E_NOCONV and r0["iters"] == [0, 1, 1, 1]
    r = P.pcg_batch_solve(bt, b, x, 1e-6, 1000)
    assert P.pcg_batch_get_form(bt) == P.PCG_FORM_ON_CHIP
    for i, d in enumerate(dims):
        if i:
            assert orc.true_relres((d[2], d[1], d[0]), host64(bt.view(b, i)), host64(bt.view(x, i))) <= 1e-6


def test_batches_and_solves_in_threads(P):
    """Two on-chip batches and three on-chip solves, from a thread each, over and
    over: every result is that of a lone call, bit for bit, and on the chip."""
    jobs = []
    for i, dims in enumerate(([(24, 24, 24), (40, 30, 20), (50, 50, 50)], [(64, 64, 64), (17, 9, 23)])):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            bt, b, x = _batch(P, dims, 35 + i, stream=s)
        s.synchronize()
        jobs.append((lambda bt=bt, b=b, x=x: P.pcg_batch_solve(bt, b, x, 1e-6, 1000),
                     lambda bt=bt, x=x: torch.cat([bt.view(x, j) for j in range(len(bt))]).cpu(),
                     lambda bt=bt: P.pcg_batch_get_form(bt)))
    for i, (nz, ny, nx) in enumerate([(32, 32, 32), (100, 96, 90), (64, 112, 300)]):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctx = P.pcg_create(nx, ny, nz, torch.float32, stream=s, x_dtype=torch.float64)
            b, _ = make_vec(37 + i, nx * ny * nz, torch.float32)
            x = torch.empty(b.numel(), dtype=torch.float64, device="cuda")
        s.synchronize()
        jobs.append((lambda c=ctx, b=b, x=x: P.pcg_solve(c, b, x, 1e-6, 1000), lambda x=x: x.cpu(),
                     lambda c=ctx: P.pcg_get_form(c)))
    want = []
    for run, out, _ in jobs:
        run()
        torch.cuda.synchronize()
        want.append(out())
    failed = []

    def work(i):
        run, out, form = jobs[i]
        try:
            for _ in range(6):
                run()
                if form() != P.PCG_FORM_ON_CHIP:
                    failed.append((i, "form"))
                if not torch.equal(out(), want[i]):
                    failed.append((i, "result"))
        except Exception as e:  # noqa: BLE001
            failed.append((i, repr(e)))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not failed, failed
