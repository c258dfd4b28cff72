"""What follows an on-chip launch whose work-groups did not come together. The
host forces it: a wait limit of 0 ticks (every kernel then ends by itself), or a
launch that it takes as late after it ended. The functions are internal C++
(mangled names)."""
import ctypes

import numpy as np
import pytest
import torch

import synthetic
from gpu_helpers import check_status, dev, host64, make_vec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _limits(P, ctx, wait=100000000, drop=0):
    fn = P.lib._ZN5pcgmi15resident_limitsEP9pcg_ctx_sxi
    fn.argtypes = [ctypes.c_void_p, ctypes.c_longlong, ctypes.c_int]
    fn.restype = None
    fn(ctx.handle, wait, drop)


def _call(P, name, handle, *args):
    fn = getattr(P.lib, name)
    fn.argtypes = [ctypes.c_void_p, ctypes.c_longlong, ctypes.c_int][:1 + len(args)]
    fn.restype = None
    fn(handle, *args)


def _retry(P, ctx):
    _call(P, "_ZN5pcgmi14resident_retryEP9pcg_ctx_s", ctx.handle)


@pytest.mark.parametrize("dtype,rtol", [(torch.float32, 1e-13), (torch.float64, 3e-15)])
def test_restart_starts_over_from_its_own_start(P, dtype, rtol):
    """The second launch of a solve (a restart, which iterates x in place)
    counts as late: the solve goes on from the x that the restart began with,
    not from what the launch left, so it takes the iterations that the
    two-kernel form takes."""
    nx, ny, nz = 64, 60, 50
    n = nx * ny * nz
    b, _ = make_vec(41, n, dtype)
    runs = []
    for opts, drop in (({}, 0), ({}, 2), ({"single_reduction": 0}, 0)):
        # use_x0 leaves the judge to the host, so each restart is a launch
        ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64, use_x0=1, max_restarts=1, **opts)
        _limits(P, ctx, drop=drop)
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        info = P.pcg_solve(ctx, b, x, rtol, 3000, raise_on_error=False)
        assert info["restarts"] == 1
        tail = len(P.pcg_get_history(ctx)) - 1  # iterations of the last start
        runs.append((info["iters"], tail, P.pcg_get_form(ctx)))
    print(runs, flush=True)
    assert [r[2] for r in runs] == [P.PCG_FORM_ON_CHIP, P.PCG_FORM_STREAMING, P.PCG_FORM_STREAMING]
    whole, late, two = runs
    assert whole[1] >= 1 and late[1] >= 1  # the restart has work to do, and it is done again
    # rounding differs between the forms: a few iterations of a restart
    assert abs(late[1] - whole[1]) <= 0.25 * whole[1] + 2
    assert abs(late[0] - two[0]) <= 0.1 * two[0]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("coef", [False, True])
@pytest.mark.parametrize("opts", [{}, {"use_x0": 1}])
@pytest.mark.parametrize("how", ["wait", "drop"])
def test_solve_after_a_late_launch(P, orc, dtype, coef, opts, how):
    """A solve whose launch was late runs in another form and is right; solves
    soon after do not try the chip, later ones do and give the first bits."""
    nx, ny, nz = 48, 40, 36  # several boxes: a wait limit of 0 always runs out
    n = nx * ny * nz
    b, b64 = make_vec(42, n, dtype)
    k = np.exp(synthetic.uniform(43, n)).astype(np.float32) if coef else None
    ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64, **opts)
    if coef:
        kd = dev(k)
        P.pcg_set_coefficients(ctx, kd)
    other = P.PCG_FORM_STREAMING if coef else P.PCG_FORM_SINGLE_REDUCTION

    def solve():
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        info = P.pcg_solve(ctx, b, x, 1e-6, 1000)
        return info, x, P.pcg_get_form(ctx)

    info0, x0, form = solve()
    assert form == P.PCG_FORM_ON_CHIP
    ref = orc.pcg((nz, ny, nx), b64, rtol=1e-6, maxit=1000, kcell=None if k is None else k.astype(np.float64))
    for _ in range(2):
        if how == "wait":
            _limits(P, ctx, wait=0)
        else:
            _limits(P, ctx, drop=1)
        info, x, form = solve()
        print(how, info["iters"], ref["iters"], form, flush=True)
        assert form == other
        assert abs(info["iters"] - ref["iters"]) <= 2
        tr = orc.true_relres((nz, ny, nx), b64, host64(x), kcell=None if k is None else k.astype(np.float64))
        assert tr <= 1e-6
        _limits(P, ctx)
        _retry(P, ctx)
        info, x, form = solve()
        assert form == P.PCG_FORM_ON_CHIP
        assert info["iters"] == info0["iters"] and torch.equal(x, x0)


def test_late_launches_are_not_tried_at_once(P):
    """A launch that lost some 15 ms is not repeated for a hundred times that:
    not by the short solves right after it."""
    nx, ny, nz = 160, 160, 160
    b, _ = make_vec(44, nx * ny * nz, torch.float32)
    x = torch.empty(b.numel(), dtype=torch.float64, device="cuda")
    ctx = P.pcg_create(nx, ny, nz, torch.float32, x_dtype=torch.float64)
    _limits(P, ctx, drop=1)
    info = P.pcg_solve(ctx, b, x, 1e-30, 2000, raise_on_error=False)
    assert info["iters"] >= 1000
    forms = [P.pcg_get_form(ctx)]
    for _ in range(3):
        P.pcg_solve(ctx, b, x, 1e-30, 2, raise_on_error=False)
        forms.append(P.pcg_get_form(ctx))
    assert forms == [P.PCG_FORM_STREAMING] * 4
    _retry(P, ctx)
    P.pcg_solve(ctx, b, x, 1e-30, 2, raise_on_error=False)
    assert P.pcg_get_form(ctx) == P.PCG_FORM_ON_CHIP


@pytest.mark.parametrize("how", ["wait", "drop"])
@pytest.mark.parametrize("use_graph", [True, False])
def test_batch_after_a_late_launch(P, orc, how, use_graph):
    """The same for a batch: the streaming kernel serves it, on arenas that the
    launch used, and the chip again later with the first bits."""
    dims = [(33, 20, 40), (17, 9, 23), (48, 40, 36), (5, 4, 3), (30, 30, 30)]
    bt = P.pcg_batch_create(dims)
    b = dev(synthetic.uniform_f32(45, bt.total))

    def solve():
        x = torch.zeros(bt.total, dtype=torch.float64, device="cuda")
        r = P.pcg_batch_solve(bt, b, x, 1e-6, 1000, use_graph=use_graph)
        return r, x, P.pcg_batch_get_form(bt)

    def limits(wait, drop):
        _call(P, "_ZN5pcgmi12batch_limitsEP11pcg_batch_sxi", bt.handle, wait, drop)

    r0, x0, form = solve()
    assert form == P.PCG_FORM_ON_CHIP
    for _ in range(2):
        limits(0 if how == "wait" else -1, 1 if how == "drop" else 0)
        r, x, form = solve()
        assert form == P.PCG_FORM_STREAMING
        for i, (nx, ny, nz) in enumerate(dims):
            b64 = host64(bt.view(b, i))
            assert abs(r["iters"][i] - orc.pcg((nz, ny, nx), b64, rtol=1e-6, maxit=1000)["iters"]) <= 2
            assert orc.true_relres((nz, ny, nx), b64, host64(bt.view(x, i))) <= 1e-6
        limits(-1, 0)
        _call(P, "_ZN5pcgmi11batch_retryEP11pcg_batch_s", bt.handle)
        r, x, form = solve()
        assert form == P.PCG_FORM_ON_CHIP
        assert r["iters"] == r0["iters"]
        for i in range(len(dims)):
            assert torch.equal(bt.view(x, i), bt.view(x0, i))
