"""Right-hand sides and limits at the edges of the on-chip form: what a solve
or a batch returns there must not depend on the form that runs it."""
import numpy as np
import pytest
import torch

import synthetic
from gpu_helpers import dev, host64, make_vec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _times_2(t, e):
    """t 2^e, exactly (torch.ldexp multiplies by a rounded power)."""
    return dev(np.ldexp(t.cpu().numpy(), e))


def _coef(seed, n):
    return dev(np.exp(synthetic.uniform(seed, n)).astype(np.float32))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("coef", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 4, 5), (50, 60, 64)])
def test_scaled_right_hand_side(P, dtype, coef, shape):
    """b 2^e for powers of two far outside the range whose squares FP32 holds:
    the solve takes the same steps as for b, so x is x(b) 2^e bit for bit."""
    nz, ny, nx = shape
    n = nx * ny * nz
    b, _ = make_vec(71, n, dtype)
    ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64)
    if coef:
        k = _coef(72, n)
        P.pcg_set_coefficients(ctx, k)
    outs = []
    for e in (0, -61, -75, -90, 63, 90):
        x = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
        info = P.pcg_solve(ctx, _times_2(b, e), x, 1e-5, 1000, raise_on_error=False)
        print(shape, dtype, coef, e, info["status"], info["iters"], info["rel_res_true_fp64"], flush=True)
        outs.append((info["status"], info["iters"], info["restarts"], np.ldexp(host64(x), -e)))
    assert outs[0][0] == P.PCG_OK
    for o in outs[1:]:
        assert o[:3] == outs[0][:3]
        assert np.array_equal(o[3], outs[0][3])


@pytest.mark.parametrize("coef", [False, True])
@pytest.mark.parametrize("e", [-61, -75, -90])
def test_scaled_right_hand_side_started_outside(P, coef, e):
    """With an FP32 x other kernels make the start and judge the result; their
    start sums squares in FP32 and may take a small b for zero (the judge then
    restarts), so only the outcome is compared: the FP64 judge accepts x."""
    nx, ny, nz = 20, 12, 9
    n = nx * ny * nz
    b, _ = make_vec(74, n, torch.float32)
    ctx = P.pcg_create(nx, ny, nz, torch.float32)
    if coef:
        k = _coef(75, n)
        P.pcg_set_coefficients(ctx, k)
    x = torch.full((n,), np.nan, dtype=torch.float32, device="cuda")
    info = P.pcg_solve(ctx, _times_2(b, e), x, 1e-5, 1000, raise_on_error=False)
    print(info, flush=True)
    assert info["status"] == P.PCG_OK and info["rel_res_true_fp64"] <= 1e-5


def test_scaled_right_hand_side_batch(P):
    """As above in a batch, each problem with another power of two."""
    dims = [(1, 1, 1), (5, 4, 3), (17, 17, 17), (33, 20, 40), (24, 24, 24)]
    bt = P.pcg_batch_create(dims)
    b = dev(synthetic.uniform_f32(73, bt.total))
    x = torch.full((bt.total,), np.nan, dtype=torch.float64, device="cuda")
    r0 = P.pcg_batch_solve(bt, b, x, 1e-6, 1000)
    want = [host64(bt.view(x, i)) for i in range(len(dims))]
    exps = [-90, -75, 90, -61, 63]
    for i, e in enumerate(exps):
        v = bt.view(b, i)
        v.copy_(_times_2(v, e))
    r = P.pcg_batch_solve(bt, b, x, 1e-6, 1000, raise_on_error=False)
    print(r, flush=True)
    assert r["status"] == P.PCG_OK
    assert r["iters"] == r0["iters"] and r["restarts"] == r0["restarts"]
    for i, e in enumerate(exps):
        assert np.array_equal(np.ldexp(host64(bt.view(x, i)), -e), want[i])


@pytest.mark.parametrize("rtol", [1.0, 2.0])
@pytest.mark.parametrize("maxit", [0, 1, 50])
def test_batch_takes_one_step_at_least(P, orc, rtol, maxit):
    """A batch iterates before it judges: with a tolerance that x = 0 meets
    every problem ends after one step (the streaming form's answer). One CG step
    in FP32: the norms and the update are good to a few 2^-24 per term."""
    dims = [(5, 4, 3), (17, 17, 17), (33, 20, 40)]
    bt = P.pcg_batch_create(dims)
    b = dev(synthetic.uniform_f32(76, bt.total))
    x = torch.full((bt.total,), np.nan, dtype=torch.float64, device="cuda")
    r = P.pcg_batch_solve(bt, b, x, rtol, maxit)
    print(r, flush=True)
    assert r["iters"] == [1, 1, 1] and r["restarts"] == [0, 0, 0]
    for i, (nx, ny, nz) in enumerate(dims):
        ref = orc.pcg((nz, ny, nx), host64(bt.view(b, i)), rtol=0.0, maxit=1)
        xi = host64(bt.view(x, i))
        assert np.linalg.norm(xi - ref["x"]) <= 32 * 2.0 ** -24 * np.linalg.norm(ref["x"])


def test_batch_in_place(P):
    """One problem with b inside x's memory: solved as with arrays of their own
    (the FP64 judge accepts x, which agrees to the solve's error)."""
    bt = P.pcg_batch_create([(33, 20, 40)])
    b = dev(synthetic.uniform_f32(77, bt.total))
    x = torch.zeros(bt.total, dtype=torch.float64, device="cuda")
    r0 = P.pcg_batch_solve(bt, b, x, 1e-6, 1000)
    y = torch.zeros_like(x)
    inside = y.view(torch.float32)[:bt.total]
    inside.copy_(b)
    r = P.pcg_batch_solve(bt, inside, y, 1e-6, 1000, raise_on_error=False)
    print(r0, r, flush=True)
    assert r["status"] == P.PCG_OK and r["relres"][0] <= 1e-6
    assert abs(r["iters"][0] - r0["iters"][0]) <= 1
    # || x - y || <= 2 cond(A) rtol ||x||, cond(A) below 500 on this grid
    assert torch.linalg.norm(x - y) <= 1e-3 * torch.linalg.norm(x)


def test_times_of_a_solve_without_iterations(P):
    """A start that other kernels judged as finished reports no iteration time,
    whatever the context solved before."""
    n = 20 * 20 * 20
    b, _ = make_vec(78, n, torch.float32)
    ctx = P.pcg_create(20, 20, 20, torch.float32, kernel_timing=1)  # FP32 x: started outside
    x = torch.empty(n, device="cuda")
    info = P.pcg_solve(ctx, b, x, 1e-4, 500)
    assert info["k1_launches"] == info["iters"] > 0 and info["k1_ms"] > 0 and info["k2_ms"] > 0
    info = P.pcg_solve(ctx, torch.zeros_like(b), x, 1e-4, 500)
    print(info, flush=True)
    assert info["iters"] == info["k1_launches"] == 0
    assert info["k1_ms"] == 0 and info["k2_ms"] == 0
    info = P.pcg_solve(ctx, b, x, 1e-4, 500)
    assert info["k1_launches"] == info["iters"] > 0 and info["k1_ms"] > 0 and info["k2_ms"] > 0


def test_phase_times_leave_out_the_start(P):
    """k1_ms and k2_ms are an iteration's two phases: a solve of one iteration,
    which reads no surfaces, reports no more than one of a hundred takes (with a
    quarter for noise, the least of ten solves): no loads, no norm before it."""
    nx, ny, nz = 128, 128, 64
    n = nx * ny * nz
    b, _ = make_vec(79, n, torch.float32)
    ctx = P.pcg_create(nx, ny, nz, torch.float32, x_dtype=torch.float64, kernel_timing=1, max_restarts=0)
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    many = [P.pcg_solve(ctx, b, x, 1e-30, 100, raise_on_error=False) for _ in range(3)]
    one = [P.pcg_solve(ctx, b, x, 1e-30, 1, raise_on_error=False) for _ in range(10)]
    each = min(i["k1_ms"] for i in many) / 100
    print("phase 1 of 100:", each, "of 1:", [i["k1_ms"] for i in one], flush=True)
    assert all(i["k1_launches"] == 1 for i in one)
    assert min(i["k1_ms"] for i in one) <= 1.25 * each


def test_coefficients_reuse_the_exchange_buffers(P):
    """The box surfaces' memory is made at creation for either operator: setting
    coefficients allocates D^-1 (8 MiB here) and nothing else, and frees nothing."""
    n = 128 ** 3
    k = torch.ones(n, device="cuda")
    ctx = P.pcg_create(128, 128, 128, torch.float32, x_dtype=torch.float64)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    P.pcg_set_coefficients(ctx, k)
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0]
    print("setting coefficients took", took, "bytes", flush=True)
    assert took <= 4 * n
