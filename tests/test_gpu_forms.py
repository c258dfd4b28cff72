"""Which form runs a solve or a batch, and the streaming forms where the
defaults would take the on-chip one: captured chunks, eager and timed launches,
cell coefficients, and the streaming batch kernel, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import synthetic
from gpu_helpers import check_status, host64, make_vec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _kfield(n, seed=6):
    return np.exp(synthetic.uniform(seed, n)).astype(np.float32)


# (nz, ny, nx), storage, cell coefficients, options, the form's name
TAKEN = [
    ((20, 20, 20), torch.float32, False, {}, "ON_CHIP"),
    ((20, 20, 20), torch.float32, True, {}, "ON_CHIP"),
    ((20, 20, 20), torch.float64, False, {}, "ON_CHIP"),
    ((20, 20, 20), torch.float64, True, {}, "ON_CHIP"),
    ((20, 20, 20), torch.float32, False, {"use_x0": 1}, "ON_CHIP"),
    ((64, 112, 512), torch.float32, False, {}, "ON_CHIP"),
    ((128, 128, 128), torch.float32, True, {}, "ON_CHIP"),
    ((20, 20, 20), torch.float32, False, {"single_reduction": 0}, "STREAMING"),
    ((20, 20, 20), torch.float32, True, {"single_reduction": 0}, "STREAMING"),
    ((20, 20, 20), torch.float32, False, {"single_reduction": 1}, "SINGLE_REDUCTION"),
    ((20, 20, 20), torch.float32, False, {"zchunk": 5}, "SINGLE_REDUCTION"),
    ((20, 20, 20), torch.float32, False, {"tile_x": 64, "tile_y": 4}, "SINGLE_REDUCTION"),
    ((20, 20, 20), torch.float32, True, {"zchunk": 5}, "STREAMING"),
    ((20, 20, 20), torch.float32, False, {"x_accum": torch.float32}, "SINGLE_REDUCTION"),
    ((20, 20, 20), torch.bfloat16, False, {}, "STREAMING"),
    ((8, 400, 400), torch.float32, False, {}, "STREAMING"),      # flat: more boxes than CUs
    ((128, 128, 128), torch.float64, True, {}, "STREAMING"),     # more points than registers
]


@pytest.mark.parametrize("shape,dtype,coef,opts,name", TAKEN)
def test_form_taken(P, shape, dtype, coef, opts, name):
    nz, ny, nx = shape
    n = nx * ny * nz
    b, _ = make_vec(11, n, dtype)
    ctx = P.pcg_create(nx, ny, nz, dtype, x_dtype=torch.float64, **opts)
    if coef:
        k = torch.from_numpy(_kfield(n)).cuda()
        P.pcg_set_coefficients(ctx, k)
    assert P.pcg_get_form(ctx) == P.PCG_FORM_NONE
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    P.pcg_solve(ctx, b, x, 1e-3, 4, raise_on_error=False)
    assert P.pcg_get_form(ctx) == getattr(P, "PCG_FORM_" + name)


def test_form_follows_the_operator(P):
    """Coefficients set and taken back change the plan; 16-bit and FP32
    refinement run their inner solves in their own forms."""
    nx, ny, nz = 160, 160, 160
    n = nx * ny * nz
    b, _ = make_vec(12, n, torch.float32)
    k = torch.ones(n, device="cuda")
    ctx = P.pcg_create(nx, ny, nz, torch.float32, x_dtype=torch.float64)
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    seen = []
    for kk in (None, k, None):
        P.pcg_set_coefficients(ctx, kk)
        P.pcg_solve(ctx, b, x, 1e-3, 4, raise_on_error=False)
        seen.append(P.pcg_get_form(ctx))
    assert seen == [P.PCG_FORM_ON_CHIP, P.PCG_FORM_STREAMING, P.PCG_FORM_ON_CHIP]
    for dtype, form in ((torch.float32, P.PCG_FORM_ON_CHIP), (torch.bfloat16, P.PCG_FORM_STREAMING)):
        ctx = P.pcg_create(24, 24, 24, dtype)
        b, _ = make_vec(13, 24 ** 3, torch.float64)
        x = torch.empty_like(b)
        P.pcg_solve_refined(ctx, b, x)
        assert P.pcg_get_form(ctx) == form


@pytest.mark.parametrize("single", [0, 1])
@pytest.mark.parametrize("chunk", [2, 16, 64])
def test_graph_eager_timing_identical_streaming(P, single, chunk):
    """Captured graph chunks, eager launches and the event-timed mode of the
    streaming forms run the same kernels in the same order: the same bits."""
    nz, ny, nx = 24, 40, 48
    n = nx * ny * nz
    b, _ = make_vec(5, n, torch.float32)
    outs = []
    for opts in ({"use_graph": 1}, {"use_graph": 0}, {"kernel_timing": 1}, {"use_graph": 1}):
        ctx = P.pcg_create(nx, ny, nz, torch.float32, x_dtype=torch.float64, chunk_iters=chunk, single_reduction=single,
                           **opts)
        x = torch.empty(n, dtype=torch.float64, device="cuda")
        info = P.pcg_solve(ctx, b, x, 1e-6, 500)
        assert P.pcg_get_form(ctx) == (P.PCG_FORM_SINGLE_REDUCTION if single else P.PCG_FORM_STREAMING)
        outs.append((info["iters"], host64(x).tobytes()))
        if opts.get("kernel_timing"):
            assert info["k1_ms"] > 0 and info["k2_ms"] > 0 and info["k1_launches"] >= info["iters"]
    assert all(o == outs[0] for o in outs)


@pytest.mark.parametrize("dtype,n,rtol", [(torch.float32, 24, 1e-6), (torch.float32, 48, 1e-6), (torch.float64, 32, 1e-10)])
def test_coefficients_two_kernels(P, orc, dtype, n, rtol):
    """The two-kernel form with cell coefficients, which serves the grids that
    do not fit the chip: iterations within 2 of the oracle, FP64 residual."""
    k32 = synthetic.coefficient_field(n, 6)
    k64 = k32.astype(np.float64)
    b, b64 = make_vec(31, n ** 3, dtype)
    ref = orc.pcg((n, n, n), b64, rtol=rtol, maxit=5000, kcell=k64)
    ctx = P.pcg_create(n, n, n, dtype, x_dtype=torch.float64, single_reduction=0)
    kd = torch.from_numpy(k32).cuda()
    P.pcg_set_coefficients(ctx, kd)
    x = torch.empty(n ** 3, dtype=torch.float64, device="cuda")
    info = P.pcg_solve(ctx, b, x, rtol, 5000, raise_on_error=False)
    assert P.pcg_get_form(ctx) == P.PCG_FORM_STREAMING
    check_status(P, info, rtol)
    assert abs(info["iters"] - ref["iters"]) <= 2
    # converged on the recursion; FP64 rounding may leave the true residual just above it
    assert orc.true_relres((n, n, n), b64, host64(x), kcell=k64) <= 1.5 * rtol


def test_streaming_batch_64_uneven(P, orc):
    """The 64 cubes in the streaming kernel, with the tile shapes that the
    default batch chose: XCD-local barriers on every group, the oracle's
    iterations (restarts off), and the default batch is on the chip."""
    sizes = synthetic.batch_sizes()
    dims = [(n, n, n) for n in sizes]
    auto = P.pcg_batch_create(dims)
    bt = P.pcg_batch_create(dims, cfgs=[p[0] for p in auto.plans])
    b = torch.zeros(bt.total, dtype=torch.float32, device="cuda")
    host = []
    for i, n in enumerate(sizes):
        v = synthetic.uniform_f32(synthetic.SEED_C4_B_BASE + i, n ** 3)
        bt.view(b, i).copy_(torch.from_numpy(v))
        host.append(v.astype(np.float64))
    x = torch.zeros(bt.total, dtype=torch.float64, device="cuda")
    assert P.pcg_batch_get_form(bt) == P.PCG_FORM_NONE
    P.pcg_batch_set_restarts(bt, 0)
    r = P.pcg_batch_solve(bt, b, x, 1e-6, 5000, raise_on_error=False)
    assert P.pcg_batch_get_form(bt) == P.PCG_FORM_STREAMING
    assert r["xcd_local"] == len(sizes)
    for i, n in enumerate(sizes):
        ref = orc.pcg((n, n, n), host[i], rtol=1e-6, maxit=5000)
        assert abs(r["iters"][i] - ref["iters"]) <= 2, (n, r["iters"][i], ref["iters"])
        tr = orc.true_relres((n, n, n), host[i], host64(bt.view(x, i)))
        assert abs(r["relres"][i] - tr) <= 1e-9 * tr + 1e-13
    P.pcg_batch_solve(auto, b, x, 1e-6, 5000)
    assert P.pcg_batch_get_form(auto) == P.PCG_FORM_ON_CHIP
