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
