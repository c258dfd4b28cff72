"""The on-chip form's host rules, on the CPU: which grids take it and how they
are cut into boxes, where a box finds its halo in the neighbours' surfaces, and
the reservation of CUs. The functions are internal C++ (mangled names).

The boxes have to cover every point of the grid once and respect the limits
the kernel is compiled for; the halo map below restates the layout (a box's
faces x-, x+ as [y][z], y-, y+ as [x][z], z-, z+ as [y][x], z pitch rounded up
to 4) and must give, for every halo point, the neighbour's surface value of
that very point.
"""
import ctypes
import threading
import time

import numpy as np
import pytest

F32, F64 = 0, 3
SHAPES = [(5, 4), (4, 4), (3, 4)]


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("nx", "ny", "nz", "lx", "ly", "bx", "by", "bz", "gx", "gy", "gz", "G",
                                            "V", "S")] + [("lds", ctypes.c_size_t)]


@pytest.fixture(scope="module")
def lib():
    from paper_2603_23343_amd import lib as L

    plan = L._ZN5pcgmi13resident_planEiiiibiPNS_7ResPlanE
    plan.argtypes = [ctypes.c_int] * 4 + [ctypes.c_bool, ctypes.c_int, ctypes.POINTER(Plan)]
    plan.restype = ctypes.c_bool
    return L


def _plan(lib, nx, ny, nz, dt=F32, var=False, wg=256):
    p = Plan()
    ok = lib._ZN5pcgmi13resident_planEiiiibiPNS_7ResPlanE(nx, ny, nz, dt, var, wg, ctypes.byref(p))
    return p if ok else None


def _most_v(dt, var):
    return (8 if var else 16) if dt == F64 else (16 if var else 32)


def _grids():
    rng = np.random.default_rng(11)
    fixed = [(1, 1, 1), (32, 32, 32), (101, 77, 59), (512, 112, 64), (128, 128, 128), (160, 160, 160), (9, 200, 3),
             (17, 33, 65), (250, 61, 130), (1, 1, 5000), (3000, 1, 1), (16, 16, 4096), (33, 17, 1)]
    drawn = [tuple(int(v) for v in np.rint(np.exp(rng.uniform(0, np.log(300), 3)))) for _ in range(200)]
    return fixed + drawn


@pytest.mark.parametrize("dt", [F32, F64])
@pytest.mark.parametrize("var", [False, True])
def test_boxes_cover_the_grid(lib, dt, var):
    taken = 0
    for nx, ny, nz in _grids():
        for wg in (256, 64, 8):
            p = _plan(lib, nx, ny, nz, dt, var, wg)
            if p is None:
                continue
            taken += 1
            tz = 512 >> (p.lx + p.ly)
            assert (p.lx, p.ly) in SHAPES and 2 <= p.V <= _most_v(dt, var)
            assert p.G == p.gx * p.gy * p.gz and 1 <= p.G <= wg
            for n, b, g, most in ((nx, p.bx, p.gx, 1 << p.lx), (ny, p.by, p.gy, 1 << p.ly), (nz, p.bz, p.gz, tz * p.V)):
                assert 1 <= b <= most and (g - 1) * b < n <= g * b  # no box is empty, none too wide
            zp = (tz * p.V + 3) // 4 * 4
            assert p.S == 2 * (zp * ((1 << p.lx) + (1 << p.ly)) + (1 << (p.lx + p.ly)))
            assert p.lds <= 156 << 10
            # halo groups per thread and their table in LDS (four at most)
            assert -(-(p.S // (4 if dt == F32 else 2)) // 512) <= 4
            # buffer offsets are 32 bits, signed
            assert nx * ny * nz * 8 < 2 ** 31 and 2 * p.G * p.S * 8 < 2 ** 31
    assert taken > 100


def test_which_grids_fit(lib):
    assert _plan(lib, 160, 160, 160) is not None
    assert _plan(lib, 256, 256, 256) is None
    assert _plan(lib, 128, 128, 128, F32, True) is not None
    assert _plan(lib, 160, 160, 160, F32, True) is None
    assert _plan(lib, 128, 128, 128, F64) is not None
    assert _plan(lib, 128, 128, 128, F64, True) is None
    assert _plan(lib, 512, 512, 8) is None  # more boxes than CUs


@pytest.mark.parametrize("dims", [(101, 77, 59), (33, 17, 65), (40, 40, 9), (65, 33, 130), (17, 33, 40)])
def test_halo_sources(lib, dims):
    nx, ny, nz = dims
    p = _plan(lib, nx, ny, nz)
    TX, TY = 1 << p.lx, 1 << p.ly
    zr = (512 >> (p.lx + p.ly)) * p.V
    ZP = (zr + 3) // 4 * 4
    NXF, NYF, NZF = TY * ZP, TX * ZP, TX * TY
    value = np.arange(nx * ny * nz, dtype=np.int64).reshape(nz, ny, nx)
    ext = {}
    surf = np.full((p.G, p.S), -1, dtype=np.int64)
    for rank in range(p.G):
        c = (rank % p.gx, rank // p.gx % p.gy, rank // (p.gx * p.gy))
        o = (c[0] * p.bx, c[1] * p.by, c[2] * p.bz)
        e = (min(p.bx, nx - o[0]), min(p.by, ny - o[1]), min(p.bz, nz - o[2]))
        ext[rank] = (c, o, e)
        box = value[o[2]:o[2] + e[2], o[1]:o[1] + e[1], o[0]:o[0] + e[0]]
        y, z = np.meshgrid(np.arange(e[1]), np.arange(e[2]), indexing="ij")
        surf[rank, y * ZP + z] = box[z, y, 0]
        surf[rank, NXF + y * ZP + z] = box[z, y, e[0] - 1]
        x, z = np.meshgrid(np.arange(e[0]), np.arange(e[2]), indexing="ij")
        surf[rank, 2 * NXF + x * ZP + z] = box[z, 0, x]
        surf[rank, 2 * NXF + NYF + x * ZP + z] = box[z, e[1] - 1, x]
        y, x = np.meshgrid(np.arange(e[1]), np.arange(e[0]), indexing="ij")
        surf[rank, 2 * (NXF + NYF) + y * TX + x] = box[0, y, x]
        surf[rank, 2 * (NXF + NYF) + NZF + y * TX + x] = box[e[2] - 1, y, x]
    seen = 0
    for rank in range(p.G):
        c, o, e = ext[rank]
        for j in range(p.S):
            if j < 2 * NXF:
                hi, k = divmod(j, NXF)
                y, z = divmod(k, ZP)
                x, step, face = (e[0] if hi else -1), (1 if hi else -1), (0 if hi else NXF)
                ok = (c[0] + 1 < p.gx if hi else c[0] > 0) and y < e[1] and z < e[2]
            elif j < 2 * (NXF + NYF):
                hi, k = divmod(j - 2 * NXF, NYF)
                x, z = divmod(k, ZP)
                y, step, face = (e[1] if hi else -1), (p.gx if hi else -p.gx), 2 * NXF + (0 if hi else NYF)
                ok = (c[1] + 1 < p.gy if hi else c[1] > 0) and x < e[0] and z < e[2]
            else:
                hi, k = divmod(j - 2 * (NXF + NYF), NZF)
                y, x = divmod(k, TX)
                z, step = (e[2] if hi else -1), (p.gx * p.gy if hi else -p.gx * p.gy)
                face = 2 * (NXF + NYF) + (0 if hi else NZF)
                ok = (c[2] + 1 < p.gz if hi else c[2] > 0) and x < e[0] and y < e[1]
            if ok:
                seen += 1
                assert surf[rank + step, face + k] == value[o[2] + z, o[1] + y, o[0] + x], (rank, j)
    assert seen > 0 or p.G == 1


class _Hold:
    def __init__(self, lib, want, cap, wait):
        self.buf = (ctypes.c_int64 * 8)()
        self.lib = lib
        ctor = lib._ZN5pcgmi6CuHoldC1Eiiid
        ctor.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_double]
        ctor.restype = None
        ctor(ctypes.addressof(self.buf), 15, want, cap, wait)
        # dev, want, ok
        self.ok = bool(ctypes.c_uint8.from_address(ctypes.addressof(self.buf) + 8).value)

    def release(self):
        dtor = self.lib._ZN5pcgmi6CuHoldD1Ev
        dtor.argtypes = [ctypes.c_void_p]
        dtor.restype = None
        dtor(ctypes.addressof(self.buf))


def test_reservation_limits(lib):
    a = _Hold(lib, 200, 256, 0.05)
    b = _Hold(lib, 56, 256, 0.05)
    c = _Hold(lib, 1, 256, 0.05)
    d = _Hold(lib, 300, 256, 0.05)  # can never fit
    assert a.ok and b.ok and not c.ok and not d.ok
    for h in (c, d, b):
        h.release()
    e = _Hold(lib, 56, 256, 0.05)
    assert e.ok
    e.release()
    a.release()
    f = _Hold(lib, 256, 256, 0.05)
    assert f.ok
    f.release()


def test_reservation_order(lib):
    """A claim on everything is served in its turn although small claims keep
    coming, and a claim that gives up leaves the queue in order."""
    first = _Hold(lib, 100, 256, 1.0)
    order = []

    def claim(name, want, wait):
        h = _Hold(lib, want, 256, wait)
        order.append((name, h.ok))
        time.sleep(0.05)
        h.release()

    ts = []
    for name, want, wait in (("gives up", 256, 0.1), ("all", 256, 10.0), ("small", 1, 10.0), ("small 2", 1, 10.0)):
        t = threading.Thread(target=claim, args=(name, want, wait))
        t.start()
        ts.append(t)
        time.sleep(0.03)
    time.sleep(0.3)
    assert order == [("gives up", False)]  # the small ones wait behind "all"
    first.release()
    for t in ts:
        t.join()
    assert order[1] == ("all", True)
    assert sorted(order[2:]) == [("small", True), ("small 2", True)]
    h = _Hold(lib, 256, 256, 0.05)
    assert h.ok
    h.release()
