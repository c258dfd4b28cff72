"""Launches on the chip beside other work of the process: claims on CUs do not
outlast the need for them."""
import threading
import time

import pytest
import torch

import synthetic
from gpu_helpers import dev, make_vec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2603_23343_amd as P

    return P


def _stream_beside_the_default():
    """A stream whose work does not queue up before the default stream's (a
    process's streams share a few hardware queues), and the cycles of a second's
    sleep of one thread there."""
    one = torch.zeros(1, device="cuda")
    for _ in range(16):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda._sleep(1000000)
            e[0].record()
            torch.cuda._sleep(1000000)
            e[1].record()
            s.synchronize()
            cycles = int(1000000 * 1000.0 / e[0].elapsed_time(e[1]))
            torch.cuda._sleep(cycles // 10)
        t = time.monotonic()
        one.add_(1)
        torch.cuda.current_stream().synchronize()
        t = time.monotonic() - t
        s.synchronize()
        if t < 0.05:
            return s, cycles
    pytest.skip("every stream shares the default stream's hardware queue")


@pytest.mark.parametrize("first", ["solve", "started outside", "batch"])
def test_a_busy_stream_holds_no_claim(P, first):
    """A solve or batch that is called behind a second of other work of its
    stream claims its CUs when that work is done: a solve in another thread,
    which would not fit beside it, is not kept waiting."""
    sa, cycles = _stream_beside_the_default()
    with torch.cuda.stream(sa):
        if first == "batch":
            bt = P.pcg_batch_create([(24, 24, 24), (40, 30, 20)], stream=sa)
            bb = dev(synthetic.uniform_f32(51, bt.total))
            bx = torch.zeros(bt.total, dtype=torch.float64, device="cuda")
            run = lambda: P.pcg_batch_solve(bt, bb, bx, 1e-3, 1000)  # noqa: E731
        else:
            big = P.pcg_create(160, 160, 160, torch.float32, stream=sa,
                               x_dtype=torch.float64 if first == "solve" else torch.float32)
            xb = torch.empty(160 ** 3, dtype=torch.float64 if first == "solve" else torch.float32, device="cuda")
            b, _ = make_vec(52, 160 ** 3, torch.float32)
            run = lambda: P.pcg_solve(big, b, xb, 1e-3, 1000)  # noqa: E731
    small = P.pcg_create(64, 64, 64, torch.float32, x_dtype=torch.float64)
    bs, _ = make_vec(53, 64 ** 3, torch.float32)
    xs = torch.empty(64 ** 3, dtype=torch.float64, device="cuda")
    run()
    P.pcg_solve(small, bs, xs, 1e-3, 1000)
    torch.cuda.synchronize()
    failed = []

    def call():
        try:
            with torch.cuda.stream(sa):
                torch.cuda._sleep(cycles)
                started.set()
                run()
            ended.append(time.monotonic())
        except Exception as ex:  # noqa: BLE001
            failed.append(repr(ex))
            started.set()

    started, ended = threading.Event(), []
    t0 = time.monotonic()
    th = threading.Thread(target=call)
    th.start()
    started.wait()
    time.sleep(0.1)  # the call is waiting for its stream by now
    t1 = time.monotonic()
    P.pcg_solve(small, bs, xs, 1e-3, 1000)
    took = time.monotonic() - t1
    th.join()
    print(first, "small solve", took, "s; call", ended[0] - t0 if ended else None, "s", flush=True)
    assert not failed, failed
    assert ended[0] - t0 >= 0.8  # it had to wait for its stream
    assert took <= 0.4
    assert P.pcg_get_form(small) == P.PCG_FORM_ON_CHIP
