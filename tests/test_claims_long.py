"""A claim on CUs that is willing to wait as long as it takes (a batch's), on
the CPU: it is served when the holder ends, in its turn, and the length of the
wait does not overflow the clock."""
import re
import os
import threading
import time

from test_onchip_plan import _Hold, lib  # noqa: F401

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_23343_amd", "csrc")


def test_a_batch_waits_for_its_claim(lib):  # noqa: F811
    text = open(os.path.join(SRC, "resident.hpp")).read()
    wait = float(re.search(r"RES_HOLD_BATCH_S = ([0-9.e]+);", text).group(1))
    # no batch launch goes on without its claim after a short wait
    claims = re.findall(r"CuHold hold\((.*)\);", open(os.path.join(SRC, "batched.hip")).read())
    assert claims and all(c.endswith("RES_HOLD_BATCH_S") for c in claims)
    first = _Hold(lib, 1, 256, 1.0)
    got = []

    def claim():
        t = time.monotonic()
        h = _Hold(lib, 256, 256, wait)
        got.append((h.ok, time.monotonic() - t))
        h.release()

    th = threading.Thread(target=claim)
    th.start()
    time.sleep(0.3)
    assert not got  # still waiting
    first.release()
    th.join(5)
    assert got and got[0][0] and got[0][1] >= 0.25
