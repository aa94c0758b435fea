"""mecefo_init() prepares every kernel (dynamic-LDS limits, the static scratch address), so that the first
call of a process can already be recorded into a HIP graph: no eager warm-up call per shape is needed."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("tile", ["auto", "L8", "S", "S4", "T", "T2"])
def test_first_call_of_a_fresh_process_under_graph_capture(tile):
    child = os.path.join(HERE, "graph_after_init_child.py")
    res = subprocess.run([sys.executable, "-u", child, tile], capture_output=True, text=True, timeout=110)
    assert res.returncode == 0, f"child failed ({res.returncode}):\n{res.stdout[-2000:]}\n{res.stderr[-4000:]}"
    assert res.stdout.strip().endswith("OK"), res.stdout[-2000:]


def test_a_repeated_init_costs_one_look_at_the_device():
    """Programs call mecefo_init wherever they make a plan: after the first call on a device it must not walk over the
    library's kernels (8.6 us for 130 of them).  Least of 300 calls through ctypes, itself below a microsecond."""
    import time

    from paper_2510_16415_amd import binding as B
    B.mecefo_init()
    call, least = B.lib().mecefo_init, 1.0
    for _ in range(300):
        t = time.perf_counter()
        assert call() == B.OK
        least = min(least, time.perf_counter() - t)
    print("repeated mecefo_init: %.2f us" % (least * 1e6))
    assert least < 3e-6
