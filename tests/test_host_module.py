"""The package's host module as its callers see it: it lets other threads run while it launches."""
import ctypes
import sys
import threading

import pytest
import torch

from paper_2503_12491_amd import _ffi
from paper_2503_12491_amd.binding import make_params, make_shape


@pytest.fixture(scope="module")
def host():
    return _ffi.host()


def _calls(host):
    """One call of every entry that launches, with arguments that the library refuses before it touches a device."""
    shape = make_shape(1, 1, 3, 2, 64, 64, 32, torch.float32)        # three query heads over two key/value heads
    params = make_params()
    plan = _ffi.cake_decode_plan(shape, ctypes.addressof(params), rank=3)
    x = torch.zeros(1, 2, 64)
    y = torch.zeros(1, 2, 32, 64)
    at = ctypes.addressof(plan)
    return [("pass_launch", lambda: host.pass_launch(0, 3, 0, 0)), ("pass_place", lambda: host.pass_place(0, 0, 0, 0)),
            ("decode_run", lambda: host.decode_run(at, x, x, x, 0)), ("cascade_stage", lambda: host.cascade_stage(0, 0, y, y, y, y, 0)),
            ("cascade_gather", lambda: host.cascade_gather(0, 1, 0, 0, 0))], (shape, params, plan)


@pytest.mark.parametrize("which", range(5))
def test_other_threads_run_while_it_launches(host, which):
    """With a switch interval of hours a waiting thread gets the interpreter only when it is given up: a thread
    started beside the calls must have had it long before they end."""
    calls, keep = _calls(host)
    name, call = calls[which]
    assert call() < 0                                                # refused, not launched
    ran = threading.Event()
    waiting = threading.Event()

    def other():
        waiting.set()
        lock.acquire()                                               # held by the main thread until its calls begin
        ran.set()

    lock = threading.Lock()
    before = sys.getswitchinterval()
    lock.acquire()
    thread = threading.Thread(target=other, daemon=True)
    thread.start()
    waiting.wait()
    sys.setswitchinterval(1e4)
    try:
        lock.release()
        done = any(call() >= 0 or ran.is_set() for _ in range(200000))
    finally:
        sys.setswitchinterval(before)
    thread.join(10)
    assert done, f"{name} kept the interpreter"
