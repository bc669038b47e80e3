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


def _without_storage(kind, shape):
    """Tensors of that shape whose memory or strides cannot be asked for."""
    if kind == "sparse":
        return torch.zeros(shape).to_sparse()
    if kind == "fake":
        from torch._subclasses.fake_tensor import FakeTensorMode
        with FakeTensorMode():
            return torch.zeros(shape)
    return torch._C._functorch._add_batch_dim(torch.zeros((2,) + shape), 0, torch._C._functorch._vmap_increment_nesting(2, "error"))


@pytest.mark.parametrize("kind", ["sparse", "fake", "vmap"])
@pytest.mark.parametrize("entry", ["decode_run", "cascade_stage", "layer_views"])
def test_tensors_without_memory_raise(entry, kind):
    """An error of the tensor library becomes a Python exception, whichever call meets it (in a process of its own:
    an exception that leaves the module ends the process)."""
    import os
    import subprocess
    code = f"""
import ctypes, numpy as np, torch, sys
sys.path.insert(0, {os.path.dirname(os.path.abspath(__file__))!r})
from test_host_module import _calls, _without_storage, _ffi
host = _ffi.host()
_, keep = _calls(host)
x, y, z = [_without_storage({kind!r}, s) for s in ((1, 2, 64), (1, 2, 32, 64), (65536,))]
rows = np.ones((1, 1), dtype=np.int32)
try:
    if {entry!r} == "decode_run": host.decode_run(ctypes.addressof(keep[2]), x, x, x, 0)
    elif {entry!r} == "cascade_stage": host.cascade_stage(0, 0, y, y, y, y, 0)
    else: host.layer_views(z, z, z, z, rows.ctypes.data, 1, 1, 2, 32, 64)
except Exception as e:
    print("raised", type(e).__name__, str(e)[:100].replace("\\n", " "))
else:
    print("returned")
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    print(r.stdout, r.stderr[-300:])
    assert r.returncode == 0, (r.returncode, r.stderr[-400:])
    if kind != "fake":                       # a fake tensor's address is 0, which the library refuses where it reads it
        assert r.stdout.startswith("raised")


def test_a_session_stage_that_is_refused_gives_its_return_code(host):
    calls, keep = _calls(host)
    shape, params, _ = keep
    session = _ffi.cake_session(shape, params, 1)
    y = torch.zeros(1, 2, 32, 64)
    stage = lambda: host.session_stage(ctypes.addressof(session), 0, y, y, y, None, y, 1, 0)
    assert stage()[0] == 0 and stage()[1] < 0 and stage()[2:] == (None,) * 5
    with pytest.raises(ValueError):
        host.session_stage(ctypes.addressof(session), 1, y, y, y, None, y, 1, 0)
    with pytest.raises(AssertionError):
        host.session_stage(ctypes.addressof(session), 0, y, y, y[:, :, :, ::2], None, y, 1, 0)
    with pytest.raises(ValueError):
        host.slab_views(torch.zeros(10), [4], [(2, 4)])
    assert [t.tolist() for t in host.slab_views(torch.arange(10), [4, 0], [(2, 3), (0, 5)])] == [[[4, 5, 6], [7, 8, 9]], []]
