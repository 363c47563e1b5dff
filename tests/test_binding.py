"""The native half of the binding reads its arguments on the host; every call here is refused by the library's own checks before
any launch (no GPU)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2605_26646_amd as umas
from paper_2605_26646_amd import binding


@pytest.fixture(scope="module")
def native():
    if not os.path.exists(umas.lib_path()):
        import __graft_entry__ as g
        g.build()
    return binding._native()


def assign(native, **kw):
    """The native routing call on a graph that the library refuses (role 1 on a model that does not exist) and its message."""
    a = dict(n_roles=2, n_models=1, role_to_model=np.array([0, 1], np.int32), traj_turn_off=np.array([0, 2], np.int32), turn_role=np.array([0, 1], np.int32),
             turn_tok_off=np.array([0, 3, 5]), mask=torch.ones(5, dtype=torch.uint8), turn_pred_off=None, turn_pred=None, traj_group=None, role_reward=None,
             turn_reward=None, traj_reward=None, w_role=None, w_turn=None, w_traj=None, place_mode=0, norm_eps=1e-6, stream=0)
    status = native.assign(*{**a, **kw}.values())
    return status, umas.load_library().umas_last_error().decode()


class Index:
    def __init__(self, value):
        self.value = value

    def __index__(self):
        return self.value


@pytest.mark.parametrize("number", [int, np.int64, np.int32, np.uint8, Index, lambda v: torch.tensor(v), lambda v: np.array(v)])
def test_integers_of_every_kind_are_taken(native, number):
    want = assign(native)
    assert want[0] == -1 and "role_to_model" in want[1]
    assert assign(native, n_roles=number(2), n_models=number(1), place_mode=number(0), stream=number(0)) == want


@pytest.mark.parametrize("value", [2.0, np.float32(2), "2", None])
def test_other_numbers_are_refused(native, value):
    with pytest.raises(TypeError):
        assign(native, n_roles=value)


def unaligned(a):
    """The same values at an odd address."""
    raw = np.empty(a.nbytes + 1, np.uint8)
    out = raw[1:].view(a.dtype)
    out[:] = a
    assert out.ctypes.data % a.itemsize
    return out


def as_view(a):
    """... behind a buffer that names its type but not where it lies."""
    return memoryview(unaligned(a).view(np.uint8)).cast(a.dtype.char)


@pytest.mark.parametrize("place", [unaligned, as_view])
def test_arrays_at_any_address_are_taken(native, place):
    want = assign(native)
    assert want[0] == -1 and "role_to_model" in want[1]
    assert assign(native, role_to_model=place(np.array([0, 1], np.int32)), turn_tok_off=place(np.array([0, 3, 5])),
                  norm_eps=1e-6, w_role=place(np.ones(2, np.float32))) == want


def streams(n_turns=2):
    """A Streams object whose tensors nobody reads: the calls below are refused first."""
    one = torch.zeros(1, dtype=torch.int64)
    return umas.Streams(0, n_turns, 1, *[one] * 16)


def test_bytes_are_no_array(native):
    # numpy reads them as text, and so did the binding before it read buffers itself
    with pytest.raises(ValueError):
        native.ready_batch(streams(), np.array([0, 2], np.int32), 0, 0, b"\x01", None, 0)
    status = native.ready_batch(streams(), np.array([0, 2], np.int32), 0, 0, bytearray(b"\x01"), None, 0)
    assert status == -1 and "n_minibatch" in umas.load_library().umas_last_error().decode()


def test_offsets_without_a_dimension(native):
    """A single number has one entry, as numpy's ascontiguousarray gives it; the offsets of trajectories and turns need a dimension."""
    error = lambda: umas.load_library().umas_last_error().decode()
    assert native.ready_batch(streams(), np.array(0, np.int32), 0, 1, None, None, 0) == -1 and "from 0 to n_turns" in error()
    for zero in (np.array(0), np.array(0, np.int32), 0):
        for name in ("traj_turn_off", "turn_tok_off"):
            with pytest.raises(TypeError):
                assign(native, **{name: zero})


def test_a_call_without_host_memory_raises():
    """The check of a trajectory order needs a byte each; without them the call raises instead of ending the process."""
    child = """
import resource
import numpy as np, torch
import paper_2605_26646_amd as umas
from paper_2605_26646_amd import binding
native, n = binding._native(), 100_000_000
s = umas.Streams(0, 0, 1, *[torch.zeros(1, dtype=torch.int64)] * 16)
off, order = np.zeros(n + 1, np.int32), np.zeros(n, np.int32)
native.ready_batch(s, off[:2], 0, 1, None, order[:1], 0)                 # refused: the workspace's address
size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + umas.load_library().umas_ready_batch_workspace_bytes(n, 1) + (64 << 20), -1))
try:
    native.ready_batch(s, off, 0, 1, None, order, 0)
except RuntimeError as e:
    print("raised", e)
"""
    done = subprocess.run([sys.executable, "-c", child], cwd=os.path.dirname(os.path.dirname(umas.lib_path())), capture_output=True, text=True)
    assert done.returncode == 0 and "raised std::bad_alloc" in done.stdout, (done.returncode, done.stdout, done.stderr[-500:])
