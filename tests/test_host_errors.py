"""What the library's host code does where a HIP call or an allocation fails,
on the library as it was built, with the HIP calls answered by
tests/c_abi/host_hip.cpp: no device, kernels counted and not run."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROLOGUE = """
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library, so that its calls land there
from paper_2106_03452_amd import _lib
I = ctypes.c_int
class State(ctypes.Structure):
    _fields_ = ([(n, I) for n in ("host_live", "event_live", "launches", "pending", "device_syncs",
                                  "host_frees_unsynced", "fail_event_sync", "fail_new", "capturing")] +
                [(n, ctypes.c_int64) for n in ("mesh_verts", "mesh_tris")])
st = State.in_dll(hip, "host_hip")
st.mesh_verts, st.mesh_tris = 300, 600
L, ctx = _lib.lib(), _lib.Context(0)
room = ctypes.create_string_buffer(1 << 20)
at = (ctypes.addressof(room) + 4095) & ~4095
def mesh(nv=None, nt=None):
    return L.psr_marching_cubes_sized(ctx.handle, at, 32, 0.0, at, at, at, 1000, at, 1000, at, nv, nt, None, None)
"""


@pytest.fixture(scope="module")
def host_hip(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_hip") / "host_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-o", out,
                    os.path.join(ROOT, "tests", "c_abi", "host_hip.cpp")], check=True, timeout=120)
    return out


def _run(host_hip, body):
    got = subprocess.run([sys.executable, "-c", PROLOGUE + body, host_hip], cwd=ROOT, capture_output=True, text=True,
                         timeout=120)
    assert got.returncode == 0, f"exit status {got.returncode}\n{got.stdout}{got.stderr}"


def test_mesh_totals_under_a_failing_allocation(host_hip):
    """No exception leaves a C entry: the call reports the lack of memory, and
    one that finds a pair in the pool needs none."""
    _run(host_hip, """
st.fail_new = 1
rc = mesh()
st.fail_new = 0
assert rc == _lib.PSR_ENOMEM and st.launches == 0, rc
nv = ctypes.c_int64(0)
assert mesh(ctypes.byref(nv)) == 0 and nv.value == 300
st.fail_new = 1
rc = mesh()
st.fail_new = 0
assert rc == 0, rc
ctx.close()
assert (st.host_live, st.event_live) == (0, 0)
""")


def test_mesh_totals_of_failed_calls_are_freed_with_the_context(host_hip):
    """A kernel of a failed call may still write its pair: kept from the pool,
    and freed once the device is idle."""
    _run(host_hip, """
assert mesh() == 0
st.fail_event_sync = 1
for _ in range(3):
    assert mesh() == _lib.PSR_EDEVICE
st.fail_event_sync = 0
live = st.host_live
assert mesh() == 0 and mesh() == 0  # a new pair, reused
assert st.host_live == live + 1, (st.host_live, live)
ctx.close()
assert (st.host_live, st.event_live, st.host_frees_unsynced) == (0, 0, 0), (st.host_live, st.event_live)
""")


def test_sized_call_under_capture_takes_nothing(host_hip):
    """Refused as before, but before anything is recorded or taken: however
    often it happens, nothing piles up."""
    _run(host_hip, """
st.capturing = 1
for _ in range(50):
    assert mesh() == _lib.PSR_EDEVICE
assert st.launches == 0 and st.host_live == 0 and st.event_live == 0, (st.launches, st.host_live)
st.capturing = 0
assert mesh() == 0
ctx.close()
assert (st.host_live, st.event_live) == (0, 0)
""")


@pytest.mark.parametrize("verts,tris,code", [(70000, 600, "PSR_ETOOBIG"), (300, 70000, "PSR_ETOOBIG"),
                                             (0, 0, "PSR_EDEGENERATE")])
def test_refused_optimisation_step_leaves_nothing_running(host_hip, verts, tris, code):
    """A step that ends at its mesh's size returns with the workspace idle: its
    caller makes a larger one or gives up, and may free this one."""
    _run(host_hip, f"st.mesh_verts, st.mesh_tris, code = {verts}, {tris}, _lib.{code}" + """
n = ctypes.c_size_t(0)
assert L.psr_opt_step_workspace_bytes(32, 100, 100, 100, 65536, 65536, ctypes.byref(n)) == 0
ws = ctypes.create_string_buffer(n.value + 256)
w = (ctypes.addressof(ws) + 255) & ~255
counts = (ctypes.c_int64 * 2)()
rc = L.psr_opt_step(ctx.handle, at, at, 100, at, at, at, at, 1, 1e-3, 0.9, 0.999, 1e-8, at, 100, at, 100, 32, 2.0,
                    65536, 65536, at, counts, w, n, None)
assert rc == code and list(counts) == [st.mesh_verts, st.mesh_tris], rc
assert st.launches > 0 and st.pending == 0, (st.launches, st.pending)
""")
