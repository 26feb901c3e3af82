"""Argument handling of the binding, without a device."""
import ctypes
import weakref

import pytest
import torch

from paper_2106_03452_amd import _lib
from paper_2106_03452_amd import function as F
from paper_2106_03452_amd import mesh as M
from paper_2106_03452_amd import optimize as O
from paper_2106_03452_amd import slab as S


@pytest.mark.parametrize("res,points", [(7, 10), (1024, 10), (64, 0)])
def test_refused_sizes_are_refused_every_time(res, points):
    for _ in range(2):
        for f in (_lib.workspace_bytes, _lib.saved_bytes):
            with pytest.raises(_lib.PSRError):
                f(res, points)


@pytest.mark.parametrize("res", [8, 64, 256, 512])
def test_kept_sizes_are_the_librarys(res):
    out = ctypes.c_size_t(0)
    for points in (1, 20000, 20001):
        for _ in range(2):
            assert _lib.lib().psr_workspace_bytes(res, points, 1, ctypes.byref(out)) == 0
            assert _lib.workspace_bytes(res, points) == out.value
            assert _lib.lib().psr_saved_bytes(res, points, ctypes.byref(out)) == 0
            assert _lib.saved_bytes(res, points) == out.value


def test_calls_without_a_context_are_refused_before_any_device_work():
    L, n = _lib.lib(), None
    assert L.psr_marching_cubes_sized(n, n, 32, 0.0, n, n, n, 10, n, 10, n, n, n, n, n) == _lib.PSR_EINVAL
    assert L.psr_chamfer_f32(n, n, 10, n, 10, n, n, n, n, n, n, 0, n) == _lib.PSR_EINVAL
    assert L.psr_chamfer_backward_scaled(n, n, 10, n, 10, n, n, n, n, n) == _lib.PSR_EINVAL


@pytest.fixture
def no_device(monkeypatch):
    """A device 0 whose context the library refuses: a call that gets that far
    raises PSRError and launches nothing, here and where there is a GPU."""
    context = type("Context", (), {"handle": None})()
    monkeypatch.setattr(_lib, "context", lambda device=0: context)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0, raising=False)


def _host_calls():
    v, f, u = torch.rand(9, 3), torch.arange(6, dtype=torch.int32).reshape(2, 3), torch.rand(5, 3)
    x, y, grid = torch.rand(6, 3), torch.rand(7, 3), torch.rand(8, 8, 8)
    raw = lambda n: torch.zeros(n, dtype=torch.uint8)
    mesh = M.Mesh(v, f, v, torch.arange(9, dtype=torch.int32), raw(M.state_bytes(8)), 8, 0.0)
    return {
        "sample": lambda: O.sample_raw(v, f, u),
        "sample layer": lambda: O.SampleFunction.apply(v, f, u),
        "chamfer": lambda: O.chamfer_raw(x, y),
        "chamfer layer": lambda: O.ChamferFunction.apply(x, y),
        "components": lambda: O.components(v, f),
        "mesh backward": lambda: M.marching_cubes_backward(grid, mesh, v),
        "slab": lambda: S.forward_raw(x, x, 16, 2.0, 1, torch.empty(16, 16, 16), raw(48),
                                      raw(S.workspace_bytes(16, 6, 1))),
        "step": lambda: O.NativeStep(torch.device("cpu", 0), 10, 10, 10, 8)(x, x, [x] * 4, 1, 1e-3, y, u, 2.0),
        "status": lambda: F.status(raw(4096)),
        "scalars": lambda: F.scalars(raw(4096)),
    }


@pytest.mark.parametrize("call", list(_host_calls()))
def test_host_tensors_are_refused(no_device, call):
    """Their addresses mean nothing to a kernel: refused as torch.cuda does, before the library is called."""
    with pytest.raises(ValueError, match="cuda device"):
        _host_calls()[call]()


class _HeldArguments:
    """Stands in for the library in optimize: a call checks that every tensor
    whose address it was given is still alive, and keeps its arguments."""

    def __init__(self, monkeypatch):
        self.refs, self.seen, real = [], [], _lib.lib()
        def address(t):
            if t is not None:
                self.refs.append(weakref.ref(t))
            return None if t is None else t.data_ptr()
        class Library:
            def __getattr__(lib, name):
                return getattr(real, name) if name.endswith("_bytes") else lambda *args: self.call(name, args)
        monkeypatch.setattr(O, "_p", address)
        monkeypatch.setattr(O, "_st", lambda dev: 0)
        monkeypatch.setattr(O, "_ctx", lambda dev: type("Context", (), {"handle": None})())
        monkeypatch.setattr(O._lib, "lib", lambda: Library())

    def call(self, name, args):
        assert all(r() is not None for r in self.refs), f"{name}: an argument was freed before the call"
        self.refs.clear()
        self.seen.append((name, args))
        return 0


def _strided(t):
    return t.t().contiguous().t()


@pytest.mark.parametrize("call", ["sample", "sample backward", "chamfer", "chamfer backward", "components"])
def test_copies_of_strided_arguments_live_until_the_call(monkeypatch, call):
    """A copy freed while the next one is made can share its memory with it."""
    held = _HeldArguments(monkeypatch)
    v, f, u = _strided(torch.rand(9, 3)), _strided(torch.arange(9, dtype=torch.int32).reshape(3, 3)), _strided(torch.rand(9, 3))
    x, y = _strided(torch.rand(7, 3)), _strided(torch.rand(7, 3))
    if call == "sample":
        O.sample_raw(v, f, u, vnormals=_strided(torch.rand(9, 3)), face_weight=torch.ones(6)[::2])
    elif call == "sample backward":
        p = O.SampleFunction.apply(v.requires_grad_(True), f, u)
        torch.autograd.grad(p, v, _strided(torch.rand(9, 3)))
    elif call == "chamfer":
        O.chamfer_raw(x, y)
    elif call == "chamfer backward":
        loss = O.ChamferFunction.apply(x.requires_grad_(True), y)
        torch.autograd.grad(loss, x)
    else:
        O.components(v, f)
    assert len(held.seen) == (2 if "backward" in call else 1)


def _ints(address, n):
    return list((ctypes.c_int32 * n).from_address(address))


@pytest.mark.parametrize("faces", ["transposed", "columns", "contiguous"])
def test_sampling_backward_reads_the_faces_of_the_forward(monkeypatch, faces):
    """The backward's scatter indexes the vertices through the faces: rows of a
    strided array must reach it as the forward saw them."""
    held = _HeldArguments(monkeypatch)
    plain = torch.tensor([[0, 1, 2], [3, 4, 5], [6, 7, 8], [2, 4, 6]], dtype=torch.int32)
    wide = torch.cat([plain, torch.full((4, 2), 1 << 30, dtype=torch.int32)], 1)
    f = {"transposed": _strided(plain), "columns": wide[:, :3], "contiguous": plain}[faces]
    rows = []
    def call(name, args, base=held.call):
        rows.append(_ints(args[4 if name == "psr_mesh_sample" else 1], 12))
        return base(name, args)
    monkeypatch.setattr(held, "call", call)
    v = torch.rand(9, 3).requires_grad_(True)
    torch.autograd.grad(O.SampleFunction.apply(v, f, torch.rand(5, 3)), v, torch.ones(5, 3))
    assert rows == [plain.reshape(-1).tolist()] * 2


class _OnDevice(torch.Tensor):
    """A host tensor that passes for one of the device and notes the streams it is recorded on."""

    streams = []
    is_cuda = property(lambda self: True)

    def record_stream(self, stream):
        self.streams.append((self.data_ptr(), stream))


@pytest.mark.parametrize("strided", [False, True])
def test_mesh_holds_its_grid_until_the_stream_is_done(monkeypatch, strided):
    """The call returns while the mesh is being written from the grid: a grid of
    another stream must not be reused before this stream has read it."""
    def sized(*args):
        args[11]._obj.value, args[12]._obj.value, args[13]._obj.value = 4, 5, 0
        return 0
    monkeypatch.setattr(M, "_device_index", lambda dev: 0)
    monkeypatch.setattr(M, "_stream", lambda dev: 0)
    monkeypatch.setattr(M._lib, "context", lambda device: type("Context", (), {"handle": None})())
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: "current")
    M.state_bytes(8)
    monkeypatch.setattr(M._lib, "lib", lambda: type("Library", (), {"psr_marching_cubes_sized": staticmethod(sized)}))
    chi = torch.rand(8, 8, 8)
    chi = (chi.permute(2, 1, 0) if strided else chi).as_subclass(_OnDevice)
    _OnDevice.streams.clear()
    mesh = M.marching_cubes(chi)
    assert (mesh.verts.shape[0], mesh.faces.shape[0]) == (4, 5)
    assert (chi.data_ptr(), "current") in _OnDevice.streams
