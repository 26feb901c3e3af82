"""Argument handling of the binding, without a device."""
import ctypes

import pytest

from paper_2106_03452_amd import _lib


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
