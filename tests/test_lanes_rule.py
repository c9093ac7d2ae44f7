"""The rule for lanes a receiver (step_lanes) and the dispatchers of the step kernels agree on
the tile shapes that have a kernel of one lane; another shape refuses it."""
import ctypes

import pytest

from paper_2002_09217_amd import pond

INVALID_VALUE = 1


class LaunchCtx(ctypes.Structure):
    _fields_ = [("dim", ctypes.c_int), ("nx", ctypes.c_int), ("ny", ctypes.c_int), ("N", ctypes.c_int),
                ("fp32", ctypes.c_int), ("st", ctypes.c_void_p), ("stream_tile", ctypes.c_int),
                ("ev_start", ctypes.c_void_p), ("ev_stop", ctypes.c_void_p), ("nz", ctypes.c_int),
                ("law", ctypes.c_int), ("fused", ctypes.c_bool), ("lanes", ctypes.c_int)]


def internal(name, *argtypes):
    f = getattr(pond.load(), name)
    f.argtypes, f.restype = argtypes, ctypes.c_int
    return f


@pytest.mark.parametrize("launcher", ["_ZN4pond13launch_streamERKNS_9LaunchCtxEPKNS_8SlotDescEii",
                                      "_ZN4pond17launch_step_fusedERKNS_9LaunchCtxEPKNS_8SlotDescEii"])
@pytest.mark.parametrize("fp32", [0, 1, 2])
def test_one_lane_only_where_there_is_a_kernel(launcher, fp32):
    launch = internal(launcher, ctypes.POINTER(LaunchCtx), ctypes.c_void_p, ctypes.c_int, ctypes.c_int)
    lanes = internal("_ZN4pond10step_lanesERKNS_9LaunchCtxEi", ctypes.POINTER(LaunchCtx), ctypes.c_int)
    for tile in range(6):
        c = LaunchCtx(dim=2, nx=64, ny=64, N=4096, fp32=fp32, stream_tile=tile, nz=1, fused="fused" in launcher, lanes=1)
        one = lanes(ctypes.byref(c), 1 << 20) == 1
        assert lanes(ctypes.byref(c), 256) == 2
        # (a launch of no workgroups, and without a device: refused in another way where there is a kernel)
        assert (launch(ctypes.byref(c), None, 0, 0) == INVALID_VALUE) == (not one), f"tile {tile}"
