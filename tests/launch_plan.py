"""The number of timesteps of each launch of a step call (host code of the library, no GPU needed)."""

import ctypes

from paper_1705_09807_amd import native as N
from paper_1705_09807_amd.sim import make_params


def launch_plan(nx, ny, n, t=0, recorded=False, cus=256, **kw):
    """Steps of the launches of step(n) at time t."""
    f = N.load().lbm_internal_launch_plan
    f.restype = ctypes.c_int64
    f.argtypes = [ctypes.POINTER(N.LbmParams), ctypes.c_int32, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32,
                  ctypes.POINTER(ctypes.c_int32), ctypes.c_int64]
    p = make_params(nx, ny, nu=2e-3, eta=3e-3, b_ref=(0.01, 0.0), **kw)
    steps = (ctypes.c_int32 * max(n, 1))()
    count = f(ctypes.byref(p), cus, n, t, int(recorded), steps, n)
    assert count >= 0, N.load().lbm_last_error()
    return list(steps[:count])
