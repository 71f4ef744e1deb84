"""GPU test of the read-outs: fields, state, grid fields and axis lineouts
come out the same into host memory (one transfer split on the host up to
8192 rings, a transfer per row beyond) and into device memory (one kernel),
with any of the outputs left out."""
import ctypes

import numpy as np
import pytest

from paper_2603_16623_amd import workloads as W
from parity import FIELDS

pytestmark = pytest.mark.gpu


def _hip_runtime():
    """The HIP runtime the library itself loaded."""
    with open("/proc/self/maps") as fh:
        paths = {ln.split()[-1] for ln in fh if "libamdhip64" in ln}
    assert paths, "libamdhip64 not loaded"
    hip = ctypes.CDLL(sorted(paths)[0])
    hip.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    hip.hipFree.argtypes = [ctypes.c_void_p]
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    return hip


class _Buf:
    """n doubles of device memory, filled with NaN."""

    def __init__(self, hip, n):
        self.hip, self.n, self.p = hip, n, ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(self.p), 8 * max(n, 1)) == 0
        nan = np.full(n, np.nan)
        assert hip.hipMemcpy(self.p, nan.ctypes.data, 8 * n, 1) == 0

    def data_ptr(self):
        return self.p.value

    def host(self):
        out = np.empty(self.n)
        assert self.hip.hipMemcpy(out.ctypes.data, self.p, 8 * self.n, 2) == 0
        assert self.hip.hipFree(self.p) == 0
        return out


@pytest.mark.parametrize("n_rings", [1, 700, 8192, 8193])
def test_host_and_device_readouts_agree(n_rings):
    from paper_2603_16623_amd import wake as wk
    wk.load()
    wk.wake_set_tiling(512, 0)
    wk.wake_set_cluster(0, 0)
    inst = W.small_instance(21, n_rings=n_rings, n_xi=12, n_peak=2.0, dxi=0.1, geometric=False)
    s = wk.WakeSolver.from_instance(inst, record_stride=5)
    s.wake_set_grid(33, 2.0)
    s.wake_solve()
    hip = _hip_runtime()
    for sl in (-1, 5):
        h = s.wake_fields(sl)
        assert all(np.all(np.isfinite(h[k])) for k in FIELDS)
        d = {k: _Buf(hip, n_rings) for k in h}
        s.wake_fields(sl, out=d, device=True)
        for k in h:
            assert np.array_equal(d[k].host(), h[k]), k
            one = {k: np.full(n_rings, np.nan)}          # one output alone
            s.wake_fields(sl, out=one)
            assert np.array_equal(one[k], h[k]), k
    g = s.wake_grid_fields(-1)
    d = {k: _Buf(hip, 33) for k in ("er_bt", "bt")}
    s.wake_grid_fields(-1, out=d, device=True)
    for k in d:
        assert np.array_equal(d[k].host(), g[k]), k
    psi, ez = s.wake_lineout()
    dp, de = _Buf(hip, inst.n_xi), _Buf(hip, inst.n_xi)
    lib = wk.load()
    assert lib.wake_lineout(s.h, dp.data_ptr(), None, 1) == 0
    assert lib.wake_lineout(s.h, None, de.data_ptr(), 1) == 0
    assert np.array_equal(dp.host(), psi) and np.array_equal(de.host(), ez)
    only = np.full(inst.n_xi, np.nan)
    assert lib.wake_lineout(s.h, None, only.ctypes.data, 0) == 0
    assert np.array_equal(only, ez)
    s.close()
