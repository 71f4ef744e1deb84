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


def test_device_outputs_that_share_memory_take_the_last_row():
    """The same device buffer for several outputs: the rows arrive in order,
    the last one whole (copies on the stream, not one kernel's stores)."""
    from paper_2603_16623_amd import wake as wk
    lib = wk.load()
    wk.wake_set_tiling(512, 0)
    wk.wake_set_cluster(0, 0)
    n = 5000
    inst = W.small_instance(21, n_rings=n, n_xi=300, n_peak=2.0, dxi=0.01, geometric=False)
    s = wk.WakeSolver.from_instance(inst)
    s.wake_set_grid(700, 2.0)
    s.wake_solve()
    hip = _hip_runtime()
    h, g, st = s.wake_fields(-1), s.wake_grid_fields(-1), s.wake_get_state()
    b = _Buf(hip, n)
    s.wake_fields(-1, out={k: b for k in h}, device=True)
    assert np.array_equal(b.host(), h["ur"])
    b = _Buf(hip, 2 * n)                    # two outputs half over one another
    p = b.data_ptr()
    assert lib.wake_fields(s.h, -1, p, p + 8 * (n // 2), None, None, None, None, 1) == 0
    got = b.host()
    assert np.array_equal(got[:n // 2], h["psi"][:n // 2])
    assert np.array_equal(got[n // 2:n // 2 + n], h["er_bt"])
    b = _Buf(hip, 700)
    s.wake_grid_fields(-1, out={k: b for k in g}, device=True)
    assert np.array_equal(b.host(), g["bt"])
    b = _Buf(hip, n)
    assert lib.wake_get_state(s.h, None, b.data_ptr(), b.data_ptr(), None, None, 1) == 0
    assert np.array_equal(b.host(), st["ur"])
    psi, ez = s.wake_lineout()
    b = _Buf(hip, inst.n_xi)
    assert lib.wake_lineout(s.h, b.data_ptr(), b.data_ptr(), 1) == 0
    assert np.array_equal(b.host(), ez)
    s.close()


# two and three of six rows: at once up to 4096 and 6144 rings, a transfer each beyond
@pytest.mark.parametrize("n_rings", [4096, 4097, 6144, 6145])
def test_some_rows_into_host_memory(n_rings):
    from paper_2603_16623_amd import wake as wk
    wk.load()
    wk.wake_set_tiling(512, 0)
    wk.wake_set_cluster(0, 0)
    s = wk.WakeSolver.from_instance(W.small_instance(21, n_rings=n_rings, n_xi=4, n_peak=2.0, dxi=0.1, geometric=False))
    s.wake_solve()
    whole = s.wake_fields(-1)
    for names in (("psi", "ur"), ("er_bt", "bt"), ("psi", "ez", "rho")):
        some = {k: np.full(n_rings, np.nan) for k in names}
        s.wake_fields(-1, out=some)
        for k in names:
            assert np.array_equal(some[k], whole[k]), (names, k)
    s.close()
