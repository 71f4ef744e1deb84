"""Slices at the sizes where the kernels' layouts change: waves without rings
and chunks of one and two rings at the wave and workgroup edges (the block
scans leave idle waves out), cooperative members whose ion-interval window is
smaller than, as long as and longer than the interval table, two-species
planes around one ring per thread, and beam tables around the entries the
two-species kernel stages in LDS.  Against the oracle, per slice, to the
tolerances of tests/parity.py."""
import dataclasses

import numpy as np
import pytest

from oracle.mobile_ions import TwoSpeciesOracle
from oracle.wake_oracle import RingOracle
from paper_2603_16623_amd import workloads as W
from parity import FIELDS, check_fields, check_state, field_scales, say

pytestmark = pytest.mark.gpu

AT = 10          # the slice compared


@pytest.fixture(scope="module")
def wk():
    from paper_2603_16623_amd import wake
    wake.load()
    yield wake
    wake.wake_set_cluster(0, 0)
    wake.wake_set_tiling(512, 0)


def _inst(n, entries=600):
    """n rings; every beam particle between slices AT and AT + 1, so that
    ``entries`` of them are in the beam table of slice AT."""
    inst = W.small_instance(9, n_rings=n, n_xi=40, n_peak=0.5, geometric=False, n_part=entries)
    b = inst.sources[0]
    inst.sources[0] = dataclasses.replace(b, xi=np.full(entries, (AT + 0.5) * inst.dxi))
    return inst


def _moved(state, rng):
    """Rings off their nodes with velocities, in order."""
    n = len(state["rho"])
    state["rho"] = np.sort(state["rho"] * np.exp(rng.normal(0, 0.02, n)))
    state["u"] = rng.normal(0, 0.02, n)
    return state


def _one(wk, inst, label):
    o = RingOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens)
    state = _moved(o.initial_state(), np.random.default_rng(inst.n_rings))
    ref, new = o.slice(AT, state, keep=True)
    say(label)
    s = wk.WakeSolver.from_instance(inst, record_stride=1)
    layout = s.layout()
    s.wake_set_state(AT, state["rho"], state["u"], state["fr"], state["fu"])
    s.wake_solve(AT, 1)
    check_fields(s.wake_fields(AT), ref, field_scales(ref), label)
    check_state(s.wake_get_state(), new, label)
    s.close()
    return layout


@pytest.mark.parametrize("n", [2, 63, 64, 65, 129, 511, 513, 1025])
@pytest.mark.parametrize("nt", [256, 512])
def test_idle_waves(wk, n, nt):
    wk.wake_set_cluster(0, 0)
    wk.wake_set_tiling(nt, 0)
    assert _one(wk, _inst(n), f"idle waves n={n} threads={nt}")[0] == 1


# members of 4 x 256 = 1024 positions, a window of 4097 nodes; the last cases
# reach over both ends of the table
@pytest.mark.parametrize("n", [1025, 4095, 4096, 4097, 6000])
def test_interval_window(wk, n):
    wk.wake_set_tiling(256, 0)
    wk.wake_set_cluster(4, 500)
    assert _one(wk, _inst(n), f"interval window n={n}") == ((n + 1023) // 1024, 4)


@pytest.mark.parametrize("n,entries", [(1, 600), (63, 831), (64, 832), (65, 833), (1023, 1), (1024, 1665),
                                       (1025, 832), (2049, 833)])
def test_two_species_sizes(wk, n, entries):
    wk.wake_set_cluster(0, 0)
    wk.wake_set_tiling(512, 0)
    inst = _inst(n, entries)
    o = TwoSpeciesOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, 1836.0, inst.sources, inst.dens)
    state = o.initial_state()
    rng = np.random.default_rng(n)
    for key in ("e", "i"):
        _moved(state[key], rng)
    ref, new = o.slice(AT, state, keep=True)
    label = f"two species n={n} beam entries={entries}"
    say(label)
    s = wk.WakeSolver(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens, record_stride=1,
                      ion_mass=1836.0)
    for sp, key in ((0, "e"), (1, "i")):
        st = state[key]
        s.wake_set_species_state(sp, AT, st["rho"], st["u"], st["fr"], st["fu"])
    s.wake_solve(AT, 1)
    sc = field_scales(ref)
    for q in FIELDS:
        sc[q] = max(sc[q], float(np.max(np.abs(ref["ion_" + q]))))
    check_fields(s.wake_species_fields(0, AT), ref, sc, label + " electrons")
    check_fields(s.wake_species_fields(1, AT), ref, sc, label + " ions",
                 want={q: ref["ion_" + q] for q in FIELDS})
    check_state(s.wake_get_species_state(0), new["e"], label)
    check_state(s.wake_get_species_state(1), new["i"], label)
    s.close()
