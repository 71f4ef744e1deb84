"""Ring order put right by the wave sorts (256 positions a wave, merged with
their neighbours) when radii are equal and rings are a few or many positions
from their places: rings of equal radius come in the order of their ids, as
in the oracle's sort, also where a run of them lies across the blocks' ends
(256 and 128 + 256) or the last, partly filled block.  The slice on the
reordered state, and the state it pushes, against the oracle to the per-slice
tolerances of tests/parity.py."""
import numpy as np
import pytest

from oracle.mobile_ions import TwoSpeciesOracle
from oracle.wake_oracle import RingOracle
from paper_2603_16623_amd import workloads as W
from parity import check_fields, check_state, field_scales, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wk():
    from paper_2603_16623_amd import wake
    wake.load()
    yield wake
    wake.wake_set_cluster(0, 0)
    wake.wake_set_tiling(512, 0)


def _mixed(r0, reach, seed):
    """Radii r0 with rings moved up to about ``reach`` positions and runs of
    equal radii around the ends of the sorted blocks."""
    rng = np.random.default_rng(seed)
    n = len(r0)
    rho = r0.copy()
    for q in range(128, n, 128):
        a, b = max(q - rng.integers(1, 5), 0), min(q + rng.integers(1, 5), n)
        rho[a:b] = rho[a]
    rho[-3:] = rho[-3]
    order = np.argsort(np.arange(n) + rng.uniform(0, reach, n), kind="stable")
    return rho[order]


def _inst(n):
    return W.small_instance(5, n_rings=n, n_xi=60, n_peak=3.0, sigma_r=0.2, geometric=False, dxi=0.02)


# members of 256, 512 and 2048 positions; up to 32 odd-even phases and beyond
@pytest.mark.parametrize("tiling,rings,n", [((256, 0), 1, 1281), ((512, 0), 1, 1400), ((512, 0), 4, 2500)])
@pytest.mark.parametrize("reach", [0.5, 6.0, 90.0])
def test_cooperative_order_with_equal_radii(wk, tiling, rings, n, reach):
    inst = _inst(n)
    o = RingOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens)
    state = o.initial_state()
    state["rho"] = _mixed(inst.r0, reach, n)
    ref, new = o.slice(10, state, keep=True)
    wk.wake_set_tiling(*tiling)
    wk.wake_set_cluster(rings, 500)
    label = f"equal radii cooperative n={n} tiling={tiling} rings={rings} reach={reach}"
    say(label)
    s = wk.WakeSolver.from_instance(inst, record_stride=1)
    assert s.layout()[0] > 1
    s.wake_set_state(10, state["rho"], state["u"], state["fr"], state["fu"])
    s.wake_solve(10, 1)
    check_fields(s.wake_fields(10), ref, field_scales(ref), label)
    check_state(s.wake_get_state(), new, label)
    s.close()


# (63 rings moved by less than a position keep both species at the same radii:
# psi is nothing but rounding there and has no scale of its own)
@pytest.mark.parametrize("n,reach", [(63, 90.0), (257, 0.5), (257, 90.0), (1025, 0.5), (1025, 90.0)])
def test_two_species_order_with_equal_radii(wk, n, reach):
    inst = _inst(n)
    o = TwoSpeciesOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, 1836.0, inst.sources, inst.dens)
    state = o.initial_state()
    state["e"]["rho"] = _mixed(inst.r0, reach, n)
    state["i"]["rho"] = _mixed(inst.r0, reach, n + 1)
    ref, new = o.slice(10, state, keep=True)
    label = f"equal radii two species n={n} reach={reach}"
    say(label)
    s = wk.WakeSolver(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens, record_stride=1,
                      ion_mass=1836.0)
    for sp, key in ((0, "e"), (1, "i")):
        st = state[key]
        s.wake_set_species_state(sp, 10, st["rho"], st["u"], st["fr"], st["fu"])
    s.wake_solve(10, 1)
    sc = field_scales(ref)
    for q in sc:
        if "ion_" + q in ref:
            sc[q] = max(sc[q], float(np.max(np.abs(ref["ion_" + q]))))
    check_fields(s.wake_species_fields(0, 10), ref, sc, label + " electrons")
    check_fields(s.wake_species_fields(1, 10), ref, sc, label + " ions",
                 want={q: ref["ion_" + q] for q in ("psi", "er_bt", "ez", "bt")})
    check_state(s.wake_get_species_state(0), new["e"], label)
    check_state(s.wake_get_species_state(1), new["i"], label)
    s.close()
