"""Ring order after a push in one workgroup: wave blocks sorted, then merged
where a junction is out of order.  Rings cross many neighbours, so that most
junctions of a slice are out of order and the merges, which move the keys at
the junctions, run on every wave: each copy of one instance in a batch, many
of them on the device at once, must come out bitwise as the same slices
marched one launch each, whose orders are found from scratch.  Rings of equal
radius come in the order of their ids, as in the oracle's sort, in the sorts
after a push of single workgroups and of cooperative members."""
import numpy as np
import pytest

from oracle.wake_oracle import RingOracle
from paper_2603_16623_amd import workloads as W
from parity import FIELDS, check_fields, field_scales, pushed_by_device, say

pytestmark = pytest.mark.gpu

AT = 10


@pytest.fixture(scope="module")
def wk():
    from paper_2603_16623_amd import wake
    wake.load()
    yield wake
    wake.wake_set_cluster(0, 0)
    wake.wake_set_tiling(512, 0)


def _inst(n):
    return W.small_instance(5, n_rings=n, n_xi=40, n_peak=2.0, geometric=False)


# a step moves a ring by 0.02 * 1.5 u, u ~ 40 spacings' worth: within a block
# pass's reach for most rings, beyond it for a few (a second round)
@pytest.mark.parametrize("nt,n", [(256, 1300), (256, 4096), (512, 3001), (512, 8192)])
def test_block_merges_in_a_batch_of_copies(wk, nt, n):
    wk.wake_set_tiling(nt, 0)
    wk.wake_set_cluster(0, 0)
    inst = _inst(n)
    state = RingOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens).initial_state()
    u = np.random.default_rng(n).normal(0, 40 * (3.0 / n) / (1.5 * inst.dxi), n)
    slices, copies = 5, 96
    say(f"block merges after a push n={n} threads={nt}")
    one = wk.WakeSolver.from_instance(inst, record_stride=1)
    assert one.layout()[0] == 1
    one.wake_set_state(AT, state["rho"], u)
    for m in range(slices):
        one.wake_solve(AT + m, 1)
    assert one.wake_status()[0] == -1
    want, end = one.wake_fields(AT + slices - 1), one.wake_get_state()
    one.close()
    solvers = [wk.WakeSolver.from_instance(inst, record_stride=1) for _ in range(copies)]
    for s in solvers:
        s.wake_set_state(AT, state["rho"], u)
    b = wk.WakeBatch(solvers)
    b.wake_batch_solve(slices)
    b.wake_batch_sync()
    for s in solvers:
        got, st = s.wake_fields(AT + slices - 1), s.wake_get_state()
        for q in FIELDS + ("rho",):
            assert np.array_equal(got[q], want[q]), q
        for q in ("rho", "ur", "f_rho", "f_u"):
            assert np.array_equal(st[q], end[q]), q
    c = solvers[0].wake_counters()
    say({k: c[k] for k in ("fixups", "general_fixups")})
    assert c["fixups"] >= slices - 1
    b.close()
    for s in solvers:
        s.close()


# single workgroups (rings per thread 0), members of 512 and 2048 positions
@pytest.mark.parametrize("tiling,rings,n", [((256, 0), 0, 1281), ((512, 0), 0, 2500), ((256, 0), 2, 1400),
                                            ((512, 0), 4, 4500)])
@pytest.mark.parametrize("places", [2.0, 70.0])
def test_equal_radii_after_a_push(wk, tiling, rings, n, places):
    inst = _inst(n)
    o = RingOracle(inst.r0, inst.dr, inst.dxi, inst.n_xi, inst.sources, inst.dens)
    state = o.initial_state()
    rng = np.random.default_rng(n)
    # runs of equal radii over the ends of the sorted and of the merged blocks;
    # rings without momentum keep their radius through the push
    for q in range(128, n, 128):
        a, b = max(q - rng.integers(1, 5), 0), min(q + rng.integers(1, 5), n)
        state["rho"][a:b] = state["rho"][a]
    state["rho"][-3:] = state["rho"][-3]
    move = rng.random(n) < 0.1
    state["u"][move] = rng.normal(0, places * (3.0 / n) / (1.5 * inst.dxi), move.sum())
    wk.wake_set_tiling(*tiling)
    wk.wake_set_cluster(rings, 500 if rings else 0)
    label = f"equal radii after a push n={n} tiling={tiling} rings={rings} places={places}"
    say(label)
    _, mid = pushed_by_device(wk, inst, AT, state)
    still = state["u"] == 0.0
    assert np.array_equal(mid["rho"][still], state["rho"][still])
    ref, _ = o.slice(AT + 1, mid, keep=True)
    s = wk.WakeSolver.from_instance(inst, record_stride=1)
    assert (s.layout()[0] > 1) == (rings > 0)
    s.wake_set_state(AT, state["rho"], state["u"], state["fr"], state["fu"])
    s.wake_solve(AT, 2)
    got = s.wake_fields(AT + 1)
    check_fields(got, ref, field_scales(ref), label)
    assert np.array_equal(got["rho"], mid["rho"])
    assert s.wake_counters()["fixups"] >= 1
    s.close()
