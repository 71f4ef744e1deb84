"""Ring order after a push in one workgroup: wave blocks sorted, then merged
where a junction is out of order.  Rings cross many neighbours, so that most
junctions of a slice are out of order and the merges, which move the keys at
the junctions, run on every wave: each copy of one instance in a batch, many
of them on the device at once, must come out bitwise as the same slices
marched one launch each, whose orders are found from scratch."""
import numpy as np
import pytest

from oracle.wake_oracle import RingOracle
from paper_2603_16623_amd import workloads as W
from parity import FIELDS, say

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
