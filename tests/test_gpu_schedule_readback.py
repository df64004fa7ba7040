"""A schedule that is read back can be set again, entry by entry, also for plans whose only lines are
those of W operators' embedded second derivatives."""
import pytest

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ops", [[("(1)W2", d, -1, 0) for d in range(3)],
                                 [("(1)W2-", d, 0) for d in range(3)] + [("(1)Q1_3[1]", 0)]])
def test_w_operators(cuda, ops):
    wl = synth.batch64(nblocks=3, nfields=2, sizes=(16, 24), ng=5, seed=77)
    plan = H.make_plan(wl, ops)
    want = {(b.n[d], int(d == 0)) for b in wl.blocks for d in range(3)}
    got = plan.get_schedule()
    assert {c[:2] for c in got["classes"]} == want
    for N, x, P in got["classes"]:
        other = 2 if P != 2 else 1
        plan.set_schedule(N=N, xlines=x, partitions=other)
        assert (N, x, other) in plan.get_schedule()["classes"]
        plan.set_schedule(N=N, xlines=x, partitions=P)
    assert plan.get_schedule()["classes"] == got["classes"]
    assert H.full_parity(plan, wl, ops, 0) <= H.ERR_F64
