"""Partitions of plans of few rounds of workgroups: the longer ones where they save a round.  17-node y and
z lines take two partitions of 12 rows or one of 24; the counts below are for 256 compute units."""
import pytest

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

D1 = [("(1)Q1_3[1]", d, -1) for d in range(3)]


@pytest.mark.parametrize("nblocks,nfields,yz", [(64, 2, 1),     # 1152 workgroups of 2 x 12 rows, 896 of 24: one round less
                                                (27, 2, 2),     # one round either way
                                                (64, 12, 2)])   # seven rounds: registers count, not rounds
def test_longer_partitions_where_they_save_a_round(cuda, nblocks, nfields, yz):
    wl = synth.batch64(nblocks=nblocks, nfields=nfields, sizes=(17,), ng=5, seed=83)
    plan = H.make_plan(wl, D1)
    assert sorted(plan.get_schedule()["classes"]) == [(17, 0, yz), (17, 1, 2)]
    assert H.full_parity(plan, wl, D1, 0) <= H.ERR_F64


def test_a_set_partition_stays(cuda):
    wl = synth.batch64(nblocks=64, nfields=2, sizes=(17,), ng=5, seed=83)
    plan = H.make_plan(wl, D1)
    plan.set_schedule(N=17, xlines=False, partitions=2)
    assert sorted(plan.get_schedule()["classes"]) == [(17, 0, 2), (17, 1, 2)]
    assert H.full_parity(plan, wl, D1, 0) <= H.ERR_F64
