"""The schedule of plans used as created: partitions by kernel class, and the XCD order only where its
queues balance in every launch and a block-field's arrays fit the L2s.  Outputs against the oracle."""
import pytest

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

XCD = 4


def _plan(sizes, nfields, ops, nblocks=1, seed=79):
    wl = synth.batch64(nblocks=nblocks, nfields=nfields, sizes=sizes, ng=5, seed=seed)
    return wl, H.make_plan(wl, ops)


def _d1(name, field=-1):
    return [(name, d, field) for d in range(3)]


@pytest.mark.parametrize("name,yz", [("(1)Q1_3[1]", 2), ("(1)QP_O8[1]", 1), ("(2)Q1_3[1]", 1)])
def test_partitions_follow_the_kernel_classes(cuda, name, yz):
    """20 nodes: 2 x 12 rows where a class without longer partitions takes them, else 24 rows."""
    wl, plan = _plan((20,), 2, _d1(name))
    assert sorted(plan.get_schedule()["classes"]) == [(20, 0, yz), (20, 1, 2)]
    assert H.full_parity(plan, wl, _d1(name), 0) <= H.ERR_F64


@pytest.mark.parametrize("n,nfields,nblocks,ops,xcd", [
    (32, 16, 1, _d1("(1)Q1_3[1]"), True),                          # 16 fields of 1 MB in 8 queues
    (32, 6, 1, _d1("(1)Q1_3[1]"), False),                          # 6 fields: two queues empty
    (64, 16, 1, _d1("(1)Q1_3[1]") + _d1("(2)Q1_3[1]"), False),     # 15.8 MB per field: beyond the L2s
    # two launches of four fields each, in different queues: each leaves half of them empty
    (32, 8, 1, sum([_d1("(1)Q1_3[1]", f) for f in range(4)] + [_d1("(2)QP_O8[1]", f) for f in range(4, 8)], []), False),
])
def test_xcd_order_only_where_it_pays(cuda, n, nfields, nblocks, ops, xcd):
    wl, plan = _plan((n,), nfields, ops, nblocks)
    assert bool(plan.get_schedule()["flags"] & XCD) == xcd
    assert H.full_parity(plan, wl, ops, 0) <= H.ERR_F64
