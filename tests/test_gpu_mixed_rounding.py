"""Symmetrised mixed derivatives 1/2 (D_i D_j + D_j D_i): the two orders are the same sum with
independent roundings, and their mean keeps the smaller error of the mean.  On a periodic box the
orders are chained from first-derivative plans; with independent roundings of equal size the mean's
rms error is 1/sqrt(2) = 0.71 of one order's, so 0.9 leaves room for correlated ones (up to 0.62) and
is failed by a single order (1)."""
import pytest
import torch

import paper_2302_14858_amd as P
import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["(1)Q1_3[1]", "(1)QP_O8[1]"])
@pytest.mark.parametrize("pair", [(0, 1), (0, 2), (1, 2)])
def test_mean_of_both_orders(cuda, name, pair):
    wl = synth.periodic_box(n=(48, 48, 48), nfields=2, seed=11)
    x = torch.as_tensor(wl.data, device="cuda").float()
    i, j = pair

    def apply(ops, v, dtype):
        plan = H.make_plan(wl, ops, dtype=dtype)
        td = torch.float64 if dtype == P.CFD_F64 else torch.float32
        out = torch.empty(plan.sizes()[1], dtype=td, device="cuda")
        plan.apply(v.to(td).contiguous(), out)
        torch.cuda.synchronize()
        return out

    def order(inner, outer, dtype):
        return apply([(name, outer, -1)], apply([(name, inner, -1)], x, dtype), dtype)

    exact = 0.5 * (order(j, i, P.CFD_F64) + order(i, j, P.CFD_F64))

    def rms(v):
        return float((v.double() - exact).square().mean().sqrt())

    mixed = rms(apply([(name, i, -1, -1, j)], x, P.CFD_F32))
    single = [rms(order(j, i, P.CFD_F32)), rms(order(i, j, P.CFD_F32))]
    assert mixed <= 0.9 * min(single), (mixed, single)
