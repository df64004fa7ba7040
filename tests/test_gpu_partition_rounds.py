"""Partitions of plans of few rounds of workgroups: the longer ones where they save a round.  17-node y and
z lines take two partitions of 12 rows or one of 24; the counts below are for 256 compute units."""
import numpy as np
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


@pytest.mark.parametrize("dtype,nfields", [(0, 15), (1, 20)])
def test_one_pass_equals_the_allocation_free_apply(cuda, dtype, nfields):
    """One operator on one block, 128 workgroups of 2 x 12 rows per field: two rounds, one with 24 rows;
    the plan's output is still that of the apply without a plan, bit for bit."""
    import torch
    import paper_2302_14858_amd as P
    n, ng = (64, 17, 256), 4
    rng = np.random.default_rng(89)
    x = torch.from_numpy(rng.standard_normal((nfields,) + tuple(v + 2 * ng for v in n[::-1]))).flatten()
    x = x.to(device="cuda", dtype=torch.float32 if dtype else torch.float64)
    block = dict(n=n, ng=ng, h=(0.01, 0.02, 0.03), boundary=(P.CFD_BOUNDARY_CLOSURE,) * 3)
    scheme = P.Scheme.named("(1)Q1_3[1]")
    y = torch.full((nfields * n[0] * n[1] * n[2],), float("nan"), dtype=x.dtype, device="cuda")
    P.cfd_apply_block_noalloc(scheme, block, 1, nfields, x, y, field=-1, dtype=dtype)
    plan = P.Plan([block], nfields, [(scheme, 1)], dtype=dtype)
    out = torch.empty_like(y)
    plan.apply(x, out)
    torch.cuda.synchronize()
    assert torch.equal(y, out)
