"""Captured applies: captures of at most four launches are replayed as plain launches, larger ones and
those with forked streams as a HIP graph.  Both kinds are replayed several times, on changed input,
with eager applies and synchronizations between the replays, and every replay is compared with the
eager result bit for bit."""
import pytest
import torch

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

# ten kernel classes: centred first degree, second degree alone, explicit, dissipation, and biased half-widths 2 to 5
MANY = ([("(1)Q1_3[1]", d, 0) for d in range(3)] + [("(2)QP_O8[1]", d, 1) for d in range(3)] +
        [("(1)E3", 0, 0), ("KO8[0.04]", 1, 0), ("(1)V1-", 0, 0), ("(1)X1", 1, -1, 0), ("(1)X2s", 2, 1), ("(1)X3+", 0, 0),
         ("(1)W2", 2, -1, 1)])
FEW = [("(1)QP_O8[1]", d) for d in range(3)]


@pytest.mark.parametrize("ops,schedule", [(MANY, {}), (MANY, {"concurrent": True}), (FEW, {}),
                                          (FEW, {"split_x": True, "concurrent": True})])
def test_replays_match_eager(cuda, ops, schedule):
    wl = synth.batch64(nblocks=3, nfields=2, sizes=(16, 24), ng=6, seed=78)
    plan = H.make_plan(wl, ops)
    if schedule:
        plan.set_schedule(**schedule)
    x = torch.from_numpy(wl.data).to("cuda")
    y = torch.full((plan.sizes()[1],), float("nan"), dtype=torch.float64, device="cuda")
    eager = torch.empty_like(y)
    plan.capture_graph(x, y)
    assert plan.graph_status() == 1
    side = torch.cuda.Stream()
    for k in range(5):
        x.mul_(-1.25)
        eager.fill_(float("nan"))
        y.fill_(float("nan"))
        if k % 2:
            side.wait_stream(torch.cuda.current_stream())
            plan.launch_graph(side)
            torch.cuda.current_stream().wait_stream(side)
        else:
            plan.launch_graph()
        plan.apply(x, eager)
        torch.cuda.synchronize()
        assert torch.isfinite(eager).all() and torch.equal(y, eager), k
    plan.set_schedule(persistent=False)   # another schedule drops the capture
    assert plan.graph_status() == 0
    with pytest.raises(Exception):
        plan.launch_graph()
