"""Hybrid closure iteration on long x lines, up to the longest that iterated closures take (128 nodes):
the end-value kernel stages 64 of them in up to 79 KB of LDS.  Against the oracle, every output node;
bars as in test_gpu_iterate.py."""
import pytest

import synth
from tests import helpers as H
from tests.test_gpu_iterate import _iter_ref, _ops, _run

pytestmark = pytest.mark.gpu


# second derivatives in FP64 only: in FP32 the input's rounding alone, 6e-8 times 4 / (h k)^2, is above the bar here
@pytest.mark.parametrize("n,names,dtype", [((64, 12, 13), ("(1)Q1_3[1]", "(2)Q1_3[1]"), 0), ((96, 9, 12), ("(1)Q1_3[1]",), 0),
                                           ((96, 9, 12), ("(1)Q1_3[1]",), 1), ((127, 8, 9), ("(1)Q1_3[1]",), 0),
                                           ((127, 8, 9), ("(1)Q1_3[1]",), 1), ((128, 9, 8), ("(1)Q1_3[1]",), 0),
                                           ((128, 9, 8), ("(1)Q1_3[1]",), 1), ((128, 8, 12), ("(2)Q1_3[1]",), 0)])
def test_long_x_lines(cuda, n, names, dtype):
    lat = (2, 2, 1)
    wl = synth.lattice(n=n, lat=lat, ng=4, nfields=2, seed=12)
    ops = _ops(names)
    plan = H.make_plan(wl, ops, dtype=dtype)
    _, ooffs = plan.offsets()
    _, nout = plan.sizes()
    for iters in (1, 3):
        plan.set_iteration(iters, *lat)
        err = H.compare_flat(_run(plan, wl, dtype), _iter_ref(wl, ops, lat, iters, ooffs, nout), wl, ops, ooffs)
        assert err <= H.tol_for(dtype), (iters, err)
