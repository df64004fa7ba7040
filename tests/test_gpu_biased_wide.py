"""x lines of more than 64 columns, ghosts included, which the biased wave kernel moves in column blocks
of 64 in kernels of their own: one column past a block and full blocks (55, 118, 119, 182 nodes with 5
ghosts), the partition counts that change the rows of a block (96, 97, 192, 193, 384, 385), planes of
fewer rows than a wave holds and more, line counts that leave a wave's last lines empty, periodic
lines, and plans whose other x lines are short (the same kernel takes them).  Against
oracle/biased.py, every output node; bars as in test_gpu_biased.py (1e-12 in FP64, 1e-5 in FP32,
relative to the largest value)."""
import pytest

import synth
from tests import helpers as H
from tests.test_gpu_biased_lengths import _block, _ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,dtype", [("(1)X2", 0), ("(1)X2", 1), ("(1)W2", 0), ("(1)W2", 1)])
@pytest.mark.parametrize("n", [(54, 9, 8), (55, 9, 8), (55, 3, 7), (64, 16, 4), (96, 8, 3), (97, 5, 5), (118, 3, 9),
                               (119, 4, 4), (182, 4, 3), (192, 6, 3), (193, 4, 3), (384, 3, 3), (385, 3, 4)])
def test_wide_x_lines(cuda, n, name, dtype):
    if "W" in name and max(n) > 192:
        n = (n[0] // 2,) + n[1:]
    wl = _block(n, 5, 74)
    ops = _ops(name)
    err = H.full_parity(H.make_plan(wl, ops, dtype=dtype), wl, ops, dtype)
    assert err <= H.tol_for(dtype), err


@pytest.mark.parametrize("name,ng", [("(1)X2", 5), ("(1)V1", 3), ("(1)W3", 5), ("(1)X3", 6)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_mixed_lengths(cuda, name, ng, dtype):
    wl = synth.batch64(nblocks=6, nfields=3, sizes=(12, 17, 25, 80), ng=ng, seed=75)
    assert any(b.n[0] == 80 for b in wl.blocks) and any(b.n[0] < 48 for b in wl.blocks)
    ops = _ops(name)
    err = H.full_parity(H.make_plan(wl, ops, dtype=dtype), wl, ops, dtype)
    assert err <= H.tol_for(dtype), err


@pytest.mark.parametrize("name,n", [("(1)X2", (65, 9, 4)), ("(1)X1", (128, 5, 6)), ("(1)W2", (96, 24, 12))])
def test_periodic_wide(cuda, name, n):
    wl = synth.periodic_box(n=n, nfields=2, seed=76)
    ops = _ops(name)
    err = H.full_parity(H.make_plan(wl, ops), wl, ops)
    assert err <= H.ERR_F64, err
