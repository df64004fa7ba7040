"""Biased operators at the line lengths where the wave kernel's split changes: one and two partitions
(12, 13 nodes), full and uneven partitions (24, 25, 48, 49, 96, 97), the longest y/z and x lines it
takes and the first ones it leaves to the sweep kernel (192, 193; 768, 769), lines of two and three
nodes, ghost widths equal to and above the stencil's half-width, periodic lines, and line counts that
leave a wave's last lines empty.  Against oracle/biased.py, every output node; bars as in
test_gpu_biased.py (1e-12 in FP64, 1e-5 in FP32, relative to the largest value)."""
import pytest

import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _block(n, ng, seed):
    wl = synth.batch64(seed=seed, nblocks=1, nfields=2, ng=ng, sizes=(8,))
    blk = wl.blocks[0]
    blk.n = n
    data, offs = synth._fill([blk], 2, lambda b, f, x, y, z: synth.eval_modes(wl.modes[f][0], x, y, z))
    return synth.Workload("lengths", [blk], 2, data, offs, wl.modes)


def _ops(name):
    ops = []
    for d in range(3):
        ops += [(name + "-", d, 0), (name + "+", d, 1), (name, d, -1, 1), (name + "s", d, 0)]
    return ops


@pytest.mark.parametrize("name,ng,dtype", [("(1)X2", 4, 0), ("(1)X2", 5, 0), ("(1)V1", 2, 0), ("(1)X3", 6, 1)])
@pytest.mark.parametrize("n", [(2, 3, 7), (12, 13, 24), (25, 48, 49), (96, 97, 5), (192, 193, 4), (5, 4, 192),
                               (768, 4, 2), (769, 3, 2)])
def test_line_lengths(cuda, n, name, ng, dtype):
    wl = _block(n, ng, 71)
    ops = _ops(name)
    err = H.full_parity(H.make_plan(wl, ops, dtype=dtype), wl, ops, dtype)
    assert err <= H.tol_for(dtype), err


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("M,n", [(2, (3, 13, 25)), (2, (49, 97, 128)), (2, (200, 5, 4)), (1, (4, 200, 3)), (3, (24, 12, 128))])
def test_embedded_line_lengths(cuda, M, n, dtype):
    wl = _block(n, M + 2, 72)
    ops = _ops(f"(1)W{M}")
    err = H.full_parity(H.make_plan(wl, ops, dtype=dtype), wl, ops, dtype)
    assert err <= H.tol_for(dtype), err


@pytest.mark.parametrize("name,n", [("(1)X2", (97, 13, 5)), ("(1)X1", (6, 193, 25)), ("(1)W2", (96, 24, 12)),
                                    ("(1)W3", (16, 256, 8))])
def test_periodic_line_lengths(cuda, name, n):
    wl = synth.periodic_box(n=n, nfields=2, seed=73)
    ops = _ops(name)
    err = H.full_parity(H.make_plan(wl, ops), wl, ops)
    assert err <= H.ERR_F64, err
