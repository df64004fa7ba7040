"""Biased operators on fields of 4 GiB and more, whose lines the wave kernel addresses with 64-bit
offsets: every line depends on its own samples alone, so slabs of the large block (its first, middle
and last lines) are compared with small blocks that hold the same samples.  Bars as in
test_gpu_biased.py.  The ghost layers beyond the scheme's reach hold NaN, which must not show."""
import pytest
import torch

import paper_2302_14858_amd as P
from tests import helpers as H

pytestmark = pytest.mark.gpu

NG = 6


def _plan(name, d, n, dtype):
    s = P.Scheme.named(name)
    blk = dict(n=n, ng=NG, h=(0.125, 0.25, 0.5), boundary=(P.CFD_BOUNDARY_CLOSURE,) * 3)
    op = (s, d, 0) if name.endswith("-") else (s, d, -1, 0)
    return P.Plan([blk], 1, [op], dtype=dtype), max(2, s.required_ghosts())   # the narrowest class reaches two


# (1)V1 and (1)X1, (1)W1: classes of half-width 2 and 3 with six ghosts; lines of one, two and four partitions
@pytest.mark.parametrize("name,d,N,dtype", [("(1)X1-", 0, 20, 0), ("(1)X1", 0, 48, 0), ("(1)V1", 0, 48, 1),
                                            ("(1)W1-", 0, 48, 0), ("(1)X2", 2, 48, 0), ("(1)W2", 1, 40, 1)])
def test_large_fields(cuda, name, d, N, dtype):
    td, es = (torch.float64, 8) if dtype == 0 else (torch.float32, 4)
    # transverse extents: the field with its ghosts, and the output, of 4 GiB and more
    m = int((2 ** 32 / es / N) ** 0.5) + 40
    n = tuple(N if k == d else m for k in range(3))
    plan, reach = _plan(name, d, n, dtype)
    assert min(plan.sizes()) * es >= 2 ** 32 and reach < NG
    shape = tuple(v + 2 * NG for v in reversed(n))
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.rand(shape, dtype=td, device="cuda", generator=g).sub_(0.4)   # the velocity takes both signs
    axis = 2 - d
    x.narrow(axis, 0, NG - reach).fill_(float("nan"))
    x.narrow(axis, NG + N + reach, NG - reach).fill_(float("nan"))
    out = torch.empty(tuple(reversed(n)), dtype=td, device="cuda")
    plan.apply(x.reshape(-1), out.reshape(-1))
    torch.cuda.synchronize()
    w = 12
    small, _ = _plan(name, d, tuple(N if k == d else w for k in range(3)), dtype)
    for at in (0, m // 2 + 1, m - w):
        xs, want = x, out
        for k in range(3):
            if k != d:
                xs = xs.narrow(2 - k, at, w + 2 * NG)
                want = want.narrow(2 - k, at, w)
        xs = xs.contiguous()
        got = torch.empty(tuple(reversed([N if k == d else w for k in range(3)])), dtype=td, device="cuda")
        small.apply(xs.reshape(-1), got.reshape(-1))
        torch.cuda.synchronize()
        assert torch.isfinite(got).all() and torch.isfinite(want).all()
        err = float((got - want).abs().max() / got.abs().max())
        assert err <= H.tol_for(dtype), (at, err)
