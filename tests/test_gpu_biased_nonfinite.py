"""How far a NaN or an infinity in the input of a biased operator reaches.  A left-biased row takes the
nodes up to the half-width h on either side (the closure row one node more to the right) and every later
row of its line; the right-biased operator is the mirror image.  So a value at node j leaves the other
lines and fields finite and, on its own line, the left-biased rows before j - h (the first two rows are
solved together), while the rows from j on are not finite; a ghost beyond the reach shows nowhere.
In the velocity a value acts at its own node alone: an infinity shows there, a NaN counts as no
velocity (fmin and fmax take their other operand)."""
import numpy as np
import pytest
import torch

import paper_2302_14858_amd as P

pytestmark = pytest.mark.gpu


def _run(name, d, n, ng, x, dtype, ops_of):
    td = torch.float64 if dtype == 0 else torch.float32
    blk = dict(n=n, ng=ng, h=(0.125, 0.25, 0.5), boundary=(P.CFD_BOUNDARY_CLOSURE,) * 3)
    ops = [(P.Scheme.named(name + t), d) + a for t, a in ops_of]
    plan = P.Plan([blk], 3, ops, dtype=dtype)
    out = torch.zeros(plan.sizes()[1], dtype=td, device="cuda")
    plan.apply(x.to(td).reshape(-1).contiguous(), out)
    torch.cuda.synchronize()
    # [operator][field][along the line][other][other]
    y = out.reshape((len(ops), 3) + tuple(reversed(n))).movedim(4 - d, 2)
    return torch.isfinite(y).cpu().numpy()


def _shapes():
    for d, N in ((0, 12), (0, 25), (0, 48), (0, 97), (1, 13), (1, 37), (1, 100), (2, 12), (2, 49), (2, 192), (2, 200)):
        yield d, N


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name,dtype", [("(1)V1", 0), ("(1)X2", 0), ("(1)X2", 1), ("(1)X3", 0), ("(1)W2", 0)])
def test_reach_of_one_value(cuda, name, dtype, bad):
    rng = np.random.default_rng(6)
    W = "W" in name
    for d, N in _shapes():
        if W and N > 128:
            continue
        h = max(2, P.Scheme.named(name + "-").required_ghosts())
        ng = h + 2
        n = tuple(N if k == d else (5, 6, 7)[k] for k in range(3))
        base = torch.from_numpy(rng.uniform(0.5, 1.5, (3,) + tuple(v + 2 * ng for v in reversed(n)))).to("cuda")
        base[1] -= 1.0   # the velocity takes both signs
        ops_of = [("-", (-1,)), ("+", (-1,)), ("s", (-1,)), ("", (-1, 1))]
        for j in (-h - 1, -h, 0, 1, N // 2, N - 2, N - 1, N + h - 1, N + h):
            x = base.clone()
            at = [int(rng.integers(0, n[k])) for k in range(3)]
            idx = [at[k] + ng for k in range(3)]
            idx[d] = j + ng
            x[(0,) + tuple(reversed(idx))] = bad
            fin = _run(name, d, n, ng, x, dtype, ops_of)
            rest = [at[k] for k in (2, 1, 0) if k != d]
            mine = fin[:, 0, :, rest[0], rest[1]].copy()
            fin[:, 0, :, rest[0], rest[1]] = True
            where = (name, d, N, j)
            assert fin.all(), where                       # other lines, other fields
            if j < -h or j >= N + h:
                assert mine.all(), where                  # a ghost beyond the reach
                continue
            if W:
                continue                                  # the embedded second derivative couples the whole line
            left, right = mine[0], mine[1][::-1]          # the right-biased operator, mirrored
            for rows, k in ((left, j), (right, N - 1 - j)):
                first = 0 if k <= h + 1 else k - h
                assert rows[:first].all(), where
                if k >= 1:
                    assert not rows[k:].any(), where


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("name", ["(1)X2", "(1)W2"])
def test_velocity(cuda, name, bad):
    rng = np.random.default_rng(7)
    for d, N in ((0, 25), (0, 97), (1, 37), (2, 48), (2, 100)):
        ng = 6
        n = tuple(N if k == d else (5, 6, 7)[k] for k in range(3))
        x = torch.from_numpy(rng.uniform(0.5, 1.5, (3,) + tuple(v + 2 * ng for v in reversed(n)))).to("cuda")
        at = [int(rng.integers(0, n[k])) for k in range(3)]
        x[(1,) + tuple(at[k] + ng for k in (2, 1, 0))] = bad
        mine = _run(name, d, n, ng, x, 0, [("", (-1, 1))])[0, 0]
        rest = [at[k] for k in (2, 1, 0) if k != d]
        assert mine[at[d], rest[0], rest[1]] == np.isnan(bad), (name, d, N)
        mine[at[d], rest[0], rest[1]] = True
        assert mine.all(), (name, d, N)
