"""Cases that stand for what a program does with this library: derivative steps on batches of mesh
blocks, shift advection with the upwind pairs, the dissipation and mixed derivatives of a Z4c
right-hand side, iterated block closures on a lattice, periodic boxes, and Runge-Kutta steps of the
first-order wave system, each through the public Python calls.

A case is a dict of plain values:

kind     "derivs"   first (and second) derivatives along x, y, z of every field
         "upwind"   c d_i f of every field along x, y, z, c the fields 0, 1, 2 (an upwind pair)
         "z4c"      Kreiss-Oliger dissipation along x, y, z and the mixed derivatives xy, xz, yz
         "iterate"  ghost exchange on a periodic lattice of equal blocks, then first derivatives with
                    the hybrid closure iteration
         "wave"     one RK4 step of the wave system on a periodic box or a lattice of blocks
scheme   "tri" (1)/(2)Q1_3[1], "penta" (1)/(2)QP_O8[1], "X2" or "W2"
second   derivs: the second derivatives as well
dtype    "f64", "f32" or "mixed" (the dense BF16 path with FP64 refinement)
blocks   extents of the blocks, "16x24x32 48x16x16", or "64 of 16,24,32,48" / "9 of 17-61": so many
         blocks whose extents are drawn along each axis (always the same ones for one case)
lattice  iterate, wave: blocks per direction (0: one periodic box)
fields   fields per block
ghosts   ghost layers (0 on periodic boxes)
periodic every line periodic instead of closed by the block closures
tuned    the plan is autotuned and its apply captured in a graph, as a long run does; otherwise the
         plan is used as created
"""
from __future__ import annotations

import math
import random
from fractions import Fraction

import numpy as np
import torch

import paper_2302_14858_amd as cfd
from paper_2302_14858_amd.wave import WaveRK4

ITERATIONS = 2          # hybrid closure iteration: iterates after the block closure
KO_HALF, KO_SIGMA = 4, 0.04
PAIRS = ((0, 1), (0, 2), (1, 2))


def listed():
    def case(name, kind, scheme, blocks, fields, dtype="f64", ghosts=4, second=False, lattice=0, periodic=False,
             tuned=False):
        return dict(name=name, kind=kind, scheme=scheme, second=second, dtype=dtype, blocks=blocks, lattice=lattice,
                    fields=fields, ghosts=ghosts, periodic=periodic, tuned=tuned)

    return [
        # one small block of one field, differentiated on its own between other work: launches and latency
        case("tiny16", "derivs", "tri", "16x16x16", 1),
        # a few uneven blocks with odd extents, several fields, first and second derivatives
        case("odd_blocks", "derivs", "penta", "33x21x45 17x48x29 40x13x61 51x37x23", 5, ghosts=5, second=True),
        # one large block of one field (a unigrid run)
        case("block128", "derivs", "tri", "128x128x128", 1, second=True),
        # the large batched step of an adaptive-mesh run: 64 uneven blocks, 22 fields, tuned once, then replayed
        case("batch64", "derivs", "penta", "64 of 16,24,32,48", 22, ghosts=5, second=True, tuned=True),
        # the same step in single precision, on a plan used as created
        case("batch64_f32", "derivs", "penta", "64 of 16,24,32,48", 22, dtype="f32", ghosts=5, second=True),
        # shift advection of every field on the same blocks
        case("upwind64", "upwind", "X2", "64 of 16,24,32,48", 22, ghosts=5),
        # shift advection with the pair that embeds a compact second derivative, single precision
        case("upwind64_w2_f32", "upwind", "W2", "64 of 16,24,32,48", 22, dtype="f32", ghosts=5),
        # shift advection on one large block, lines longer than 64 nodes
        case("upwind_long", "upwind", "X2", "128x96x80", 6),
        # dissipation and mixed derivatives of a Z4c right-hand side
        case("z4c64", "z4c", "penta", "64 of 16,24,32,48", 22, ghosts=5),
        # a lattice of equal blocks: refresh the ghosts, then derivatives with iterated closures
        case("lattice_iter", "iterate", "tri", "32x32x32", 5, lattice=4),
        # a periodic box on the matrix cores: dense mixed-precision derivatives
        case("periodic256_mixed", "derivs", "tri", "256x256x256", 4, dtype="mixed", ghosts=0, periodic=True),
        # one time step of a wave evolution on a periodic box
        case("wave192", "wave", "tri", "192x192x192", 5, ghosts=0, periodic=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    c = dict(kind=rng.choice(("derivs", "derivs", "derivs", "upwind", "upwind", "z4c", "iterate", "wave")), scheme="tri",
             second=False, dtype=rng.choice(("f64", "f64", "f32")), blocks="", lattice=0, fields=log_int(1, 24), ghosts=4,
             periodic=False, tuned=False)
    budget = 1.6e7          # interior nodes x fields of a drawn case, at most
    kind = c["kind"]
    if kind == "derivs" and rng.random() < 0.4:       # a periodic box
        c.update(periodic=True, ghosts=0, second=rng.random() < 0.4)
        if rng.random() < 0.4:
            c.update(dtype="mixed", second=False)
            n = [32 * rng.randint(1, 8) for _ in range(3)]
        else:
            n = [rng.choice((16, 24, 32, 48, 64, 96, 128)) for _ in range(3)]
        c["blocks"] = "x".join(map(str, n))
        nodes = n[0] * n[1] * n[2]
    elif kind in ("derivs", "upwind", "z4c"):
        if kind == "derivs":
            c.update(scheme=rng.choice(("tri", "penta")), second=rng.random() < 0.6, tuned=rng.random() < 0.3)
            longest = 96 if c["scheme"] == "penta" else 128
        elif kind == "upwind":
            c.update(scheme=rng.choice(("X2", "X2", "W2")), fields=max(3, c["fields"]))
            longest = 144 if c["scheme"] == "X2" else 112
        else:
            c.update(scheme="penta")
            longest = 64
        c["ghosts"] = 5
        if rng.random() < 0.4:                        # one block
            n = [log_int(12, longest) for _ in range(3)]
            if c["second"]:                           # closed lines of 49 or 65 to 73 nodes: no kernel for both degrees
                n = [48 if v == 49 else 64 if 64 < v < 74 else v for v in n]
            c["blocks"] = "x".join(map(str, n))
            nodes = n[0] * n[1] * n[2]
        else:
            lo = log_int(12, 24)
            hi = rng.randint(lo + 4, 48 if c["second"] else 56)
            c["blocks"] = "%d of %d-%d" % (log_int(2, 64), lo, hi)
            nodes = sum(math.prod(n) for n in extents(c))
    elif kind == "iterate":
        c.update(lattice=rng.randint(2, 4), ghosts=4, fields=log_int(1, 8))
        n = [rng.randint(12, 40) for _ in range(3)]
        c["blocks"] = "x".join(map(str, n))
        nodes = n[0] * n[1] * n[2] * c["lattice"] ** 3
    else:
        c.update(fields=5)
        if rng.random() < 0.5:
            c.update(lattice=rng.randint(2, 4))
            n = [rng.randint(13, 40)] * 3
            nodes = n[0] ** 3 * c["lattice"] ** 3
        else:
            c.update(periodic=True, ghosts=0)
            n = [rng.choice((32, 48, 64, 96, 128))] * 3
            nodes = n[0] ** 3
        c["blocks"] = "x".join(map(str, n))
    if kind != "wave":
        least = 3 if kind == "upwind" else 1
        c["fields"] = max(least, min(c["fields"], int(budget // nodes)))
    return c


# ---------------------------------------------------------------------------
# Layout and inputs
# ---------------------------------------------------------------------------

def extents(case):
    """Interior extents (nx, ny, nz) of every block."""
    text = case["blocks"]
    if " of " in text:
        count, sizes = text.split(" of ")
        rng = random.Random("extents " + text)
        if "-" in sizes:
            lo, hi = map(int, sizes.split("-"))
            return [tuple(rng.randint(lo, hi) for _ in range(3)) for _ in range(int(count))]
        sizes = [int(v) for v in sizes.split(",")]
        return [tuple(rng.choice(sizes) for _ in range(3)) for _ in range(int(count))]
    each = [tuple(map(int, t.split("x"))) for t in text.split()]
    return each * max(1, case["lattice"]) ** 3


def spacing(case):
    """h per direction: the box [0, 2 pi) on periodic boxes and lattices, 1/64 on other blocks."""
    if case["periodic"] or case["lattice"]:
        n = extents(case)[0]
        return tuple(2 * math.pi / (n[d] * max(1, case["lattice"])) for d in range(3))
    return (1.0 / 64,) * 3


def dtype_of(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def modes(rng, case):
    """(amplitudes, wave vectors, phases) of one field."""
    if case["periodic"] or case["lattice"]:
        n = extents(case)[0]
        J = 16
        top = [max(1, int(0.4 * n[d] * max(1, case["lattice"]) / (1 if case["kind"] == "derivs" else 4))) for d in range(3)]
        k = np.stack([rng.integers(0, t + 1, J) for t in top], axis=1).astype(np.float64)
    else:
        J = 8
        k = 2 * math.pi * rng.integers(1, 7, (J, 3))
    return rng.uniform(-1, 1, J), k, rng.uniform(0, 2 * math.pi, J)


def sample(A, k, phi, axes):
    """sum_j A_j sin(k_j . x + phi_j) on the tensor grid axes = (x, y, z), as [z][y][x]."""
    A, k, phi = (torch.as_tensor(v, dtype=torch.float64, device="cuda") for v in (A, k, phi))
    xy = (k[:, 1:2] * axes[1][None, :])[:, :, None] + (k[:, 0:1] * axes[0][None, :])[:, None, :]
    zz = k[:, 2:3] * axes[2][None, :] + phi[:, None]
    J = A.numel()
    f = (A[:, None] * torch.sin(zz)).T @ torch.cos(xy).reshape(J, -1) + (A[:, None] * torch.cos(zz)).T @ torch.sin(xy).reshape(J, -1)
    return f.reshape(axes[2].numel(), axes[1].numel(), axes[0].numel())


def inputs(case, seed):
    """The input in 64 bits, per block a tensor [field][z][y][x] with ghosts, and the block descriptions."""
    rng = np.random.default_rng([seed, 2302])
    g, h = case["ghosts"], spacing(case)
    per_field = [modes(rng, case) for _ in range(case["fields"])]
    wave = case["kind"] == "wave"
    if wave:                                          # a solution's state: phi, Pi and the gradient of phi
        A, k, phi = per_field[0]
        w = np.sqrt((k * k).sum(axis=1))
        per_field = [(A, k, phi), (-A * w, k, phi + math.pi / 2)] + [(A * k[:, d], k, phi + math.pi / 2) for d in range(3)]
    out, blocks = [], []
    L = case["lattice"]
    for b, n in enumerate(extents(case)):
        if L:
            at = (b % L, (b // L) % L, b // (L * L))
            org = [at[d] * n[d] * h[d] for d in range(3)]
        elif case["periodic"]:
            org = [0.0] * 3
        else:
            org = rng.uniform(0, 1, 3)
        axes = [org[d] + h[d] * torch.arange(-g, n[d] + g, dtype=torch.float64, device="cuda") for d in range(3)]
        f = torch.stack([sample(*m, axes) for m in per_field])
        if L:                                         # ghosts as an update of the interior leaves them: not yet refreshed
            keep = torch.zeros_like(f)
            i = slice(g, -g)
            keep[:, i, i, i] = f[:, i, i, i]
            f = keep
        out.append(f)
        blocks.append(dict(n=n, ng=g, h=h, boundary=((cfd.CFD_BOUNDARY_PERIODIC if case["periodic"] else cfd.CFD_BOUNDARY_CLOSURE),) * 3))
    return out, blocks


def operators(case):
    """The operators of the plan, in output order."""
    kind, s = case["kind"], case["scheme"]
    if kind == "upwind":
        scheme = cfd.Scheme.named("(1)" + s)
        return [(scheme, d, -1, d) for d in range(3)]
    name = "QP_O8[1]" if s == "penta" else "Q1_3[1]"
    d1 = cfd.Scheme.named("(1)" + name)
    if kind == "z4c":
        ko = cfd.Scheme.dissipation(KO_HALF, KO_SIGMA)
        return [(ko, d) for d in range(3)] + [(d1, i, -1, -1, j) for i, j in PAIRS]
    ops = [(d1, d) for d in range(3)]
    if case["second"]:
        d2 = cfd.Scheme.named("(2)" + name)
        ops += [(d2, d) for d in range(3)]
    return ops


def time_step(case):
    return 0.25 * spacing(case)[0]


# ---------------------------------------------------------------------------
# Preparation and one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    data, blocks = inputs(case, seed)
    flat = torch.cat([f.reshape(-1) for f in data]).to(dtype_of(case))
    del data
    code = {"f64": cfd.CFD_F64, "f32": cfd.CFD_F32, "mixed": cfd.CFD_MIXED_BF16}[case["dtype"]]
    L = (case["lattice"],) * 3
    if case["kind"] == "wave":
        rk = WaveRK4(blocks, cfd.Scheme.named("(1)Q1_3[1]"), time_step(case), dtype=code, lattice=L if case["lattice"] else None)
        rk.load(flat)
        rk.capture()
        rk.load(flat)
        return {"kind": "wave", "rk": rk}
    plan = cfd.Plan(blocks, case["fields"], operators(case), dtype=code)
    out = torch.empty(plan.sizes()[1], dtype=flat.dtype, device="cuda")
    state = {"kind": case["kind"], "plan": plan, "x": flat, "out": out, "tuned": case["tuned"]}
    if case["kind"] == "iterate":
        state["lattice"] = L
        plan.set_iteration(ITERATIONS, *L)
    if case["tuned"]:
        plan.autotune(flat, out)
        plan.capture_graph(flat, out)
    return state


def run(state):
    if state["kind"] == "wave":
        state["rk"].run(1)
        return state["rk"].u
    plan = state["plan"]
    if state["kind"] == "iterate":
        plan.halo_exchange(state["x"], *state["lattice"])
        plan.apply(state["x"], state["out"])
        return {"x": state["x"], "out": state["out"]}
    if state["tuned"]:
        plan.launch_graph()
    else:
        plan.apply(state["x"], state["out"])
    return state["out"]


# ---------------------------------------------------------------------------
# What one pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: the interior and the ghosts that the operators reach, read once, and every output written
    once (a wave step: the state read and written by each of its four stages, which follow one another).
    Flops: stencils, eliminations and combinations of every value."""
    es = 8 if case["dtype"] == "f64" else 4
    g, nf = case["ghosts"], case["fields"]
    nodes = ghost = edge = 0
    for nx, ny, nz in extents(case):
        nodes += nx * ny * nz
        ghost += 2 * g * (nx * ny + nx * nz + ny * nz)
        edge += 4 * g * g * (nx + ny + nz)
    if case["kind"] == "wave":
        return {"bytes": 4 * 2 * 5 * nodes * es, "flops": 4 * nodes * (6 * 15 + 5 * 4 + 2)}
    each = {"tri": 15, "penta": 20, "X2": 2 * 20 + 6, "W2": 2 * 18 + 6 + 14}[case["scheme"]]
    if case["kind"] == "z4c":
        return {"bytes": nf * es * (nodes + ghost + edge + 6 * nodes), "flops": nf * nodes * (3 * 14 + 3 * (4 * each + 2))}
    if case["kind"] == "iterate":                     # the ghosts: read from the neighbours and written, and read by the operators
        return {"bytes": nf * es * (nodes + 2 * ghost + 3 * nodes), "flops": nf * nodes * 3 * each}
    ops = 6 if case["second"] else 3
    return {"bytes": nf * es * (nodes + ghost + ops * nodes), "flops": nf * nodes * ops * each}


# ---------------------------------------------------------------------------
# The same outputs in plain 64-bit torch, from the schemes' coefficients
# ---------------------------------------------------------------------------

F = Fraction
# centred schemes: degree, implicit coefficients alpha_0.., stencil a_0.. and closure stencil c_0.. (symmetric for
# the second degree, antisymmetric for the first)
CENTRED = {
    "(1)Q1_3[1]": (1, (1.0, 0.3798792289490848), (0.0, 0.7816566024124237, 0.052602255439511914, -0.002327294780787575),
                   (0.0, 0.8003696892928448, -0.20036968929284477, 0.038253676363600136, -0.0035978349494889122)),
    "(2)Q1_3[1]": (2, (1.0, 0.24246602513914975),
                   (-2.1834088330241115, 0.954451443436913, 0.1409592301669797, -0.0037062570918369297),
                   (-2.8492210880518036, 1.601599092663665, -0.20079954633183247, 0.025625267205920392, -0.00181426951185116)),
    "(1)QP_O8[1]": (1, (1.0, 0.504298413487875, 0.05171936539514997),
                    (0.0, 0.7058259254654063, 0.17240249810185493, 0.0017956190713029143),
                    (0.0, 0.8333672533232381, -0.23813400379798638, 0.05954561523160544, -0.00992709587109297,
                     0.0007944584124580498)),
    "(2)QP_O8[1]": (2, (1.0, 0.37745582706749753, 0.02496879172226591),
                    (-1.7530389164115057, 0.5758180139313329, 0.2954563549643172, 0.005245089310102781),
                    (-2.9274983624345836, 1.6668967835103012, -0.23822673343445788, 0.039731850434747105,
                     -0.004971275405252443, 0.00031855611195381574)),
    "(2)P1_2": (2, (1.0, F(2, 11)), (F(-51, 22), F(12, 11), F(3, 44)),
                (F(-763, 270), F(2137, 1350), F(-517, 2700), F(31, 1350), F(-1, 675))),
}
# left-biased schemes: alpha, stencil a_-m..a_m, weight of the embedded h^2 f'', closure stencil c_-4..c_5
BIASED = {
    "X2": (F(407, 600),
           (F(-43, 56000), F(1523, 126000), F(-857, 6000), F(-39697, 36000), F(245, 288), F(2723, 6000), F(-1459, 18000),
            F(2899, 252000), F(-43, 56000)), F(0),
           (F(194871521, 170360232000), F(-242883881, 17036023200), F(3813668231, 42590058000), F(-8537761009, 18252882000),
            F(-3401756057, 4056196000), F(40137795113, 36505764000), F(507715327, 3650576400), F(-338742841, 42590058000),
            F(-458269213, 511080696000), F(16295059, 63885087000))),
    "W2": (F(829, 1200),
           (F(29, 12000), F(-877, 12000), F(-24271, 14400), F(151, 80), F(-307, 2400), F(-167, 36000), F(29, 24000)),
           F(71, 200),
           (F(638561861, 555773535000), F(-773306021, 55577353500), F(24069573467, 277886767500),
            F(-1015672928093, 2223094140000), F(-480625731203, 555773535000), F(4974276451727, 4446188280000),
            F(1867414306, 13894338375), F(-7783562141, 2223094140000), F(-159391966, 69471691875),
            F(1913697589, 4446188280000))),
}


def centred_rows(name, N, g, periodic):
    """(A, B) of A f~ = B f at unit spacing on a line of N nodes with g ghosts either side."""
    d, lhs, rhs, clo = CENTRED[name]
    odd = -1.0 if d == 1 else 1.0
    A, B = np.zeros((N, N)), np.zeros((N, N + 2 * g))
    nl = len(lhs) - 1
    for k in range(N):
        closed = not periodic and min(k, N - 1 - k) < nl
        A[k, k] += 1.0
        if not closed:
            for j in range(1, nl + 1):
                A[k, (k + j) % N] += float(lhs[j])
                A[k, (k - j) % N] += float(lhs[j])
        for m, a in enumerate(clo if closed else rhs):
            at = [(k + m, 1.0), (k - m, odd)] if m else [(k, 1.0)]
            for col, sign in at:
                B[k, (col % N if periodic else col) + g] += sign * float(a)
    return A, B


def centred(name, N, g, periodic):
    return np.linalg.solve(*centred_rows(name, N, g, periodic))


def biased(name, bias, N, g, periodic):
    """The line operator of one bias at unit spacing; the right-biased one is the left-biased one mirrored."""
    alpha, a, a2, c = BIASED[name]
    A, B = np.eye(N), np.zeros((N, N + 2 * g))
    half = (len(a) - 1) // 2
    for k in range(N):
        if k == 0 and not periodic:
            A[0, 1] += float(alpha)
            for m, v in enumerate(c):
                B[0, m - 4 + g] += float(v)
            continue
        A[k, (k - 1) % N] += float(alpha)
        for m, v in enumerate(a):
            col = k + m - half
            B[k, (col % N if periodic else col) + g] += float(v)
    if a2:
        first = 0 if periodic else 1
        B[first:] += float(a2) * centred("(2)P1_2", N, g, periodic)[first:]
    D = np.linalg.solve(A, B)
    return D if bias < 0 else -D[::-1, ::-1].copy()


def along(D, f, d):
    """D along direction d (0 x, 1 y, 2 z) of f [..., z, y, x]."""
    D = torch.as_tensor(D, dtype=torch.float64, device="cuda")
    f = f.transpose(-1 - d, -1)
    return (f.reshape(-1, f.shape[-1]) @ D.T).reshape(f.shape[:-1] + (D.shape[0],)).transpose(-1 - d, -1)


def inner(f, g, dirs):
    """f without its ghosts along the directions in dirs."""
    if g:
        for d in dirs:
            f = f.narrow(f.dim() - 1 - d, g, f.shape[-1 - d] - 2 * g)
    return f


def refreshed(case, data):
    """The lattice's blocks with their face ghosts taken from the neighbours."""
    L, g = case["lattice"], case["ghosts"]
    out = [f.clone() for f in data]
    for b, f in enumerate(out):
        at = [b % L, (b // L) % L, b // (L * L)]
        for d in range(3):
            others = [e for e in range(3) if e != d]
            n = f.shape[-1 - d] - 2 * g
            for step, dst, src in ((-1, 0, n), (1, n + g, g)):
                to = list(at)
                to[d] = (to[d] + step) % L
                src_f = data[(to[2] * L + to[1]) * L + to[0]]
                inner(f, g, others).narrow(f.dim() - 1 - d, dst, g).copy_(
                    inner(src_f, g, others).narrow(f.dim() - 1 - d, src, g))
    return out


def iterated(case, lines, h, N):
    """First derivatives of lines [block along the lattice][line][N + 2 g] after the closure iterations."""
    g, c = case["ghosts"], 2
    x = lines @ torch.as_tensor(centred("(1)Q1_3[1]", N, g, False), device="cuda").T / h
    d, lhs, rhs, _ = CENTRED["(1)Q1_3[1]"]
    E = N + 2 * (c - 1)
    A, B = np.eye(E), np.zeros((E, N + 2 * g))
    for k in range(E):
        for j in (k - 1, k + 1):
            if 0 <= j < E:
                A[k, j] += lhs[1]
        for m in range(1, len(rhs)):
            B[k, k - (c - 1) + g + m] += rhs[m]
            B[k, k - (c - 1) + g - m] -= rhs[m]
    inv = torch.as_tensor(np.linalg.inv(A), device="cuda")
    r0 = lines @ torch.as_tensor(B, device="cuda").T / h
    for _ in range(ITERATIONS):
        r = r0.clone()
        r[..., 0] -= lhs[1] * x.roll(1, 0)[..., N - c]
        r[..., -1] -= lhs[1] * x.roll(-1, 0)[..., c - 1]
        x = (r @ inv.T)[..., c - 1:c - 1 + N]
    return x


def exact(case, seed):
    data, _ = inputs(case, seed)
    data = [f.to(dtype_of(case)).double() for f in data]       # what the pass reads
    g, per, h, kind = case["ghosts"], case["periodic"], spacing(case), case["kind"]
    made = {}

    def matrix(fn, *args):
        if (fn, args) not in made:
            made[(fn, args)] = torch.as_tensor(fn(*args), dtype=torch.float64, device="cuda")
        return made[(fn, args)]

    def line(name, f, d, ghosts):
        """The centred operator along d of f, whose lines along d hold `ghosts` ghosts either side."""
        power = CENTRED[name][0]
        return along(matrix(centred, name, f.shape[-1 - d] - 2 * ghosts, ghosts, per), f, d) / h[d] ** power

    if kind == "wave":
        return exact_wave(case, data, line)
    out = []
    if kind == "iterate":
        data = refreshed(case, data)
        L, (nx, ny, nz) = case["lattice"], extents(case)[0]
        grid = torch.stack(data).reshape((L, L, L) + data[0].shape)       # [bz][by][bx][field][z][y][x]
        per_dir = []
        for d in range(3):
            f = inner(grid, g, [e for e in range(3) if e != d]).movedim((2 - d, 6 - d), (0, -1))
            got = iterated(case, f.reshape(L, -1, f.shape[-1]), h[d], f.shape[-1] - 2 * g)
            per_dir.append(got.reshape(f.shape[:-1] + (-1,)).movedim((0, -1), (2 - d, 6 - d)))
        y = torch.stack(per_dir, dim=3)                                    # [bz][by][bx][op][field][z][y][x]
        return {"x": torch.stack(data).reshape(-1), "out": y.reshape(-1)}
    for f in data:
        def others(d):
            return inner(f, g, [e for e in range(3) if e != d])
        if kind == "upwind":
            for d in range(3):
                lines = others(d)
                N = lines.shape[-1 - d] - 2 * g
                c = inner(f, g, range(3))[d]
                left, right = (along(matrix(biased, case["scheme"], s, N, g, per), lines, d) / h[d] for s in (-1, 1))
                out.append(torch.clamp(c, max=0.0) * right + torch.clamp(c, min=0.0) * left)
        elif kind == "z4c":
            for d in range(3):
                lines = others(d)
                N = lines.shape[-1 - d] - 2 * g
                q = 0.0
                for m in range(-KO_HALF, KO_HALF + 1):
                    w = (-1) ** (KO_HALF + m) * math.comb(2 * KO_HALF, KO_HALF + m)
                    q = q + w * lines.narrow(lines.dim() - 1 - d, g + m, N)
                out.append(q * (-(-1) ** KO_HALF * KO_SIGMA / 4 ** KO_HALF / h[d]))
            for i, j in PAIRS:
                third = inner(f, g, [3 - i - j])
                one = line("(1)QP_O8[1]", line("(1)QP_O8[1]", third, j, g), i, g)
                two = line("(1)QP_O8[1]", line("(1)QP_O8[1]", third, i, g), j, g)
                out.append(0.5 * (one + two))
        else:
            name = "QP_O8[1]" if case["scheme"] == "penta" else "Q1_3[1]"
            for degree in (1, 2) if case["second"] else (1,):
                out += [line("(%d)%s" % (degree, name), others(d), d, g) for d in range(3)]
    return torch.cat([v.reshape(-1) for v in out])


def exact_wave(case, data, line):
    g, dt = case["ghosts"], time_step(case)

    def whole(parts):
        """Interiors with ghosts around them, refreshed on a lattice."""
        if not g:
            return parts
        out = []
        for f, old in zip(parts, data):
            new = torch.zeros_like(old)
            new[:, g:-g, g:-g, g:-g] = f
            out.append(new)
        return refreshed(case, out)

    def slope(parts):
        k = []
        for f in whole(parts):
            def D(field, d):
                return line("(1)Q1_3[1]", inner(f[field], g, [e for e in range(3) if e != d]), d, g)
            k.append(torch.stack([inner(f[1], g, range(3)), D(2, 0) + D(3, 1) + D(4, 2), D(1, 0), D(1, 1), D(1, 2)]))
        return k

    u = [inner(f, g, range(3)) for f in data]
    k1 = slope(u)
    k2 = slope([a + dt / 2 * b for a, b in zip(u, k1)])
    k3 = slope([a + dt / 2 * b for a, b in zip(u, k2)])
    k4 = slope([a + dt * b for a, b in zip(u, k3)])
    new = [a + dt / 6 * (p + 2 * q + 2 * r + s) for a, p, q, r, s in zip(u, k1, k2, k3, k4)]
    return torch.cat([f.reshape(-1) for f in whole(new)])
