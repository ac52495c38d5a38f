"""Performance cases of the compressible Navier-Stokes residual and RK3 path.

A case is one call (or one short sequence of calls) that a program using this
package makes: advancing a solve by some RK3 steps in one of the three
algorithm classes, evaluating the residual, reading the diagnostics, or
advancing a batch of independent solves.  The states are Taylor-Green vortices
with a seeded smooth perturbation and some white noise, so that every stencil
tap carries a value of its own.

``listed`` names the cases, ``draw`` gives more of the same ranges,
``prepare`` makes a solve's state and workspace on the device, ``run`` makes
the call, ``work`` says what the call cannot do without and ``exact``
evaluates the same call with plain torch operations in double precision.
"""
from __future__ import annotations

import math

import torch

import paper_1709_09713_amd as ns

GAMMA = 1.4
PRANDTL = 0.71

# Grid sizes of the batched workload (32^3 to 128^3).
BATCH_SIZES = (32, 48, 64, 96, 128)


def _dt(n, mach):
    """Stable time step of a grid whose finest direction has n points."""
    return min(3.385e-3, 3.385e-3 * (64.0 / n) * 11.0 * mach / (1.0 + mach))


def _case(name, kind, n, *, algo="fused", precision="fp64", steps=1, diag=False,
          reynolds=1600.0, mach=0.1, members=0):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], algo=algo, precision=precision, steps=steps,
             diag=diag, reynolds=reynolds, mach=mach, members=members)
    if name:
        c["name"] = name
    return c


def listed():
    cube = lambda n: (n, n, n)  # noqa: E731
    return [
        # the smallest workload, one step per call with its diagnostics, as a
        # program that watches the solve calls it: launches and latency
        _case("step_16_diag", "step", cube(16), steps=1, diag=True),
        # a small served request in FP32 storage, one scheduling quantum
        _case("step_48_fp32", "step", cube(48), precision="fp32", steps=25, reynolds=900.0, mach=0.2),
        # an ordinary small solve
        _case("step_64", "step", cube(64), steps=10),
        # odd extents in every direction, with diagnostics
        _case("step_odd_diag", "step", (101, 77, 53), steps=4, diag=True, mach=0.2),
        # FP32 storage at the paper's grid
        _case("step_256_fp32", "step", cube(256), precision="fp32", steps=2),
        # the paper's workload: the 256^3 Taylor-Green vortex, per-step diagnostics
        _case("step_256_diag", "step", cube(256), steps=2, diag=True),
        # the largest solve of the benchmark, per-step diagnostics
        _case("step_512_diag", "step", cube(512), steps=1, diag=True),
        # one residual evaluation for a program with its own time integrator
        _case("residual_odd", "residual", (161, 97, 119), reynolds=800.0, mach=0.3),
        # the baseline class that stores every derivative, at the paper's grid
        _case("stored_256", "step", cube(256), algo="stored", steps=1),
        # the intermediate-storage class at the paper's grid
        _case("some_256", "step", cube(256), algo="some", steps=1),
        # kinetic energy, enstrophy and the conserved totals of a state
        _case("diagnostics_256", "diagnostics", cube(256)),
        # many independent solves of mixed sizes advanced together
        _case("batch_20_fp32", "batch", cube(128), precision="fp32", steps=8, members=20),
    ]


def _spread(rng, lo, hi):
    """An extent between lo and hi, spread over its logarithm, odd or even."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _grid(rng, lo, hi):
    """Three extents near one side: a cube, an even box or a ragged box."""
    side = _spread(rng, lo, hi)
    shape = rng.choice(("cube", "even", "ragged"))
    if shape == "cube":
        return (side, side, side)
    n = [max(lo, min(hi, int(round(side * rng.uniform(0.75, 1.3))))) for _ in range(3)]
    if shape == "even":
        n = [x + x % 2 for x in n]
        n = [x if x <= hi else x - 2 for x in n]
    return tuple(n)


def draw(rng):
    reynolds = round(rng.uniform(400.0, 3200.0), 3)
    mach = round(rng.uniform(0.05, 0.4), 4)
    kind = rng.choice(("fp64", "fp64", "fp64", "fp32", "fp32", "residual", "stored", "some",
                       "diagnostics", "batch"))
    kw = dict(reynolds=reynolds, mach=mach)
    if kind in ("fp64", "fp32"):
        n = _grid(rng, 16, 400)
        points = n[0] * n[1] * n[2]
        steps = max(1, min(rng.choice((1, 2, 10, 25)), (1 << 25) // points))
        return _case(None, "step", n, precision=kind, steps=steps, diag=rng.random() < 0.5, **kw)
    if kind == "residual":
        return _case(None, "residual", _grid(rng, 16, 320), algo=rng.choice(("fused", "fused", "stored", "some")),
                     **kw)
    if kind in ("stored", "some"):
        return _case(None, "step", _grid(rng, 16, 240), algo=kind, steps=1, diag=rng.random() < 0.3, **kw)
    if kind == "diagnostics":
        return _case(None, "diagnostics", _grid(rng, 16, 400), **kw)
    side = rng.choice((64, 96, 128))
    return _case(None, "batch", (side, side, side), precision=rng.choice(("fp32", "fp32", "fp64")),
                 steps=rng.choice((2, 4, 8)), members=rng.randint(4, 24), **kw)


# ---------------------------------------------------------------------------
# inputs

def _device():
    return torch.device("cuda")


def _state(n, mach, seed):
    """A Taylor-Green vortex with perturbed velocity, pressure and
    temperature: smooth low modes and white noise, drawn from the seed."""
    nx, ny, nz = n
    g = torch.Generator(device="cpu")
    g.manual_seed(int(seed))
    d = _device()
    gd = torch.Generator(device=d)
    gd.manual_seed(int(seed))
    ax = [torch.arange(k, dtype=torch.float64, device=d) * (2.0 * math.pi / k) for k in (nx, ny, nz)]
    X, Y, Z = ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]

    def rough(smooth, noise):
        f = (torch.rand((nz, ny, nx), dtype=torch.float64, device=d, generator=gd) - 0.5) * (2.0 * noise)
        for _ in range(2):
            k = torch.randint(-2, 3, (3,), generator=g).tolist()
            ph, a = (torch.rand(2, generator=g, dtype=torch.float64)).tolist()
            s = k[0] * X + ph * 2.0 * math.pi
            f += (smooth * a) * (torch.cos(s) * torch.cos(k[1] * Y) * torch.cos(k[2] * Z))
        return f

    gm2 = GAMMA * mach * mach
    Q = torch.empty((5, nz, ny, nx), dtype=torch.float64, device=d)
    p = 1.0 / gm2 + (torch.cos(2.0 * X) + torch.cos(2.0 * Y)) * (2.0 + torch.cos(2.0 * Z)) / 16.0
    p = p + rough(0.02, 0.002)
    Q[0] = gm2 * p / (1.0 + rough(0.01, 0.001))
    ke = torch.zeros_like(p)
    for a in range(3):
        u = rough(0.1, 0.005)
        if a == 0:
            u += torch.sin(X) * torch.cos(Y) * torch.cos(Z)
        elif a == 1:
            u -= torch.cos(X) * torch.sin(Y) * torch.cos(Z)
        Q[1 + a] = Q[0] * u
        ke += 0.5 * Q[1 + a] * u
    Q[4] = p / (GAMMA - 1.0) + ke
    return Q


def _members(case, seed):
    """(side, Reynolds, Mach, time step) of each solve of a batch."""
    g = torch.Generator(device="cpu")
    g.manual_seed(int(seed) + 977)
    sizes = [s for s in BATCH_SIZES if s <= case["nx"]]
    out = []
    for k in range(case["members"]):
        n = sizes[k % len(sizes)]
        r = torch.rand(2, generator=g, dtype=torch.float64).tolist()
        re, mach = 400.0 + 2800.0 * r[0], 0.05 + 0.35 * r[1]
        out.append((n, re, mach, _dt(n, mach)))
    return out


def prepare(case, seed):
    n = (case["nx"], case["ny"], case["nz"])
    st = dict(case=case)
    if case["kind"] == "batch":
        b = ns.Batch(case["members"], case["precision"])
        st["batch"], st["states"] = b, []
        for k, (side, re, mach, dt) in enumerate(_members(case, seed)):
            Q = _state((side,) * 3, mach, seed * 1000 + k)
            b.add(side, reynolds=re, mach=mach, dt=dt, steps=2000000000, state=Q, init_tgv=False)
            st["states"].append(Q)
        return st
    s = ns.Solver(n, reynolds=case["reynolds"], mach=case["mach"], algo=case["algo"],
                  precision=case["precision"])
    s.set_state(_state(n, case["mach"], seed))
    st["solver"] = s
    st["dt"] = _dt(max(n), case["mach"])
    if case["diag"]:
        st["diag"] = torch.zeros((case["steps"], 8), dtype=torch.float64, device=_device())
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        state["batch"].step(case["steps"])
        return state["states"]
    s = state["solver"]
    if case["kind"] == "residual":
        return s.residual()
    if case["kind"] == "diagnostics":
        d = s.diagnostics()
        return [d[k] for k in ns.DIAG_NAMES]
    s.step(state["dt"], case["steps"], diag=state.get("diag"))
    return [s.state, state["diag"]] if case["diag"] else [s.state]


def work(case):
    """A residual reads a state and writes one, an RK3 step reads and writes
    the state once, diagnostics read it once.  Operations per point of one
    residual: 13 for the primitive values, 14 for the fluxes, 39 first
    derivatives of 5, 12 second derivatives of 7, 6 mixed ones of 5, and about
    140 to combine them and to update the stage; the diagnostics take 9 first
    derivatives and about 20 more."""
    if case["kind"] == "batch":
        sizes = [s for s in BATCH_SIZES if s <= case["nx"]]
        points = sum(sizes[k % len(sizes)] ** 3 for k in range(case["members"]))
    else:
        points = case["nx"] * case["ny"] * case["nz"]
    per_residual = 480.0
    if case["kind"] == "diagnostics":
        return {"bytes": 40.0 * points, "flops": 65.0 * points}
    if case["kind"] == "residual":
        return {"bytes": 80.0 * points, "flops": per_residual * points}
    return {"bytes": 80.0 * points * case["steps"],
            "flops": (3 * per_residual + (65.0 if case["diag"] else 0.0)) * points * case["steps"]}


# ---------------------------------------------------------------------------
# the same calls in plain torch, double precision

_DIM = {0: 2, 1: 1, 2: 0}


def _first(f, d, h):
    ax = _DIM[d]
    out = torch.roll(f, -1, ax)
    out -= torch.roll(f, 1, ax)
    out *= 8.0
    far = torch.roll(f, -2, ax)
    far -= torch.roll(f, 2, ax)
    out -= far
    out /= 12.0 * h[d]
    return out


def _second(f, d, h):
    ax = _DIM[d]
    out = torch.roll(f, -1, ax)
    out -= f
    out += torch.roll(f, 1, ax)
    out -= f
    out *= 16.0
    far = torch.roll(f, -2, ax)
    far -= f
    far += torch.roll(f, 2, ax)
    far -= f
    out -= far
    out /= 12.0 * h[d] ** 2
    return out


def _spacing(Q):
    return [2.0 * math.pi / Q.shape[3 - d] for d in range(3)]


def _residual(Q, reynolds, mach):
    h = _spacing(Q)
    rho, E = Q[0], Q[4]
    u = [Q[1 + a] / rho for a in range(3)]
    p = (GAMMA - 1.0) * (E - 0.5 * (Q[1] * u[0] + Q[2] * u[1] + Q[3] * u[2]))
    T = GAMMA * mach ** 2 * p / rho
    inv_re = 0.0 if math.isinf(reynolds) else 1.0 / reynolds
    kappa = inv_re / ((GAMMA - 1.0) * mach ** 2 * PRANDTL)
    # derivatives of the pressure and the energy do not see their means;
    # without them less is lost to cancellation
    p0 = 1.0 / (GAMMA * mach ** 2)
    E0 = p0 / (GAMMA - 1.0)
    dp, dE = p - p0, E - E0
    G = [[_first(u[i], j, h) for j in range(3)] for i in range(3)]
    div = G[0][0] + G[1][1] + G[2][2]
    R = torch.empty_like(Q)
    for f in range(5):
        q = Q[f]
        acc = torch.zeros_like(rho)
        if f < 4:
            for j in range(3):
                if f == 0:
                    acc += _first(Q[1 + j], j, h)
                else:
                    acc += _first(q * u[j], j, h)
                acc += u[j] * _first(q, j, h)
            acc += q * div
            R[f] = -0.5 * acc
        else:
            for j in range(3):
                acc += _first(dE * u[j], j, h)
                acc += u[j] * _first(dE, j, h)
            acc += dE * div + 2.0 * E0 * div
            R[4] = -0.5 * acc
            for j in range(3):
                R[4] -= _first(dp * u[j], j, h)
            R[4] -= p0 * div
    work = torch.zeros_like(rho)
    for i in range(3):
        V = _second(u[i], i, h)
        for k in range(3):
            if k != i:
                V += _first(G[k][k], i, h)
        V /= 3.0
        for j in range(3):
            V += _second(u[i], j, h)
        R[1 + i] -= _first(dp, i, h)
        R[1 + i] += inv_re * V
        work += u[i] * V
    for i in range(3):
        for j in range(3):
            work += G[i][j] * (G[i][j] + G[j][i])
    work -= (2.0 / 3.0) * div * div
    R[4] += inv_re * work
    for j in range(3):
        R[4] += kappa * _second(T, j, h)
    return R


def _diagnostics(Q, reynolds):
    h = _spacing(Q)
    vol, rho = h[0] * h[1] * h[2], Q[0]
    u = [Q[1 + a] / rho for a in range(3)]
    ke = 0.5 * (Q[1] * u[0] + Q[2] * u[1] + Q[3] * u[2])
    w2 = (_first(u[2], 1, h) - _first(u[1], 2, h)) ** 2
    w2 += (_first(u[0], 2, h) - _first(u[2], 0, h)) ** 2
    w2 += (_first(u[1], 0, h) - _first(u[0], 1, h)) ** 2
    ens = (0.5 * rho * w2).mean()
    return torch.stack([vol * Q[0].sum(), vol * Q[1].sum(), vol * Q[2].sum(), vol * Q[3].sum(),
                        vol * Q[4].sum(), ke.mean(), ens, ens * (2.0 / reynolds)])


def _rk3(Q, reynolds, mach, dt, steps, diag):
    rec = []
    for _ in range(steps):
        if diag:
            rec.append(_diagnostics(Q, reynolds))
        acc, cur = Q.clone(), Q
        for a, b in ((2.0 / 3.0, 1.0 / 4.0), (5.0 / 12.0, 3.0 / 20.0), (3.0 / 5.0, 3.0 / 5.0)):
            R = _residual(cur, reynolds, mach)
            cur = acc + (a * dt) * R
            acc += (b * dt) * R
        Q = cur
    return [Q, torch.stack(rec)] if diag else [Q]


def exact(case, seed):
    if case["kind"] == "batch":
        return [_rk3(_state((side,) * 3, mach, seed * 1000 + k), re, mach, dt, case["steps"], False)[0]
                for k, (side, re, mach, dt) in enumerate(_members(case, seed))]
    n = (case["nx"], case["ny"], case["nz"])
    Q = _state(n, case["mach"], seed)
    if case["kind"] == "residual":
        return _residual(Q, case["reynolds"], case["mach"])
    if case["kind"] == "diagnostics":
        return _diagnostics(Q, case["reynolds"]).tolist()
    return _rk3(Q, case["reynolds"], case["mach"], _dt(max(n), case["mach"]), case["steps"], case["diag"])
