"""Workloads of the time step: what a program has the library do, through the
package's public entry points, from one small channel to 134 million
populations, with a plain 64-bit evaluation of each.

A pass of a channel workload is one stretch of a run: a number of RK-3 steps,
then the state and its moments read out.  The state goes on from pass to pass,
as it does in a program's own loop.
"""
from __future__ import annotations

import math
from decimal import Decimal, getcontext, localcontext
from functools import lru_cache

import numpy as np
import torch

DEVICE = "cuda"


def listed():
    return [
        # the small validation channel (barometric closed form): one channel
        # of two windows, replayed graphs; every launch counts
        dict(name="small_channel", kind="flow", quad="half", Q=4, channels=1, Nx_min=64, Nx_max=64, adv="upwind3",
             chi=True, stretch=0.0, Kn_min=0.1, Kn_max=0.1, g=-0.1, T_right=1.0, dt=5e-4, form="fp64",
             graph=64, steps=64, monitor=False, draw=0),
        # the steady-state study on the stretched grid, half-range model, plain
        # launches (the default)
        dict(name="channel_hhlb8", kind="flow", quad="half", Q=8, channels=1, Nx_min=512, Nx_max=512, adv="weno5",
             chi=True, stretch=0.9, Kn_min=0.1, Kn_max=0.1, g=-0.5, T_right=2.0, dt=-0.5, form="fp64",
             graph=0, steps=16, monitor=False, draw=0),
        # its full-range comparison model, replayed graphs
        dict(name="channel_hlb16", kind="flow", quad="full", Q=16, channels=1, Nx_min=512, Nx_max=512, adv="weno5",
             chi=True, stretch=0.9, Kn_min=0.1, Kn_max=0.1, g=-0.5, T_right=2.0, dt=-0.5, form="fp64",
             graph=64, steps=64, monitor=False, draw=0),
        # a parameter sweep watched for its steady state: steps, then moments,
        # masses, wall densities and residuals
        dict(name="sweep_monitored", kind="flow", quad="half", Q=12, channels=64, Nx_min=300, Nx_max=700, adv="weno5",
             chi=True, stretch=0.9, Kn_min=0.01, Kn_max=1.0, g=-0.5, T_right=1.5, dt=-0.5, form="fp64",
             graph=0, steps=16, monitor=True, draw=1),
        # thousands of uneven channels (orders 4, 8 and 12) in one solver
        dict(name="batch_fp64", kind="flow", quad="half", Q=0, channels=4096, Nx_min=64, Nx_max=1024, adv="weno5",
             chi=True, stretch=0.0, Kn_min=1e-3, Kn_max=10.0, g=-1.0, T_right=2.0, dt=-0.5, form="fp64",
             graph=0, steps=4, monitor=False, draw=0),
        # the same batch in the mixed form
        dict(name="batch_mixed_f32", kind="flow", quad="half", Q=0, channels=4096, Nx_min=64, Nx_max=1024, adv="weno5",
             chi=True, stretch=0.0, Kn_min=1e-3, Kn_max=10.0, g=-1.0, T_right=2.0, dt=-0.5, form="mixed_f32",
             graph=0, steps=2, monitor=False, draw=0),
        # the large workload: 256 stretched channels of 16384 cells
        dict(name="large_fp64", kind="flow", quad="half", Q=16, channels=256, Nx_min=16384, Nx_max=16384, adv="weno5",
             chi=True, stretch=0.9, Kn_min=0.005, Kn_max=0.05, g=-1.0, T_right=1.5, dt=-0.5, form="fp64",
             graph=0, steps=4, monitor=False, draw=0),
        # the same with the force block on BF16 matrix cores
        dict(name="large_mixed_bf16", kind="flow", quad="half", Q=16, channels=256, Nx_min=16384, Nx_max=16384,
             adv="weno5", chi=True, stretch=0.9, Kn_min=0.005, Kn_max=0.05, g=-1.0, T_right=1.5, dt=-0.5,
             form="mixed_bf16", graph=0, steps=2, monitor=False, draw=0),
        # the ballistic study: eight collisionless channels of 24 cells, large
        # velocity sets (half range, then the full-range comparison)
        dict(name="ballistic_hhlb200", kind="flow", quad="half", Q=200, channels=8, Nx_min=24, Nx_max=24, adv="weno5",
             chi=False, stretch=0.99, Kn_min=0.0, Kn_max=0.0, g=-0.1, T_right=0.6, dt=1e-4, form="fp64",
             graph=0, steps=16, monitor=False, draw=0),
        dict(name="ballistic_hlb500", kind="flow", quad="full", Q=500, channels=8, Nx_min=24, Nx_max=24, adv="weno5",
             chi=False, stretch=0.99, Kn_min=0.0, Kn_max=0.0, g=-0.1, T_right=0.6, dt=1e-4, form="fp64",
             graph=0, steps=16, monitor=False, draw=0),
        # the homogeneous gas on a three-axis product set, a million points
        dict(name="gas_3d", kind="gas", axes="half:4 full:4 full:4", points=1000000, Kn=0.1, dt=1e-3, steps=4,
             workspace=True),
        # a few points on a two-axis set, without a workspace
        dict(name="gas_2d_small", kind="gas", axes="half:8 full:8", points=2048, Kn=0.1, dt=1e-3, steps=8,
             workspace=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pick = rng.random()
    if pick < 0.2:   # product sets of the homogeneous gas
        axes, steps = rng.choice(("half:4 full:4 full:4", "half:8 full:8", "half:3 half:3 full:4", "half:8 full:8 full:4",
                                  "half:12 full:4", "full:6 half:4 laguerre:3", "half:10 half:10 full:2")), rng.randint(1, 4)
        V = math.prod(a.V for a in _axes(axes))
        workspace = rng.random() < 0.7
        most = 1.28e8 / V if workspace else 15.0 * 2 ** 20 / (8 * V)
        return dict(kind="gas", axes=axes, points=_log_int(rng, 100, most), Kn=round(10 ** rng.uniform(-1.5, 0.5), 4),
                    dt=1e-3, steps=steps, workspace=workspace)
    if pick < 0.35:  # large velocity sets, few cells
        quad = rng.choice(("half", "full"))
        Q = _log_int(rng, 18, 200) if quad == "half" else 2 * _log_int(rng, 9, 250)
        Nx = _log_int(rng, 16, 200)
        return dict(kind="flow", quad=quad, Q=Q, channels=rng.randint(1, 12), Nx_min=Nx, Nx_max=Nx,
                    adv=rng.choice(("weno5", "weno5", "upwind3")), chi=rng.random() < 0.4, stretch=rng.choice((0.0, 0.9)),
                    Kn_min=0.0 if rng.random() < 0.5 else 0.1, Kn_max=1.0, g=-0.1, T_right=round(rng.uniform(0.6, 1.5), 3),
                    dt=2e-5, form="fp64", graph=rng.choice((0, 16)), steps=16, monitor=False,
                    draw=rng.randint(2, 10 ** 6))
    quad = rng.choice(("half", "half", "half", "half", "full", "laguerre"))
    Q = rng.choice((4, 8, 16)) if quad == "full" else rng.choice((3, 4, 6, 8, 12, 16))
    if quad == "half" and rng.random() < 0.3:
        Q = 0    # orders 4, 8 and 12 in one solver
    V = {"full": Q}.get(quad, 2 * (Q or 8))
    hi = _log_int(rng, 40, 16384)
    lo = hi if rng.random() < 0.4 else max(24, hi // rng.randint(2, 8))
    most = int(min(4096, max(1, 1.2e8 / (V * hi))))
    channels = _log_int(rng, 1, most) if most > 1 else 1
    size = channels * hi * V
    steps = max(1, min(64, int(2e8 / size)))
    form = rng.choice(("fp64", "fp64", "fp64", "mixed_f32", "mixed_bf16", "mixed_f16")) if quad == "half" else "fp64"
    if form != "fp64":
        steps = min(steps, 2)
    graph = min(16, steps) if rng.random() < 0.3 else 0
    return dict(kind="flow", quad=quad, Q=Q, channels=channels, Nx_min=lo, Nx_max=hi,
                adv=rng.choice(("weno5", "weno5", "weno5", "upwind3")), chi=rng.random() < 0.85,
                stretch=rng.choice((0.0, 0.9)), Kn_min=0.01, Kn_max=round(10 ** rng.uniform(-1.5, 1), 3),
                g=-round(rng.uniform(0.05, 1.0), 3), T_right=round(rng.uniform(1.0, 2.0), 3), dt=-0.5, form=form,
                graph=graph, steps=steps, monitor=rng.random() < 0.25, draw=rng.randint(2, 10 ** 6))


# ---- what a program has in hand ---------------------------------------------

P0_LAGUERRE = {3: 0.5, 4: 0.4, 6: 0.35, 8: 0.3, 12: 0.2, 16: 0.2}   # momentum scales that hold T = 1 .. 2


def _channels(case):
    """The channels of a flow case, as plain parameters."""
    rng = np.random.default_rng(case["draw"])
    out = []
    for _ in range(case["channels"]):
        Q = case["Q"] or int(rng.choice([4, 8, 12]))
        Nx = int(rng.integers(case["Nx_min"], case["Nx_max"] + 1))
        u = rng.random(3)
        Kn = math.inf if case["Kn_min"] == 0.0 else case["Kn_min"] * (case["Kn_max"] / case["Kn_min"]) ** u[0]
        many = case["channels"] > 1
        g = case["g"] * (0.1 + 0.9 * u[1]) if many else case["g"]
        TR = 1.0 + (case["T_right"] - 1.0) * u[2] if many else case["T_right"]
        TL = 1.4 if case["T_right"] < 1.0 else 1.0
        p0 = P0_LAGUERRE[Q] if case["quad"] == "laguerre" else 1.0
        out.append(dict(Q=Q, N=min(20, Q - 1), Nx=Nx, Kn=Kn, g=float(g), TL=TL, TR=float(TR), p0=p0))
    return out


class _Axis:
    def __init__(self, quad, Q):
        self.quad, self.Q, self.N, self.p0 = quad, Q, Q - 1, 0.6 if quad == "laguerre" else 1.0
        self.V = Q if quad == "full" else 2 * Q


def _axes(text):
    return [_Axis(a.split(":")[0], int(a.split(":")[1])) for a in text.split()]


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _flow_start(case, seed):
    """f and chi in the library's layout: the equilibrium at rest, every row
    (node of a channel) times a smooth modulation of its own, as a developed
    flow has it."""
    g = _generator(seed)
    chans = _channels(case)
    f, rows_n, amp = [], [], 0.05
    unit = {}
    for c in chans:
        key = (case["quad"], c["Q"], c["N"], c["p0"])
        if key not in unit:
            R = _rule(*key[:2])
            one = torch.ones(1, dtype=torch.float64)
            unit[key] = _equilibrium(R, c["N"], c["p0"], one * 0.0, one)[:, 0]
        f.append(unit[key])
        rows_n.append(np.full(len(unit[key]), c["Nx"], dtype=np.int64))
    f = torch.cat(f).to(DEVICE)
    rows_n = torch.from_numpy(np.concatenate(rows_n)).to(DEVICE)
    rows = len(f)
    first = torch.cumsum(rows_n, 0) - rows_n
    total = int(rows_n.sum())
    if case["Q"] > 16:
        # a large set's force matrix differentiates in p: the modulation is
        # smooth in p too (one per channel)
        per = torch.tensor([(c["Q"] if case["quad"] == "full" else 2 * c["Q"]) for c in chans], device=DEVICE)
        amp = 0.02
    else:
        per = torch.ones(rows, dtype=torch.int64, device=DEVICE)
    row = torch.repeat_interleave(torch.arange(rows, device=DEVICE), rows_n, output_size=total)
    x = (torch.arange(total, device=DEVICE) - first[row] + 0.5) / rows_n[row]
    out = []
    for fn in range(2 if case["chi"] else 1):
        m = torch.randint(1, 4, (len(per),), generator=g, device=DEVICE).to(torch.float64).repeat_interleave(per)
        phi = (2 * math.pi) * torch.rand(len(per), generator=g, dtype=torch.float64, device=DEVICE).repeat_interleave(per)
        y = x * (2 * math.pi * m)[row]
        y += phi[row]
        y = y.sin_().mul_(amp).add_(1.0).mul_(f[row])
        out.append(y)
    return out[0], (out[1] if case["chi"] else None)


def _gas_start(case, seed):
    """Populations of points at densities, velocities and temperatures of
    their own, a little off equilibrium."""
    g = _generator(seed)
    axes, n = _axes(case["axes"]), case["points"]

    def uniform(*shape):
        return torch.rand(*shape, generator=g, dtype=torch.float64, device=DEVICE)

    dens, T, u = 0.8 + 0.4 * uniform(n), 0.8 + 0.4 * uniform(n), 0.3 * (uniform(n, len(axes)) - 0.5)
    f = _gas_equilibrium(axes, dens, u, T).contiguous()
    f *= 1.0 + 0.1 * uniform(n, f.shape[1])
    return f


GAS_FORCE = (0.3, -0.2, 0.5)


def prepare(case, seed):
    import paper_1708_03249_amd as H
    quads = {"half": H.HALF_HERMITE, "full": H.FULL_HERMITE, "laguerre": H.HALF_LAGUERRE}
    if case["kind"] == "gas":
        axes = [H.Axis(quad=quads[a.quad], Q=a.Q, N=a.N, p0=a.p0) for a in _axes(case["axes"])]
        f0 = _gas_start(case, seed)
        s = H.MultiSolver(axes, case["points"], GAS_FORCE[:len(axes)], case["Kn"]) if case["workspace"] else None
        return dict(case=case, H=H, axes=axes, f0=f0, f=torch.empty_like(f0), solver=s)
    s = H.Solver([H.Channel(quad=quads[case["quad"]], Q=c["Q"], N=c["N"], Nx=c["Nx"],
                            adv=H.WENO5 if case["adv"] == "weno5" else H.UPWIND3, transverse_dof=2 if case["chi"] else 0,
                            L=1.0, stretch_A=case["stretch"], Kn=c["Kn"], g=c["g"], T_left=c["TL"], T_right=c["TR"],
                            p0=c["p0"], dt=case["dt"]) for c in _channels(case)], precision=case["form"])
    f, chi = _flow_start(case, seed)
    s.set_state(f, chi)
    if case["graph"]:
        s.set_graph_steps(case["graph"])
    return dict(case=case, solver=s)


def run(state):
    case, s = state["case"], state["solver"]
    if case["kind"] == "gas":
        f = state["f"].copy_(state["f0"])
        if s is not None:
            s.step(f, case["dt"], case["steps"])
        else:
            axes = state["axes"]
            state["H"].multi_step_noalloc(axes, f, GAS_FORCE[:len(axes)], case["Kn"], case["dt"], case["steps"])
        return f
    s.step(case["steps"])
    f, chi = s.get_state()
    n, u, T = s.moments()
    out = dict(f=f, n=n, u=u, T=T)
    if case["chi"]:
        out["chi"] = chi
    if case["monitor"]:
        out["n_wall"], out["mass"], out["nonfinite"], out["residual"] = s.diagnostics(residual=True)
    return _kept(case, out)


def _kept(case, out):
    """What a program keeps of the results: a mixed run's are FP32 at heart
    (increments of about 1e-7) and are kept as such."""
    if case["form"] == "fp64":
        return out
    return {k: v.float() if v.is_floating_point() else v for k, v in out.items()}


def work(case):
    """The state in and out once, and the operations of the steps."""
    if case["kind"] == "gas":
        axes, pts = _axes(case["axes"]), case["points"]
        V = math.prod(a.V for a in axes)
        coeff = sum(_coefficient_flops(a.quad, a.Q, a.N) + 2 * a.V * (a.N + 1) for a in axes)
        stage = V * (sum(2 * a.V for a in axes) + 4 * len(axes) + 15) + coeff
        return dict(bytes=16.0 * V * pts, flops=3.0 * case["steps"] * stage * pts)
    nf = 2 if case["chi"] else 1
    byts = flops = 0.0
    for c in _channels(case):
        V = c["Q"] if case["quad"] == "full" else 2 * c["Q"]
        rows = V if case["quad"] == "full" else V // 2
        face = 70 if case["adv"] == "weno5" else 8
        stage = V * nf * (face + 12 + 2 * rows)
        if c["Kn"] != math.inf:
            stage += V * (2 * (c["N"] + 1) + 4 * nf) + _coefficient_flops(case["quad"], c["Q"], c["N"])
        byts += 8.0 * c["Nx"] * (2 * V * nf + 3)
        flops += 3.0 * case["steps"] * stage * c["Nx"]
    return dict(bytes=byts, flops=flops)


def _coefficient_flops(quad, Q, N):
    """Operations of one cell's equilibrium coefficients: a three-term
    recurrence at the points of the exact rule."""
    return 6.0 * N if quad == "full" else 2 * 7.0 * (N + 1) * ((N + 2) // 2)


# ---- the same in plain 64-bit arithmetic ------------------------------------

@lru_cache(maxsize=None)
def _recurrence(quad, n):
    """Coefficients a_0..a_n, b_0..b_n of the monic orthogonal polynomials."""
    if quad == "full":
        return [Decimal(0)] * (n + 1), [Decimal(max(1, l)) for l in range(n + 1)]
    if quad == "laguerre":
        return [Decimal(2 * l + 1) for l in range(n + 1)], [Decimal(max(1, l * l)) for l in range(n + 1)]
    with localcontext() as ctx:
        ctx.prec = 60 + 4 * n
        m = [Decimal(1) / 2, 1 / (2 * _pi(ctx.prec + 10)).sqrt()]
        for s in range(2, 2 * n + 2):
            m.append((s - 1) * m[s - 2])
        a, b = [m[1] / m[0]], [m[0]]     # the Chebyshev algorithm
        old, cur = [Decimal(0)] * (2 * n + 2), m
        for k in range(1, n + 1):
            new = [Decimal(0)] * (2 * n + 2)
            for l in range(k, 2 * n - k + 2):
                new[l] = cur[l + 1] - a[k - 1] * cur[l] - (b[k - 1] * old[l] if k > 1 else 0) if l + 1 < 2 * n + 2 else 0
            a.append(new[k + 1] / new[k] - cur[k] / cur[k - 1] if k + 1 < 2 * n + 2 else Decimal(0))
            b.append(new[k] / cur[k - 1])
            old, cur = cur, new
    with localcontext() as ctx:
        ctx.prec = 50
        return [+x for x in a], [+x for x in b]


@lru_cache(maxsize=None)
def _pi(prec):
    with localcontext() as ctx:     # Machin's formula
        ctx.prec = prec

        def arctan_inv(k):
            term, total, d, sign = Decimal(1) / k, Decimal(0), 1, 1
            while abs(term) > Decimal(10) ** -prec:
                total += sign * term / d
                term, d, sign = term / (k * k), d + 2, -sign
            return total

        return 4 * (4 * arctan_inv(5) - arctan_inv(239))


class _Rule:
    pass


@lru_cache(maxsize=None)
def _rule(quad, Q):
    """Nodes, weights and the orthonormal polynomials at the nodes; for the
    momentum derivative its matrix K (p0 = 1)."""
    a, b = _recurrence(quad, Q)
    J = np.diag([float(x) for x in a[:Q]])
    for l in range(1, Q):
        J[l, l - 1] = J[l - 1, l] = math.sqrt(float(b[l]))
    guess = np.linalg.eigvalsh(J)
    z, h = [], []
    with localcontext() as ctx:
        ctx.prec = 50
        sb = [x.sqrt() for x in b]

        def ortho(x):
            v = [1 / sb[0]]
            for l in range(Q):
                v.append(((x - a[l]) * v[l] - (sb[l] * v[l - 1] if l else 0)) / sb[l + 1])
            return v

        for x in guess[Q // 2:] if quad == "full" else guess:
            x = Decimal(float(x))
            for _ in range(3):   # Newton on p_Q / p_Q'
                p, d, pm, dm = 1 / sb[0], Decimal(0), Decimal(0), Decimal(0)
                for l in range(Q):
                    t = x - a[l]
                    s = sb[l] if l else Decimal(0)
                    p, d, pm, dm = (t * p - s * pm) / sb[l + 1], (p + t * d - s * dm) / sb[l + 1], p, d
                x -= p / d
            z.append(x)
            h.append(ortho(x))
        h0 = ortho(Decimal(0))
        w = [1 / sum(v * v for v in row[:Q]) for row in h]
        w0 = 1 / (2 * _pi(60)).sqrt() if quad == "half" else Decimal(1)    # weight function at 0

    def ld(rows):
        return np.array([[np.longdouble(str(v)) for v in r] for r in rows])

    R = _Rule()
    R.quad, R.Q, R.H = quad, Q, len(z)
    R.V = Q if quad == "full" else 2 * Q
    hz, wl, zl, h0 = ld(h), ld([w])[0], ld([z])[0], ld([h0])[0]
    sbl = ld([sb])[0]
    if quad == "full":
        sign = np.array([(-1.0) ** l for l in range(Q + 1)])
        hz = np.concatenate([hz, hz * sign])
        zl, wl = np.concatenate([zl, -zl]), np.concatenate([wl, wl])
        K = -wl[:, None] * ((hz[:, 1:Q] * np.sqrt(np.arange(1, Q).astype(np.longdouble))) @ hz[:, :Q - 1].T)
    else:
        terms = h0[:Q] * hz[:, :Q]
        tail = np.cumsum(terms[:, ::-1], axis=1)[:, ::-1] - terms     # sum over s > l
        A = h0[:Q] * np.longdouble(str(w0)) * tail
        if quad == "half":
            A[:, :Q - 1] -= sbl[1:Q] * hz[:, 1:Q]
        inner = A[:, :Q - 1] @ hz[:, :Q - 1].T
        phi = terms.sum(axis=1)
        cross = -wl[:, None] * np.longdouble(str(w0)) / 2 * phi[:, None] * phi[None, :]
        inner = wl[:, None] * inner
        K = np.block([[inner + cross, cross], [-cross, -inner - cross]])
        zl, wl = np.concatenate([zl, -zl]), np.concatenate([wl, wl])
    R.z, R.w, R.K = (torch.from_numpy(x.astype(np.float64)) for x in (zl, wl, K))
    R.wh = torch.from_numpy((wl[:, None] * np.concatenate([hz, hz]) if quad != "full" else wl[:, None] * hz)[:, :Q].astype(np.float64))
    R.a = [float(x) for x in a]
    R.sb = [float(x) for x in sb]
    R.on = {}
    return R


def _on(R, device):
    """The rule's tables on a device."""
    if str(device) not in R.on:
        R.on[str(device)] = {k: getattr(R, k).to(device) for k in ("z", "w", "K", "wh")}
    return R.on[str(device)]


def _equilibrium(R, N, p0, u, T):
    """Truncated expansion of the unit-density Maxwellian, [V, cells]."""
    t = _on(R, u.device)
    if R.quad == "full":
        ub, aa = u / p0, T / p0 ** 2 - 1.0
        G = [torch.ones_like(u), ub]
        for l in range(1, N):
            G.append((ub * G[l] + math.sqrt(l) * aa * G[l - 1]) / math.sqrt(l + 1))
        return t["wh"][:, :N + 1] @ torch.stack(G[:N + 1])
    sT = T.sqrt()
    main = _rule("half", (N + 2) // 2)
    xs, ls = np.polynomial.legendre.leggauss(24)
    out = []
    for sg in (1.0, -1.0):
        G = torch.zeros((N + 1,) + u.shape, dtype=u.dtype, device=u.device)

        def add(x, wt):
            hm, h = torch.zeros_like(x), torch.full_like(x, 1 / R.sb[0])
            G[0].add_(wt * h)
            for l in range(N):
                hm, h = h, ((x - R.a[l]) * h - (R.sb[l] if l else 0.0) * hm) / R.sb[l + 1]
                G[l + 1].add_(wt * h)

        for z, w in zip(main.z[:main.H].tolist(), main.w[:main.H].tolist()):
            add((sg * u + sT * z) / p0, w)
        y0 = -u / sT      # the shift of the half axis, an interval [y0, 0]
        for x, lam in zip(xs, ls):
            s = 0.5 * (x + 1.0)
            e = y0 * (0.5 * lam / math.sqrt(2 * math.pi)) * torch.exp(-0.5 * (y0 * s) ** 2)
            add(sg * u / p0 * (1.0 - s), -sg * e)
        out.append(t["wh"][:R.H, :N + 1] @ G)
    return torch.cat(out)


def _grid(Nx, A):
    if A == 0.0:
        return np.full(Nx, 1.0 / Nx)
    d = np.longdouble(2.0) / Nx * np.arctanh(np.longdouble(A))
    i = np.arange(Nx).astype(np.longdouble)
    hi, lo = (i + 1 - np.longdouble(Nx) / 2) * d, (i - np.longdouble(Nx) / 2) * d
    return (np.sinh(d) / (2 * np.longdouble(A)) / (np.cosh(hi) * np.cosh(lo))).astype(np.float64)


def _weno5(a, b, c, d, e):
    s = [13 / 12 * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2,
         13 / 12 * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2,
         13 / 12 * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2]
    big = torch.maximum(s[0], torch.maximum(s[1], s[2]))
    big = torch.where(big > 0, big, torch.ones_like(big))
    q = [(x / big) ** 2 for x in s]
    w = [0.1 * q[1] * q[2], 0.6 * q[0] * q[2], 0.3 * q[0] * q[1]]
    flat = w[0] + w[1] + w[2] <= 1e-250
    w = [torch.where(flat, torch.where(x < 1e-125, k, 0.0).to(x.dtype), y) for x, y, k in zip(q, w, (0.1, 0.6, 0.3))]
    F = [(2 * a - 7 * b + 11 * c) / 6, (-b + 5 * c + 2 * d) / 6, (2 * c + 5 * d - e) / 6]
    return (w[0] * F[0] + w[1] * F[1] + w[2] * F[2]) / (w[0] + w[1] + w[2])


def _face(adv, a, b, c, d, e):
    return _weno5(a, b, c, d, e) if adv == "weno5" else (-b + 5 * c + 2 * d) / 6


class _Flow:
    """Channels of one order on a flat axis of cells, three ghosts on either
    side of each channel."""

    def __init__(self, case, chans, offsets, cells):
        self.case, self.c0 = case, chans[0]
        self.R = R = _rule(case["quad"], self.c0["Q"])
        self.t = _on(R, DEVICE)
        Nx = np.array([c["Nx"] for c in chans])
        first = np.concatenate([[0], np.cumsum(Nx + 6)])[:-1]
        ch = np.repeat(np.arange(len(chans)), Nx)
        i = np.arange(Nx.sum()) - np.repeat(np.cumsum(Nx) - Nx, Nx)
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEVICE)  # noqa: E731
        self.M = int((Nx + 6).sum())
        self.pos = dev(first[ch] + 3 + i)                  # of each cell on the ghosted axis
        self.left, self.right = dev(first + 3), dev(first + 2 + Nx)
        self.cell = dev(np.array(cells)[ch] + i)           # of each cell in the per-cell outputs
        self.at, self.step = dev(np.array(offsets)[ch] + i), dev(Nx[ch])
        p = R.z * self.c0["p0"]
        self.p = dev(p.numpy())
        vmax = float(p.abs().max())
        dx = [_grid(c["Nx"], case["stretch"]) for c in chans]
        dts = []
        for c, d in zip(chans, dx):
            dt = case["dt"]
            if dt < 0:
                dt = -dt * d.min() / vmax
                if math.isfinite(c["Kn"]):
                    dt = min(dt, 0.5 * c["Kn"])
            dts.append(dt)
        self.dx, self.dt, self.dts = dev(np.concatenate(dx)), dev(np.array(dts)[ch]), dev(np.array(dts))
        self.g = dev(np.array([c["g"] for c in chans])[ch])
        self.inv_Kn = dev(np.array([1.0 / c["Kn"] for c in chans])[ch])
        self.collide = math.isfinite(self.c0["Kn"])
        self.ch, self.n_ch = dev(ch), len(chans)
        T = lambda k: dev(np.array([c[k] for c in chans]))  # noqa: E731
        self.TL, self.TR = T("TL"), T("TR")
        H = R.V // 2
        self.gL, self.gR = (_equilibrium(R, self.c0["N"], self.c0["p0"], 0 * x, x) for x in (self.TL, self.TR))
        self.DL, self.DR = (self.p[:H, None] * self.gL[:H]).sum(0), (self.p[H:, None] * self.gR[H:]).sum(0)

    def take(self, flat):
        k = torch.arange(self.R.V, device=DEVICE)[:, None]
        return flat[self.at + k * self.step]

    def put(self, flat, y):
        k = torch.arange(self.R.V, device=DEVICE)[:, None]
        flat[self.at + k * self.step] = y

    def moments(self, f, chi):
        n = f.sum(0)
        u = (self.p[:, None] * f).sum(0) / n
        e = sum(((self.p[k] - u) ** 2 * f[k] for k in range(len(f))), 0.0 * u)
        Dt = 2 if chi is not None else 0
        if Dt:
            e = e + 2 * chi.sum(0)
        return n, u, e / ((1 + Dt) * n)

    def rhs(self, f, chi):
        adv, H, V = self.case["adv"], self.R.V // 2, self.R.V
        n, u, T = self.moments(f, chi)
        geq = _equilibrium(self.R, self.c0["N"], self.c0["p0"], u, T) if self.collide else None
        out, nL = [], None
        for fn, y in enumerate((f,) if chi is None else (f, chi)):
            L = (self.t["K"] / self.c0["p0"]) @ y
            L *= -self.g
            if geq is not None:
                L -= (y - (n if fn == 0 else n * T) * geq) * (n * self.inv_Kn)
            Y = torch.zeros((V, self.M), dtype=y.dtype, device=y.device)
            Y[:, self.pos] = y
            # incoming ghosts, extrapolated quadratically; the wall-face flux
            # of the incoming nodes balances the emergent one
            wl = [Y[H:, self.left + k] for k in range(3)]
            wr = [Y[:H, self.right - k] for k in range(3)]
            for w, rows, at, d in ((wl, slice(H, V), self.left, -1), (wr, slice(0, H), self.right, 1)):
                for k, c in enumerate(((3, -3, 1), (6, -8, 3), (10, -15, 6)), 1):
                    Y[rows, at + d * k] = c[0] * w[0] + c[1] * w[1] + c[2] * w[2]
            if fn == 0:
                gl = [3 * w[0] - 3 * w[1] + w[2] for w in (wl, wr)], [6 * w[0] - 8 * w[1] + 3 * w[2] for w in (wl, wr)]
                fl = _face(adv, wl[2], wl[1], wl[0], gl[0][0], gl[1][0])
                fr = _face(adv, wr[2], wr[1], wr[0], gl[0][1], gl[1][1])
                nL, nR = -(self.p[H:, None] * fl).sum(0) / self.DL, -(self.p[:H, None] * fr).sum(0) / self.DR
            eL, eR = nL * self.gL[:H] * (1 if fn == 0 else self.TL), nR * self.gR[H:] * (1 if fn == 0 else self.TR)
            for k in range(1, 4):
                Y[:H, self.left - k], Y[H:, self.right + k] = eL, eR
            for k0 in range(0, V, H):      # faces i+1/2, at most a gigabyte at a time
                rows = max(1, int(2 ** 26 // self.M))
                for k in range(k0, k0 + H, rows):
                    y5 = Y[k:min(k + rows, k0 + H)]
                    F = torch.zeros_like(y5)
                    if k0 == 0:
                        F[:, 2:-2] = _face(adv, y5[:, :-4], y5[:, 1:-3], y5[:, 2:-2], y5[:, 3:-1], y5[:, 4:])
                        F[:, self.left - 1] = eL[k:k + len(F)]
                    else:
                        F[:, 1:-3] = _face(adv, y5[:, 4:], y5[:, 3:-1], y5[:, 2:-2], y5[:, 1:-3], y5[:, :-4])
                        F[:, self.right] = eR[k - H:k - H + len(F)]
                    F *= self.p[k:k + len(F), None]
                    L[k:k + len(F)] -= (F[:, self.pos] - F[:, self.pos - 1]) / self.dx
            out.append(L)
        self.walls = torch.stack([nL, nR], 1)
        return out

    def run(self, f, chi, steps):
        def stage(y, a, base, b):
            ls = self.rhs(*y)
            return [None if x is None else b * (x + self.dt * ls[k]) + (a * base[k] if a else 0.0) for k, x in enumerate(y)]

        y = [f, chi]
        for _ in range(steps):
            y1 = stage(y, 0.0, y, 1.0)
            y2 = stage(y1, 0.75, y, 0.25)
            y = stage(y2, 1 / 3, y, 2 / 3)
        return y

    def per_channel(self, x, what):
        r = torch.zeros(self.n_ch, dtype=x.dtype, device=x.device)
        return r.index_add_(0, self.ch, x) if what == "sum" else r.index_reduce_(0, self.ch, x, "amax")


def _flow_exact(case, seed):
    f0, c0 = _flow_start(case, seed)
    chans = _channels(case)
    V = [c["Q"] if case["quad"] == "full" else 2 * c["Q"] for c in chans]
    off = np.concatenate([[0], np.cumsum([v * c["Nx"] for v, c in zip(V, chans)])])
    cell = np.concatenate([[0], np.cumsum([c["Nx"] for c in chans])])
    new = lambda k: torch.zeros(int(k), dtype=torch.float64, device=DEVICE)  # noqa: E731
    out = dict(f=torch.empty_like(f0), n=new(cell[-1]), u=new(cell[-1]), T=new(cell[-1]))
    if case["chi"]:
        out["chi"] = torch.empty_like(f0)
    if case["monitor"]:
        out.update(n_wall=new(2 * len(chans)).view(-1, 2), mass=new(len(chans)),
                   nonfinite=torch.zeros(1, dtype=torch.int32, device=DEVICE), residual=new(len(chans)))
    for Q in sorted({c["Q"] for c in chans}):
        who = [k for k, c in enumerate(chans) if c["Q"] == Q]
        F = _Flow(case, [chans[k] for k in who], [off[k] for k in who], [cell[k] for k in who])
        f, chi = F.run(F.take(f0), F.take(c0) if case["chi"] else None, case["steps"])
        F.put(out["f"], f)
        if case["chi"]:
            F.put(out["chi"], chi)
        n, u, T = F.moments(f, chi)
        for k, v in (("n", n), ("u", u), ("T", T)):
            out[k][F.cell] = v
        if case["monitor"]:
            who = torch.tensor(who, device=DEVICE)
            out["n_wall"][who] = F.walls
            out["mass"][who] = F.per_channel(n * F.dx, "sum")
            res = new(len(who))
            for y, L in zip((f, chi), F.rhs(f, chi)):
                res = torch.maximum(res, F.per_channel(L.abs().amax(0), "max") / F.per_channel(y.abs().amax(0), "max"))
            out["residual"][who] = res
    return _kept(case, out)


def _gas_equilibrium(axes, n, u, T):
    f = n[:, None]
    for a, ax in enumerate(axes):
        g = _equilibrium(_rule(ax.quad, ax.Q), ax.N, ax.p0, u[:, a].contiguous(), T)
        f = (f[:, :, None] * g.T[:, None, :]).reshape(len(n), -1)
    return f


def _gas_rhs(axes, f, F, Kn):
    shape, d = [len(f)] + [a.V for a in axes], len(axes)
    y, L = f.view(shape), torch.zeros_like(f).view(shape)
    n, c2 = f.sum(1), 0.0
    u = []
    for a, ax in enumerate(axes):
        R = _rule(ax.quad, ax.Q)
        t = _on(R, f.device)
        m = y.sum([k + 1 for k in range(d) if k != a])     # the axis' marginal
        p = t["z"] * ax.p0
        u.append((m * p).sum(1) / n)
        c2 = c2 + (m * (p - u[a][:, None]) ** 2).sum(1)
        L -= F[a] / ax.p0 * (y.movedim(a + 1, -1) @ t["K"].T.contiguous()).movedim(-1, a + 1)
    T = c2 / (d * n)
    return L.reshape(f.shape) - (f - _gas_equilibrium(axes, n, torch.stack(u, 1), T)) * (n / Kn)[:, None]


def _gas_exact(case, seed):
    axes, dt = _axes(case["axes"]), case["dt"]
    f0, out = _gas_start(case, seed), []
    for f in f0.split(max(1, 2 ** 25 // f0.shape[1])):
        for _ in range(case["steps"]):
            y1 = f + dt * _gas_rhs(axes, f, GAS_FORCE, case["Kn"])
            y2 = 0.75 * f + 0.25 * (y1 + dt * _gas_rhs(axes, y1, GAS_FORCE, case["Kn"]))
            f = f / 3 + 2 / 3 * (y2 + dt * _gas_rhs(axes, y2, GAS_FORCE, case["Kn"]))
        out.append(f)
    return torch.cat(out)


def exact(case, seed):
    if case["kind"] == "gas":
        return _gas_exact(case, seed)
    return _flow_exact(case, seed)


getcontext().prec = 50
