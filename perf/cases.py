"""Timed workloads of the CRKSPH path, and their values in 64 bits.

Each case is one call (or one forward and its adjoint) that a hydro or
calibration program makes through the public entry points: the evaluation
(``Context.forward``), its gradient (``Context.backward`` or autograd through
``CRKSPHFunction``), the time steps, the cooling update and the subgrid
deposition. Sizes, kernels and particle sets are those of the benchmark, the
synthetic sets and the tests (``lattice16``, ``sedov64_v``, the clump sets,
random sets with unequal masses), with odd sizes between them.

A program keeps one context per particle set, so ``prepare`` makes the
context with the inputs and ``run`` is a call on it. The FP32 form's
accelerations, du/dt and gradients are handed on in FP32 like the velocities
and energies they update; the FP64 form's in FP64.

``exact`` is a plain torch evaluation in float64 of the same inputs: pairs by
brute force over slabs, gradients by autograd, the solved h differentiated at
its root.
"""
import math

import torch
from torch.utils.checkpoint import checkpoint

from paper_2511_21921_amd import (CUBIC_SPLINE, FP32, FP64, WENDLAND_C4, Context,
                                  CRKSPHFunction, Params)

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # the unit-test lattice: a single evaluation of a small box, where the
        # call's own latency counts
        {"name": "eval_lattice_4k", "op": "eval", "set": "lattice", "n": 4096, "precision": "fp32",
         "kernel": "cubic", "n_h": 1.9695, "h_mode": 0},
        # gradient check and small-box calibration: FP64, unequal masses, a
        # ragged size, through autograd with the viscosity coefficients
        {"name": "autograd_random_1001_fp64", "op": "autograd", "set": "random", "n": 1001,
         "precision": "fp64", "kernel": "cubic", "n_h": 2.4814, "h_mode": 1, "masses": "spread"},
        # a calibration box at the paper's gas resolution (~268 neighbours),
        # the moments kept for the adjoint, the adjoint without allocation
        {"name": "grad_random_33k_c4", "op": "grad", "set": "random", "n": 33333,
         "precision": "fp32", "kernel": "c4", "n_h": 4.0, "h_mode": 1, "store": True,
         "noalloc": True},
        # the 64^3 gradient workload of the benchmark, in both precisions
        {"name": "grad_sedov_262k", "op": "grad", "set": "sedov", "n": 262144,
         "precision": "fp32", "kernel": "cubic", "n_h": 2.4814, "h_mode": 1},
        {"name": "grad_sedov_262k_fp64", "op": "grad", "set": "sedov", "n": 262144,
         "precision": "fp64", "kernel": "cubic", "n_h": 2.4814, "h_mode": 1},
        # the same particles at the paper's gas resolution
        {"name": "grad_sedov_262k_c4", "op": "grad", "set": "sedov", "n": 262144,
         "precision": "fp32", "kernel": "c4", "n_h": 4.0, "h_mode": 1},
        # strongly clustered gas: 128^3 and the benchmark's headline 256^3
        {"name": "grad_clumps_2m", "op": "grad", "set": "clumps", "n": 2097152,
         "precision": "fp32", "kernel": "cubic", "n_h": 2.4814, "h_mode": 1},
        {"name": "grad_clumps_17m", "op": "grad", "set": "clumps", "n": 16777216,
         "precision": "fp32", "kernel": "cubic", "n_h": 2.4814, "h_mode": 1},
        # time integration: a single-level step of an odd-sized box with
        # unequal masses, and a big step of the timestep hierarchy at 64^3
        {"name": "kdk_lattice_100k", "op": "kdk", "set": "lattice", "n": 100003,
         "precision": "fp32", "kernel": "cubic", "n_h": 2.4814, "h_mode": 0, "masses": "spread"},
        {"name": "hkdk_hotspot_262k", "op": "hkdk", "set": "hotspot", "n": 262144,
         "precision": "fp32", "kernel": "cubic", "n_h": 2.4814, "h_mode": 0},
        # radiative cooling of a large volume, and one subgrid deposition
        {"name": "cool_17m", "op": "cool", "n": 16777216, "precision": "fp32", "nodes": 2001},
        {"name": "deposit_2m", "op": "deposit", "n": 2097152, "sources": 65536,
         "precision": "fp32", "kernel": "c4"},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["eval", "autograd", "grad", "grad", "grad", "grad", "clumps", "clumps", "kdk",
                     "hkdk", "cool", "deposit"])
    precision = rng.choice(["fp32", "fp32", "fp64"])
    if op == "cool":
        return {"op": "cool", "n": size(10 ** 4, 16777216), "precision": precision,
                "nodes": rng.choice([501, 2001, 4001])}
    if op == "deposit":
        n = size(2 * 10 ** 4, 2097152)
        return {"op": "deposit", "n": n, "sources": max(32, int(n * rng.uniform(0.002, 0.03))),
                "precision": precision, "kernel": rng.choice(["cubic", "c4"])}
    c4 = rng.random() < 0.3
    case = {"precision": precision, "kernel": "c4" if c4 else "cubic",
            "n_h": 4.0 if c4 else rng.choice([1.9695, 2.4814])}
    if op == "clumps":
        case.update(op=rng.choice(["eval", "grad", "grad"]), set="clumps", n=size(20000, 2097152),
                    h_mode=1, n_h=2.4814, kernel="cubic")
        return case
    if op in ("kdk", "hkdk"):
        case.update(op=op, n=size(4000 if op == "kdk" else 30000, 262144), h_mode=0,
                    set="hotspot" if op == "hkdk" else "lattice",
                    masses=rng.choice(["equal", "spread"]))
        return case
    case.update(op=op, set=rng.choice(["random", "lattice", "sedov"]),
                n=size(4000 if c4 else 800, 262144), h_mode=rng.choice([0, 1, 1]),
                masses=rng.choice(["equal", "equal", "spread"]), store=rng.random() < 0.3)
    if op == "grad" and case["n"] <= 65536:
        case["noalloc"] = rng.random() < 0.3
    return case


# ------------------------------------------------------------------ inputs --


def real_of(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def params_of(case, h_mode=None):
    return Params(n_h=case.get("n_h", 2.4814),
                  kernel=WENDLAND_C4 if case.get("kernel") == "c4" else CUBIC_SPLINE,
                  precision=FP64 if case["precision"] == "fp64" else FP32,
                  h_mode=case.get("h_mode", 1) if h_mode is None else h_mode,
                  store_corrections=1 if case.get("store") else 0)


def lattice_sites(n, g):
    """The first n sites of a cubic lattice (a random choice of them when n is
    no cube), jittered by a tenth of the spacing."""
    side = math.ceil(round(n ** (1.0 / 3.0), 6))
    i = torch.arange(side ** 3, device=DEV)
    if side ** 3 > n:
        i = torch.sort(torch.randperm(side ** 3, generator=g, device=DEV)[:n])[0]
    x = torch.stack([i // (side * side), (i // side) % side, i % side]).to(F64) / side
    return torch.remainder(x + (0.2 * torch.rand(3, n, generator=g, device=DEV, dtype=F64) - 0.1) / side,
                           1.0)


def clump_sites(n, g):
    """Half uniform, half in Plummer spheres: one clump per 4096 particles,
    log-normal clump masses (sigma 1 dex), scale radii U(0.002, 0.02)."""
    clumps = max(4, n // 4096)
    mass = 10.0 ** torch.randn(clumps, generator=g, device=DEV, dtype=F64)
    centre = torch.rand(3, clumps, generator=g, device=DEV, dtype=F64)
    a = 0.002 + 0.018 * torch.rand(clumps, generator=g, device=DEV, dtype=F64)
    n_cl = n - n // 2
    edge = torch.cumsum(mass, 0) / mass.sum() * n_cl
    c = torch.searchsorted(edge, torch.arange(n_cl, device=DEV, dtype=F64) + 0.5).clamp_(max=clumps - 1)
    q = torch.rand(n_cl, generator=g, device=DEV, dtype=F64) * (100.0 / 101.0) ** 1.5
    r = a[c] / torch.sqrt(q.clamp_min(1e-12) ** (-2.0 / 3.0) - 1.0)
    d = torch.randn(3, n_cl, generator=g, device=DEV, dtype=F64)
    d = centre[:, c] + r * d / d.norm(dim=0)
    return torch.remainder(torch.cat([torch.rand(3, n // 2, generator=g, device=DEV, dtype=F64), d], 1),
                           1.0)


def gas(case, seed):
    """x, v, m, u, the first h (or the fixed one) and the loss weights."""
    n, R = case["n"], real_of(case)
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["set"]
    if kind in ("lattice", "sedov", "hotspot"):
        x = lattice_sites(n, g)
    elif kind == "clumps":
        x = clump_sites(n, g)
    else:
        x = torch.rand(3, n, generator=g, device=DEV, dtype=F64)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=F64)

    v = (0.05 if kind == "clumps" else 0.1) * normal(3, n)
    if kind == "clumps":
        u = 10.0 ** (0.5 * normal(n))
    elif kind == "random":
        u = 10.0 ** (0.3 * normal(n))
    elif kind == "hotspot":
        # a warm region with a small hot core: few particles on the fine levels
        r2 = ((x - 0.5) ** 2).sum(0)
        u = 10.0 ** (0.1 * normal(n))
        u = torch.where(r2 < 0.1 ** 2, 4.0 * u, u)
        u = torch.where(r2 < 0.05 ** 2, 4.0 * u, u)
    else:
        u = torch.ones(n, device=DEV, dtype=F64)
        if kind == "sedov":
            u *= 1e-2
            u[((x - 0.5) ** 2).sum(0).argsort()[:27]] = 1e4
    m = torch.full((n,), 1.0 / n, device=DEV, dtype=F64)
    if case.get("masses") == "spread":
        m = m * 10.0 ** (0.6 * torch.rand(n, generator=g, device=DEV, dtype=F64) - 0.3)
    h = torch.full((n,), case["n_h"] * n ** (-1.0 / 3.0), device=DEV, dtype=F64)
    w = {"w_a": normal(3, n), "w_u": normal(n)} if case["op"] in ("grad", "autograd") else {}
    return {"x": x, **{k: a.to(R).contiguous() for k, a in (("v", v), ("m", m), ("u", u), ("h", h))},
            **w}


def levels_of(s):
    """Timestep levels from the signal speed c + |v|, as a CFL condition sets them."""
    sig = torch.sqrt(10.0 / 9.0 * s["u"].double()) + s["v"].double().norm(dim=0)
    return torch.ceil(torch.log2(sig / sig.median())).clamp(0, 3).to(torch.int32)


STEP = {"kdk": 2e-6, "hkdk": 4e-6}  # well inside the CFL condition of these sets


def cool_table(case):
    """A broken power law with a stable zero (heating below, cooling above), 8 decades."""
    K = case["nodes"]
    k = torch.arange(K, dtype=F64)
    lu0, dex = -3.0, 8.0 / (K - 1)
    uk = 10.0 ** (lu0 + dex * k)
    return lu0, dex, (uk ** 1.5 - 0.123 ** 1.5) * torch.exp(0.3 * torch.sin(0.02 * k * 2001 / K))


def cool_gas(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, R = case["n"], real_of(case)
    u = 10.0 ** (7.0 * torch.rand(n, generator=g, device=DEV, dtype=F64) - 2.5)
    rho = 10.0 ** (2.0 * torch.rand(n, generator=g, device=DEV, dtype=F64) - 1.0)
    return {"rho": rho.to(R), "u": u.to(R), "dt": 1e-3}


N_H_SRC = 2.25


def deposit_sets(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    ng, ns, R = case["n"], case["sources"], real_of(case)

    def uni(*s):
        return torch.rand(*s, generator=g, device=DEV, dtype=F64)

    def normal(*s):
        return torch.randn(*s, generator=g, device=DEV, dtype=F64)

    h0 = (32 / (4 * math.pi / 3) / ng) ** (1 / 3)
    gas_ = {"h": h0 * (1 + 0.2 * (2 * uni(ng) - 1)), "V": (1 + 0.2 * (2 * uni(ng) - 1)) / ng,
            "m": (1 + 0.1 * (2 * uni(ng) - 1)) / ng, "u": 10.0 ** (0.3 * normal(ng)),
            "v": 0.1 * normal(3, ng)}
    gas_["mZ"] = 0.04 * uni(ng) * gas_["m"]
    src = {"dM": 0.05 * (0.5 + uni(ns)) / ng, "dE": 0.05 * (0.5 + uni(ns)) / ng,
           "v": 0.2 * normal(3, ns)}
    src["dMZ"] = 0.01 * src["dM"]
    gas_ = {k: a.to(R).contiguous() for k, a in gas_.items()}
    src = {k: a.to(R).contiguous() for k, a in src.items()}
    gas_["x"], src["x"] = uni(3, ng), uni(3, ns)
    return gas_, src


# --------------------------------------------------------- prepare and run --


def prepare(case, seed):
    op = case["op"]
    if op == "cool":
        ctx = Context(Params(precision=FP64 if case["precision"] == "fp64" else FP32))
        lu0, dex, lam = cool_table(case)
        ctx.cooling_table(lu0, dex, lam.numpy())
        s = cool_gas(case, seed)
        return {"op": op, "ctx": ctx, "u_now": torch.empty_like(s["u"]), **s}
    if op == "deposit":
        gas_, src = deposit_sets(case, seed)
        return {"op": op, "ctx": Context(params_of(case)), "gas": gas_, "src": src}
    s = gas(case, seed)
    s.update(op=op, real=real_of(case), noalloc=bool(case.get("noalloc")),
             ctx=Context(params_of(case)))
    if op == "autograd":
        s["ab"] = torch.tensor([1.0, 2.0], dtype=F64)
        for k in ("x", "v", "u", "ab"):
            s[k].requires_grad_(True)
    if op in ("kdk", "hkdk"):
        # the evaluation at the start of the step
        s["out"] = s["ctx"].forward(s["x"], s["v"], s["m"], s["u"], s["h"])
        s["levels"] = levels_of(s)
    if op in ("eval", "grad"):
        n = case["n"]
        rows = {"h": 0, "V": 0, "rho": 0, "A": 0, "B": 3, "gradA": 3, "gradB": 9, "gradv": 9}
        s["out"] = {k: torch.empty((r, n) if r else (n,), dtype=s["real"], device=DEV)
                    for k, r in rows.items()}
        s["out"]["accel"] = torch.empty(3, n, dtype=F64, device=DEV)
        s["out"]["dudt"] = torch.empty(n, dtype=F64, device=DEV)
    return s


def run(s):
    op, ctx = s["op"], s["ctx"]
    if op == "cool":
        return ctx.cool(s["rho"], s["u_now"].copy_(s["u"]), s["dt"])
    if op == "deposit":
        out = ctx.deposit(s["gas"], s["src"], N_H_SRC)
        return {**{"s_" + k: out[k] for k in out}, **{k: s["gas"][k] for k in ("m", "mZ", "u", "v")}}
    R = s["real"]
    if op == "autograd":
        accel, dudt, h, rho, V, A, B, gA, gB, gv = CRKSPHFunction.apply(
            s["x"], s["v"], s["u"], s["ab"], s["m"], s["h"], ctx)
        g = torch.autograd.grad((accel, dudt), (s["x"], s["v"], s["u"], s["ab"]),
                                (s["w_a"], s["w_u"]))
        return {"accel": accel.detach().to(R), "dudt": dudt.detach().to(R), "h": h, "rho": rho,
                "V": V, "A": A, "B": B, "gradA": gA, "gradB": gB, "gradv": gv,
                "g_x": g[0].to(R), "g_v": g[1], "g_u": g[2], "g_alpha_beta": g[3].to(R)}
    out = s["out"]
    if op == "kdk":
        ctx.kdk_step(s["x"], s["v"], s["m"], s["u"], out, STEP[op])
    elif op == "hkdk":
        ctx.hkdk_step(s["x"], s["v"], s["m"], s["u"], out, s["levels"], STEP[op])
    else:
        ctx.forward(s["x"], s["v"], s["m"], s["u"], s["h"], out=out)
    r = dict(out)
    if op in ("kdk", "hkdk"):
        r.update(x=s["x"], v=s["v"], u=s["u"])
    if op == "grad":
        g = ctx.backward(s["w_a"], s["w_u"], noalloc=s["noalloc"])
        r.update({k: a.to(R) for k, a in g.items()})
    r["accel"], r["dudt"] = out["accel"].to(R), out["dudt"].to(R)
    return r


def work(case):
    """Inputs read and outputs written once; the pair sums' operations (FMA = 2)."""
    n, op = case["n"], case["op"]
    w = 8 if case["precision"] == "fp64" else 4
    if op == "cool":
        return {"bytes": 3 * w * n, "flops": 22 * n}
    if op == "deposit":
        s = case["sources"]
        # per source ~32 gas in each of its two sums, and the gas that receive
        return {"bytes": n * (24 + 12 * w) + s * (24 + 9 * w), "flops": s * 40.0 * (30 + 30 + 45)}
    gather = 4.18879 * case["n_h"] ** 3 * n * (0.87 if case["set"] == "clumps" else 1.0)
    force = gather * (1.19 if case["set"] == "clumps" else 1.12)
    # h and volume (five sums), moments, density and grad v, force
    fwd = gather * (5 * 12.0 + 109.0 + 94.0) + force * 216.0
    state = n * (24 + 6 * w + 28 * w + 4 * w)  # x, v, m, u, h; the outputs
    if op in ("grad", "autograd"):
        bwd = force * 680.0 + gather * (473.0 + 109.0 + 527.0 + 60.0)
        return {"bytes": state + n * (4 * 8 + 7 * w), "flops": fwd + bwd}
    if op == "kdk":
        return {"bytes": state + n * (24 + 4 * w + 32), "flops": fwd}
    if op == "hkdk":
        # every particle once a big step, the finer levels' more often
        return {"bytes": state + n * (24 + 4 * w + 32), "flops": 1.5 * fwd}
    return {"bytes": state, "flops": fwd}


# ------------------------------------------------------- values in 64 bits --


def shape(kernel, q):
    """w(q) and w'(q) of W(r, h) = C h^-3 w(r / h), support q < 1."""
    t = (1.0 - q).clamp_min(0.0)
    if kernel == "c4":
        return (t ** 6 * (1 + 6 * q + 35.0 / 3.0 * q * q),
                -56.0 / 3.0 * q * (1 + 5 * q) * t ** 5)
    inner = q <= 0.5
    return (torch.where(inner, 1 + q * q * (6 * q - 6), 2 * t ** 3),
            torch.where(inner, q * (18 * q - 12), -6 * t ** 2))


def norm_of(kernel):
    return 495.0 / (32.0 * math.pi) if kernel == "c4" else 8.0 / math.pi


def image(d):
    return d - torch.round(d)


def pairs_within(x, radius, rows, y=None):
    """All (i, j) with |x_i - y_j| < radius_i for i in rows (j != i when y is x)."""
    same = y is None
    y = x if same else y
    order = rows[torch.argsort(x[0, rows])]
    got_i, got_j = [], []
    step = 512
    for k in range(0, order.numel(), step):
        i = order[k:k + step]
        lo, hi, reach = x[0, i[0]], x[0, i[-1]], radius[i].max()
        near = (image(y[0] - 0.5 * (lo + hi)).abs() <= 0.5 * (hi - lo) + reach).nonzero()[:, 0]
        d2 = sum(image(x[a, i][:, None] - y[a, near][None, :]) ** 2 for a in range(3))
        hit = (d2 < (radius[i] ** 2)[:, None]).nonzero()
        a, b = i[hit[:, 0]], near[hit[:, 1]]
        if same:
            keep = a != b
            a, b = a[keep], b[keep]
        got_i.append(a)
        got_j.append(b)
    return torch.cat(got_i), torch.cat(got_j)


def rows_sum(n, i, vals):
    """vals [k, pairs] summed into [k, n] by i."""
    return torch.zeros(vals.shape[0], n, dtype=F64, device=vals.device).index_add(1, i, vals)


def over_pairs(f, i, j, *tensors):
    """The sum of f(i, j, *tensors) over blocks of pairs; a block's
    intermediates are computed again for its gradient."""
    total = None
    for k in range(0, max(1, i.numel()), 1 << 22):
        a, b = i[k:k + (1 << 22)], j[k:k + (1 << 22)]
        part = checkpoint(f, a, b, *tensors, use_reentrant=False)
        total = part if total is None else total + part
    return total


def thacker(kernel, x, m, h, i, j):
    """sum_j (m_j / m_i) w(r / h_i) and its derivative in h, self included."""
    n = m.numel()

    def f(a, b, x, m, h):
        r = image(x[:, a] - x[:, b]).square().sum(0).sqrt()
        w, dw = shape(kernel, r / h[a])
        return rows_sum(n, a, torch.stack([m[b] / m[a] * w, -m[b] / m[a] * dw * r / h[a] ** 2]))

    s = over_pairs(f, i, j, x, m, h)
    return s[0] + 1.0, s[1]


def solve_h(kernel, n_h, x, m):
    """The roots of C sum (m_j / m_i) w(r / h) = n_h^3, and the pairs they gather."""
    n = m.numel()
    C = norm_of(kernel)
    radius = torch.full_like(m, min(0.49, 1.25 * n_h * n ** (-1.0 / 3.0)))
    if n <= 70000:  # clustered sets: near the distance that holds twice the target count
        k = min(n - 1, int(2.2 * 4.18879 * n_h ** 3))
        for s in range(0, n, 512):
            d2 = sum(image(x[a, s:s + 512, None] - x[a, None, :]) ** 2 for a in range(3))
            radius[s:s + 512] = d2.topk(k + 1, 1, largest=False).values[:, -1].sqrt()
    radius.clamp_(max=0.49)
    todo = torch.arange(n, device=x.device)
    pi, pj = [], []
    while todo.numel():
        i, j = pairs_within(x, radius, todo)
        short = torch.zeros(n, dtype=torch.bool, device=x.device)
        short[todo] = (C * thacker(kernel, x, m, radius, i, j)[0] <= n_h ** 3)[todo]
        ok = ~short[i]
        pi.append(i[ok])
        pj.append(j[ok])
        todo = short.nonzero()[:, 0]
        radius[todo] = (radius[todo] * 1.3).clamp(max=0.499)
    i, j = torch.cat(pi), torch.cat(pj)
    lo, hi = torch.zeros_like(m), radius.clone()
    h = 0.8 * radius
    for _ in range(80):
        s, ds = thacker(kernel, x, m, h, i, j)
        f, fp = C * s - n_h ** 3, C * ds
        lo, hi = torch.where(f > 0, lo, h), torch.where(f > 0, h, hi)
        nt = h - f / fp.clamp_min(1e-300)
        new = torch.where((nt > lo) & (nt < hi), nt, 0.5 * (lo + hi))
        done = ((new - h).abs() <= 1e-15 * h).all()
        h = new
        if done:
            break
    keep = image(x[:, i] - x[:, j]).square().sum(0).sqrt() < h[i]
    return h, i[keep], j[keep]


SYM = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]


def corrected(kernel, d, h, A, B, dA, dB):
    """W^R = A (1 + B.x) W and its gradient for separations d, at h and the
    corrections of the evaluation point (dB rows: the derivative's axis)."""
    r = d.square().sum(0).sqrt()
    w, dw = shape(kernel, r / h)
    C = norm_of(kernel)
    W, f = C / h ** 3 * w, C / h ** 4 * dw / r
    s = 1.0 + (B * d).sum(0)
    g = [dA[a] * s * W + A * ((dB[3 * a:3 * a + 3] * d).sum(0) + B[a]) * W + A * s * f * d[a]
         for a in range(3)]
    return A * s * W, torch.stack(g)


def evaluate(case, x, v, m, u, h, ab, pairs=None, passive=None):
    """The evaluation in plain torch, h given or solved; pairs: (i, j) holding at
    least every r < h_i; passive: a mask and the V, rho, gradv, A, B, gradA, gradB
    that its particles keep."""
    kernel, n_h, n = case["kernel"], case["n_h"], m.numel()
    C = norm_of(kernel)
    if case["h_mode"] == 1:
        with torch.no_grad():
            root, i, j = solve_h(kernel, n_h, x, m)
        f, _ = thacker(kernel, x, m, root, i, j)
        with torch.no_grad():
            _, fp = thacker(kernel, x, m, root, i, j)
        h = root - (f - f.detach()) / fp  # the root's own derivative
    else:
        with torch.no_grad():
            i, j = pairs if pairs else pairs_within(x, h, torch.arange(n, device=x.device))
            near = image(x[:, i] - x[:, j]).square().sum(0).sqrt() < h[i]
            i, j = i[near], j[near]
    keep = (lambda name, new: new) if passive is None else \
        (lambda name, new: torch.where(passive["mask"], passive[name], new))
    s, _ = thacker(kernel, x, m, h, i, j)
    V = keep("V", h ** 3 / (C * s))

    def moments(a, b, x, h, V):
        d = image(x[:, a] - x[:, b])
        r = d.square().sum(0).sqrt()
        w, dw = shape(kernel, r / h[a])
        VW, Vf = V[b] * C / h[a] ** 3 * w, V[b] * C / h[a] ** 4 * dw / r
        p = [torch.ones_like(r)] + [d[k] for k in range(3)] + [d[k] * d[l] for k, l in SYM]
        out = rows_sum(n, a, torch.stack([VW * t for t in p]))
        for g in range(3):
            out = torch.cat([out, rows_sum(n, a, torch.stack([Vf * d[g] * t for t in p]))])
        return out

    M = over_pairs(moments, i, j, x, h, V)
    m0 = M[0] + V * C / h ** 3
    full = [[SYM.index((min(k, l), max(k, l))) for l in range(3)] for k in range(3)]
    m1, m2 = M[1:4].T, torch.stack([torch.stack([M[4 + full[k][l]] for l in range(3)], -1)
                                    for k in range(3)], -2)
    B = -torch.linalg.solve(m2, m1)
    A = 1.0 / (m0 + (B * m1).sum(1))
    dAs, dBs = [], []
    for g in range(3):
        o = 10 * (g + 1)
        dm0 = M[o]
        dm1 = torch.stack([M[o + 1 + k] + (m0 if k == g else 0.0) for k in range(3)], -1)
        dm2 = torch.stack([torch.stack([M[o + 4 + full[k][l]] + (m1[:, l] if k == g else 0.0) +
                                        (m1[:, k] if l == g else 0.0) for l in range(3)], -1)
                           for k in range(3)], -2)
        dBg = -torch.linalg.solve(m2, dm1 + (dm2 @ B[:, :, None])[:, :, 0])
        dBs.append(dBg.T)
        dAs.append(-A * A * (dm0 + (dBg * m1).sum(1) + (B * dm1).sum(1)))
    A, B, dA, dB = keep("A", A), keep("B", B.T), keep("gradA", torch.stack(dAs)), \
        keep("gradB", torch.cat(dBs))

    def density(a, b, x, v, h, V, A, B, dA, dB):
        WR, g = corrected(kernel, image(x[:, a] - x[:, b]), h[a], A[a], B[:, a], dA[:, a], dB[:, a])
        dv = v[:, a] - v[:, b]
        return rows_sum(n, a, torch.stack([m[b] * V[b] * WR, V[b] ** 2 * WR] +
                                          [-V[b] * dv[k] * g[l] for k in range(3) for l in range(3)]))

    D = over_pairs(density, i, j, x, v, h, V, A, B, dA, dB)
    self_w = A * C / h ** 3
    rho = keep("rho", (D[0] + m * V * self_w) / (D[1] + V * V * self_w))
    gv = keep("gradv", D[2:])
    P, cs = 2.0 / 3.0 * rho * u, torch.sqrt(10.0 / 9.0 * u)

    with torch.no_grad():  # every pair with r < max(h_i, h_j) once
        r = image(x[:, i] - x[:, j]).square().sum(0).sqrt()
        once = (i < j) | ~(r < h[j])
        fi, fj = i[once], j[once]

    def force(a, b, x, v, h, V, A, B, dA, dB, rho, P, cs, gv, ab):
        d = image(x[:, a] - x[:, b])
        _, gi = corrected(kernel, d, h[a], A[a], B[:, a], dA[:, a], dB[:, a])
        _, gj = corrected(kernel, -d, h[b], A[b], B[:, b], dA[:, b], dB[:, b])
        ga = torch.stack([(gv[3 * k:3 * k + 3, a] * d).sum(0) for k in range(3)])
        gb = torch.stack([(gv[3 * k:3 * k + 3, b] * d).sum(0) for k in range(3)])
        na, nb = (d * ga).sum(0), (d * gb).sum(0)
        sq = (na + nb) ** 2
        phi = torch.where(sq > 0, 4 * na * nb / torch.where(sq > 0, sq, 1.0), 0.0).clamp(0.0, 1.0)
        dv = v[:, a] - v[:, b]
        vx = ((dv - 0.5 * phi * (ga + gb)) * d).sum(0)
        r2 = d.square().sum(0)
        Q = 0.0
        for k in (a, b):
            mu = (vx * h[k] / (r2 + 0.01 * h[k] ** 2)).clamp(max=0.0)
            Q = Q + rho[k] * (-ab[0] * cs[k] * mu + ab[1] * mu * mu)
        F = -0.5 * V[a] * V[b] * (P[a] + P[b] + Q) * (gi - gj)
        work_ = -0.5 * (dv * F).sum(0)
        to_a = torch.stack([*(F / m[a]), work_ / m[a]])
        to_b = torch.stack([*(-F / m[b]), work_ / m[b]])
        return rows_sum(n, a, to_a) + rows_sum(n, b, to_b)

    S = over_pairs(force, fi, fj, x, v, h, V, A, B, dA, dB, rho, P, cs, gv, ab)
    return {"h": h, "V": V, "rho": rho, "A": A, "B": B, "gradA": dA, "gradB": dB, "gradv": gv,
            "accel": S[:3], "dudt": S[3]}


def exact_kdk(case, s, ab):
    dt, lam, n_h = STEP["kdk"], 0.5, case["n_h"]
    x, v, m, u, h = (s[k].double() for k in ("x", "v", "m", "u", "h"))
    o = evaluate(case, x, v, m, u, h, ab)
    vh, uh = v + 0.5 * dt * o["accel"], u + 0.5 * dt * o["dudt"]
    div = o["gradv"][0] + o["gradv"][4] + o["gradv"][8]
    delta = n_h * o["V"] ** (1.0 / 3.0) / h
    x = torch.remainder(x + dt * vh, 1.0)
    h = h * torch.exp(lam * (delta - 1.0) + div * dt / 3.0)
    r = evaluate(case, x, vh + 0.5 * dt * o["accel"], m, uh + 0.5 * dt * o["dudt"], h, ab)
    return {**r, "x": x, "v": vh + 0.5 * dt * r["accel"], "u": uh + 0.5 * dt * r["dudt"]}


def exact_hkdk(case, s, ab):
    lam, n_h = 0.5, case["n_h"]
    x, v, m, u, h = (s[k].double() for k in ("x", "v", "m", "u", "h"))
    lev = levels_of(s).long()
    top = int(lev.max())
    nsub = 1 << top
    dt = STEP["hkdk"] / nsub
    per = torch.bitwise_left_shift(torch.ones_like(lev), top - lev)
    span = per * dt
    # (nothing moves by a hundredth of h within the big step)
    pairs = pairs_within(x, 1.05 * h, torch.arange(m.numel(), device=x.device))
    st = evaluate(case, x, v, m, u, h, ab, pairs)
    start = torch.zeros_like(lev)
    vh, uh, hdot = torch.zeros_like(v), torch.zeros_like(u), torch.zeros_like(h)

    def div():
        return st["gradv"][0] + st["gradv"][4] + st["gradv"][8]

    opening = torch.ones_like(lev, dtype=torch.bool)
    for k in range(nsub):
        vh = torch.where(opening, v + 0.5 * span * st["accel"], vh)
        uh = torch.where(opening, u + 0.5 * span * st["dudt"], uh)
        rate = h * lam * (n_h * st["V"] ** (1.0 / 3.0) / h - 1.0) / span + h * div() / 3.0
        hdot = torch.where(opening, rate, hdot)
        start = torch.where(opening, k, start)
        x = torch.remainder(x + dt * (vh + st["accel"] * ((k - start) * dt + 0.5 * (dt - span))), 1.0)
        h = h * torch.exp(hdot * dt / h)
        st["V"], st["rho"] = (h / n_h) ** 3, st["rho"] * torch.exp(-div() * dt)
        active = (k + 1 - start) == per
        t = (k + 1 - start) * dt - 0.5 * span
        o = evaluate(case, x, vh + st["accel"] * t, m, uh + st["dudt"] * t, h, ab,
                     pairs, passive={**st, "mask": ~active})
        v = torch.where(active, vh + 0.5 * span * o["accel"], v)
        u = torch.where(active, uh + 0.5 * span * o["dudt"], u)
        st = {q: torch.where(active, o[q], st[q]) for q in st}
        opening = active
    return {**st, "h": h, "x": x, "v": v, "u": u}


def exact_cool(case, seed):
    s = cool_gas(case, seed)
    lu0, dex, lam = cool_table(case)
    lam = lam.to(DEV)
    K = lam.numel()
    ln_u = (math.log(10.0) * (lu0 + dex * torch.arange(K, device=DEV, dtype=F64)))
    u_k = torch.exp(ln_u)
    width = math.log(10.0) * dex
    zero = int((lam < 0).sum()) - 1  # the bin [zero, zero + 1] holds the sign change
    ueq = u_k[zero] - lam[zero] * (u_k[zero + 1] - u_k[zero]) / (lam[zero + 1] - lam[zero])
    # per bin: (1 - slope) and u / lam at its lower node; int du / |lam| over the bin
    om = 1.0 - torch.log((lam[1:] / lam[:-1]).abs()) / width
    c = u_k[:-1] / lam[:-1].abs()

    def inside(k, t):  # int of du / |lam| over the first t (in ln u) of bin k
        return c[k] * torch.where(om[k] == 0, t, torch.expm1(om[k] * t) / om[k])

    def inverse(k, g):
        y = g / c[k]
        return torch.where(om[k] == 0, y, torch.log1p(om[k] * y) / om[k])

    bins = torch.arange(K - 1, device=DEV)
    cost = inside(bins, torch.full_like(c, width))
    cost[zero] = 0.0
    cool_G = torch.cat([torch.zeros(1, device=DEV, dtype=F64), torch.cumsum(cost, 0)])
    out = torch.empty_like(s["u"], dtype=F64)
    for k0 in range(0, s["u"].numel(), 1 << 22):
        u = s["u"][k0:k0 + (1 << 22)].double().clamp(float(u_k[0]), float(u_k[-1]))
        left = s["rho"][k0:k0 + (1 << 22)].double() * s["dt"]
        t = torch.log(u)
        k = torch.floor((t - ln_u[0]) / width).long().clamp(0, K - 2)
        G = cool_G[k] + inside(k, t - ln_u[k])
        down = k > zero
        # cooling goes down to the upper node of the zero's bin, heating up to its lower node
        goal = torch.where(down, G - left, G + left)
        stop = torch.where(down, cool_G[zero + 1], cool_G[zero])
        over = torch.where(down, stop - goal, goal - stop)
        kk = (torch.searchsorted(cool_G, goal, right=True) - 1).clamp(0, K - 2)
        kk = torch.where(down, kk.clamp(min=zero + 1), kk.clamp(max=zero - 1))
        moved = torch.exp(ln_u[kk] + inverse(kk, goal - cool_G[kk]))
        mag = torch.maximum(lam[zero].abs(), lam[zero + 1].abs())
        edge = torch.where(down, u_k[zero + 1], u_k[zero])
        from_zero = torch.where(k == zero, u, edge)
        rest = torch.where(k == zero, left, over) * mag
        slid = from_zero + (ueq - from_zero).sign() * torch.minimum(rest, (ueq - from_zero).abs())
        out[k0:k0 + (1 << 22)] = torch.where((k == zero) | (over > 0), slid, moved)
    return out


def exact_deposit(case, seed):
    g, s = deposit_sets(case, seed)
    g, s = {k: a.double() for k, a in g.items()}, {k: a.double() for k, a in s.items()}
    kernel, ns, ng = case["kernel"], s["dM"].numel(), g["m"].numel()
    C = norm_of(kernel)
    rows = torch.arange(ns, device=DEV)

    def W(i, j, h):
        r = image(s["x"][:, i] - g["x"][:, j]).square().sum(0).sqrt()
        return torch.where(r < h, C / h ** 3 * shape(kernel, r / h)[0], 0.0)

    i, j = pairs_within(s["x"], g["h"].max().expand(ns), rows, g["x"])
    total = rows_sum(ns, i, W(i, j, g["h"][j])[None])[0]
    V = torch.where(total > 0, (1.0 - C / N_H_SRC ** 3) / total, 0.0)
    h = N_H_SRC * V ** (1.0 / 3.0)
    i, j = pairs_within(s["x"], h, rows, g["x"])
    w = g["V"][j] * W(i, j, h[i])
    total = rows_sum(ns, i, w[None])[0]
    A = torch.where(total > 0, 1.0 / total, 0.0)
    f = A[i] * w
    d = rows_sum(ng, j, torch.stack([f * s["dM"][i], f * s["dMZ"][i], f * s["dE"][i],
                                     *(f * s["dM"][i] * s["v"][:, i])]))
    m = g["m"] + d[0]
    return {"s_V": V, "s_h": h, "s_A": A, "m": m, "mZ": g["mZ"] + d[1],
            "u": (g["m"] * g["u"] + d[2]) / m, "v": (g["m"] * g["v"] + d[3:]) / m}


def exact(case, seed):
    op = case["op"]
    if op == "cool":
        return exact_cool(case, seed)
    if op == "deposit":
        return exact_deposit(case, seed)
    if case["n"] > 70000 if case["set"] == "clumps" else case["n"] * case["n_h"] ** 3 > 5e6:
        return None  # too many pairs for a brute-force search
    s = gas(case, seed)
    ab = torch.tensor([1.0, 2.0], dtype=F64, device=DEV)
    if op in ("kdk", "hkdk"):
        with torch.no_grad():
            return exact_kdk(case, s, ab) if op == "kdk" else exact_hkdk(case, s, ab)
    x, v, m, u, h = (s[k].double() for k in ("x", "v", "m", "u", "h"))
    if op == "eval":
        with torch.no_grad():
            return evaluate(case, x, v, m, u, h, ab)
    for a in (x, v, u, ab):
        a.requires_grad_(True)
    r = evaluate(case, x, v, m, u, h, ab)
    g = torch.autograd.grad((r["accel"], r["dudt"]), (x, v, u, ab), (s["w_a"], s["w_u"]))
    r = {k: a.detach() for k, a in r.items()}
    return {**r, **dict(zip(("g_x", "g_v", "g_u", "g_alpha_beta"), g))}
