"""The pair passes on either side of their choice of lanes per particle.

Up to 16,384 particles a pass gives each particle 16 lanes, beyond that 4: a
set at each side of that line and two small ones (fewer particles than a block
takes; a ragged last wave), on the cell list and on the tree, equal and unequal
masses, against the FP64 oracle; and at each side of 65,536, from where on the
outputs and gradients go through records in sorted order. The sets are jittered lattices with sites left
out, ~64 neighbours: second moments stay well conditioned, so every output's
relative L2 error is held to the forward's bounds, 1e-11 in FP64 and 2e-5 in
FP32 (accel and du/dt 1e-5). The gradient g along a normal direction d is held
to |g.d - jvp| <= 1e-9 |g| in FP64 and 1e-5 |g| in FP32: an error dg of the
gradient gives a difference of standard deviation |dg|, so 1e-5 is five sigma
of a relative L2 error of 2e-6 (|jvp| itself, a sum of 49,000 terms of either
sign, may be small by chance). The FP32 gradient is taken without viscosity:
among 600,000 pairs one or two lie within FP32 rounding of the limiter's clamp
or of the switch of mu, where the gradient jumps.
"""
import dataclasses
import math

import numpy as np
import pytest

import oracle
import synth
from paper_2511_21921_amd import FP32, FP64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from tests import _gpu  # noqa: E402
from tests.test_gpu_backward import _directions  # noqa: E402


def _set(n, spread):
    """n sites of a jittered lattice, u near 1, masses spread by 10^U(-spread, spread)."""
    ps = synth.sedov(math.ceil(round(n ** (1 / 3), 6)), k=4, with_velocity=True)
    rng = np.random.default_rng(n)
    pick = np.sort(rng.choice(ps.n, n, replace=False))
    m = 10.0 ** rng.uniform(-spread, spread, n) / n
    return dataclasses.replace(ps, x=ps.x[:, pick], v=ps.v[:, pick], m=m,
                               u=10.0 ** rng.normal(0.0, 0.1, n), h=ps.h[pick],
                               w_a=ps.w_a[:, pick], w_u=ps.w_u[pick])


@pytest.mark.parametrize("n,search,spread", [(343, 1, 0.0), (1003, 2, 0.1), (16384, 1, 0.1),
                                             (16384, 2, 0.0), (16385, 1, 0.0), (16385, 2, 0.1),
                                             (65535, 1, 0.0), (65536, 1, 0.1), (65536, 2, 0.0)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_lanes_per_particle(n, search, spread, precision):
    print("case n=%d search=%d spread=%g precision=%d" % (n, search, spread, precision),
          flush=True)
    ps = _set(n, spread)
    visc = {} if precision == FP64 else {"alpha": 0.0, "beta": 0.0}
    g, ctx = _gpu.run(ps, precision, search=search)
    o = oracle.forward(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps), nbr_mode=0 if n < 2000 else 1)
    e = {k: _gpu.rel_l2(g[k], o[k]) for k in ("h", "V", "rho", "A", "B", "gradA", "gradB", "gradv",
                                              "accel", "dudt")}
    print({k: "%.2e" % v for k, v in e.items()}, flush=True)
    for k, v in e.items():
        assert v <= (1e-11 if precision == FP64 else 1e-5 if k in ("accel", "dudt") else 2e-5), k
    _, ctx = _gpu.run(ps, precision, search=search, **visc)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_gpu.DEV)
    g = {k: a.cpu().numpy() for k, a in ctx.backward(t(ps.w_a), t(ps.w_u)).items()}
    for name, dx, dv, du, da, db in _directions(ps):
        j = oracle.jvp(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps, **visc), dx, dv, du, da, db,
                       nbr_mode=0 if n < 2000 else 1)
        jl = float((ps.w_a * j["d_accel"]).sum() + (ps.w_u * j["d_dudt"]).sum())
        gl = float((g["g_x"] * dx).sum() + (g["g_v"] * dv).sum() + (g["g_u"] * du).sum() +
                   g["g_alpha_beta"][0] * da + g["g_alpha_beta"][1] * db)
        norm = {"x": np.linalg.norm(g["g_x"]), "v": np.linalg.norm(g["g_v"]),
                "u": np.linalg.norm(g["g_u"] * ps.u), "ab": np.linalg.norm(g["g_alpha_beta"])}[name]
        print("  %s: %.2e of |g|" % (name, abs(gl - jl) / norm), flush=True)
        assert abs(gl - jl) <= (1e-9 if precision == FP64 else 1e-5) * norm, name


@pytest.mark.parametrize("n,n_h,spread", [(32768, None, 0.0), (32769, None, 0.1), (65536, None, 0.1),
                                          (65537, None, 0.0), (131072, None, 0.1),
                                          (131073, None, 0.0), (131073, 3.25, 0.1)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_lanes_of_the_search(n, n_h, spread, precision):
    """Either side of the sizes where the passes over the candidates leave the
    16-lane rows, and larger sets (n_h 3.25: ~140 neighbours)."""
    print("case n=%d n_h=%s spread=%g precision=%d" % (n, n_h, spread, precision), flush=True)
    ps = _set(n, spread)
    more = {} if n_h is None else {"n_h": n_h}
    if n_h is not None:
        ps = dataclasses.replace(ps, h=ps.h * (n_h / oracle.params_for(ps).n_h))
    g, _ = _gpu.run(ps, precision, search=1, **more)
    o = oracle.forward(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps, **more), nbr_mode=1)
    for k in ("h", "V", "rho", "accel", "dudt"):
        e = _gpu.rel_l2(g[k], o[k])
        print("  %s: %.2e" % (k, e), flush=True)
        assert e <= (1e-11 if precision == FP64 else 1e-5 if k in ("accel", "dudt") else 2e-5), k


@pytest.mark.parametrize("n,wide", [(700, 0), (5000, 0), (65536, 0), (65537, 0), (80000, 9)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_tree_walks(n, wide, precision):
    """The tree's walk from its lowest levels (700: the leaves; 5000: the level
    above), with a wave per particle (65,536) and per four of them (65,537, a
    last wave with one), and depth first (fixed h of 0.45 boxes for 9 of 80,000
    particles: their spheres reach more than 64 nodes of a level)."""
    print("case n=%d wide=%d precision=%d" % (n, wide, precision), flush=True)
    ps = _set(n, 0.1)
    more = {}
    if wide:
        h = ps.h.copy()
        h[:: n // wide][:wide] = 0.45
        ps = dataclasses.replace(ps, h=h)
        more = {"h_mode": 0}
    g, _ = _gpu.run(ps, precision, search=2, **more)
    o = oracle.forward(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps, **more),
                       nbr_mode=0 if n < 2000 else 1)
    for k in ("h", "V", "rho") + (("accel", "dudt") if precision == FP64 or not wide else ()):
        e = _gpu.rel_l2(g[k], o[k])
        print("  %s: %.2e" % (k, e), flush=True)
        assert e <= (1e-11 if precision == FP64 else 1e-5 if k in ("accel", "dudt") else 2e-5), k


@pytest.mark.parametrize("n,scale,bits", [(110592, 1.0, 16), (200003, 1.0, 17), (300000, 0.75, 19)])
def test_sort_digits(n, scale, bits):
    """Cell lists whose keys take the sort two passes of 8, 9 and 10 bits, with
    a ragged last block and empty cells (fixed h, `scale` times the set's)."""
    print("case n=%d bits=%d" % (n, bits), flush=True)
    ps = _set(n, 0.1)
    ps = dataclasses.replace(ps, h=ps.h * scale)
    g, _ = _gpu.run(ps, FP64, search=1, h_mode=0)
    grid = g["stats"]["grid"]
    print("  grid %d" % grid, flush=True)
    assert math.ceil(math.log2(grid ** 3)) == bits
    o = oracle.forward(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps, h_mode=0), nbr_mode=1)
    assert g["stats"]["n_pairs_gather"] == o["pairs_gather"]
    for k in ("V", "rho", "accel", "dudt"):
        e = _gpu.rel_l2(g[k], o[k])
        print("  %s: %.2e" % (k, e), flush=True)
        assert e <= 1e-11, k


@pytest.mark.parametrize("n,n_h,clump", [(64, 1.5, 0), (125, 2.2, 0), (512, 3.0, 0), (3000, 2.4814, 1800)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_candidate_runs(n, n_h, clump, precision):
    """Cell runs that wrap once and twice (grids of a few cells), and more than
    2048 particles within a stencil (`clump` of them in a tenth of the box)."""
    print("case n=%d n_h=%g clump=%d precision=%d" % (n, n_h, clump, precision), flush=True)
    ps = _set(n, 0.1)
    x = ps.x.copy()
    x[:, :clump] = 0.95 + 0.1 * x[:, :clump]
    ps = dataclasses.replace(ps, x=x % 1.0, h=ps.h * (n_h / ps.n_h))
    g, _ = _gpu.run(ps, precision, search=1, h_mode=0)
    print("  grid %d candidates %d" % (g["stats"]["grid"], g["stats"]["n_candidates"]), flush=True)
    o = oracle.forward(ps.x, ps.v, ps.m, ps.u, ps.h, oracle.params_for(ps, h_mode=0))
    if precision == FP64:  # (a pair within FP32 rounding of h counts either way)
        assert g["stats"]["n_pairs_gather"] == o["pairs_gather"]
    for k in ("V", "rho"):
        e = _gpu.rel_l2(g[k], o[k])
        print("  %s: %.2e" % (k, e), flush=True)
        assert e <= (1e-11 if precision == FP64 else 2e-5), k
