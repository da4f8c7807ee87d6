"""The sorted records of large sets: from 65,536 particles on, outputs and
gradients are kept by sorted slot and fetched by the caller's index, through
the inverse permutation that every forward of that size writes."""
import dataclasses

import numpy as np
import pytest

from paper_2511_21921_amd import FP32, FP64, Context, Params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from tests import _gpu  # noqa: E402
from tests.test_gpu_pairs import _set  # noqa: E402


@pytest.mark.parametrize("search", [1, 2])
@pytest.mark.parametrize("own_forward", [True, False])
def test_gradient_after_a_big_step_of_level_zero(own_forward, search):
    """A big step with every level 0 moves most particles to other cells; the
    gradient after it is that after the same single-level step (the two states
    agree to 1e-11, measured 1e-14; without viscosity the gradient is smooth, and
    1e-9 of its norm leaves a factor 100). The state before the step comes from
    the context's own forward, or from another context's."""
    n, dt, lam = 70001, 2e-4, 0.5
    print("case n=%d own_forward=%d search=%d" % (n, own_forward, search), flush=True)
    ps = _set(n, 0.1)
    # a common velocity: every particle moves by (0.03, 0.018, 0.012) of the box
    ps = dataclasses.replace(ps, h_mode=0, v=ps.v + np.array([[150.0], [90.0], [60.0]]))
    p = _gpu.params_for(ps, FP64, search=search, alpha=0.0, beta=0.0)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_gpu.DEV)

    def grads(step, first):
        ctx = Context(p)
        x, v, m, u, h = _gpu.to_dev(ps, FP64)
        out = (first or ctx).forward(x, v, m, u, h)
        step(ctx, x, v, m, u, out)
        torch.cuda.synchronize()
        g = ctx.backward(t(ps.w_a), t(ps.w_u))
        return x.cpu().numpy(), {k: a.cpu().numpy() for k, a in g.items()}

    x0, want = grads(lambda c, x, v, m, u, out: c.kdk_step(x, v, m, u, out, dt, lam), None)
    assert np.mean(np.any(np.floor(x0 * 40) != np.floor(ps.x * 40), axis=0)) > 0.5
    levels = torch.zeros(n, dtype=torch.int32, device=_gpu.DEV)
    _, got = grads(lambda c, x, v, m, u, out: c.hkdk_step(x, v, m, u, out, levels, dt, lam),
                   None if own_forward else Context(p))
    for k in ("g_x", "g_v", "g_u"):
        e = _gpu.rel_l2(got[k], want[k])
        print("  %s: %.2e" % (k, e), flush=True)
        assert e <= 1e-9, k


@pytest.mark.parametrize("precision", [FP32, FP64])
def test_records_take_no_memory_of_their_own(precision):
    """Workspace of a context for 4,194,304 particles. Per particle, with R bytes a
    Real and the first capacities: keys and indices 20 and the sort's histogram 1,
    position and velocity 8 R, m, u, h and V 4 R, state and correction records 32 R,
    counts and cells 16, lists 4 (128 + 32), candidates 192 (4 + R). The 17 blocks
    are rounded up to 2 MiB at most, another 9 bytes a particle; the output records
    (16 R + 32 bytes) would come on top."""
    n, R = 1 << 22, 8 if precision == FP64 else 4
    print("case reserve n=%d precision=%d" % (n, precision), flush=True)
    ctx = Context(Params(precision=precision))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx.reserve(n)
    got = (before - torch.cuda.mem_get_info()[0]) / n
    want = 21 + 44 * R + 16 + 4 * 160 + 192 * (4 + R)
    print("  %.1f bytes a particle, %d by the list" % (got, want), flush=True)
    assert got <= want + 9 + 2


@pytest.mark.parametrize("precision", [FP64, FP32])
def test_noalloc_adjoint_of_its_largest_set(precision):
    """65,536 particles: the one size whose gradients go through the records inside
    the static workspace. The same kernels on the same state: equal bits."""
    ps = _set(65536, 0.1)
    print("case noalloc n=%d precision=%d" % (ps.n, precision), flush=True)
    _, ctx = _gpu.run(ps, precision)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_gpu.DEV)
    wa, wu = t(ps.w_a), t(ps.w_u)
    a = ctx.backward(wa, wu, noalloc=True)
    b = ctx.backward(wa, wu)
    for k in a:
        assert bool(torch.isfinite(a[k]).all()) and torch.equal(a[k], b[k]), k
