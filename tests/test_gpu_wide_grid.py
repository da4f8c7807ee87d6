"""Forwards that settle on a wider cell grid than their first.

The roots of a random set's h scatter beyond the candidate radius of the grid
that its first h suggests, so every forward widens the grid. From the third on
it starts on the settled grid; the results have to be those of a new context,
bit for bit, also when the input then changes (h that needs no wider grid,
other positions, a crowded set).
"""
import numpy as np
import pytest

from paper_2511_21921_amd import CUBIC_SPLINE, FP32, FP64, WENDLAND_C4, Context, Params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a HIP device", allow_module_level=True)


def _random(n, precision, spread, seed, clump=0):
    g = np.random.default_rng(seed)
    R = torch.float64 if precision == FP64 else torch.float32
    t = lambda a, dt=R: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda:0")
    x = g.random((3, n))
    x[:, :clump] = 0.95 + 0.1 * x[:, :clump]
    m = 10.0 ** g.uniform(-spread, spread, n) / n
    return (t(x % 1.0, torch.float64), t(0.1 * g.normal(size=(3, n))), t(m),
            t(10.0 ** g.normal(0.0, 0.1, n)))


def _same(a, b):
    for k in ("h", "V", "rho", "A", "B", "gradA", "gradB", "gradv", "accel", "dudt"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("n,kernel,n_h,spread,search", [(1001, CUBIC_SPLINE, 2.4814, 0.3, 0),
                                                        (20000, CUBIC_SPLINE, 2.4814, 0.0, 1),
                                                        (70000, WENDLAND_C4, 3.0, 0.3, 0)])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_settled_wider_grid(n, kernel, n_h, spread, search, precision):
    print("case n=%d precision=%d search=%d" % (n, precision, search), flush=True)
    p = Params(n_h=n_h, kernel=kernel, h_mode=1, precision=precision, search=search)

    def run(ctx, s, h):
        h = torch.full_like(s[2], h) if isinstance(h, float) else h.clone()
        return ctx.forward(s[0], s[1], s[2], s[3], h, stats=True)

    a = _random(n, precision, spread, 1)
    h0 = float(0.8 * n_h * n ** (-1.0 / 3.0))  # (short of every root)
    ctx = Context(p)
    want = run(Context(p), a, h0)
    grids = []
    for _ in range(4):
        got = run(ctx, a, h0)
        grids.append((got["stats"]["grid"], got["stats"]["speculative"]))
        _same(got, want)
    print("  grids %s" % grids, flush=True)
    assert [g[1] for g in grids] == [0, 0, 1, 1] and len({g[0] for g in grids}) == 1
    for s, h in ((a, want["h"]), (a, h0), (_random(n, precision, spread, 2), h0), (a, 2.0 * h0),
                 (_random(n, precision, spread, 3, n // 2), h0), (a, h0)):
        _same(run(ctx, s, h), run(Context(p), s, h))
