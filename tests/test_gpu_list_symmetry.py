"""The neighbour lists are symmetric: r_ij is the same number from both sides, so
that j gathers i exactly when r_ij < h_j whichever of the two asks, and every
force pair is on both particles' lists. Counted over all particles such pairs
are then even in number, on the cell list and on the tree.

The sets are lattices whose sites are moved by a few units in the last place of
the distances, with h at the distance of a shell of neighbours (24 of sqrt 6
spacings, or others), so that tens of thousands of pairs lie within a rounding of
h: one that is decided differently from its two sides leaves an odd count in
half of the draws.
"""
import dataclasses

import numpy as np
import pytest

import synth
from paper_2511_21921_amd import FP32, FP64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a HIP device", allow_module_level=True)

from tests import _gpu  # noqa: E402

SIDE = 28  # (not a power of two: the offsets from the cells' centres are rounded)


def _shell(shell, seed, precision):
    """SIDE^3 sites moved by a few roundings of r = sqrt(shell) spacings, h = r."""
    rng = np.random.default_rng(seed)
    h = np.sqrt(shell) / SIDE
    a = 4.0 * np.spacing(np.float32(h) if precision == FP32 else h)
    site = np.stack(np.meshgrid(*[np.arange(SIDE)] * 3, indexing="ij")).reshape(3, -1)
    ps = synth.random_small(SIDE ** 3, seed, mass_spread=0.1)
    x = (site + 0.37) / SIDE + rng.uniform(-a, a, size=site.shape)
    return dataclasses.replace(ps, x=x % 1.0, h=np.full(ps.n, h), h_mode=0)


@pytest.mark.parametrize("search", [1, 2])
@pytest.mark.parametrize("precision", [FP32, FP64])
def test_pairs_at_the_edge_of_h_are_on_both_lists(search, precision):
    odd = []
    for seed in range(12):
        shell = (5, 6, 9)[seed % 3]
        ps = _shell(shell, 500 + seed, precision)
        print("case shell=%d seed=%d search=%d precision=%d" % (shell, seed, search, precision),
              flush=True)
        s = _gpu.run(ps, precision, search=search)[0]["stats"]
        print("  gather %d force %d" % (s["n_pairs_gather"], s["n_pairs_force"]), flush=True)
        assert s["n_pairs_force"] == s["n_pairs_gather"]  # (one h: no scatter-only entry)
        odd.append(s["n_pairs_gather"] % 2)
    assert not any(odd), odd


@pytest.mark.parametrize("search", [1, 2])
@pytest.mark.parametrize("precision", [FP32, FP64])
def test_force_pairs_of_solved_h_are_on_both_lists(search, precision):
    for seed in range(4):
        ps = synth.random_small(30000, 520 + seed, mass_spread=0.1)
        print("case random30000 seed=%d search=%d precision=%d" % (seed, search, precision),
              flush=True)
        s = _gpu.run(ps, precision, search=search)[0]["stats"]
        assert s["n_pairs_force"] > s["n_pairs_gather"]
        assert s["n_pairs_force"] % 2 == 0, s
