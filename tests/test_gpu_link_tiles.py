"""The walk of the per-link restriction over more than one LDS tile of 2048 class
links: L = 10 has 5000 (two full tiles and one of 904), windows so narrow that the
arc sampler draws links in every tile.  One class pass from the imported state
against the oracle's.

FP64: the running energies of the two sides differ by the rounding of 5000 sums
near 3.3e4, at most 5000 x 1.8e-12 = 9e-9, far below every decision's margin (asserted: 1e-7).
Links drawn by the sampler see staples and random numbers only: within 1e-11, ten
times the whole sweep's bar, as moduli R of a few hundredths divide the ulp-level
differences of sine, cosine and arctangent.  The arc sampler starts at
x_a = acos((hi - E + ...) / R), whose slope 1 / (R sin x_a) carries the energies'
difference into the angle: 1e-6 leaves it a slope of 100.

FP32: the bars of the existing class-pass test (median 1e-6, largest 1e-3, energy
1e-3), on the chains and sweep indices whose decisions in the oracle's walk all
have a margin of 1e-4."""
import numpy as np
import pytest

import oracle
from tests.inputs import circ_dist
from tests.test_gpu_link import SEED, _ctx, _states

pytestmark = pytest.mark.gpu

L, N, DE = 10, 8, 16.0
TILES = [(0, 2048), (2048, 4096), (4096, 5000)]


@pytest.mark.parametrize("colour", [0, 5])
def test_class_pass_fp64(colour):
    from paper_1509_08391_amd import llr
    th, E = _states(L, N, 1300)
    a = 0.98 + 0.005 * np.arange(N)
    ctx = _ctx(llr, llr.FP64, L, th, E - 0.5 * DE, DE, a)
    E0 = ctx.get_energy(0)[0]
    ctx.class_pass(1, colour, mode=llr.MODE_LINK, sweep_index=11)
    got, Eg = ctx.export_state(0).cpu().numpy(), ctx.get_energy(0)[0]
    fixes, arcs = ctx.link_stats()
    ctx.close()
    par = np.array([sum((s // L ** m) % L for m in range(4)) % 2 for s in range(L ** 4)])
    mine = np.nonzero(par == (colour & 1))[0]   # the class's sites in half-index order
    for k in range(N):
        t = th[k].copy()
        Eo, mg, how = oracle.link_pass(4, L, t, colour, a[k], E[k] - 0.5 * DE, E[k] + 0.5 * DE, E0[k], SEED, sweep=11,
                                       interval=k)
        assert np.all(how > 0) and mg.min() > 1e-7
        assert all((how[lo:hi] == 2).any() for lo, hi in TILES)
        assert arcs[k] == (how == 2).sum() and fixes[k] >= arcs[k]
        dist = circ_dist(got[k], t)
        cls = dist[colour >> 1, mine]
        assert np.max(cls[how == 1]) < 1e-11 and np.max(cls[how == 2]) < 1e-6, (k, np.max(cls[how == 1]), np.max(cls))
        dist[colour >> 1, mine] = 0.0
        assert not dist.any()                   # no other link is touched
        assert abs(Eg[k] - Eo) < 1e-7, (k, Eg[k] - Eo)


@pytest.mark.parametrize("colour,sweep,k", [(0, 15, 4), (0, 35, 4), (0, 47, 6), (0, 50, 3), (5, 54, 6)])
def test_class_pass_fp32(colour, sweep, k):
    from paper_1509_08391_amd import llr
    th, E = _states(L, N, 1300, np.float32)
    ctx = _ctx(llr, llr.FP32, L, th, E - 0.5 * DE, DE, np.full(N, 1.0))
    ctx.class_pass(1, colour, mode=llr.MODE_LINK, sweep_index=sweep)
    got, Eg = ctx.export_state(0).cpu().numpy().astype(np.float64), ctx.get_energy(0)[0]
    ctx.close()
    t = th[k].copy()
    Eo, mg, how = oracle.link_pass(4, L, t, colour, 1.0, E[k] - 0.5 * DE, E[k] + 0.5 * DE, E[k], SEED, sweep=sweep,
                                   interval=k, f32=True)
    assert np.all(how > 0) and mg.min() >= 1e-4
    assert all((how[lo:hi] == 2).any() for lo, hi in TILES)
    dist = circ_dist(got[k], t)
    assert np.median(dist) < 1e-6 and np.max(dist) < 1e-3, np.max(dist)
    assert abs(Eg[k] - Eo) < 1e-3
