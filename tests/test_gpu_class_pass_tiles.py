"""Tiles of the class passes at sizes that always take them (lattices above L = 8
are never kept in LDS).  L = 10 and 14 leave two links over in the last tile of
four: every choice of links per thread gives the same bits, in every order of the
passes and with the restriction per link, and four links per thread agree with the
oracle after a sweep with every class accepted, to the bars of the batched FP64
test (bits equal, energies within 1e-9 relative, angles within 1e-11)."""
import numpy as np
import pytest

import oracle
from tests.inputs import circ_dist, random_state

pytestmark = pytest.mark.gpu

SEED = 1509083910
ORDERS = {"grouped": 0, "interleaved": 1, "staggered": 2}


def _states(L, n, dtype, seed):
    th = np.concatenate([random_state(4, L, 1, seed=seed + k, u_target=0.55 + 0.02 * k, dtype=dtype)
                         for k in range(n)]).astype(np.float64)
    E = np.array([oracle.energy(4, L, t) for t in th])
    o = np.argsort(E)
    return np.ascontiguousarray(th[o]), E[o]


def _context(llr, prec, L, th, E_low, dE, order):
    import torch
    ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64)
    ctx.set_params(seed=SEED)
    ctx.add_lattice(L, E_low, dE)
    ctx.bind_state()
    ctx.set_a(0, np.linspace(0.95, 1.05, len(th)))
    if order in ORDERS:
        ctx.set_sweep_order((llr.SWEEP_GROUPED, llr.SWEEP_INTERLEAVED, llr.SWEEP_STAGGERED)[ORDERS[order]])
    ctx.import_state(0, torch.from_numpy(th.astype(np.float32 if prec == "f32" else np.float64)))
    return ctx


@pytest.mark.parametrize("order", ["grouped", "interleaved", "staggered", "link"])
@pytest.mark.parametrize("L,prec", [(10, "f32"), (10, "f64"), (14, "f32")])
def test_every_tile_gives_the_same_bits(L, prec, order):
    from paper_1509_08391_amd import llr
    n = 3
    th, E = _states(L, n, np.float32 if prec == "f32" else np.float64, 40 * L)
    mode = llr.MODE_LINK if order == "link" else llr.MODE_RESTRICTED
    # windows of half the smallest distance of the states' energies, around each
    dE = 0.5 * float(np.min(np.diff(E)))
    got = []
    for tiles in [(1, 1), (2, 2), (4, 4), (4, 1), (1, 4), None]:
        ctx = _context(llr, prec, L, th, E - 0.5 * dE, dE, order)
        if tiles is None:
            ctx.autotune()
        else:
            ctx.set_tiles(*tiles)
        out = [ctx.sweeps(2, sweep0=3, mode=llr.MODE_FREE if order != "link" else mode), ctx.sweeps(2, sweep0=5, mode=mode)]
        out += [ctx.export_state(0).cpu().numpy(), ctx.get_energy(0)[0], *ctx.stats()[:2], *ctx.link_stats()]
        got.append(out)
        ctx.close()
    for o in got[1:]:
        for x, y in zip(o, got[0]):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("order", ["grouped", "interleaved", "staggered"])
def test_four_links_per_thread_against_the_oracle(order):
    from paper_1509_08391_amd import llr
    L, n = 10, 3
    th, E = _states(L, n, np.float64, 900)
    width = 0.3 * np.sqrt(6 * L ** 4)
    E_low = E - 0.45 * width
    a = np.linspace(0.95, 1.05, n)
    ctx = _context(llr, "f64", L, th, E_low, width, order)
    ctx.set_tiles(4, 4)
    bits = ctx.sweeps(1, sweep0=11, mode=llr.MODE_FREE)
    got, Eg = ctx.export_state(0).cpu().numpy(), ctx.get_energy(0)[0]
    ctx.close()
    ref = th.copy()
    Er, br = oracle.sweeps(4, L, ref, a, E_low, E_low + width, np.arange(n), E, 1, 11,
                           mode=oracle.MODE_FREE, seed=SEED, order=ORDERS[order])
    assert np.array_equal(bits.astype(np.int64), br.astype(np.int64))
    assert np.max(circ_dist(got, ref)) < 1e-11
    assert np.max(np.abs(Eg - Er) / np.abs(Er)) < 1e-9
