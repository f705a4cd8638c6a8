"""Chain-resident sweeps (small lattices, one block per chain in LDS) against
the class-pass kernels, which the library runs while per-kernel timing is on
and which the other GPU tests hold to the oracle.  Both perform the same
operations per link and sum the same integers, so every result is equal bit
for bit: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(L, n):
    v6 = 6 * L ** 4
    lo, hi = {2: (0.1, 0.9), 4: (0.45, 0.75), 6: (0.50, 0.72)}.get(L, (0.55, 0.71))
    dE = (hi - lo) / n * v6
    return L, lo * v6 + dE * np.arange(n), dE


def _context(llr, lats, prec, order, replica, class_passes):
    ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64, device=0)
    ctx.set_params(n_th=3, n_a=9, n_rm=2, seed=77, replica_exchange=replica, overlap=1.0, recompute_every=5,
                   approach_cap=4000)
    if order == "link":
        ctx.set_restriction(True)
    else:
        ctx.set_sweep_order({"grouped": llr.SWEEP_GROUPED, "interleaved": llr.SWEEP_INTERLEAVED,
                             "staggered": llr.SWEEP_STAGGERED}[order])
    for L, E_low, dE in lats:
        ctx.add_lattice(L, E_low, dE)
    ctx.bind_state()
    ctx.set_timing(class_passes)
    ctx.hot_start()
    return ctx


def _state(ctx, n_lat):
    out = [ctx.export_state(i).cpu().numpy() for i in range(n_lat)]
    out += [ctx.get_energy(i)[j] for i in range(n_lat) for j in (0, 1)]
    out += [ctx.get_a(i)[0] for i in range(n_lat)]
    return out + list(ctx.stats()) + [ctx.health()[1], *ctx.link_stats()]


CASES = [  # lattices (L, chains): one link to several per thread, idle lanes, mixed sizes, more chains than CUs
    ([(4, 1)], "f64", "grouped", False),
    ([(4, 5)], "f32", "staggered", True),
    ([(4, 7)], "f64", "interleaved", True),     # four lanes per link
    ([(2, 3), (4, 4)], "f32", "interleaved", False),
    ([(4, 257)], "f32", "grouped", True),
    ([(4, 513)], "f64", "grouped", False),
    ([(6, 3)], "f64", "interleaved", True),
    ([(6, 5), (4, 3)], "f32", "grouped", False),
    ([(8, 3)], "f32", "interleaved", False),
    ([(6, 3), (4, 2)], "f64", "staggered", False),
    ([(8, 3), (6, 2), (4, 2)], "f64", "staggered", False),   # L = 8 in FP64: class passes
    ([(8, 5)], "f64", "grouped", True),
    ([(8, 257)], "f32", "grouped", False),
    ([(8, 257)], "f32", "interleaved", True),
    ([(4, 3)], "f64", "link", True),
    ([(6, 2)], "f64", "link", False),
    ([(8, 3), (4, 2)], "f32", "link", False),
    ([(8, 2)], "f64", "link", False),
]


@pytest.mark.parametrize("sizes,prec,order,replica", CASES)
def test_algorithm1_equals_the_class_passes(sizes, prec, order, replica):
    from paper_1509_08391_amd import llr
    lats = [_lattice(L, n) for L, n in sizes]
    got = []
    for class_passes in (False, True):
        ctx = _context(llr, lats, prec, order, replica, class_passes)
        ctx.enable_bits_log(4096)
        ap = ctx.approach()
        ctx.run()
        bits = ctx.get_bits_log()
        got.append([ap, bits, *ctx.observables(3, 2, 500)] + _state(ctx, len(lats)))
        ctx.close()
    assert got[0][1].any()
    for x, y in zip(*got):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("L,n,prec", [(2, 3, "f32"), (2, 2, "f64"), (4, 2, "f32"), (6, 2, "f64"), (8, 2, "f32")])
def test_free_and_multicanonical_sweeps_equal_the_class_passes(L, n, prec):
    from paper_1509_08391_amd import llr
    lats = [_lattice(L, n)]
    got = []
    for class_passes in (False, True):
        ctx = _context(llr, lats, prec, "grouped", False, class_passes)
        bits = ctx.sweeps(70, sweep0=3, mode=llr.MODE_FREE)      # more than one launch's sweeps
        ctx.muca_begin([0.9])
        E = ctx.muca_sweeps(66, sweep0=100)
        got.append([bits, E] + _state(ctx, 1))
        ctx.close()
    for x, y in zip(*got):
        assert np.array_equal(x, y)
