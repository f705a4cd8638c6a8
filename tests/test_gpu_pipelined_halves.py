"""Sweeps with the chains in two halves on two streams (large runs) against the class passes one after another, which the library
runs while per-kernel timing is on.  The sequence of every chain is the same, so
every result is equal bit for bit: no tolerance.  The sizes lie just above the
rule's 760 000 class links (FP64 ones count four times), with odd numbers of chains,
a lattice of a single chain, and recomputes inside and at the end of the run;
the last three have halves just above the 240 MB from which they run in parts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(L, n):
    v6 = 6 * L ** 4
    dE = 0.10 / n * v6
    return L, 0.58 * v6 + dE * np.arange(n), dE


CASES = [
    ([(16, 25)], "f32", "grouped", True),
    ([(16, 25)], "f32", "staggered", True),
    ([(14, 17), (16, 1), (12, 39)], "f32", "grouped", False),
    ([(14, 11)], "f64", "grouped", True),
    ([(10, 39)], "f64", "staggered", False),
    ([(14, 17), (16, 1), (12, 39)], "f32", "interleaved", True),
    ([(14, 11)], "f64", "interleaved", False),
    ([(20, 93), (14, 3)], "f32", "interleaved", True),
    ([(20, 93), (14, 3)], "f32", "grouped", True),
    ([(20, 48)], "f64", "staggered", True),
]


@pytest.mark.parametrize("sizes,prec,order,replica", CASES)
def test_halves_equal_the_class_passes(sizes, prec, order, replica):
    from paper_1509_08391_amd import llr
    lats = [_lattice(L, n) for L, n in sizes]
    assert sum(n * L ** 4 // 2 for L, n in sizes) * (4 if prec == "f64" else 1) >= 760000
    got = []
    for class_passes in (False, True):
        ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64, device=0)
        ctx.set_params(n_th=3, n_a=8, n_rm=2, seed=91, replica_exchange=replica, overlap=1.0, recompute_every=4,
                       approach_cap=4000)
        ctx.set_sweep_order({"grouped": llr.SWEEP_GROUPED, "interleaved": llr.SWEEP_INTERLEAVED,
                             "staggered": llr.SWEEP_STAGGERED}[order])
        for L, E_low, dE in lats:
            ctx.add_lattice(L, E_low, dE)
        ctx.bind_state()
        ctx.set_tiles(2, 2)
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(class_passes)
        ctx.enable_bits_log(64)
        ctx.run()
        out = [ctx.get_bits_log()]
        ctx.muca_begin([0.99] * len(lats))
        out += [ctx.muca_sweeps(9, sweep0=1000), ctx.sweeps(5, sweep0=2000, mode=llr.MODE_FREE)]
        for i in range(len(lats)):
            out += [ctx.get_a(i)[0], *ctx.get_energy(i), ctx.export_state(i).cpu().numpy()]
        out += [*ctx.stats(), ctx.health()[1]]
        rates = ctx.rates()
        out.append(np.array([rates["sweeps"], rates["or_class_passes"], rates["link_updates"]]))
        got.append(out)
        ctx.close()
    assert got[0][0].any()
    for x, y in zip(*got):
        assert np.array_equal(x, y)
