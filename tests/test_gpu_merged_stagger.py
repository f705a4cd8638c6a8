"""Staggered sweeps on one stream (runs too small for two halves beside each
other), where the halves' overrelaxation passes of neighbouring sweeps are one
launch, against the staggered class passes on two streams, which the library runs
while per-kernel timing is on.  The sequence of every chain is the same, so every
result is equal bit for bit: no tolerance.  Odd chain counts, a lattice whose
second half is empty, recomputes inside, at the end and not at the end of a run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(L, n):
    v6 = 6 * L ** 4
    dE = 0.10 / n * v6
    return L, 0.58 * v6 + dE * np.arange(n), dE


@pytest.mark.parametrize("sizes,prec,replica,every", [
    ([(12, 5)], "f32", True, 4),
    ([(10, 3), (14, 1)], "f32", False, 3),
    ([(10, 1)], "f64", False, 100),
    ([(8, 7)], "f64", True, 1),
])
def test_one_stream_equals_two(sizes, prec, replica, every):
    from paper_1509_08391_amd import llr
    lats = [_lattice(L, n) for L, n in sizes]
    got = []
    for two_streams in (False, True):
        ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64, device=0)
        ctx.set_params(n_th=3, n_a=8, n_rm=2, seed=37, replica_exchange=replica, overlap=1.0, recompute_every=every,
                       approach_cap=4000)
        ctx.set_sweep_order(llr.SWEEP_STAGGERED)
        for L, E_low, dE in lats:
            ctx.add_lattice(L, E_low, dE)
        ctx.bind_state()
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(two_streams)
        ctx.enable_bits_log(64)
        ctx.run()
        out = [ctx.get_bits_log()]
        ctx.muca_begin([0.99] * len(lats))
        out += [ctx.muca_sweeps(7, sweep0=1000), ctx.sweeps(5, sweep0=2000, mode=llr.MODE_FREE)]
        out.append(ctx.sweeps(1, sweep0=3000, mode=llr.MODE_FREE))
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
