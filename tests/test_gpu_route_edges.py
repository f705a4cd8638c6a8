"""Edges of the routes a run can take, each against the class passes one after
another (the route while per-kernel timing is on), all equal bit for bit: halves with four
links per thread, Robbins-Monro iterations longer than one chain-resident launch,
a caller's own stream, and histories longer than one block of device rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context(llr, lats, prec, order, stream=None, replica=False, **params):
    ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64, stream=stream)
    p = dict(n_th=3, n_a=8, n_rm=2, seed=57, recompute_every=4, approach_cap=4000)
    p.update(params)
    ctx.set_params(replica_exchange=replica, **p)
    if order == "link":
        ctx.set_restriction(True)
    else:
        ctx.set_sweep_order({"grouped": llr.SWEEP_GROUPED, "interleaved": llr.SWEEP_INTERLEAVED,
                             "staggered": llr.SWEEP_STAGGERED}[order])
    for L, n in lats:
        v6 = 6 * L ** 4
        lo, hi = (0.5, 0.72) if L <= 8 else (0.58, 0.68)
        dE = (hi - lo) / n * v6
        ctx.add_lattice(L, lo * v6 + dE * np.arange(n), dE)
    ctx.bind_state()
    return ctx


def _results(ctx, lats):
    out = [*ctx.stats(), ctx.health()[1]]
    for i in range(len(lats)):
        out += [ctx.get_a(i)[0], ctx.get_history(i), *ctx.get_energy(i), ctx.export_state(i).cpu().numpy()]
    return out


def _equal(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("order", ["grouped", "interleaved", "staggered"])
@pytest.mark.parametrize("lats,prec", [([(20, 11)], "f32"), ([(14, 33), (10, 30)], "f32"), ([(14, 11)], "f64")])
def test_halves_with_four_links_per_thread(lats, prec, order):
    from paper_1509_08391_amd import llr
    assert sum(n * L ** 4 // 2 for L, n in lats) * (4 if prec == "f64" else 1) >= 760000
    got = []
    for timing in (False, True):
        ctx = _context(llr, lats, prec, order, replica=True)
        ctx.set_tiles(4, 4)
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(timing)
        ctx.run()
        got.append(_results(ctx, lats))
        ctx.close()
    _equal(*got)


@pytest.mark.parametrize("order", ["grouped", "interleaved", "staggered", "link"])
@pytest.mark.parametrize("lats,prec,n_th,n_a", [([(4, 3)], "f64", 70, 80), ([(6, 2), (4, 2)], "f32", 20, 130),
                                                ([(4, 2)], "f32", 64, 64), ([(4, 2)], "f64", 63, 66)])
def test_iterations_longer_than_one_launch(lats, prec, n_th, n_a, order):
    from paper_1509_08391_amd import llr
    got = []
    for timing in (False, True):
        ctx = _context(llr, lats, prec, order, n_th=n_th, n_a=n_a, recompute_every=7)
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(timing)
        ctx.run()
        got.append(_results(ctx, lats))
        ctx.close()
    _equal(*got)


@pytest.mark.parametrize("lats,prec,order", [([(4, 5)], "f64", "grouped"), ([(10, 5)], "f32", "interleaved"),
                                             ([(10, 5)], "f32", "staggered"), ([(14, 44)], "f32", "grouped"),
                                             ([(14, 44)], "f32", "staggered")])
def test_callers_own_stream(lats, prec, order):
    import torch
    from paper_1509_08391_amd import llr
    got = []
    for own in (False, True):
        s = torch.cuda.Stream() if own else None
        ctx = _context(llr, lats, prec, order, stream=s, replica=True)
        ctx.hot_start()
        ctx.approach()
        ctx.run()
        out = [*ctx.observables(2, 2, 60), ctx.sweeps(3, sweep0=70, mode=llr.MODE_FREE)]
        ctx.muca_begin([1.0])
        out.append(ctx.muca_sweeps(6, sweep0=90))
        cen = np.linspace(0.59, 0.67, 40) * 6e4
        a = 1.0 + 1e-3 * np.sin(np.arange(40))
        out += [*ctx.beta_c(cen, a, cen[1] - cen[0], 6e4, 0.98, 1.02), *ctx.reconstruct(cen, a, cen[1] - cen[0], 6e4, [1.0])]
        got.append(out + _results(ctx, lats))
        ctx.close()
    _equal(*got)


def test_histories_of_several_blocks_resident():
    """4 MB of device rows hold 256 sweeps of E, 1024 of accept bits and 128
    measurements of 2048 chains."""
    from paper_1509_08391_amd import llr
    L, n = 2, 2048
    v6 = 6.0 * L ** 4
    got = []
    for timing in (False, True):
        ctx = llr.Context(precision=llr.FP64)
        ctx.set_params(seed=3, recompute_every=50)
        # windows of the whole range: nothing binds, any state lies inside
        ctx.add_lattice(L, -v6 + 1e-3 * np.arange(n), 2 * v6 - 3.0)
        ctx.bind_state()
        ctx.set_a(0, 0.9)
        ctx.hot_start()
        ctx.set_timing(timing)
        out = [ctx.sweeps(1100, sweep0=1, mode=llr.MODE_FREE), *ctx.observables(150, 1, 2000)]
        out += [ctx.export_state(0).cpu().numpy(), ctx.get_energy(0)[0]]
        got.append(out)
        ctx.close()
    assert np.ptp(got[0][1][:, 0]) > 0
    _equal(*got)


@pytest.mark.parametrize("order", ["grouped", "staggered"])
def test_histories_of_several_blocks_in_halves(order):
    """160 chains: 3276 sweeps of E to a block of 4 MB."""
    from paper_1509_08391_amd import llr
    lats = [(10, 160)]
    got = []
    for timing in (False, True):
        ctx = _context(llr, lats, "f32", order, recompute_every=100)
        ctx.hot_start()
        ctx.set_timing(timing)
        ctx.muca_begin([1.0])
        got.append([ctx.muca_sweeps(3300, sweep0=5), ctx.export_state(0).cpu().numpy(), ctx.get_energy(0)[0]])
        ctx.close()
    assert np.ptp(got[0][0][:, 0]) > 0
    _equal(*got)


@pytest.mark.parametrize("n,replica", [(3, True), (130, True), (258, True), (514, False)])
def test_interleaved_l8_on_either_route(n, replica):
    """Kept in LDS (130 chains with exchange), class passes (3, 258) or halves (514)."""
    from paper_1509_08391_amd import llr
    lats = [(8, n)]
    got = []
    for timing in (False, True):
        ctx = _context(llr, lats, "f32", "interleaved", replica=replica)
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(timing)
        ctx.run()
        out = [ctx.sweeps(3, sweep0=50, mode=llr.MODE_FREE)]
        got.append(out + _results(ctx, lats))
        ctx.close()
    _equal(*got)


@pytest.mark.parametrize("lats,prec", [([(4, 3)], "f64"), ([(6, 2), (4, 3)], "f32")])
def test_class_pass_bits_reach_the_next_sweep(lats, prec):
    """A single class pass leaves its accept bit for the next sweep's record, whichever
    route that sweep takes, and for that one only."""
    from paper_1509_08391_amd import llr
    got = []
    for timing in (False, True):
        ctx = _context(llr, lats, prec, "grouped", n_th=1, n_a=2)
        ctx.hot_start()
        ctx.approach()
        ctx.set_timing(timing)
        ctx.enable_bits_log(64)
        out = []
        for colour in (2, 5):
            ctx.class_pass(1, colour, mode=llr.MODE_FREE, sweep_index=900 + colour)
            out.append(ctx.sweeps(3, sweep0=10 * colour))
            ctx.class_pass(1, colour, mode=llr.MODE_FREE, sweep_index=920 + colour)
            ctx.approach_begin()
            out.append(ctx.approach_continue(10)[0])
            out.append(ctx.sweeps(1, sweep0=100, mode=llr.MODE_APPROACH))
        ctx.class_pass(1, 7, mode=llr.MODE_FREE, sweep_index=940)
        ctx.rm_begin()
        ctx.rm_step(1)
        out += [ctx.get_bits_log(), ctx.export_state(0).cpu().numpy(), *ctx.get_energy(0)]
        got.append(out)
        ctx.close()
    assert np.all(got[0][0][0] & 4)
    _equal(*got)
