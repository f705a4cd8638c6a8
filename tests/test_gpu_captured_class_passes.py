"""Captured sweeps at a size that runs them: L = 10 with a few chains is neither
kept in LDS nor large enough for two halves, so its grouped and interleaved sweeps
are class passes replayed from HIP graphs.  Replays over several Robbins-Monro
iterations, with the host's reads in between, against direct launches, and a
switch of the order or of the restriction between iterations: the same launches,
so every result is equal bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L, N = 10, 5


def _context(prec, replica, graphs, n_rm=4):
    from paper_1509_08391_amd import llr
    v6 = 6 * L ** 4
    dE = 0.02 * v6
    ctx = llr.Context(precision=llr.FP32 if prec == "f32" else llr.FP64)
    ctx.set_params(n_th=2, n_a=5, n_rm=n_rm, seed=23, replica_exchange=replica, recompute_every=3, approach_cap=4000)
    ctx.add_lattice(L, 0.6 * v6 + dE * np.arange(N), dE)
    ctx.bind_state()
    ctx.set_a(0, 1.0)
    ctx.set_graphs(graphs)
    ctx.hot_start()
    ctx.approach()
    ctx.set_tiles(4, 2)
    ctx.enable_bits_log(64)
    return ctx


def _results(ctx):
    return [ctx.get_history(0), ctx.get_bits_log(), ctx.export_state(0).cpu().numpy(), *ctx.get_energy(0), *ctx.stats()]


@pytest.mark.parametrize("replica", [False, True])
@pytest.mark.parametrize("order", ["grouped", "interleaved"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_replays_equal_direct_launches(prec, order, replica):
    from paper_1509_08391_amd import llr
    got = []
    for graphs in (True, False):
        ctx = _context(prec, replica, graphs)
        ctx.set_sweep_order({"grouped": llr.SWEEP_GROUPED, "interleaved": llr.SWEEP_INTERLEAVED}[order])
        ctx.rm_begin()
        E = []
        for _ in range(4):
            ctx.rm_step(1)
            E.append(ctx.get_energy(0)[0])
            ctx.recompute_energy()
        got.append([np.array(E)] + _results(ctx))
        ctx.close()
    assert got[0][2].any()
    for x, y in zip(*got):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("switch", ["order", "restriction"])
def test_switch_between_iterations(switch, prec):
    from paper_1509_08391_amd import llr
    got = []
    for graphs in (True, False):
        ctx = _context(prec, True, graphs)
        ctx.rm_begin()
        ctx.rm_step(1)
        for on in (True, False, True):
            if switch == "order":
                ctx.set_sweep_order(llr.SWEEP_INTERLEAVED if on else llr.SWEEP_GROUPED)
            else:
                ctx.set_restriction(on)
            ctx.rm_step(1)
        got.append(_results(ctx))
        ctx.close()
    for x, y in zip(*got):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("order", ["grouped", "interleaved", "staggered"])
def test_short_iterations_of_a_large_run(order):
    """Two sweeps an iteration: too short for halves, so captured whole; the staggered
    order's graph holds both streams' launches and their fork and join."""
    from paper_1509_08391_amd import llr
    L, n = 14, 40
    v6 = 6 * L ** 4
    dE = 0.1 / n * v6
    got = []
    for graphs in (True, False):
        ctx = llr.Context(precision=llr.FP32)
        ctx.set_params(n_th=1, n_a=1, n_rm=5, seed=29, replica_exchange=True, recompute_every=3, approach_cap=4000)
        ctx.set_sweep_order({"grouped": llr.SWEEP_GROUPED, "interleaved": llr.SWEEP_INTERLEAVED,
                             "staggered": llr.SWEEP_STAGGERED}[order])
        ctx.add_lattice(L, 0.58 * v6 + dE * np.arange(n), dE)
        ctx.bind_state()
        ctx.set_a(0, 1.0)
        ctx.set_graphs(graphs)
        ctx.hot_start()
        ctx.approach()
        ctx.set_tiles(2, 2)
        ctx.enable_bits_log(32)
        ctx.rm_begin()
        E = []
        for _ in range(5):
            ctx.rm_step(1)
            E.append(ctx.get_energy(0)[0])
            ctx.recompute_energy()
        out = [np.array(E), ctx.sweeps(2, sweep0=40, mode=llr.MODE_FREE)]
        got.append(out + _results(ctx))
        ctx.close()
    for x, y in zip(*got):
        assert np.array_equal(x, y)
