"""Reconstruction at the edges of its kernels: terms per lane (16 and 64 lanes),
the largest row held in registers (512 intervals) and the block-wide path beyond
it, the ln rho recursion over several LDS pieces, and many rows at once; against
the oracle with the bars of the existing reconstruction test."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

V6 = 6.0 * 20 ** 4
SIZES = [2, 15, 16, 17, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 700]


def _curve(n, seed):
    dE = 0.064 / n * V6
    c = 0.6 * V6 + dE * (np.arange(n) + 0.5)
    x = (c / V6 - 0.632) / 0.032
    a = 1.010 + 0.002 * (x ** 3 - 0.5 * x) + 1e-5 * np.random.default_rng(seed).normal(size=n)
    return c, a, dE


@pytest.fixture(scope="module")
def ctx():
    from paper_1509_08391_amd import llr
    c = llr.Context(precision=llr.FP64)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1] + SIZES)
def test_moments(ctx, n):
    c, a, dE = _curve(n, n)
    beta = np.linspace(1.008, 1.012, 21)
    lr, u, cv = ctx.reconstruct(c, a, dE, V6, beta)
    lro, uo, cvo = oracle.reconstruct(c, a, dE, V6, beta)
    assert np.max(np.abs(lr - lro)) <= 1e-9 * np.max(np.abs(lro))
    assert np.max(np.abs(u - uo)) < 1e-12
    assert np.max(np.abs(cv - cvo)) <= 1e-9 * np.max(np.abs(cvo))


@pytest.mark.parametrize("n", SIZES)
def test_beta_c(ctx, n):
    c, a, dE = _curve(n, n)
    bc, pk = ctx.beta_c(c, a, dE, V6, 1.008, 1.012)
    bco, pko = oracle.beta_c(c, a, dE, V6, 1.008, 1.012)
    assert abs(bc - bco) < 1e-8
    assert abs(pk - pko) < 1e-9 * pko


@pytest.mark.parametrize("n,n_boot", [(65, 63), (65, 64), (128, 70), (513, 3)])
def test_bootstrap_rows(ctx, n, n_boot):
    runs = np.array([_curve(n, 100 + k)[1] for k in range(3)])
    c, _, dE = _curve(n, 0)
    bc, pk = ctx.bootstrap(c, runs, dE, V6, 1.008, 1.012, n_boot, 5)
    bco, pko = oracle.bootstrap(c, runs, dE, V6, 1.008, 1.012, n_boot, 5)[:2]
    assert np.max(np.abs(bc - bco)) < 1e-8
    assert np.max(np.abs(pk - pko) / pko) < 1e-9


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049])
def test_ln_rho_in_pieces(ctx, n):
    c, a, dE = _curve(n, n)
    lr = ctx.reconstruct(c, a, dE, V6, [])[0]
    lro = oracle.ln_rho(a, dE)
    assert np.max(np.abs(lr - lro)) <= 1e-12 * np.max(np.abs(lro))
