"""Infinite inputs the analysis and training calls accept: the values that do not
depend on the infinity stay what they are in 64 bits, at sizes on both sides of the
kernels' blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OW2, OW3 = 192, 4352   # offsets of W2[64][64] and W3[64] in the parameter vector


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [1, 63, 64, 65])
def test_gradient_with_an_infinite_weight(n, bf16):
    """W2[3][5] = inf saturates hidden unit 3 at h = sign(h1_5), so dL/dW3[3] is the
    sum of dy h over the samples.  FP32 products and sums of n terms: 1e-6 of the
    terms' sum (a rounding each of 6e-8, n <= 65 added in sequence, of random sign)."""
    from paper_1509_08391_amd import llr
    ctx = llr.Context(precision=llr.FP32)
    rng = np.random.default_rng(n)
    u = rng.uniform(0.55, 0.7, n).astype(np.float32)
    inv_l = np.full(n, 1.0 / 12, dtype=np.float32)
    a = 1.2 + 0.1 * rng.normal(size=n)
    w = ctx.mlp_init(5)
    w[OW2 + 64 * 3 + 5] = np.inf
    loss, g = ctx.mlp_loss_grad(w, u, inv_l, a, bf16=bf16)
    pred = ctx.mlp_predict(w, u, inv_l, bf16=bf16)
    ctx.close()
    x0, x1 = (u.astype(np.float64) - 0.6) / 0.1, (inv_l.astype(np.float64) - 0.0875) / 0.0375
    h1 = np.tanh(float(w[10]) * x0 + float(w[11]) * x1)       # W1[5], b1 = 0
    assert np.all(np.abs(h1) > 1e-5)                            # of one sign in either precision
    terms = 0.2 * (pred - a) / n * np.sign(h1)
    assert np.isfinite(loss)
    assert abs(g[OW3 + 3] - terms.sum()) < 1e-6 * np.abs(terms).sum()


@pytest.mark.parametrize("n", [1, 5, 16, 512, 513, 1100])
def test_ln_rho_with_an_infinite_width(n):
    """ln rho of the first interval is 0 by definition, whatever the width; the others
    then lie infinitely below it, and every moment is the first interval's."""
    from paper_1509_08391_amd import llr
    ctx = llr.Context(precision=llr.FP64)
    c = 0.6 + 0.01 * np.arange(n)
    lr, u, cv = ctx.reconstruct(c, np.full(n, 1.01), np.inf, 1.0, [1.0])
    ctx.close()
    assert lr[0] == 0.0 and np.all(lr[1:] == -np.inf)
    assert u[0] == c[0] and cv[0] == 0.0
