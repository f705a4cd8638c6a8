"""The losses of a training longer than one block of epochs (256): each epoch's loss
is that of the weights before its step, as a shorter training and the gradient call
compute it, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 600])   # the Adam step inside the next epoch's launch, and in its own
def test_loss_history_over_blocks(n):
    from paper_1509_08391_amd import llr
    rng = np.random.default_rng(n)
    u = rng.uniform(0.55, 0.7, n).astype(np.float32)
    inv_l = (1.0 / rng.choice([8, 12, 16], n)).astype(np.float32)
    a = 1.0 + 0.3 * (u.astype(np.float64) - 0.6) + 0.2 * inv_l
    ctx = llr.Context(precision=llr.FP32)
    w0 = ctx.mlp_init(3)
    kw = dict(lr=1e-3, bf16=True)
    w, hist = ctx.mlp_train(w0, u, inv_l, a, epochs=600, **kw)
    for k in (1, 255, 256, 257, 511, 512, 513, 599):
        wk, hk = ctx.mlp_train(w0, u, inv_l, a, epochs=k, **kw)
        assert np.array_equal(hk, hist[:k])
        assert hist[k] == ctx.mlp_loss_grad(wk, u, inv_l, a, bf16=True)[0]
    ctx.close()
    assert hist[-1] < hist[0]
