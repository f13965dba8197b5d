"""Gradients of the proposal network against the oracle network at the edges of
the grouped products: one row and one unit, rows and widths that are not multiples
of four (element-wise operand reads) or of a tile, batches on both sides of the
fused forward pass (256 rows), a last product split over K (the loss in a kernel of
its own), products with one split and with several; and a training step's parameters
from the same gradients."""
import numpy as np
import pytest

from oracle import mlp as OM
from paper_1808_00128_amd import workloads as W
from test_gpu_learned import B, host_ctx, say, varied_params  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,H,batch", [(1, 16, 1), (3, 16, 33), (52, 256, 256), (50, 256, 257), (7, 48, 511),
                                       (50, 512, 300), (64, 1024, 70), (33, 128, 2050), (12, 272, 1021)])
def test_gradients_and_step(B, n, H, batch):  # noqa: F811
    say(f"mlp gradients n={n} H={H} batch={batch}")
    ctx = host_ctx(B)
    p = varied_params(n, H, seed=40 + n)
    net = B.MLP(ctx, n, H, batch, p)
    ref = OM.MLPRef(p, n, H)
    rng = np.random.default_rng(41)
    x = W.random_bitstrings(n, batch, rng)
    t = W.random_bitstrings(n, batch, rng) & W.random_bitstrings(n, batch, rng)
    eloss, eg = ref.loss_and_grad(x, t)
    for _ in range(2):
        loss, g = net.loss_grad(x, t)
        assert abs(loss - eloss) <= 1e-5 * abs(eloss)
        for k in OM.PARAM_ORDER:
            a, e = np.asarray(g[k], np.float64), np.asarray(eg[k], np.float64)
            assert np.linalg.norm(a - e) <= 3e-3 * np.linalg.norm(e) + 1e-9, k
    assert all(np.array_equal(net.params()[k], p[k]) for k in OM.PARAM_ORDER)  # gradients alone move nothing
    tl = net.train(x, t, batch=batch, epochs=1, lr=1e-3)
    assert abs(tl[0] - eloss) <= 1e-5 * abs(eloss)
    got = net.params()
    for k in OM.PARAM_ORDER:  # the first Adam step: lr g / (|g| + eps')
        gk = np.asarray(g[k], np.float64)
        want = np.asarray(p[k], np.float64) - 1e-3 * gk / (np.abs(gk) + 1e-8)
        assert np.max(np.abs(got[k] - want)) <= 2e-6 * max(1.0, np.max(np.abs(p[k]))), k
    net.close()
    ctx.close()
