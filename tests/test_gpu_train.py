"""Training kernels of the learned correction at the sizes where their
splits can go wrong: the weight gradients' block partials and pixel chunks
(few crops and many, narrow planes whose chunks cross rows and crops), the
sum over them with the Adam update, and the queue of optimisation steps of
swe_lc_fit.  Oracle: FP64 convolution gradients of the stored bf16 values."""
import sys

import numpy as np
import pytest

from oracle import learned as LN
from paper_1705_00614_amd import learned as LC
from paper_1705_00614_amd import scenarios as S

pytestmark = pytest.mark.gpu

swe = pytest.importorskip("paper_1705_00614_amd.swe")


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[gpu] %s" % request.node.nodeid, flush=True)
    sys.stdout.flush()
    yield


def _conv_grads(a, g):
    """dW, db of a valid 3x3 convolution in FP64, tap by tap."""
    so = g.shape[1]
    gm = g.reshape(-1, g.shape[-1])
    dw = np.empty((g.shape[-1], a.shape[-1], 3, 3))
    for ky in range(3):
        for kx in range(3):
            dw[:, :, ky, kx] = gm.T @ a[:, ky:ky + so, kx:kx + so].reshape(-1, a.shape[-1])
    return dw, gm.sum(axis=0)


# chunks of 16 pixels and one partial block (1 x 2^2 outputs), chunks over
# several crops of narrow planes, a chunk count just past a staging round of
# k_opt, the default tile with a ragged last chunk, wide rows
@pytest.mark.parametrize("tile,n", [(1, 1), (1, 40), (2, 97), (8, 26), (16, 7), (32, 3), (32, 40), (64, 2)])
def test_weight_gradients_match_oracle(tile, n):
    rng = np.random.default_rng(100 * tile + n)
    so = tile + 1
    x = rng.normal(size=(n, so + 8, so + 8, 6))
    y = rng.normal(size=(n, so, so, 6))
    mask = (rng.uniform(size=y.shape) > 0.2).astype(float)
    net = swe.Net(tile, n, np.ones(6), np.ones(6))
    net.set_params(LC.initial_params(7))
    loss = net.train_step(x, y, mask, 0.0)
    dW, db = swe.lc_unpack(net.grads())
    out = net.forward(x)
    want = 0.5 * (mask * (out - y) ** 2).sum() / mask.sum()
    assert abs(loss - want) <= 1e-5 * want
    net.train_step(x, y, mask, 0.0)
    for l in range(4):
        a, g = net.layer(l, n), net.layer(4 + l, n)
        dw, dbb = _conv_grads(a, g)
        adw, adb = _conv_grads(np.abs(a), np.abs(g))
        # FP32 sums of k terms in any order: k 2^-24 of the sum of magnitudes
        bar = max(g.shape[0] * g.shape[1] * g.shape[2], 16) * 2.0 ** -24
        assert np.all(np.abs(dW[l] - dw) <= bar * adw + 1e-30), l
        assert np.all(np.abs(db[l] - dbb) <= bar * adb + 1e-30), l
    # Adam after the gradient of the same step
    p0 = net.params()
    net.train_step(x, y, mask, 1e-3)
    p1 = LN.Adam([p0], lr=1e-3).step([p0], [net.grads()])[0]
    assert np.abs(net.params() - p1).max() <= 2e-6


@pytest.mark.parametrize("iters,batch", [(3, 7), (257, 1)])
def test_fit_equals_single_training_steps(iters, batch):
    """swe_lc_fit queues its steps (256 at a time); it must compute bit for
    bit what one training step per minibatch computes."""
    fine = S.floodplain(n=256, h=25.0, seed=5, t_peak=1800.0, sigma_t=600.0)
    net = LC.make_net(32, 16)
    net.data(64)
    LC.collect(net, fine, 4, 4, intervals=6, gap=4)
    n = net.data_count()
    assert n >= batch
    x, y, mask, _ = net.get_data(0, n)
    net.set_params(LC.initial_params(3))
    losses = net.fit(iters, batch, 1e-3, seed=11)
    ref = swe.Net(32, 16, np.ones(6), np.ones(6))
    ref.set_params(LC.initial_params(3))
    M = (1 << 64) - 1
    st = (11 * 6364136223846793005 + 1442695040888963407) & M
    perm = list(range(n))
    for it in range(iters):
        pick = []
        for b in range(batch):
            st = (st * 6364136223846793005 + 1442695040888963407) & M
            j = b + (st >> 33) % (n - b)
            perm[b], perm[j] = perm[j], perm[b]
            pick.append(perm[b])
        want = ref.train_step(x[pick], y[pick], mask[pick], 1e-3)
        assert losses[it] == want, it
    assert np.array_equal(net.params(), ref.params())
