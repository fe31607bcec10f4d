"""Edges of a training step of the learned proposal: the largest batch, weights that are not
finite."""
import numpy as np
import pytest

from oracle import nn_oracle as nn
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def samples(n, seed=4):
    g = np.random.default_rng(seed)
    alpha = (0.5 * 60.0 ** g.random(n)).astype(np.float32)
    return alpha, g.uniform(-0.999, 0.999, n).astype(np.float32)


@pytest.mark.parametrize("batch", [2 ** 31 - 1, 2 ** 31 - 512 * 64])
def test_batch_past_the_sample_index_is_refused(su2, batch):
    """512 workgroups of 64 samples step past the batch by at most 32768: from 2^31 - 32768
    on the kernel's int index would wrap, and the call is refused before any launch."""
    announce(f"nn batch {batch} refused")
    with su2.NN(seed=3) as net:
        net.set_data(*samples(100))
        p = net.params
        for call in (lambda: net.loss_grad(0, batch), lambda: net.train(1, batch),
                     lambda: net.train(1, batch, 1e-3, lr_end=1e-4)):
            with pytest.raises(su2.SU2Error) as e:
                call()
            assert e.value.code == su2.SU2_EINVAL
        np.testing.assert_array_equal(net.params, p)
        assert np.isfinite(net.loss_grad(0, 100)[0])


def params(seed):
    return (np.random.default_rng(seed).standard_normal(2671) * 0.1).astype(np.float32)


# batches that end inside a tile of 64 samples (1, 36, 63 lanes with one), and whole tiles
@pytest.mark.parametrize("batch", [1, 100, 127, 128, 700])
@pytest.mark.parametrize("index", [0, 40, 64, 1090], ids=["W1", "b1", "W2", "b2"])
def test_infinite_weights_saturate(su2, batch, index):
    """An infinite weight of a hidden layer saturates its unit: loss and gradient are the oracle's,
    finite wherever its are, also where lanes of the last tile have no sample."""
    announce(f"nn infinite weight {index} batch {batch}")
    p, (al, x) = params(5), samples(1000)
    p[index] = np.inf
    with su2.NN(params=p) as net:
        net.set_data(al, x)
        loss, g = net.loss_grad(0, batch)
    wl, wg = nn.loss_and_grad(p, al[:batch].astype(np.float64), x[:batch].astype(np.float64))
    np.testing.assert_array_equal(np.isfinite(g), np.isfinite(wg))
    if np.isfinite(wl):
        assert loss == pytest.approx(wl, rel=1e-5)
    # per tensor, the bound that the gradient of finite weights has against the oracle
    for lo, hi in ((0, 32), (32, 64), (64, 1088), (1088, 1120), (1120, 2624), (2624, 2671)):
        w, ok = wg[lo:hi], np.isfinite(wg[lo:hi])
        bound = 1e-3 * np.abs(w[ok]) + 1e-4 * np.linalg.norm(w[ok])
        assert np.all(np.abs(g[lo:hi][ok] - w[ok]) <= bound), (lo, hi)


@pytest.mark.parametrize("batch", [1, 64, 700])
def test_nan_activation_reaches_every_row(su2, batch):
    """A NaN in the hidden layers makes every gradient of a weight NaN, among them those of
    the derivative outputs that no sample's bin touches."""
    announce(f"nn NaN weight batch {batch}")
    p = params(5)
    p[3] = np.nan  # W1
    with su2.NN(params=p) as net:
        net.set_data(*samples(1000))
        loss, g = net.loss_grad(0, batch)
        assert np.isnan(loss) and np.isnan(g[:2624]).all()
        net.train(2, batch)
        assert np.isnan(net.params[:2624]).all()
