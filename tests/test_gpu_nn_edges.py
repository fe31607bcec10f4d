"""Edges of a training step of the learned proposal: the largest batch."""
import numpy as np
import pytest

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
