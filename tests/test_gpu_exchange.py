"""The host exchange (get/set links) against the documented device layout: array
(mu*2 + parity) holds U_mu at the half-site s >> 1 of every site of that
parity.  Values are moved, and rounded or widened where the host type is not
the lattice's, so every comparison is exact."""
import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def classes(dims, links):
    """float[V][4][4] in site order -> float[8][V/2][4]."""
    x, y, z, t = (np.arange(n) for n in dims)
    par = ((t[:, None, None, None] + z[:, None, None] + y[:, None] + x) & 1).reshape(-1)
    sites = [np.flatnonzero(par == p) for p in (0, 1)]  # in half-site order
    return np.stack([links[sites[p], mu] for mu in range(4) for p in (0, 1)])


# the smallest lattice, ragged ones, and one of more sites than the staging buffer holds
# (32 MB: 524288 sites in FP32, 262144 in FP64)
@pytest.mark.parametrize("dims", [[2, 2, 2, 2], [4, 6, 2, 10], [10, 6, 14, 8], [32, 32, 32, 18]],
                         ids=["2^4", "4x6x2x10", "10x6x14x8", "32^3x18"])
def test_exchange_follows_the_device_layout(su2, dims):
    import torch
    announce(f"host exchange dims={dims}")
    links = inputs.random_links(dims, 70 + sum(dims), spread=0.6)
    with su2.Lattice(dims, 2.3, 1) as lat:
        lat.set_links(links)
        dev = lat.links_t.view(torch.float32).view(8, -1, 4).cpu().numpy()
        np.testing.assert_array_equal(dev, classes(dims, links))
        np.testing.assert_array_equal(lat.get_links(), links)
    wide = inputs.as_f64(links) * (1.0 + 2.0 ** -40)
    with su2.Lattice64(dims, 2.3, 1) as lat:
        lat.set_links(wide)
        np.testing.assert_array_equal(lat.get_links(), wide)
        np.testing.assert_array_equal(su2.su2_get_links(lat.h, lat.volume),
                                      wide.astype(np.float32))
        su2.su2_set_links(lat.h, links)
        np.testing.assert_array_equal(lat.get_links(), links.astype(np.float64))


def test_exchange_of_batch_replicas(su2):
    announce("host exchange of a batch's replicas")
    dims = [[4, 4, 4, 4], [8, 6, 10, 4], [2, 4, 6, 8]]
    with su2.Batch(dims, 2.0, su2.SU2_COLD, 5) as b:
        want = [inputs.random_links(d, 90 + r, spread=0.6) for r, d in enumerate(dims)]
        for r in (2, 0, 1):
            b.set_links(r, want[r])
        for r in range(3):
            np.testing.assert_array_equal(b.get_links(r), want[r])
