"""The host exchange where the host rearranges the links itself (up to 4096 sites in FP32, 1400 in
FP64) and just past it: every value in its place, whatever the two types, and the time of a small
lattice."""
import time

import numpy as np
import pytest

from tests import inputs
from tests.gpu_util import announce
from tests.test_gpu_exchange import classes

pytestmark = pytest.mark.gpu


# 16, 480 and 1200 sites, 2800, 4096 and 4160
@pytest.mark.parametrize("dims", [[2, 2, 2, 2], [4, 6, 2, 10], [10, 10, 2, 6], [10, 10, 14, 2],
                                  [16, 16, 4, 4], [26, 10, 4, 4]])
def test_exchange_on_both_sides_of_the_line(su2, dims):
    import torch
    announce(f"small host exchange dims={dims}")
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


def test_small_lattice_is_exchanged_faster(su2):
    """512 sites take a third of the time of 6400 (two thirds with a launch and a staging
    buffer)."""
    announce("small host exchange: time")
    med = {}
    for dims in ([4, 4, 4, 8], [10, 10, 8, 8]):
        with su2.Lattice(dims, 2.3, 1, su2.SU2_HOT) as lat:
            t = []
            for _ in range(400):
                a = time.perf_counter()
                links = lat.get_links()
                lat.set_links(links)
                t.append(time.perf_counter() - a)
            med[dims[0]] = float(np.median(t))
    print(f"[gpu-test] get + set {1e6 * med[4]:.1f} us (512 sites), {1e6 * med[10]:.1f} (6400)",
          flush=True)
    assert med[4] < 0.5 * med[10]
