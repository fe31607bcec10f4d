"""Whole sweeps of batches of the smallest lattices on both sides of the lines between the field in
LDS and in the caches: the same links and sums (both kernels sum per site), and the rate of a large
batch."""
import time

import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


# replicas a CU: one (256), two (257, 512), three (513); V/2 64, 96, 128, 192 and 288 in calls of
# one sweep and of sixteen
@pytest.mark.parametrize("n,dims", [(256, [4, 4, 4, 4]), (257, [4, 4, 4, 4]), (257, [6, 4, 4, 4]),
                                    (512, [4, 4, 4, 2]), (513, [4, 4, 4, 2]), (513, [6, 4, 4, 2]),
                                    (513, [6, 6, 4, 4])])
def test_batches_on_both_sides_of_the_line(su2, n, dims):
    """A batch of n replicas is the single lattices with their replica ids; the first, the last and
    some in between are run by themselves."""
    announce(f"batch line {n} x {dims}")
    betas = np.linspace(1.8, 2.8, n)
    calls = ((1, 3, 0), (16, 1, 5), (1, 2, 0), (16, 3, 0))
    with su2.Batch([dims] * n, betas, su2.SU2_HOT, 3) as b:
        h = np.concatenate([b.sweep_measure(ns, su2.SU2_KP, re, meas).cpu().numpy()
                            for ns, meas, re in calls])
        links = {r: b.get_links(r) for r in (0, 1, n // 2, 255, n - 1)}
    for r, got in links.items():
        with su2.Lattice(dims, betas[r], 3, su2.SU2_COLD) as lat:
            with su2.Batch([dims] * n, betas, su2.SU2_HOT, 3) as fresh:
                lat.set_links(fresh.get_links(r))
            lat.set_replica(r)
            hr = np.concatenate([lat.sweep_measure(ns, su2.SU2_KP, re, meas).cpu().numpy()
                                 for ns, meas, re in calls])
            np.testing.assert_array_equal(lat.get_links(), got)
            np.testing.assert_array_equal(hr, h[:, r])


def test_large_batch_sustains_its_rate(su2):
    """2048 x 4^4 with the plaquette: 5.8e10 link updates/s in the caches, 2.9e10 in LDS."""
    import torch
    announce("2048 x 4^4: rate")
    n, ns = 2048, 8
    with su2.Batch([[4, 4, 4, 4]] * n, np.linspace(1.8, 2.8, n), su2.SU2_HOT, 3) as b:
        hist = torch.zeros((ns, n, 3), dtype=torch.float64, device="cuda")
        t = []
        for _ in range(30):
            torch.cuda.synchronize()
            a = time.perf_counter()
            b.sweep_measure(ns, meas=su2.SU2_MEAS_PLAQ, hist=hist)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
    rate = n * 1024 * ns / float(np.median(t))
    print(f"[gpu-test] {rate:.3g} link updates/s", flush=True)
    assert rate > 4.2e10
