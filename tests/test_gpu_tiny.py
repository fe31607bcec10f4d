"""Whole sweeps with the field in LDS (the smallest lattices, V/2 <= 312): the
links of the per-pass launches bit for bit, whatever the shape, the coupling
(both branches of the a0 sampler, many trials) and the reunitarisation; the
plaquette's sum in per-site fixed point (2^-28 per site: below 1e-8 on a mean).
The per-pass Polyakov kernel multiplies t-segments and then their products, so
the loops are compared with the FP64 product of the links instead: Nt FP32
products of unit quaternions, each off by at most 4 roundings of 2^-24."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


# V/2: 8 (part of a wave), 64, 128 (384 threads), 132 and 192 (three and more
# waves a role), 312 (the largest), 320 (past it: the kernel for larger ones)
@pytest.mark.parametrize("dims", [[2, 2, 2, 2], [4, 4, 2, 4], [4, 4, 4, 4], [2, 6, 2, 22],
                                  [4, 6, 4, 4], [2, 26, 6, 2], [4, 4, 10, 4]],
                         ids=["2^4", "4x4x2x4", "4^4", "2x6x2x22", "4x6x4x4", "2x26x6x2",
                              "4x4x10x4"])
@pytest.mark.parametrize("beta,reunit,ns", [(2.3, 3, 7), (0.0, 0, 2), (40.0, 1, 3), (0.8, 2, 1)])
def test_tiny_sweeps_equal_pass_launches(su2, orc, dims, beta, reunit, ns):
    announce(f"sweeps in LDS dims={dims} beta={beta}")
    got = []
    for flags in (1, 1 | 4):
        with su2.Lattice(dims, beta, 31, su2.SU2_HOT) as lat:
            lat.set_launch(256, flags)
            lat.set_sweep(1)
            lat.heatbath_sweep(1)
            h = lat.sweep_measure(ns, reunit_every=reunit, meas=3).cpu().numpy()
            got.append((lat.get_links(), h, lat.sweep))
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert got[0][2] == got[1][2] == 2 + ns
    assert np.abs(got[0][1] - got[1][1])[:, 0].max() < 1e-8
    for links, h, _ in got:
        L, _ = orc.polyakov(dims, links.astype(np.float64))
        assert abs(h[-1, 1] - L) < dims[3] * 4 * 2.0 ** -24 + 2.0 ** -28
        assert h[-1, 2] == abs(h[-1, 1])


def test_tiny_batch_and_replay(su2):
    import torch
    announce("sweeps in LDS: uneven batch, graph replay")
    dims = [[4, 4, 4, 4], [2, 2, 4, 6], [6, 4, 4, 6], [2, 2, 2, 2]]
    betas = [2.0, 0.5, 2.6, 8.0]
    with torch.cuda.stream(torch.cuda.Stream()):
        b = su2.Batch(dims, betas, su2.SU2_HOT, 7)
    hist = torch.zeros((12, 4, 3), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    b.capture(4, reunit_every=4, meas=1, hist=hist)
    for k in range(3):
        b.replay(1)
        torch.cuda.synchronize()  # the program's own work between replays
        hist[4 * k:4 * k + 4].clone().sum().item()
    got = hist.cpu().numpy()
    with su2.Batch(dims, betas, su2.SU2_HOT, 7) as fresh:
        start = [fresh.get_links(r) for r in range(4)]
    for r, d in enumerate(dims):
        with su2.Lattice(d, betas[r], 7) as lat:
            lat.set_replica(r)
            lat.set_launch(256, 1 | 4)
            lat.set_links(start[r])
            h = lat.sweep_measure(12, reunit_every=4, meas=1).cpu().numpy()
            np.testing.assert_array_equal(lat.get_links(), b.get_links(r))
        assert np.abs(h - got[:, r]).max() < 1e-8
    b.close()
