"""Sweeps of small lattices by teams of workgroups, one XCD each (V/2 up to 3072,
launch not set): links and sums are bit for bit those of the whole-sweep kernel
(V/2 <= 2048) and of the pass launches, for every sweep kind, under capture, with
several lattices in flight on streams of their own, and in batches."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

OR = 2  # SU2_KP_OR


def run(su2, dims, mode, reunit, ns, launch, n_or=1):
    with su2.Lattice(dims, 2.3, 19, su2.SU2_HOT) as lat:
        if launch:
            lat.set_launch(*launch)
        lat.set_hb_overrelax(n_or)
        lat.set_sweep(1)
        lat.heatbath_sweep(1, mode)
        h = lat.sweep_measure(ns, mode, reunit, 3).cpu().numpy()
        lat.heatbath_sweep(0, mode)
        return lat.get_links(), h, lat.sweep


# V/2 320 and 768 (the heat bath in one workgroup), 800 (in a team), up to 2048 sums
# per site, ragged last tiles, 3072 (the largest), and past it
@pytest.mark.parametrize("dims", [[4, 4, 4, 10], [2, 2, 12, 32], [2, 2, 10, 40], [8, 8, 8, 8],
                                  [2, 2, 10, 102], [10, 6, 8, 10], [16, 16, 6, 4],
                                  [10, 6, 14, 8]],
                         ids=["320", "768", "800", "2048", "2040", "2400", "3072", "3360"])
@pytest.mark.parametrize("mode,reunit,ns,n_or", [(0, 3, 7, 0), (0, 0, 2, 0), (OR, 2, 5, 2),
                                                 (OR, 1, 2, 0)])
def test_team_equals_the_set_launch(su2, dims, mode, reunit, ns, n_or):
    announce(f"team sweeps dims={dims} mode={mode}")
    small = mode == 0 and np.prod(dims) <= 4096
    got = run(su2, dims, mode, reunit, ns, None, n_or)
    want = run(su2, dims, mode, reunit, ns, (256, 1 if small else 1 | 4), n_or)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    assert got[2] == want[2] == 2 + ns


def test_team_replays_and_many_sweeps(su2):
    import torch
    announce("team sweeps: replay, more sweeps than one launch takes")
    dims = [6, 8, 6, 8]
    with torch.cuda.stream(torch.cuda.Stream()):
        lat = su2.Lattice(dims, 2.3, 5, su2.SU2_HOT)
    hist = torch.zeros((12, 3), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    lat.capture(4, su2.SU2_KP, 2, 3, hist)
    for k in range(3):
        lat.replay(1)
        torch.cuda.synchronize()  # the program's own work between replays
        hist[4 * k:4 * k + 4].clone().sum().item()
    with su2.Lattice(dims, 2.3, 5, su2.SU2_HOT) as ref:
        ref.set_launch(256, 1)
        h = ref.sweep_measure(12, su2.SU2_KP, 2, 3).cpu().numpy()
        np.testing.assert_array_equal(hist.cpu().numpy(), h)
        np.testing.assert_array_equal(lat.get_links(), ref.get_links())
        ref.heatbath_sweep(4100)
        lat.heatbath_sweep(4100)
        np.testing.assert_array_equal(lat.get_links(), ref.get_links())
    lat.close()


def test_teams_on_several_streams(su2):
    import torch
    announce("team sweeps: 12 lattices in flight")
    dims = [[8, 8, 8, 8], [10, 8, 8, 8], [4, 6, 8, 10]] * 4
    lats = []
    for k, d in enumerate(dims):
        with torch.cuda.stream(torch.cuda.Stream()):
            lats.append(su2.Lattice(d, 2.0 + 0.05 * k, k, su2.SU2_HOT))
    torch.cuda.synchronize()
    for _ in range(3):
        for lat in lats:
            lat.heatbath_sweep(20)
    torch.cuda.synchronize()
    for k, (d, lat) in enumerate(zip(dims, lats)):
        with su2.Lattice(d, 2.0 + 0.05 * k, k, su2.SU2_HOT) as ref:
            ref.set_launch(256, 1 | 4)
            ref.heatbath_sweep(60)
            np.testing.assert_array_equal(lat.get_links(), ref.get_links())
        lat.close()


@pytest.mark.parametrize("n,dims", [(2, [[8, 8, 8, 8], [4, 4, 4, 6]]), (11, [[8, 8, 8, 6]]),
                                    (7, [[10, 8, 8, 8], [6, 6, 6, 8], [4, 4, 4, 4]]),
                                    (16, [[16, 16, 4, 4], [6, 6, 6, 6]]),
                                    (17, [[16, 16, 4, 4], [6, 6, 6, 6]]),
                                    (32, [[6, 6, 6, 6]])],
                         ids=["2-mixed", "11", "7-mixed", "16-mixed", "17-mixed", "32"])
@pytest.mark.parametrize("mode,reunit", [(0, 3), (0, 0), (OR, 2)])
def test_team_batches_equal_the_set_launch(su2, n, dims, mode, reunit):
    import torch
    announce(f"team batch n={n} dims={dims} mode={mode}")
    stream = torch.cuda.Stream()
    dims = [dims[r % len(dims)] for r in range(n)]
    small = mode == 0 and max(np.prod(d) for d in dims) <= 4096
    out = []
    for launch in (None, (256, 1 if small else 1 | 4)):
        with torch.cuda.stream(stream), su2.Batch(dims, np.linspace(1.8, 2.8, n),
                                                  [su2.SU2_HOT] * n, 3) as b:
            if launch:
                b.set_launch(*launch)
            b.sweep(1, mode)
            h = b.sweep_measure(7, mode, reunit, 3).cpu().numpy()
            b.capture(2, mode)
            b.replay(2)
            out.append((h, [b.get_links(r) for r in range(n)]))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    for got, want in zip(out[0][1], out[1][1]):
        np.testing.assert_array_equal(got, want)
