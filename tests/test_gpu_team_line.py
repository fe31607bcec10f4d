"""Where teams of workgroups begin, by the length of the call and what it measures: links and sums
are those of the set launches on both sides, also with calls of both kinds in one chain."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

OR = 2  # SU2_KP_OR


# V/2 800 and 832 (the Polyakov loop from 12 sweeps), 840 and 1024 (measured from 2), 1032
@pytest.mark.parametrize("dims", [[2, 2, 10, 40], [26, 4, 4, 4], [10, 6, 14, 2], [8, 8, 8, 4],
                                  [2, 2, 12, 44]],
                         ids=["800", "832", "840", "1024", "1056"])
def test_calls_of_every_length(su2, dims):
    announce(f"team line dims={dims}")
    out = []
    for launch in (None, (256, 1), (256, 1 | 4)):
        with su2.Lattice(dims, 2.3, 19, su2.SU2_HOT) as lat:
            if launch:
                lat.set_launch(*launch)
            h = []
            for ns, meas, reunit in ((1, 3, 0), (1, 1, 1), (2, 3, 0), (2, 1, 2), (11, 3, 3),
                                     (12, 3, 5), (1, 2, 0)):
                h.append(lat.sweep_measure(ns, su2.SU2_KP, reunit, meas).cpu().numpy())
                lat.heatbath_sweep(1)
            out.append((np.concatenate(h), lat.get_links(), lat.sweep))
    for _, links, sweep in out[1:]:
        np.testing.assert_array_equal(out[0][1], links)
        assert out[0][2] == sweep
    # the sums of one workgroup (the passes multiply Polyakov loops in segments)
    np.testing.assert_array_equal(out[0][0], out[1][0])


# two and three replicas on an XCD, of three and four tiles
@pytest.mark.parametrize("n,dims", [(16, [8, 8, 8, 4]), (17, [8, 8, 8, 4]), (24, [6, 6, 6, 8]),
                                    (24, [6, 6, 6, 6])])
def test_overrelaxed_batches(su2, n, dims):
    announce(f"team line, over-relaxed batch {n} x {dims}")
    out = []
    for launch in (None, (256, 1 | 4)):
        with su2.Batch([dims] * n, np.linspace(1.8, 2.8, n), su2.SU2_HOT, 3) as b:
            if launch:
                b.set_launch(*launch)
            h = b.sweep_measure(3, OR, 2, 3).cpu().numpy()
            out.append((h, [b.get_links(r) for r in (0, 7, n - 1)]))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    for got, want in zip(out[0][1], out[1][1]):
        np.testing.assert_array_equal(got, want)
