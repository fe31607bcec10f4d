"""The batch orders on replicas of really different sizes: block counts that differ, XCDs that fill
unequally within the tenth that the unset launch allows (padding workgroups), every replica too
large for a team.  Links and sums are those of the plain forward order."""
import numpy as np
import pytest

from tests.gpu_util import announce
from tests.test_gpu_affine import sweep

pytestmark = pytest.mark.gpu

A, B = [12, 12, 8, 8], [12, 12, 10, 8]      # V/2 4608 and 5760: 18 and 23 blocks of 256
C, D = [12, 10, 8, 8], [10, 10, 10, 8]      # 3840 and 4000: 15 and 16, the last one ragged


@pytest.mark.parametrize("dims", [[[16, 8, 8, 8]] * 8, [A, B] * 8, [A, B, C] * 7 + [B, A, D],
                                  [D, A] * 4 + [B] * 3],
                         ids=["8-equal", "16-two-sizes", "24-padded", "11-too-uneven"])
def test_orders_of_uneven_replicas(su2, dims):
    announce(f"batch order, uneven, n={len(dims)}")
    betas = np.linspace(1.5, 3.0, len(dims))
    for over in (False, True):
        want = sweep(su2, dims, betas, (256, 1 | 2 | 4), over)
        for launch in (None, (256, 1 | 4), (256, 64 | 4), (256, 64 | 2 | 4), (128, 64 | 4)):
            h, links = sweep(su2, dims, betas, launch, over)
            for r in range(len(dims)):
                np.testing.assert_array_equal(links[r], want[1][r])
            if launch is None or launch[0] == 256:  # sums are per workgroup
                np.testing.assert_array_equal(h, want[0])


# 9 blocks a replica (forward, as 9 is no multiple of 8), 8 and 16 (in reverse), too few or
# too uneven for one replica per XCD
@pytest.mark.parametrize("dims,n", [([12, 10, 6, 6], 5), ([8, 8, 8, 8], 3), ([16, 8, 8, 8], 9)],
                         ids=["9-blocks", "8-blocks", "16-blocks"])
def test_su3_orders(su2, dims, n):
    announce(f"SU(3) batch order, n={n} dims={dims}")
    betas = np.linspace(5.2, 6.2, n)
    with su2.Batch3(dims, betas, 13, su2.SU2_HOT) as b:
        start = [b.get_links(r) for r in range(n)]
        h = b.heatbath_sweep(2, reunit_every=2, history=True)
        b.overrelax(1)
        links = [b.get_links(r) for r in range(n)]
    for r in (0, 1, n - 1):
        with su2.Lattice3(dims, betas[r], 13, su2.SU2_COLD) as lat:
            lat.set_replica(r)
            lat.set_links(start[r])
            np.testing.assert_array_equal(lat.heatbath_sweep(2, 2, history=True), h[:, r])
            lat.overrelax(1)
            np.testing.assert_array_equal(lat.get_links(), links[r])


def test_switching_between_affine_launches(su2):
    """The affine map lies in the batch's scratch (128- and 256-thread workgroups, the unset launch)
    or in an allocation of its own (64 threads, with the work queue's flag), and moves between
    them."""
    announce("batch order: switching launches")
    dims = [A, B] * 4
    betas = np.linspace(1.5, 3.0, len(dims))
    with su2.Batch(dims, betas, su2.SU2_HOT, 11) as a, su2.Batch(dims, betas, su2.SU2_HOT, 11) as b:
        b.set_launch(256, 1 | 2 | 4)
        unset = a.launch()
        for launch in ((64, 64 | 4), (256, 257), (64, 64 | 4, 1, 1, 64), (128, 64 | 4),
                       (256, 64 | 8), (256, 64 | 4), (64, 66 | 4), (256, 1 | 4), (256, 257)):
            a.set_launch(*launch)
            for x in (a, b):
                x.sweep(1)
                x.sweep(1, su2.SU2_KP_OR)
        assert a.launch() == unset
        for r in range(len(dims)):
            np.testing.assert_array_equal(a.get_links(r), b.get_links(r))
