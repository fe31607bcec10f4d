"""Launch order of batches: replicas one after the other on an XCD each where
they fill the XCDs evenly, and reversed odd passes that take the replicas in
reverse order too.  Neither changes a bit of the links or of the sums."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


def sweep(su2, dims, betas, launch, mode_or=False):
    with su2.Batch(dims, betas, su2.SU2_HOT, 11) as b:
        if launch is not None:
            b.set_launch(*launch)
        mode = su2.SU2_KP_OR if mode_or else su2.SU2_KP
        h = b.sweep_measure(5, mode, reunit_every=2, meas=3).cpu().numpy()
        return h, [b.get_links(r) for r in range(b.n)]


# even (8 and 16 equal replicas), uneven sizes that still fill the XCDs evenly,
# and too uneven for it (9 replicas); V/2 with a ragged last workgroup
@pytest.mark.parametrize("dims", [[[8, 8, 6, 14]] * 8, [[10, 6, 8, 12]] * 16,
                                  [[12, 12, 6, 6], [6, 6, 12, 12]] * 12, [[8, 8, 8, 10]] * 9],
                         ids=["8", "16", "24-uneven", "9"])
def test_unset_launch_equals_the_plain_one(su2, dims):
    announce(f"batch order n={len(dims)}")
    betas = np.linspace(1.5, 3.0, len(dims))
    want = sweep(su2, dims, betas, (256, 1 | 2 | 4))  # plain, every pass forward
    for launch in (None, (256, 1 | 4), (128, 64 | 4), (256, 64 | 4, 0, 0, 16)):
        h, links = sweep(su2, dims, betas, launch)
        for r in range(len(dims)):
            np.testing.assert_array_equal(links[r], want[1][r])
        if launch is None or launch[0] == 256:  # sums are per workgroup
            np.testing.assert_allclose(h, want[0], rtol=0, atol=1e-8)
    want = sweep(su2, dims, betas, (256, 1 | 2 | 4), True)
    h, links = sweep(su2, dims, betas, None, True)
    for r in range(len(dims)):
        np.testing.assert_array_equal(links[r], want[1][r])
    np.testing.assert_array_equal(h, want[0])


# 8 and 16 replicas, 15 (one padding replica) and 9 (too uneven: plain order)
@pytest.mark.parametrize("dims,n", [([6, 4, 8, 6], 8), ([8, 6, 4, 4], 16), ([4, 10, 6, 4], 15),
                                    ([4, 4, 6, 4], 9)], ids=["8", "16", "15", "9"])
def test_su3_batch_order(su2, dims, n):
    announce(f"SU(3) batch order n={n}")
    betas = np.linspace(5.2, 6.2, n)
    with su2.Batch3(dims, betas, 13, su2.SU2_HOT) as b:
        h = b.heatbath_sweep(3, reunit_every=2, history=True)
        b.overrelax(1)
        pl, po = b.plaquette(), b.polyakov()
        links = [b.get_links(r) for r in range(n)]
    for r in range(n):
        with su2.Lattice3(dims, betas[r], 13, su2.SU2_COLD) as lat:
            lat.set_replica(r)
            with su2.Batch3(dims, betas, 13, su2.SU2_HOT) as fresh:
                lat.set_links(fresh.get_links(r))
            np.testing.assert_array_equal(lat.heatbath_sweep(3, 2, history=True), h[:, r])
            lat.overrelax(1)
            np.testing.assert_array_equal(lat.get_links(), links[r])
            assert lat.plaquette() == pl[r] and tuple(po[r]) == lat.polyakov()
