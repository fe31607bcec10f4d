"""Single lattices whose launch was not set: one-wave workgroups in the passes
that measure nothing below a size limit (V/2 = 131072 in FP32, 524288 in FP64),
the descriptor as a kernel argument.  Links and sums are those of the set
default launch, bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


# ragged last workgroups; just below, at and above the FP32 limit
@pytest.mark.parametrize("dims", [[10, 6, 14, 8], [32, 32, 16, 16], [32, 32, 16, 18]],
                         ids=["10x6x14x8", "V/2=131072", "V/2=147456"])
@pytest.mark.parametrize("prec", ["f32", "f32-or", "f64"])
def test_unset_launch_equals_the_set_default(su2, dims, prec):
    announce(f"single lattice launch dims={dims} {prec}")
    mode = su2.SU2_KP_OR if prec == "f32-or" else su2.SU2_KP
    got = []
    for launch in (None, (256, 1 | 4, 8, 8, 0)):
        with (su2.Lattice64 if prec == "f64" else su2.Lattice)(dims, 2.3, 17, su2.SU2_HOT) as lat:
            if launch:
                lat.set_launch(*launch)
            h = lat.sweep_measure(3, mode, reunit_every=2, meas=3).cpu().numpy()
            lat.set_beta(1.1)  # a new descriptor
            lat.set_replica(5)
            lat.heatbath_sweep(1, mode)
            got.append((lat.get_links(), h))
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
