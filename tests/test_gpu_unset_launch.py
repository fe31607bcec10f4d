"""The unset launch as a launch of its own: reported with flag 256, set back, chosen and cached by
the autotuner where it is the fastest."""
import json

import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

UNSET = 256


def make(su2, kind):
    if kind == "batch":
        return su2.Batch([[8, 6, 12, 4], [4, 4, 6, 10]] * 3, np.linspace(1.8, 2.8, 6), su2.SU2_HOT, 5)
    cls = su2.Lattice64 if kind == "f64" else su2.Lattice
    return cls([8, 6, 12, 4], 2.3, 5, su2.SU2_HOT)


@pytest.mark.parametrize("kind", ["single", "f64", "batch"])
def test_unset_launch_is_reported_and_set_back(su2, kind):
    announce(f"unset launch round trip, {kind}")
    with make(su2, kind) as a:
        unset = a.launch()
        assert unset["flags"] == UNSET | 1 and unset["block"] == 256 and unset["grid_cap"] == 0
        a.set_launch(**unset)
        assert a.launch() == unset
        a.set_launch(128, 1 | 4, 1, 2)
        assert a.launch()["flags"] == 1 | 4 and a.launch()["block"] == 128
        for bad in ((128, UNSET | 1), (256, UNSET), (256, UNSET | 1 | 4), (256, UNSET | 3),
                    (256, UNSET | 1 | 8), (256, UNSET | 1, 8, 8, 64), (256, 512 | 1),
                    (256, UNSET | 1, 3)):
            with pytest.raises(su2.SU2Error) as e:
                a.set_launch(*bad)
            assert e.value.code == su2.SU2_EINVAL
            assert a.launch()["flags"] == 1 | 4  # kept
        a.set_launch(**unset)
        assert a.launch() == unset
        with make(su2, kind) as b:
            ha = a.sweep_measure(3, reunit_every=2, meas=3).cpu().numpy()
            hb = b.sweep_measure(3, reunit_every=2, meas=3).cpu().numpy()
            np.testing.assert_array_equal(ha, hb)


def test_autotuner_chooses_and_caches_the_unset_launch(su2, tmp_path):
    """Teams of workgroups run 16 x 8^4 in two thirds of the next best launch's time; only the
    unset launch holds them."""
    announce("autotune 16 x 8^4: the unset launch")
    cache = str(tmp_path / "tune.jsonl")
    dims, betas = [[8, 8, 8, 8]] * 16, np.linspace(1.8, 2.8, 16)
    with su2.Batch(dims, betas, su2.SU2_HOT, 5) as a:
        unset = a.launch()
        a.set_launch(256, 1 | 4)
        us = a.autotune(cache)
        assert a.launch() == unset
    with open(cache) as f:
        assert json.loads(f.readline())["flags"] == UNSET | 1
    with su2.Batch(dims, betas, su2.SU2_HOT, 5) as a:
        a.set_launch(128, 3)
        assert a.autotune(cache) == pytest.approx(us, abs=1e-3)
        assert a.launch() == unset
