"""A bounded wait of a team launch that runs out is reported, as a team's, and the batch runs on: the
launch drains, the teams are cleared, and later sweeps equal those of a batch that never failed."""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


# heat bath with per-site sums (V/2 2048), over-relaxation with reunitarisation sweeps between
@pytest.mark.parametrize("n,dims,mode", [(5, [8, 8, 8, 8], 0), (3, [6, 6, 8, 8], 2)])
def test_team_wait_limit_is_reported(su2, n, dims, mode):
    announce(f"team launch: bounded wait runs out, {n} x {dims} mode {mode}")
    betas = np.linspace(1.8, 2.8, n)
    with su2.Batch([dims] * n, betas, su2.SU2_HOT, 3) as b, \
            su2.Batch([dims] * n, betas, su2.SU2_HOT, 3) as ref:
        links = [b.get_links(r) for r in range(n)]
        b.test_spin_limit(0)
        b.sweep(20, mode)
        with pytest.raises(su2.SU2Error) as e:
            b.synchronize()
        assert e.value.code == su2.SU2_EHIP and "team launch" in str(e.value)
        b.sweep_measure(4, mode, 2, 3)
        with pytest.raises(su2.SU2Error) as e:
            b.observables()
        assert e.value.code == su2.SU2_EHIP
        b.test_spin_limit(1 << 22)
        ref.sweep(20, mode)
        ref.sweep_measure(4, mode, 2, 3)
        for r in range(n):  # as if nothing had run, but for the sweep index
            b.set_links(r, links[r])
            ref.set_links(r, links[r])
        ref.set_launch(256, 1 if mode == 0 else 1 | 4)
        got, want = (x.sweep_measure(5, mode, 2, 3).cpu().numpy() for x in (b, ref))
        np.testing.assert_array_equal(got, want)
        for r in range(n):
            np.testing.assert_array_equal(b.get_links(r), ref.get_links(r))
        for got, want in zip(b.observables(), ref.observables()):
            np.testing.assert_array_equal(got, want)
