"""Health of domains that step alone in a batch: a state that turns non-finite
during a run of steps is flagged by the direct steps after the run, whatever the
run's length (16 steps, 18 where a launch takes three)."""
import numpy as np
import pytest

from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2101_06769_amd import mplb


@pytest.mark.parametrize("n", [(130, 140, 1), (64, 96, 1), (400, 300, 1)])
def test_blow_up_inside_a_run_is_flagged(n):
    params = params_for(2, n, (0, 1, 0))
    phi, u, p = inputs.random_state(params, seed=3, u_amp=1.0)  # far beyond stability
    a = mplb.Solver(params, storage="fp32")
    a.init(phi, u, p)
    a.step(1)
    assert np.isfinite(a.read(mplb.FIELD_PHI)).all()  # the check before the run passes
    a.step(16)
    assert not np.isfinite(a.read(mplb.FIELD_PHI)).all()
    b = mplb.Batch(2, "fp32", capacity=2, max_tiles=1 << 12)
    b.set_solo_cells(0)
    s = mplb.Solver(params, storage="fp32", stream=b.stream)
    s.init(phi, u, p)
    slot = b.attach(s, 32)
    b.step(32)  # one step, a run, then direct steps
    assert b.status()[slot] == mplb.EUNSTABLE
