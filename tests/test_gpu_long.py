"""2-D lattices of one very long row or column (80 GB): 2^29 cells and more, past
the 32-bit byte offsets of double fields and, for tiles of 8 by 32 cells, past
2^32 threads, alone and in a batch.  The state repeats with a period of 4096
cells, so every field after any number of steps is that of a lattice of one
period, bit for bit."""
import numpy as np
import pytest

from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    from paper_2101_06769_amd import mplb

PERIOD, REPEATS = 4096, (1 << 17) + 2


def check_repeats(axis, batch=False):
    one = [1, 1, 1]
    one[axis] = PERIOD
    many = list(one)
    many[axis] *= REPEATS
    params = params_for(2, one, (0, 0, 0))
    phi = inputs.random_state(params, seed=5)[0].reshape(-1)
    s = mplb.Solver(params, storage="fp32")
    s.init(phi, np.zeros((2, PERIOD)))
    shared = None
    if batch:
        # 2^27 tiles is what a column is counted as: 64 by 4 cells each
        shared = mplb.Batch(2, "fp32", capacity=1, max_tiles=1 << 28)
        shared.set_solo_cells(1 << 31)
    b = mplb.Solver(params_for(2, many, (0, 0, 0)), storage="fp32", stream=shared and shared.stream)
    b.init(np.tile(phi, REPEATS), np.zeros((2, PERIOD * REPEATS)))
    for steps in (0, 3):
        s.step(steps)
        if shared and steps:
            shared.attach(b, steps)
            shared.step(steps)
        else:
            b.step(steps)
        for field in (mplb.FIELD_PHI, mplb.FIELD_UX + axis):
            want = s.read(field).reshape(-1)
            assert (b.read(field).reshape(REPEATS, PERIOD) == want).all(), (axis, steps, field)
    del b, shared
    torch.cuda.empty_cache()


def test_long_row():
    check_repeats(0)


@pytest.mark.parametrize("batch", [False, True])
def test_long_column(batch):
    check_repeats(1, batch)
