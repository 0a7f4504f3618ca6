"""mplb_read into page-locked memory (the field kernel writes over the bus) and
into pageable memory (a staging array and a copy): the same bits, for every
field and storage format, on the forms the field kernels take (2-D tiles of
64 cells and narrower, 3-D rows, packed planes and the general form), into the
middle of a larger buffer whose surroundings stay untouched; and after steps
the values of the FP64 oracle."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for
from tests.test_gpu_parity import gpu_solver, noisy_state

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2101_06769_amd import mplb

LATTICES = [(2, (65, 9, 1), (2, 1, 0)), (2, (20, 31, 1), (0, 0, 0)), (3, (64, 5, 4), (0, 0, 1)),
            (3, (37, 6, 5), (0, 0, 2)), (3, (9, 8, 7), (1, 2, 0))]


def read_into(s, field, ptr):
    mplb.check(mplb.load_library().mplb_read(s.h, field, ctypes.cast(ptr, ctypes.POINTER(ctypes.c_double))))


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s", "fp16s_all"])
@pytest.mark.parametrize("dim,n,bc", LATTICES)
def test_page_locked_equals_pageable(storage, dim, n, bc):
    import torch

    params = params_for(dim, n, bc)
    s = mplb.Solver(params, storage=storage)
    s.init(*inputs.random_state(params, seed=12))
    s.step(3)
    pad = 17
    pin = torch.full((s.N + 2 * pad,), -7.0, dtype=torch.float64, pin_memory=True)
    for field in range(6):
        want = s.read(field).reshape(-1)
        read_into(s, field, pin.data_ptr() + 8 * pad)
        got = pin.numpy()
        assert np.array_equal(got[pad:-pad], want), field
        assert (got[:pad] == -7.0).all() and (got[-pad:] == -7.0).all()


@pytest.mark.parametrize("dim,n,bc", LATTICES)
def test_fields_against_the_oracle(dim, n, bc):
    params = params_for(dim, n, bc)
    po, f, g = noisy_state(params, *inputs.random_state(params, seed=31), seed=2)
    s = gpu_solver(params, "fp64", state=(f, g))
    want, got = oracle.fields(po, f, g), s.fields()
    for k in ("phi", "rho", "u", "p"):
        # a few dozen roundings of values bounded by the array's largest
        assert np.abs(got[k] - want[k]).max() <= 1e-12 * max(np.abs(want[k]).max(), 1e-300), k
