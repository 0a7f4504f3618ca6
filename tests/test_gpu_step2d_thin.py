"""2-D lattices of few columns or few rows, whose tiles are one to 32 cells wide
and up to 256 high, or 32 to 256 wide and one to eight high: one step against the
FP64 oracle at the one-step bars (FP64 1e-12, FP32 2e-6) over all boundary
mixes; bit for bit the columns (rows) of a wide (high) lattice with the same
state in each of them, and long rows bit for bit their own period, in every
format; and a batch of all of them bit for bit the solvers alone."""
import numpy as np
import pytest

import oracle
from paper_2101_06769_amd import inputs
from tests.helpers import from_abi, gpu_available, rel_err
from tests.test_gpu_degenerate import params_for
from tests.test_gpu_parity import TOL1, gpu_solver, noisy_state
from tests.test_gpu_step2d import BCS

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2101_06769_amd import mplb

# edges of the tiles: 256, 128 and 64 rows by 1, 2 and 4 columns, and few rows
SIZES = [(1, 255), (1, 257), (1, 600), (2, 128), (2, 129), (3, 200), (4, 64), (4, 65), (5, 33), (8, 70),
         (255, 1), (257, 1), (600, 1), (65, 1), (128, 2), (129, 2), (300, 2), (65, 3), (130, 5), (97, 6),
         (96, 7), (65, 8), (100, 9)]
# rows of more than 65536 cells: tiles of 256 x 1, 128 x 2 and 32 x 8
LONG = [(65601, 1), (65600, 2), (65537, 5), (65664, 6)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("bc", BCS)
def test_one_step_against_the_oracle(storage, bc):
    for i, (nx, ny) in enumerate(SIZES):
        params = params_for(2, (nx, ny, 1), bc + (0,))
        params["collision"] = i % 2
        phi, u, p = inputs.random_state(params, seed=5 + i)
        po, f, g = noisy_state(params, phi, u, p, seed=i)
        s = gpu_solver(params, storage, state=(f, g))
        s.step(1)
        f1, g1 = oracle.step(po, f, g, 1)
        ef = rel_err(from_abi(2, s.get_populations(0)), f1)
        eg = rel_err(from_abi(2, s.get_populations(1)), g1)
        assert ef < TOL1[storage] and eg < TOL1[storage], (nx, ny, bc, ef, eg)


@pytest.mark.parametrize("bcy", [0, 1, 2])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s", "fp16s_all"])
@pytest.mark.parametrize("ny", [1, 2, 5, 6])
def test_long_rows_repeat_short_ones(storage, ny, bcy):
    times = 110  # 600 cells a period: tiles of 64 x 4, and of 256 x 1, 128 x 2, 32 x 8
    for collision in (0, 1):
        params = dict(params_for(2, (600, ny, 1), (0, bcy, 0)), collision=collision)
        fields = inputs.random_state(params, seed=13)
        short = mplb.Solver(params, storage=storage)
        short.init(*fields)
        long = mplb.Solver(dict(params, n=(600 * times, ny, 1)), storage=storage)
        long.init(*(np.concatenate([f] * times, -1) for f in fields))
        for _ in range(3):
            short.step(1)
            long.step(1)
        for w in (0, 1):
            parts = np.split(long.get_populations(w), times, -1)
            want = short.get_populations(w)
            assert all(np.array_equal(part, want) for part in parts), (collision, w)


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s", "fp16s_all"])
@pytest.mark.parametrize("axis,thick,length", [(0, 1, 700), (0, 2, 300), (0, 3, 150), (0, 5, 90), (1, 1, 700),
                                               (1, 2, 300), (1, 5, 200), (1, 7, 130), (1, 1, 65601),
                                               (1, 2, 65665), (1, 5, 65600), (1, 6, 65537)])
def test_thin_equals_a_slice_of_thick(storage, bc, axis, thick, length):
    # nothing varies along `axis`, which is periodic; bc along the other
    for collision in (0, 1):
        n, wide = [length, length, 1], [length, length, 1]
        n[axis], wide[axis] = thick, 128 if axis == 0 else 12
        bcs = [bc, bc, 0]
        bcs[axis] = 0
        line = list(n)
        line[axis] = 1
        fields = inputs.random_state(params_for(2, line, bcs), seed=11)
        states = []
        for size in (n, wide):
            params = dict(params_for(2, size, bcs), collision=collision)
            s = mplb.Solver(params, storage=storage)
            numpy_axis = 2 - axis
            phi, p = (np.repeat(a, size[axis], numpy_axis) for a in (fields[0], fields[2]))
            s.init(phi, np.repeat(fields[1], size[axis], numpy_axis + 1), p)
            for _ in range(5):
                s.step(1)
            states.append([s.get_populations(w) for w in (0, 1)])
        for thin, thicker in zip(*states):
            cut = [slice(None)] * 4
            cut[3 - axis] = slice(0, thick)
            assert np.array_equal(thin, thicker[tuple(cut)]), (collision, n, bc)


@pytest.mark.parametrize("collision,cac_edf", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s", "fp16s_all"])
def test_batch_equals_alone_bitwise(storage, collision, cac_edf):
    b = mplb.Batch(2, storage, capacity=len(SIZES + LONG), max_tiles=1 << 14)
    b.set_graph_chunk(4)
    pairs = []
    for i, (nx, ny) in enumerate(SIZES + LONG):
        params = params_for(2, (nx, ny, 1), BCS[i % len(BCS)] + (0,))
        params.update(collision=collision, cac_edf=cac_edf)
        fields = inputs.random_state(params, seed=40 + i)
        a = mplb.Solver(params, storage=storage)
        s = mplb.Solver(params, storage=storage, stream=b.stream)
        a.init(*fields)
        s.init(*fields)
        a.step(7)
        b.attach(s, 7)
        pairs.append((a, s))
    b.step(7)
    for (nx, ny), (a, s) in zip(SIZES + LONG, pairs):
        for w in (0, 1):
            assert np.array_equal(a.get_populations(w), s.get_populations(w)), (nx, ny, w)
