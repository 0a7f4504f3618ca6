"""The one-launch 2-D step where its tiles can go wrong: rows
and columns at and beside the tile widths (8 to 64 cells by 256 threads), one
cell wide or high, every mix of periodic axes, walls and symmetry planes, and
both collision operators; one step against the FP64 oracle at the one-step
bars (FP64 1e-12, FP32 2e-6); runs of steps (several a launch on small lattices)
bit for bit the same steps one by one; and a batch of all of them, empty slots between
them, bit for bit the solvers alone over steps launched one by one and as
graphs."""
import numpy as np
import pytest

import oracle
from paper_2101_06769_amd import inputs
from tests.helpers import from_abi, gpu_available, rel_err
from tests.test_gpu_degenerate import params_for
from tests.test_gpu_parity import TOL1, gpu_solver, noisy_state

pytestmark = pytest.mark.gpu

if gpu_available():
    from paper_2101_06769_amd import mplb

SIZES = [(1, 1), (1, 33), (2, 5), (7, 9), (8, 32), (9, 31), (16, 17), (31, 8), (32, 9), (33, 4),
         (63, 3), (64, 4), (64, 1), (65, 5), (127, 2), (130, 12)]
BCS = [(0, 0), (0, 1), (0, 2), (1, 0), (1, 1), (1, 2), (2, 0), (2, 1), (2, 2)]


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


# two, three and four steps a launch (blocks of 16, 12 and 8 cells a side), and single steps
RUN_SIZES = [(1, 1), (1, 40), (3, 2), (8, 8), (9, 7), (17, 25), (64, 64), (130, 130), (131, 97),
             (200, 200), (245, 210), (400, 300)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("bc", BCS)
def test_runs_equal_single_steps_bitwise(storage, bc):
    for i, (nx, ny) in enumerate(RUN_SIZES):
        params = params_for(2, (nx, ny, 1), bc + (0,))
        params["collision"] = i % 2
        params["cac_edf"] = int(i % 5 == 4)
        fields = inputs.random_state(params, seed=70 + i)
        a, b = (mplb.Solver(params, storage=storage) for _ in range(2))
        a.init(*fields)
        b.init(*fields)
        for _ in range(43):
            a.step(1)
        for n in (2, 1, 40):  # direct launches, then graphs from either level and a rest
            b.step(n)
        assert a.steps_done() == b.steps_done() == 43
        for w in (0, 1):
            assert np.array_equal(a.get_populations(w), b.get_populations(w)), (nx, ny, bc, w)


@pytest.mark.parametrize("storage", ["fp16s", "fp16s_all"])
@pytest.mark.parametrize("bc", [(0, 0), (0, 1), (1, 2), (2, 1)])
def test_fp16_checkpoints_at_either_level(storage, bc):
    # the references of a level lie in one of two arrays; a state saved at
    # either resumes bit for bit, and fields and populations read between
    # steps leave it alone
    for i, (nx, ny) in enumerate(SIZES):
        params = params_for(2, (nx, ny, 1), bc + (0,))
        params["collision"] = i % 2
        fields = inputs.random_state(params, seed=90 + i)
        a, b = (mplb.Solver(params, storage=storage) for _ in range(2))
        a.init(*fields)
        a.step(7 + i % 2)
        b.load(a.save())
        assert np.array_equal(a.read(mplb.FIELD_UX), b.read(mplb.FIELD_UX))
        a.reduce()
        a.step(5)
        b.step(5)
        for w in (0, 1):
            assert np.array_equal(a.get_populations(w), b.get_populations(w)), (nx, ny, w)


@pytest.mark.parametrize("collision,cac_edf", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s", "fp16s_all"])
def test_batch_equals_alone_bitwise(storage, collision, cac_edf):
    cases = []
    for i, (nx, ny) in enumerate(SIZES):
        params = params_for(2, (nx, ny, 1), BCS[i % len(BCS)] + (0,))
        params.update(collision=collision, cac_edf=cac_edf)
        cases.append((params,) + tuple(inputs.random_state(params, seed=40 + i)))
    b = mplb.Batch(2, storage, capacity=80, max_tiles=1 << 12)
    solvers, alone = [], []
    for params, phi, u, p in cases * 4:  # more domains than one load of tile counts
        s = mplb.Solver(params, storage=storage, stream=b.stream)
        s.init(phi, u, p)
        solvers.append((s, b.attach(s, 21)))
    for k in (0, 5, 6, 40, 63):  # empty slots
        b.detach(solvers[k][1])
    b.step(37)
    for k, (s, _) in enumerate(solvers):
        if k < len(cases):
            a = mplb.Solver(cases[k][0], storage=storage)
            a.init(*cases[k][1:])
            a.step(21)
            alone.append([a.get_populations(w) for w in (0, 1)])
        steps = 0 if k in (0, 5, 6, 40, 63) else 21
        assert s.steps_done() == steps
        if steps:
            want = alone[k % len(cases)]
            assert all(np.array_equal(s.get_populations(w), want[w]) for w in (0, 1)), k
