"""Batches whose domains do not fit the Infinity Cache (256 MiB for both levels of
the populations) together: they advance in groups that do, domains beyond it in
one more, and all together where there would be more than 32 groups.  Every
domain bit for bit itself alone, over graph chunks and the steps left of one,
with windows that end in between and domains that leave and come."""
import numpy as np
import pytest

from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    from paper_2101_06769_amd import mplb

CACHE = 256 << 20


def populations(dim, storage, n):
    per = {"fp64": 16, "fp32": 8, "fp16s": 6, "fp16s_all": 4}[storage] * 2 * (9 if dim == 2 else 27)
    return per * ((int(np.prod(n)) + 63) // 64 * 64)


def check_batch(dim, storage, sizes, bc, steps, chunk, leave=None):
    """Domains of these sizes for these numbers of steps each; `leave`: one that is
    detached after the first call and comes back for the rest of its steps."""
    cases = []
    for i, n in enumerate(sizes):
        params = params_for(dim, n, bc)
        cases.append((params, inputs.random_state(params, seed=30 + i)))
    want = []
    for (params, fields), k in zip(cases, steps):
        s = mplb.Solver(params, storage=storage)
        s.init(*fields)
        s.step(k)
        want.append([s.get_populations(w) for w in (0, 1)])
        del s
    b = mplb.Batch(dim, storage, capacity=len(sizes) + 3, max_tiles=1 << 18)
    b.set_graph_chunk(chunk)
    b.set_solo_cells(1 << 40)  # all share launches
    solvers, slots = [], []
    for (params, fields), k in zip(cases, steps):
        s = mplb.Solver(params, storage=storage, stream=b.stream)
        s.init(*fields)
        solvers.append(s)
        slots.append(b.attach(s, k))
    b.step(chunk + 3)
    if leave is not None:
        b.detach(slots[leave])
        b.step(2)  # the others, regrouped
        slots[leave] = b.attach(solvers[leave], steps[leave] - (chunk + 3))
    b.step(max(steps))
    for i, (s, k) in enumerate(zip(solvers, steps)):
        assert s.steps_done() == k, i
        for w in (0, 1):
            assert np.array_equal(s.get_populations(w), want[i][w]), (storage, sizes[i], w)
    del solvers, b
    torch.cuda.empty_cache()


@pytest.mark.parametrize("leave", [None, 0, 2, 3])
@pytest.mark.parametrize("storage,sizes", [
    ("fp32", [(1000, 1001, 1), (90, 50, 1), (997, 1000, 1), (1400, 1400, 1), (30, 200, 1)]),
    ("fp64", [(700, 700, 1), (90, 50, 1), (705, 701, 1), (1100, 900, 1), (70, 50, 1)]),
    ("fp16s", [(1200, 1101, 1), (90, 50, 1), (1201, 1100, 1), (1700, 1500, 1), (20, 70, 1)]),
])
def test_2d_groups(storage, sizes, leave):
    total = [populations(2, storage, n) for n in sizes]
    assert total[0] + total[2] > CACHE >= max(total[0], total[2]) and total[3] > CACHE
    check_batch(2, storage, sizes, (0, 1, 0), [13, 8, 17, 15, 17], 4, leave)


@pytest.mark.parametrize("leave", [None, 0, 1, 3])
@pytest.mark.parametrize("storage,sizes", [
    # the phi-summing update (64-cell rows), packed planes, a domain beyond the cache
    ("fp32", [(64, 64, 90), (48, 80, 90), (20, 9, 8), (96, 96, 72), (128, 8, 9)]),
    ("fp64", [(64, 40, 70), (48, 50, 80), (20, 9, 8), (64, 64, 90), (128, 8, 9)]),
    ("fp16s_all", [(64, 100, 100), (80, 80, 110), (20, 9, 8), (100, 100, 130), (128, 8, 9)]),
])
def test_3d_groups(storage, sizes, leave):
    total = [populations(3, storage, n) for n in sizes]
    assert total[0] + total[1] > CACHE >= max(total[0], total[1]) and total[3] > CACHE
    check_batch(3, storage, sizes, (0, 0, 1), [13, 17, 8, 15, 17], 4, leave)


def test_more_groups_than_there_may_be():
    # 34 domains, each more than half the cache: one streamed group
    n = (1000, 950, 1)
    assert CACHE // 2 < populations(2, "fp32", n) <= CACHE
    params = params_for(2, n, (0, 1, 0))
    fields = [inputs.random_state(params, seed=50 + i) for i in range(2)]
    steps = [5, 7, 10]
    want = {}
    for i in range(2):
        for k in steps:
            s = mplb.Solver(params, storage="fp32")
            s.init(*fields[i])
            s.step(k)
            want[i, k] = s.get_populations(1)
    b = mplb.Batch(2, "fp32", capacity=34, max_tiles=1 << 18)
    b.set_graph_chunk(4)
    solvers = []
    for i in range(34):
        s = mplb.Solver(params, storage="fp32", stream=b.stream)
        s.init(*fields[i % 2])
        b.attach(s, steps[i % 3])
        solvers.append(s)
    b.step(10)
    for i, s in enumerate(solvers):
        assert s.steps_done() == steps[i % 3]
        assert np.array_equal(s.get_populations(1), want[i % 2, steps[i % 3]]), i
    del solvers, b
    torch.cuda.empty_cache()
