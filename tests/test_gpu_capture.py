"""mplb_step captured by its caller: an even number of steps ends at the level it
began at, so the graph can be replayed, each replay advancing the state by as
many steps.  Lattices that take four, three, two and one steps a launch, plain
and FP16 storage, and a 3-D one; every replay against the same steps of a solver
of its own, with reads and other device work between the replays."""
import numpy as np
import pytest

from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    from paper_2101_06769_amd import mplb

LATTICES = [("fp64", 2, (64, 96, 1)), ("fp32", 2, (130, 140, 1)), ("fp32", 2, (200, 200, 1)),
            ("fp32", 2, (400, 300, 1)), ("fp16s_all", 2, (64, 96, 1)), ("fp32", 3, (48, 10, 12))]


@pytest.mark.parametrize("steps", [2, 4, 6])
@pytest.mark.parametrize("storage,dim,n", LATTICES)
def test_replays_of_captured_steps(storage, dim, n, steps):
    params = params_for(dim, n, (0, 1, 0))
    fields = inputs.random_state(params, seed=21)
    stream = torch.cuda.Stream()
    a = mplb.Solver(params, storage=storage, stream=stream)
    b = mplb.Solver(params, storage=storage)
    for s in (a, b):
        s.init(*fields)
        s.step(9)
    a.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(steps)
    for rep in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        b.step(steps)
        assert float(torch.ones(1 << 16, device="cuda").sum()) == 1 << 16
        for w in (0, 1):
            assert np.array_equal(a.get_populations(w), b.get_populations(w)), (rep, w)
