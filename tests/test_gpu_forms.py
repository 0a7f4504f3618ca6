"""Addressing forms against each other, bit for bit: a 3-D domain alone takes
packed planes (ragged rows, x and y periodic) or rows, and in a batch the form
that all its domains share, so the same domain is compared packed against
rows and the general form, in every format and with both collision operators;
and lattices on either side of the Infinity Cache's size, where the same state
repeats along one axis and the kernels differ in how they store it."""
import numpy as np
import pytest

from paper_2101_06769_amd import inputs
from tests.helpers import gpu_available
from tests.test_gpu_degenerate import params_for

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch

    from paper_2101_06769_amd import mplb

FORMATS = ["fp64", "fp32", "fp16s", "fp16s_all"]


def domain(n, bc, seed, collision, cac_edf=0, dim=3):
    params = params_for(dim, n, bc)
    params.update(collision=collision, cac_edf=cac_edf)
    return params, inputs.random_state(params, seed=seed)


def state(s):
    return [s.get_populations(w) for w in (0, 1)]


def alone(params, fields, storage, steps, partials=1):
    s = mplb.Solver(params, storage=storage)
    s.set_phi_partials(partials)
    s.init(*fields)
    s.step(steps)
    return state(s)


def batch_equals_alone(domains, storage, steps, partials=1, chunk=4):
    """Every domain in one batch against the same domain alone."""
    b = mplb.Batch(3, storage, capacity=len(domains), max_tiles=1 << 14)
    b.set_graph_chunk(chunk)
    solvers = []
    for params, fields in domains:
        s = mplb.Solver(params, storage=storage, stream=b.stream)
        s.set_phi_partials(partials)
        s.init(*fields)
        b.attach(s, steps)
        solvers.append(s)
    b.step(steps)
    for s, (params, fields) in zip(solvers, domains):
        for got, want in zip(state(s), alone(params, fields, storage, steps, partials)):
            assert np.array_equal(got, want), (storage, params["n"], params["bc"])


# the domain beside a packed one that takes the batch out of the packed form:
# walls in y (rows for all) and walls in x (the general form for all)
BESIDE = {"rows": ((70, 6, 5), (0, 1, 0)), "general": ((70, 6, 5), (1, 0, 0))}


@pytest.mark.parametrize("cac_edf", [0, 1])
@pytest.mark.parametrize("collision", [0, 1])
@pytest.mark.parametrize("storage", FORMATS)
@pytest.mark.parametrize("beside", BESIDE)
def test_packed_alone_equals_rows_and_general_in_a_batch(storage, beside, collision, cac_edf):
    n, bc = BESIDE[beside]
    domains = [domain((21, 10, 9), (0, 0, 1), 1, collision, cac_edf),
               domain((100, 5, 4), (0, 0, 2), 2, collision, cac_edf),
               domain((36, 7, 6), (0, 0, 0), 3, collision, cac_edf),
               domain(n, bc, 4, collision, cac_edf)]
    batch_equals_alone(domains, storage, 7)


@pytest.mark.parametrize("collision", [0, 1])
@pytest.mark.parametrize("storage", FORMATS)
def test_rows_alone_equal_packed_in_a_batch(storage, collision):
    # rows of whole wavefronts, phi from the pulled values: rows alone, packed
    # beside the ragged domain
    domains = [domain((64, 6, 5), (0, 0, 1), 5, collision), domain((128, 5, 4), (0, 0, 0), 6, collision),
               domain((48, 7, 6), (0, 0, 2), 7, collision)]
    batch_equals_alone(domains, storage, 7, partials=0)


@pytest.mark.parametrize("collision", [0, 1])
@pytest.mark.parametrize("storage", FORMATS)
def test_phi_summing_domains_beside_a_packed_one(storage, collision):
    # the packed phi stage merges the partial sums of the two domains whose
    # update sums phi
    domains = [domain((64, 8, 5), (0, 0, 1), 8, collision), domain((128, 4, 6), (0, 0, 0), 9, collision),
               domain((48, 7, 6), (0, 0, 1), 10, collision)]
    for params, fields in domains:
        s = mplb.Solver(params, storage=storage)
        s.init(*fields)
        assert s.uses_phi_partials() == (params["n"][0] % 64 == 0)
    batch_equals_alone(domains, storage, 9)


# one period, the axis it repeats along, and how often: the populations of the
# repeated lattice exceed 256 MiB in every format, those of the period do not
LARGE = [(2, (24, 500, 1), (0, 0, 0), 1, 320), (2, (24, 500, 1), (1, 0, 0), 1, 320),
         (2, (100, 500, 1), (2, 0, 0), 1, 80), (2, (128, 500, 1), (0, 0, 0), 1, 64),
         (2, (100, 500, 1), (0, 0, 0), 1, 80),
         (2, (65, 500, 1), (1, 0, 0), 1, 130), (2, (193, 300, 1), (0, 0, 0), 1, 70),
         (2, (75, 400, 1), (2, 0, 0), 1, 130), (2, (129, 300, 1), (0, 0, 0), 1, 100),
         (3, (36, 10, 31), (0, 0, 0), 2, 120), (3, (36, 10, 31), (0, 1, 0), 2, 120),
         (3, (64, 8, 31), (0, 0, 0), 2, 80), (3, (128, 6, 31), (0, 1, 0), 2, 60)]


@pytest.mark.parametrize("collision", [0, 1])
@pytest.mark.parametrize("storage", FORMATS)
@pytest.mark.parametrize("dim,n,bc,axis,times", LARGE)
def test_beyond_the_cache_equals_within(storage, dim, n, bc, axis, times, collision):
    params, fields = domain(n, bc, 11, collision, dim=dim)
    small = mplb.Solver(params, storage=storage)
    small.init(*fields)
    big_n = list(n)
    big_n[axis] *= times
    big_params = dict(params, n=tuple(big_n))
    numpy_axis = 2 - axis  # fields are [z][y][x]
    phi, u, p = (np.repeat(a[None], times, 0) for a in fields)
    phi, p = (np.concatenate(list(a), numpy_axis) for a in (phi, p))
    u = np.concatenate(list(u), numpy_axis + 1)
    big = mplb.Solver(big_params, storage=storage)
    assert big.nbytes > (256 << 20) > small.nbytes
    big.init(phi, u, p)
    big.step(3)
    small.step(3)
    for field in (mplb.FIELD_PHI, mplb.FIELD_UX, mplb.FIELD_UY, mplb.FIELD_P):
        got, want = big.read(field), small.read(field)
        for part in np.split(got, times, numpy_axis):
            assert np.array_equal(part, want), field
    torch.cuda.empty_cache()
