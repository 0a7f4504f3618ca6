"""Decisions of the host code that need no device, built here with g++: when
mplb_read writes into the caller's memory itself, when a batch's captured graph
outlives a change of its domains, which domains of a batch advance together, and
which lattices take which launch shapes."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from tests.helpers import ROOT


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    out = str(tmp_path_factory.mktemp("plan") / "hostplan.so")
    subprocess.run([cxx, "-std=c++20", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2101_06769_amd", "csrc"),
                    os.path.join(ROOT, "tests", "hostplan.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def direct(plan, host, bytes_, ranges, pending=0):
    flat = [v for r in ranges for v in r]
    plan.direct_address.restype = ctypes.c_uint64
    asked = ctypes.c_int(0)
    got = plan.direct_address(ctypes.c_uint64(host), ctypes.c_uint64(bytes_), pending,
                              (ctypes.c_uint64 * len(flat))(*flat), len(ranges), ctypes.byref(asked))
    return got, asked.value


A, B, P = 0x10000, 0x40000, 0x1000  # two ranges, a page


@pytest.mark.parametrize("host,bytes_,ranges,want", [
    (A, 4 * P, [(A, A, 4 * P, 1)], A),                     # the whole range
    (A + 8, 4 * P - 8, [(A, A, 4 * P, 1)], A + 8),         # to its end
    (A + 8, 4 * P, [(A, A, 4 * P, 1)], 0),                 # one value beyond it
    (A, 8, [(A, A, 4 * P, 1)], A),                         # one value
    (A + 4, 8, [(A, A, 4 * P, 1)], 0),                     # not aligned
    (A, 4 * P, [(A, B, 4 * P, 1)], B),                     # seen elsewhere by the device
    (A, 4 * P, [(A, A, 4 * P, 0)], 0),                     # pageable or managed
    (A, 4 * P, [], 0),                                     # unknown to the runtime
    # locked at both ends, pageable between them
    (A, B + P - A, [(A, A, P, 1), (B, B, P, 1)], 0),
    # two ranges side by side: two registrations, which need not be seen side by side
    (A, 2 * P, [(A, A, P, 1), (A + P, A + P, P, 1)], 0),
    (A, 0xffffffffffffff00, [(A, A, 4 * P, 1)], 0),        # no wrap-around
])
def test_reads_write_into_one_page_locked_range_only(plan, host, bytes_, ranges, want):
    assert direct(plan, host, bytes_, ranges)[0] == want


def test_a_pending_error_is_left_for_the_launch_to_report(plan):
    # no query, whose own error would be cleared and the caller's with it
    assert direct(plan, A, 8, [(A, A, P, 1)], pending=1) == (0, 0)


def test_launches_of_a_batch_cover_every_tile(plan):
    for tiles in list(range(1, 300)) + [4095, 4096, 4097, 99999, (1 << 24) + 1, 0x3fffffff, 0x7fffffff // 2]:
        n = plan.launch_blocks(tiles)
        assert tiles <= n <= tiles + tiles // 8 and plan.blocks_serve(n, tiles)
        assert not plan.blocks_serve(tiles - 1, tiles)
        assert not plan.blocks_serve(2 * tiles + 33, tiles)
    # a kernel is launched exactly where it has tiles
    assert plan.launch_blocks(0) == 0
    assert plan.blocks_serve(0, 0) and not plan.blocks_serve(16, 0) and not plan.blocks_serve(0, 1)


@pytest.mark.parametrize("domains", [4, 5, 8, 12, 20, 60])
@pytest.mark.parametrize("tiles", [1, 7, 33, 250, 4000])
def test_one_domain_may_leave_and_come_back(plan, domains, tiles):
    # the graph captured for all of them serves the others, and all of them again
    blocks = plan.launch_blocks(domains * tiles)
    assert plan.blocks_serve(blocks, (domains - 1) * tiles)
    assert plan.blocks_serve(blocks, domains * tiles)


def groups_of(plan, cells, limit, most=32):
    group, kept = (ctypes.c_int * len(cells))(*[-1] * len(cells)), (ctypes.c_int * (most + 1))()
    n = plan.cache_groups((ctypes.c_int64 * len(cells))(*cells), len(cells), ctypes.c_int64(limit), most,
                          group, kept)
    return n, list(group), list(kept)


def check_groups(plan, cells, limit, most=32):
    n, group, kept = groups_of(plan, cells, limit, most)
    assert 0 <= n <= most
    load = [sum(c for c, k in zip(cells, group) if k == j) for j in range(n)]
    assert all(0 <= k < n for k in group) and all(x > 0 for x in load)
    for j in range(n):
        assert load[j] <= limit if kept[j] else j == n - 1, (j, load)
    return n, load, kept


def test_cache_groups_of_a_batch(plan):
    assert groups_of(plan, [], 100)[0] == 0
    assert check_groups(plan, [100], 100)[0] == 1
    n, load, kept = check_groups(plan, [101], 100)
    assert n == 1 and not kept[0]
    # as few and as even as the largest-first rule makes them
    n, load, kept = check_groups(plan, [60, 50, 40, 30, 10], 100)
    assert n == 2 and sorted(load) == [90, 100]
    # a domain beyond the cache in a group of its own, the last one
    n, load, kept = check_groups(plan, [30, 500, 60, 40], 100)
    assert n == 3 and load[2] == 500 and kept[:3] == [1, 1, 0]
    # as many groups as there may be, and one too many: all of them together
    n, load, kept = check_groups(plan, [90] * 32, 100)
    assert n == 32 and all(kept[:32])
    for cells in ([90] * 33, [90] * 32 + [500]):
        n, load, kept = check_groups(plan, cells, 100)
        assert n == 1 and not kept[0] and load == [sum(cells)]
    rng = random.Random(3)
    for _ in range(300):
        cells = [rng.randint(1, rng.choice([20, 100, 150])) for _ in range(rng.randint(1, 70))]
        check_groups(plan, cells, 100, rng.choice([2, 5, 32]))


def pow2(v, cap):
    b = 1
    while b < v and b < cap:
        b *= 2
    return b


def default_block(nx, ny, nz):
    bx = pow2(nx, 256)
    by = pow2(ny, 256 // bx)
    return bx, by, pow2(nz, 256 // (bx * by))


def packs(plan, n, storage, kept=1, block=None):
    a = (ctypes.c_int * 6)(*n, *(block or default_block(*n)))
    plan.lanes.restype = ctypes.c_int64
    return bool(plan.packs_planes(a, storage, kept)), plan.lanes(a, 1), plan.lanes(a, 0)


def test_packed_planes_do_not_multiply_the_lanes(plan):
    # planes of few cells: a block of 256 threads each
    for n in [(1, 1, 300000), (2, 1, 150000), (3, 1, 100000), (1, 10, 30000), (16, 1, 18750), (3, 3, 33333)]:
        for storage in range(4):
            assert not packs(plan, n, storage)[0], (n, storage)
    for nx in [1, 2, 3, 5, 9, 16, 20, 24, 33, 48, 63, 65, 100, 127, 129, 200, 300]:
        for ny in [1, 2, 3, 7, 10, 50]:
            for nz in [1, 7, 1000]:
                for storage in range(4):
                    took, packed, blocks = packs(plan, (nx, ny, nz), storage)
                    assert not took or packed <= (8 if storage < 2 else 4) * blocks
    # what packed planes are for
    for n in [(97, 96, 200), (48, 48, 192), (32, 32, 128), (100, 3, 1000), (9, 10, 3333), (20, 10, 1500)]:
        for storage in range(4):
            assert packs(plan, n, storage)[0], (n, storage)
    # FP16S_ALL with a single relaxation time: where they save a fifth of the lanes
    for n in [(63, 178, 178), (100, 3, 1000), (129, 1, 2325), (127, 125, 125)]:
        assert not packs(plan, n, 4, kept=0)[0] and not packs(plan, n, 4)[0], n
    assert packs(plan, (96, 96, 384), 4, kept=0)[0] and packs(plan, (200, 100, 50), 4)[0]
    assert not packs(plan, (128, 64, 64), 1)[0] and not packs(plan, (96, 96, 384), 1, kept=0)[0]
    assert packs(plan, (128, 64, 64), 1, block=(8, 4, 1))[0]  # not whole wavefronts wide


def test_narrow_blocks_only_where_they_fill(plan):
    def narrow(n, storage, kept):
        return bool(plan.narrow_blocks((ctypes.c_int * 6)(*n, *default_block(*n)), storage, kept))

    for storage in range(4):
        for kept in (0, 1):
            assert narrow((320, 79, 79), storage, kept) and narrow((160, 111, 111), storage, kept)
            assert not narrow((200, 50, 50), storage, kept) and not narrow((64, 50, 50), storage, kept)
            assert not narrow((40, 40, 40), storage, kept) and not narrow((65, 40, 40), storage, kept)
            assert not narrow((300, 10, 10), storage, kept) and not narrow((320, 9, 9), storage, kept)
        # a third wavefront of one cell
        assert not narrow((129, 124, 124), storage, 0) and not narrow((129, 27, 27), storage, 1)
        assert narrow((129, 48, 48), storage, 1) == (storage < 2)


def test_2d_rows_are_covered_by_their_tiles(plan):
    for nx in list(range(33, 1100)) + [65537, 100000, 1 << 29, 2 ** 31 - 65]:
        tiles = (nx - 1) // 64 + 1
        for kept in (0, 1):
            for stay in ((1,) if kept else (0, 1)):
                cols = plan.tile_columns2d(nx, stay, kept)
                assert 1 <= cols <= 64 and (tiles - 1) * cols < nx <= tiles * cols, (nx, kept, stay, cols)
                assert stay or cols == 64
    assert plan.tile_columns2d(65, 1, 1) == 33 and plan.tile_columns2d(129, 1, 1) == 64
    assert plan.tile_columns2d(100, 1, 0) == 50 and plan.tile_columns2d(100, 1, 1) == 64
    for nx, elem, want in [(65, 4, 1), (80, 4, 0), (72, 4, 1), (72, 8, 0), (64, 2, 0), (80, 2, 1), (2 ** 31 - 65, 8, 1)]:
        assert plan.stores_stay2d(nx, elem, 0) == want and plan.stores_stay2d(nx, elem, 1) == 1
