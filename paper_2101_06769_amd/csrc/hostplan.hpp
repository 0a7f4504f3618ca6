// Decisions of the host code that need no device: plain C++, so that they can be
// compiled and tested without one.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace mplb {

// What the runtime says of one address of host memory: whether it is
// page-locked, where the device sees it, and the allocation or registration
// around it in device addresses.
struct HostRange {
    bool page_locked = false;
    uintptr_t device = 0, start = 0;
    size_t bytes = 0;
};

// The device address of `bytes` of host memory at `host`, or 0 where a kernel
// must not write there itself: pageable or managed memory, memory that is
// not 8-byte aligned, or a buffer that one page-locked range does not hold to
// its end.  Both ends alone say nothing: the device commonly sees page-locked
// memory at its host address, so two ranges with pageable memory between them
// look like one.  query: HostRange of an address, false where the runtime
// cannot tell.
// pending: an earlier error that the caller of the library has yet to see; nothing is
// asked then, since the answer could take that error's place.
template <class Query>
uintptr_t direct_address(uintptr_t host, size_t bytes, bool pending, Query &&query)
{
    HostRange r;
    if (pending || host % 8 != 0 || !query(host, r) || !r.page_locked || r.device == 0) return 0;
    if (r.device < r.start) return 0;
    const size_t before = r.device - r.start;
    return before <= r.bytes && bytes <= r.bytes - before ? r.device : 0;
}

// Launch sizes of the batched kernels (surplus blocks find no tile and exit).
// A captured graph holds its sizes, so it outlives a change of the domains only
// where the old size serves the new count of tiles: enough blocks, and
// at most half more than needed (one of four equal domains or more may go and
// come; the surplus cost nothing measurable: 24 2-D domains of 64 to 200 a side
// less 8 of them 12.8 us a step with either size).
inline int launch_blocks(int tiles)
{
    int step = 1;  // up by at most an eighth
    while (step <= tiles / 16) step <<= 1;
    return (tiles + step - 1) / step * step;
}
inline bool blocks_serve(int blocks, int tiles)
{
    return tiles == 0 ? blocks == 0 : blocks >= tiles && blocks - tiles <= tiles / 2 + 32;
}

// The domains that share a batch's launches in groups whose populations (both
// levels) fit the Infinity Cache together, as few and as even as the
// largest-first rule makes them.  A group takes a chunk of steps while its
// values stay in the cache; stepped all at once, every step would stream all of
// them from HBM.  Domains too large for it share one more group, and so does
// everything when the groups would exceed max_groups.  cells: per domain;
// fits: whether a number of cells fits.
struct CacheGroup {
    bool kept;                // its populations stay in the cache
    std::vector<int> members;  // indices of cells, ascending
    long long cells;
};
template <class Fits>
std::vector<CacheGroup> cache_groups(const std::vector<long long> &cells, size_t max_groups, Fits &&fits)
{
    std::vector<int> small, large;
    for (int i = 0; i < int(cells.size()); ++i) (fits(cells[i]) ? small : large).push_back(i);
    std::stable_sort(small.begin(), small.end(), [&](int x, int y) { return cells[x] > cells[y]; });
    const size_t most = max_groups - (large.empty() ? 0 : 1);
    std::vector<CacheGroup> out;
    for (size_t n = small.empty() ? 0 : 1; n <= most; ++n) {
        out.assign(n, CacheGroup{true, {}, 0});
        bool ok = true;
        for (int i : small) {
            CacheGroup *to = &out[0];
            for (CacheGroup &c : out)
                if (c.cells < to->cells) to = &c;
            to->members.push_back(i);
            to->cells += cells[i];
            ok = ok && fits(to->cells);
        }
        if (ok) break;
        if (n == most) {
            out.clear();
            large.insert(large.end(), small.begin(), small.end());
        }
    }
    if (!large.empty()) out.push_back(CacheGroup{false, large, 0});
    for (CacheGroup &c : out) std::sort(c.members.begin(), c.members.end());
    return out;
}

// Packed planes on 3-D lattices periodic in x and y, the arrays within 32-bit
// indices, where rows would leave lanes idle.  Per step, rows and packed: FP32
// 97 x 96 x 200 282 and 201 us, 200 x 100 x 150 409 and 326, 300 x 100 x 100 541 and
// 350, 320 x 128 x 160 850 and 694; FP64 96 x 96 x 200 405 and 386; FP16S_ALL
// 96 x 96 x 384 334 and 282.  Rows stay where they fill 3/4 of their blocks and
// start at cache lines in FP32, which a packed wavefront's would straddle
// (96 x 96 x 384 364 and 374, 576 x 100 x 100 586 and 594).
// A plane of few cells fills little of its block: the block's own form stays where
// packed planes would take more lanes than pack_fifths / 5 times its own.
constexpr long long PACK_BLOCK = 256;
struct Shape3 {
    long long nx, ny, nz, bx, by, bz;  // lattice and block
    bool plain, fp32, kept;            // storage FP64 or FP32; FP32; populations in the cache
    bool pulls_twice;                  // FP16S_ALL with a single relaxation time
};
inline long long up_to(long long n, long long b) { return (n + b - 1) / b * b; }
inline long long block_lanes(const Shape3 &s)
{
    return up_to(s.nx, s.bx) * up_to(s.ny, s.by) * up_to(s.nz, s.bz);
}
inline long long pack_lanes(const Shape3 &s) { return up_to(s.nx * s.ny, PACK_BLOCK) * s.nz; }
// Rows: 4 times in plain storage and as many in the FP16 formats (100 x 1 x 3000,
// twice the lanes, FP32 39 and 33 us a step, FP16S_ALL 40 and 48; 33 x 3 x 3030, as
// many, FP16S_ALL 57 and 50), four fifths where the update pulls its FP16 codes
// twice (single relaxation time, as many lanes: 63 x 178 x 178 276 and 308, 100 x 3
// x 1000 67 and 79).  Per-lane blocks (not whole wavefronts wide), of more integer
// work a lane: 8 and 4 times (32 x 1 x 9375, 8 times, FP32 48 and 43, FP16S_ALL 54
// and 64; 9 x 3 x 11111, 4 times, FP16S_ALL 102 and 80; 16 x 1 x 18750, 16 times,
// FP32 48 and 75; 1 x 1 x 300000, 256 times, FP32 48 and 1017).
inline long long pack_fifths(const Shape3 &s)
{
    if (s.bx % 64 != 0) return s.plain ? 40 : 20;
    return s.plain ? 20 : s.pulls_twice ? 4 : 5;
}
inline bool packs_planes(const Shape3 &s)
{
    if (5 * pack_lanes(s) > pack_fifths(s) * block_lanes(s)) return false;
    if (s.bx % 64 != 0) return true;
    if (s.kept) return s.nx % 64 != 0;
    const long long wide = up_to(s.nx, s.bx);
    return wide != s.nx && !(s.fp32 && s.nx % 32 == 0 && 4 * s.nx >= 3 * wide);
}

// Whether blocks a wavefront wide take the place of a lattice's own, whose rows
// would fill less than 3/4 of it: from 50 000 cells (less do not fill the chip
// either way; 300 x 10 x 10 FP16S_ALL 13.3 us a step and 14.2 with them) where
// whole wavefronts are at least 4/5 full (320 cells take two blocks of 256), and
// on plain lattices of 200 000 cells and more in the Infinity Cache.  Lattices with walls or symmetry planes in x or y:
// the others are packed.  Per step, wide and narrow: 320 x 79 x 79 FP32 257 and
// 207 us, FP16S_ALL 219 and 177; 160 x 111 x 111 FP64 460 and 427; 129 x 48 x 48 FP32
// 53 and 47; but 129 x 124 x 124 FP32 331 and 395, FP16S_ALL 294 and 361, 129 x 48 x
// 48 49 and 59, FP32 129 x 27 x 27 20 and 24, 129 x 7 x 7 12 and 18 (a third
// wavefront of one cell, and rows that are cut inside cache lines).
inline bool takes_narrow_blocks(const Shape3 &s)
{
    const long long wide = up_to(s.nx, s.bx), waves = up_to(s.nx, 64);
    const long long cells = s.nx * s.ny * s.nz;
    if (4 * s.nx >= 3 * wide || waves >= wide || cells < 50000) return false;
    return 5 * s.nx >= 4 * waves || (s.plain && s.kept && cells >= 200000);
}

// Whether the 2-D step stores its populations with ordinary stores: where they
// stay in the Infinity Cache (kept), and where rows do not start at 64-byte
// boundaries.  Lines that two rows or tiles share are then completed in L2;
// stored non-temporally, their parts went to HBM one by one.  elem: bytes of a value
// of g.  Beyond the cache, per step, non-temporal and ordinary: 129 x 46511 FP32
// 311 and 224 us, FP64 488 and 404, FP16S 291 and 228, FP16S_ALL 244 and 203; with
// 64-byte rows 400 x 7500 FP32 101 and 103, 96 x 31250 101 and 105, 200 x 15000
// FP64 194 and 206.
inline bool stores_stay2d(int nx, int elem, bool kept) { return kept || (long long)nx * elem % 64 != 0; }
// Columns of a tile of whole wavefronts.  An even number of tiles per row, with
// ordinary stores, shares the row evenly where the last one would otherwise be
// narrow, and beyond the cache in any case: with tiles of 64 and 1 column a step
// of 65 x 307 FP16S took 8.3 us, of 33 and 32 5.4; 65 x 92307 FP32 298 and 249,
// 100 x 60000 271 and 264, 200 x 1500 13.8 and 11.8.  Not an odd number (129 x
// 46511 FP32 224 and 238), nor with non-temporal stores (120 x 25000 FP64 183 and
// 201).
inline int tile_columns2d(int nx, bool stay, bool kept)
{
    const int tiles = (nx - 1) / 64 + 1, last = nx - (tiles - 1) * 64;
    return tiles % 2 == 0 && stay && (last < 32 || !kept) ? (nx - 1) / tiles + 1 : 64;
}

}  // namespace mplb
