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

}  // namespace mplb
