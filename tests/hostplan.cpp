// The host decisions of csrc/hostplan.hpp behind C functions, for
// test_hostplan.py (built with g++, no device).
#include "hostplan.hpp"

extern "C" {

// n ranges of host memory (host address, device address, bytes, page-locked): the
// address that a read of `bytes` at `host` writes to, 0 for the staging array.
// asked: how often the ranges were looked up.
uint64_t direct_address(uint64_t host, uint64_t bytes, int pending, const uint64_t *ranges, int n, int *asked)
{
    return mplb::direct_address(host, bytes, pending != 0, [&](uintptr_t at, mplb::HostRange &r) {
        ++*asked;
        for (int i = 0; i < n; ++i) {
            const uint64_t *q = ranges + 4 * i;
            if (at < q[0] || at >= q[0] + q[2]) continue;
            r.page_locked = q[3] != 0;
            r.device = q[1] + (at - q[0]);
            r.start = q[1];
            r.bytes = q[2];
            return true;
        }
        return false;
    });
}

int launch_blocks(int tiles) { return mplb::launch_blocks(tiles); }
int blocks_serve(int blocks, int tiles) { return mplb::blocks_serve(blocks, tiles); }

// The cache groups of n domains where `limit` cells fit: per domain its group in
// group[], per group whether it is kept in kept[]; the number of groups.
int cache_groups(const int64_t *cells, int n, int64_t limit, int max_groups, int *group, int *kept)
{
    const auto out = mplb::cache_groups(std::vector<long long>(cells, cells + n), size_t(max_groups),
                                        [&](long long c) { return c <= limit; });
    for (size_t k = 0; k < out.size(); ++k) {
        kept[k] = out[k].kept;
        for (size_t j = 0; j < out[k].members.size(); ++j) {
            const int i = out[k].members[j];
            if (group[i] >= 0 || (j > 0 && i <= out[k].members[j - 1])) return -1;
            group[i] = int(k);
        }
    }
    return int(out.size());
}

// shape: nx, ny, nz, bx, by, bz; storage 0 FP64, 1 FP32, 2 FP16S, 3 FP16S_ALL, 4 the
// last with a single relaxation time.
static mplb::Shape3 shape_of(const int *n, int storage, int kept)
{
    return mplb::Shape3{n[0], n[1], n[2], n[3], n[4], n[5], storage < 2, storage == 1, kept != 0,
                        storage == 4};
}
int packs_planes(const int *n, int storage, int kept) { return mplb::packs_planes(shape_of(n, storage, kept)); }
int64_t lanes(const int *n, int packed)
{
    const mplb::Shape3 s = shape_of(n, 0, 1);
    return packed ? mplb::pack_lanes(s) : mplb::block_lanes(s);
}
int narrow_blocks(const int *n, int storage, int kept)
{
    return mplb::takes_narrow_blocks(shape_of(n, storage, kept));
}
int stores_stay2d(int nx, int elem, int kept) { return mplb::stores_stay2d(nx, elem, kept != 0); }
int tile_columns2d(int nx, int stay, int kept) { return mplb::tile_columns2d(nx, stay != 0, kept != 0); }
}
