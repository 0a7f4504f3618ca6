// The one-launch step of one 2-D domain (see step2d.hpp).
#include <algorithm>

#include "step2d.hpp"

namespace mplb {

// Blocks are dealt to the eight XCDs in turn; XCD k takes the k-th eighth of
// the tiles, so that the rows two tiles share are read through one L2
// (1024 x 1024 FP32: 38.2 -> 36.9 us, 800 x 400: 15.0 -> 13.4 us with an earlier
// form of the kernel).
template <class P, int COLL, int TILE, bool KEPT>
__global__ void __launch_bounds__(STEP2D_THREADS)
k_step2d(Geom g, Phys<typename P::T> ph, Ptrs p, int lbx, int cols, int ntx, int nt, int first)
{
    constexpr int SLOTS = step2d_slots(TILE == TILE_WIDE || TILE == TILE_ROW);
    __shared__ typename std::conditional<P::F::shifted, unsigned long long, typename P::T>::type lds[SLOTS];
    const int bid = tile_of<true>(first + int(blockIdx.x), nt);
    const int x0 = (bid % ntx) * cols, y0 = (bid / ntx) * (STEP2D_THREADS >> lbx);
    step2d_any<P, COLL, KEPT, TILE>(g, ph, p, lds, lbx, cols, x0, y0, nullptr);
}

int step2d_tiles(const Geom &g, int storage)
{
    const int lbx = step2d_width(g, storage == ST_FP16S || storage == ST_FP16S_ALL), by = STEP2D_THREADS >> lbx;
    return ((g.nx + (1 << lbx) - 1) >> lbx) * ((g.ny + by - 1) / by);
}

hipError_t launch_step2d(const Ctx &c)
{
    const int lbx = step2d_width(c.g, c.storage == ST_FP16S || c.storage == ST_FP16S_ALL);
    const int ntx = (c.g.nx + (1 << lbx) - 1) >> lbx, nt = step2d_tiles(c.g, c.storage);
    const bool kept = kept_in_cache(2, c.storage, c.g.np);
    const bool stay = stores_stay2d(c.g.nx, c.storage == ST_FP64 ? 8 : c.storage == ST_FP16S_ALL ? 2 : 4, kept);
    const int cols = lbx == 6 ? tile_columns2d(c.g.nx, stay, kept) : 1 << lbx;
    return dispatch(c, [&]<int D, class P>() -> hipError_t {
        if constexpr (D != 2) {
            return hipErrorInvalidValue;
        } else {
            auto launch = [&](auto kernel) {
                hipError_t e = hipSuccess;
                for (int first = 0; first < nt && e == hipSuccess; first += GRID_ROW) {
                    hipLaunchKernelGGL(kernel, dim3(std::min(nt - first, GRID_ROW)), dim3(STEP2D_THREADS), 0,
                                       c.stream, c.g, to_phys<typename P::T>(c.ph), c.p, lbx, cols, ntx, nt,
                                       first);
                    e = hipGetLastError();
                }
                return e;
            };
            return with_coll(coll_code(c.ph), [&](auto cc) {
                constexpr int COLL = decltype(cc)::value;
                auto by_tile = [&]<int TILE>() {
                    return stay ? launch(k_step2d<P, COLL, TILE, true>) : launch(k_step2d<P, COLL, TILE, false>);
                };
                const int form = step2d_form<P>(c.g, lbx);
                if constexpr (P::F::shifted) {
                    if (form == TILE_ROW) return by_tile.template operator()<TILE_ROW>();
                }
                return form == TILE_NARROW ? by_tile.template operator()<TILE_NARROW>()
                                           : by_tile.template operator()<TILE_WIDE>();
            });
        }
    });
}

}  // namespace mplb
