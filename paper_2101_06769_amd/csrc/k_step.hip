// The step kernels of one domain: the order-parameter pass and the cell
// update (see device.hpp).
#include "device.hpp"

namespace mplb {

template <int D, class P, class NB, int FORM>
__global__ void __launch_bounds__(256) k_phi(Geom g, Ptrs p)
{
    int x, y, z;
    if (!block_cell<FORM, is_kept<NB>>(g, x, y, z)) return;
    phi_cell<D, P, NB>(g, p, x, y, z);
}

template <int D, class P, int COLL, class NB, int FORM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(collide_waves<D, P, COLL>())))
k_collide(Geom g, Phys<typename P::T> ph, Ptrs p)
{
    int x, y, z;
    if (!block_cell<FORM, is_kept<NB>>(g, x, y, z)) return;
    collide_cell<D, P, COLL, NB>(g, ph, p, x, y, z);
}

// Row-form addressing: every wavefront inside one x-row of the block, x
// periodic, population arrays of fewer than 2^31 elements.
bool row_form_ok(int dim, const Geom &g, dim3 block)
{
    const long long Q = dim == 2 ? 9 : 27;
    return block.x % 64 == 0 && g.bcx == BC_PER && Q * g.np < (1ll << 31);
}

// Whether both levels of the populations of np cells stay in the 256 MiB
// Infinity Cache from one step to the next.  Then they are stored with
// ordinary stores: a non-temporal store goes to HBM, and the next step reads
// it back from there (1024 x 1024 FP32, 151 MB: 35.3 against 24.9 us a step;
// 1792 x 1024, 264 MB: 57.0 against 41.5).  Beyond that size cached stores only
// displace what the step has yet to read (2048 x 1024, 302 MB: 64.1 against
// 65.0 us; 2048 x 2048: 124 against 130), but for 2-D rows that do not start at
// cache lines (stores_stay2d).
bool kept_in_cache(int dim, int storage, long long np)
{
    const long long f = storage == ST_FP64 ? 8 : storage == ST_FP32 ? 4 : 2;
    const long long gg = storage == ST_FP64 ? 8 : storage == ST_FP16S_ALL ? 2 : 4;
    return 2 * (dim == 2 ? 9 : 27) * np * (f + gg) <= (256ll << 20);
}

hipError_t launch_phi(const Ctx &c)
{
    return dispatch(c, [&]<int D, class P>() {
        return with_form<D, P>(c, [&]<class NB, int FORM>(dim3 grid, dim3 block) {
            hipLaunchKernelGGL((k_phi<D, P, NB, FORM>), grid, block, 0, c.stream, c.g, c.p);
            return hipGetLastError();
        });
    });
}

hipError_t launch_collide(const Ctx &c)
{
    return dispatch(c, [&]<int D, class P>() -> hipError_t {
        using T = typename P::T;
        if constexpr (D == 2) {
            return hipErrorInvalidValue;  // one launch: launch_step2d
        } else {
            return with_coll(coll_code(c.ph), [&](auto cc) {
                constexpr int COLL = decltype(cc)::value;
                return with_form<D, P>(c, [&]<class NB, int FORM>(dim3 grid, dim3 block) {
                    // dynamic LDS: single relaxation time's flow values (3-D)
                    const size_t lds = srt_lds_bytes<D, P, COLL>(block.x * block.y * block.z);
                    hipLaunchKernelGGL((k_collide<D, P, COLL, NB, FORM>), grid, block, lds, c.stream, c.g,
                                       to_phys<T>(c.ph), c.p);
                    return hipGetLastError();
                });
            });
        }
    });
}

}  // namespace mplb
