// The batched update that sums the next order parameter (see device.hpp,
// "batches" and "next order parameter").
#include "device.hpp"

namespace mplb {

// Batched phi-summing update for domains with rows of BX cells (64, 128,
// 192, 256 or 512): the ntiles[4 + 2k] tiles from index ntiles[3 + 2k], k =
// nphi_group(BX) (domain, rows y0 .. y0 + nphi_by - 1 of plane z0), each an
// nphi_tile of its domain.  (A loop over several planes
// per tile keeps the tile's pointers and parameters live across the update
// and spills: measured slower even for one plane.)  FP32: at most 80 VGPRs (six
// wavefronts per SIMD), so that three tiles fit a CU as in the
// single-domain kernel.
// Not where the group stays in the Infinity Cache: its update holds the pulled
// phase-field values, which would spill.
template <class P, int COLL, class NB>
constexpr int kb_nphi_waves()
{
    return collide_waves<3, P, COLL>() == 4 && !is_kept<NB> ? 6 : collide_waves<3, P, COLL>();
}

template <class P, int COLL, int BX, class NB>
__global__ void __launch_bounds__(NPHI_THREADS) __attribute__((amdgpu_waves_per_eu(kb_nphi_waves<P, COLL, NB>())))
kb_collide_nphi(const BatchDom *__restrict__ doms, const BatchTile *__restrict__ tiles,
                const int *ntiles, const long long *tbase, int step_off)
{
    using T = typename P::T;
    extern __shared__ double nphi_lds[];
    constexpr int k = nphi_group(BX);
    const long long t = *tbase + step_off;
    const int n0 = ntiles[3 + 2 * k], nt = ntiles[4 + 2 * k];
    const int block = flat_block();
    if (block >= nt) return;
    const BatchTile tl = tiles[n0 + block];
    const Geom g = doms[tl.dom].g;  // by value, see kb_step
    const long long first = doms[tl.dom].first, last = doms[tl.dom].last;
    if (t < first || t >= last) return;  // the whole block
    const Ptrs p = batch_ptrs(doms[tl.dom], int((t - first) & 1), t >= doms[tl.dom].hist_from);
    const Phys<T> ph = to_phys<T>(doms[tl.dom].ph);
    const NextPhi q{doms[tl.dom].npart, doms[tl.dom].nedge, doms[tl.dom].nphi_by};
    const int tid = int(threadIdx.x);
    const int ty = __builtin_amdgcn_readfirstlane(tid / BX);
    nphi_tile<P, COLL, BX, NB>(g, ph, p, q, reinterpret_cast<T *>(nphi_lds), BX, tl.y0 / q.by, ty,
                               tid - ty * BX, tl.z0, ty < q.by);
}

// One launch per row length present (grid[2 + k] blocks for row length k); a
// group's tiles have the threads its row length takes alone.
hipError_t launch_batch_nphi(int storage, int collision, bool kept, const BatchDom *doms,
                             const BatchTile *tiles, const int *ntiles, const long long *tbase,
                             int step_off, const int *grid, hipStream_t stream)
{
    Ctx c{};
    c.dim = 3;
    c.storage = storage;
    return dispatch(c, [&]<int D, class P>() -> hipError_t {
        if constexpr (D != 3) {
            return hipErrorInvalidValue;
        } else {
            return with_coll(collision, [&](auto cc) -> hipError_t {
                constexpr int COLL = decltype(cc)::value;
                auto one = [&](auto kernel, int k) {
                    if (grid[2 + k] == 0) return hipSuccess;
                    const int threads = nphi_threads(storage, nphi_group_width(k));
                    const size_t lds = size_t(26) * threads * sizeof(typename P::T);
                    hipLaunchKernelGGL(kernel, flat_grid(grid[2 + k]), dim3(threads), lds, stream, doms, tiles,
                                       ntiles, tbase, step_off);
                    return hipGetLastError();
                };
                auto all = [&]<class NB>() {
                    hipError_t e = one(kb_collide_nphi<P, COLL, 64, NB>, 0);
                    if (e == hipSuccess) e = one(kb_collide_nphi<P, COLL, 128, NB>, 1);
                    if (e == hipSuccess) e = one(kb_collide_nphi<P, COLL, 192, NB>, 2);
                    if (e == hipSuccess) e = one(kb_collide_nphi<P, COLL, 256, NB>, 3);
                    if constexpr (sizeof(typename P::T) == 4) {
                        if (e == hipSuccess) e = one(kb_collide_nphi<P, COLL, 512, NB>, 4);
                    } else {
                        if (e == hipSuccess && grid[6]) e = hipErrorInvalidValue;
                    }
                    return e;
                };
                if constexpr (!P::F::shifted) {
                    if (kept) return all.template operator()<Kept<NbRow>>();
                }
                return all.template operator()<NbRow>();
            });
        }
    });
}

}  // namespace mplb
