// Batched kernels: many independent domains in the same launches (see
// device.hpp, "batches").
#include "step2d.hpp"

namespace mplb {

// The phi stage or the update of one step of a group of 3-D domains.  NB: the
// form of the block kernels (a Kept form: the group stays in the Infinity
// Cache).
template <class P, int COLL, bool PHI, class NB, int FORM>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(PHI ? 1 : collide_waves<3, P, COLL>()))) kb_step(const BatchDom *__restrict__ doms,
                                               const BatchTile *__restrict__ tiles,
                                               const int *ntiles, const long long *tbase,
                                               int step_off, int *status)
{
    using T = typename P::T;
    const long long t = *tbase + step_off;
    // the phi stage covers every domain, the update those without nphi_by;
    // the phi stage also flags a domain whose order parameter is not finite
    // (status[dom] != 0): a non-finite population of either set reaches phi
    // within a step
    const int nt = PHI ? ntiles[2] : ntiles[1];
    const int block = flat_block();
    if (block >= nt) return;
    const BatchTile tl = tiles[ntiles[0] + tile_of<is_kept<NB>>(block, nt)];
    // the domain's record by value: read once, not re-read after every
    // population store the compiler cannot prove to be elsewhere
    const Geom g = doms[tl.dom].g;
    const long long first = doms[tl.dom].first, last = doms[tl.dom].last;
    if (t < first || t >= last) return;
    const Ptrs p = batch_ptrs(doms[tl.dom], int((t - first) & 1), t >= doms[tl.dom].hist_from);
    const int tid = int(threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z));
    int x, y;
    const int z = tl.z0;
    if constexpr (FORM == FORM_PACK) {
        const int c = tl.x0 + tid;
        if (c >= g.nx * g.ny) return;
        y = c / g.nx;
        x = c - y * g.nx;
    } else {
        // the tile is tl.w cells wide in x and (block threads) / tl.w rows
        // high, one plane deep; the width is the domain's own (a multiple of
        // 64 in the row form, so that each wavefront lies in one x-row)
        x = tl.x0 + tid % tl.w;
        y = tl.y0 + tid / tl.w;
        if constexpr (FORM == FORM_ROW) y = __builtin_amdgcn_readfirstlane(y);
        if (x >= g.nx || y >= g.ny) return;
    }
    const int nby = doms[tl.dom].nphi_by;
    if constexpr (PHI) {
        // (packed: the rows of a phi-summing domain are whole wavefronts)
        const int yw = FORM == FORM_PACK ? __builtin_amdgcn_readfirstlane(y) : y;
        const T ph = (nby && t >= doms[tl.dom].nphi_from)
                         ? nphi_merge_cell<P, NB>(g, p, NextPhi{doms[tl.dom].npart, doms[tl.dom].nedge, nby}, x,
                                                  yw, z)
                         : phi_cell<3, P, NB>(g, p, x, y, z);
        if (!__builtin_isfinite(ph)) atomicOr(status + tl.dom, 1);
    } else {
        const Phys<T> ph = to_phys<T>(doms[tl.dom].ph);
        collide_cell<3, P, COLL, NB>(g, ph, p, x, y, z);
    }
}

// Batched form of the one-launch 2-D step over one cache group (see
// launch_batch_step2d): block b takes tile b of the group's running counts (in
// eighths per XCD, as k_step2d); every wavefront finds the domain with one load
// of 64 counts at a time.  FEW: all blocks of the launch are resident at once
// (FP16 formats only, see below).
template <class P, int COLL, bool KEPT, bool FEW>
__global__ void __launch_bounds__(STEP2D_THREADS)
kb_step2d(const BatchDom *__restrict__ doms, const int *__restrict__ table, int capacity, int group,
          const long long *tbase, int step_off, int *status)
{
    using T = typename P::T;
    __shared__ typename std::conditional<P::F::shifted, unsigned long long, T>::type lds[step2d_slots(false)];
    const int pos = table[2 * group], n = table[2 * group + 1];
    const int *ids = table + 2 * BATCH_GROUPS + pos, *tile0 = table + 2 * BATCH_GROUPS + capacity + pos + group;
    const int nt = tile0[n];
    const int block = flat_block();
    if (block >= nt) return;
    const int bid = tile_of<true>(block, nt);
    // the last domain whose tiles begin at or before bid
    int at = -1;
    for (int d0 = 0; d0 < n; d0 += 64) {
        const int d = d0 + int(threadIdx.x & 63);
        const int begins = __popcll(__ballot(d < n && tile0[d] <= bid));
        at += begins;
        if (begins < 64) break;
    }
    at = __builtin_amdgcn_readfirstlane(at);
    const int dom = ids[at];
    const long long t = *tbase + step_off;
    const long long first = doms[dom].first, last = doms[dom].last;
    if (t < first || t >= last) return;  // the whole block
    const Geom g = doms[dom].g;  // by value, see kb_step
    const Ptrs p = batch_ptrs(doms[dom], int((t - first) & 1), t >= doms[dom].hist_from);
    const Phys<T> ph = to_phys<T>(doms[dom].ph);
    const int lbx = step2d_width(g, P::F::shifted), by = STEP2D_THREADS >> lbx;
    const int ntx = (g.nx + (1 << lbx) - 1) >> lbx, k = bid - tile0[at];
    const int x0 = (k % ntx) << lbx, y0 = (k / ntx) * by;
    // the fast tile form of the format, and one for all other domains: in the
    // FP16 formats the one of fewest registers, since both bodies share the
    // kernel's (NbLane 64, NbFlat 98; 24 domains FP16S 42 and 47 us a step), but
    // the one of fewest instructions where occupancy does not matter (FEW: one
    // domain of 20 to 60 cells a side 9.6 and 7.0, forty 12.0 and 9.6)
    constexpr int FAST = P::F::shifted ? TILE_ROW : TILE_WIDE;
    constexpr int OTHER = P::F::shifted && !FEW ? TILE_LANE : TILE_NARROW;
    if (step2d_form<P>(g, lbx) == FAST)
        step2d_any<P, COLL, KEPT, FAST>(g, ph, p, lds, 6, 64, x0, y0, status + dom);
    else
        step2d_any<P, COLL, KEPT, OTHER>(g, ph, p, lds, lbx, 1 << lbx, x0, y0, status + dom);
}

hipError_t launch_batch_step2d(int storage, int collision, bool kept, const BatchDom *doms,
                               const int *table, int capacity, int group, const long long *tbase,
                               int step_off, int grid, int *status, hipStream_t stream)
{
    Ctx c{};
    c.dim = 2;
    c.storage = storage;
    return dispatch(c, [&]<int D, class P>() -> hipError_t {
        if constexpr (D != 2) {
            return hipErrorInvalidValue;
        } else {
            return with_coll(collision, [&](auto cc) {
                constexpr int COLL = decltype(cc)::value;
                auto go = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, flat_grid(grid), dim3(STEP2D_THREADS), 0, stream, doms, table, capacity,
                                       group, tbase, step_off, status);
                    return hipGetLastError();
                };
                if constexpr (P::F::shifted) {
                    // four blocks a CU: five fit with NbFlat's registers
                    if (kept && grid <= 1024) return go(kb_step2d<P, COLL, true, true>);
                }
                return kept ? go(kb_step2d<P, COLL, true, false>) : go(kb_step2d<P, COLL, false, false>);
            });
        }
    });
}

__global__ void k_set_i64(long long *ptr, long long v) { *ptr = v; }

__global__ void __launch_bounds__(256) k_fill_i32(int *ptr, int n, int v)
{
    const int i = int(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) ptr[i] = v;
}

hipError_t launch_batch_step(int storage, int collision, int form, bool kept,
                             const BatchDom *doms, const BatchTile *tiles, const int *ntiles,
                             const long long *tbase, int step_off, dim3 block, const int *grid,
                             int *status, hipStream_t stream)
{
    Ctx c{};
    c.dim = 3;
    c.storage = storage;
    auto step = [&]<class P, class NB, int FORM>() -> hipError_t {
        auto go = [&](auto k, int nblk, size_t lds) {
            if (nblk == 0) return hipSuccess;
            hipLaunchKernelGGL(k, flat_grid(nblk), block, lds, stream, doms, tiles, ntiles, tbase, step_off,
                               status);
            return hipGetLastError();
        };
        hipError_t e = go(kb_step<P, 0, true, NB, FORM>, grid[0], 0);
        if (e != hipSuccess) return e;
        return with_coll(collision, [&](auto cc) -> hipError_t {
            constexpr int COLL = decltype(cc)::value;
            // dynamic LDS: single relaxation time's flow values (3-D)
            return go(kb_step<P, COLL, false, NB, FORM>, grid[1],
                      srt_lds_bytes<3, P, COLL>(block.x * block.y * block.z));
        });
    };
    return dispatch(c, [&]<int D, class P>() -> hipError_t {
        if constexpr (D == 2) {
            return hipErrorInvalidValue;  // one launch: launch_batch_step2d
        } else {
            auto by_form = [&]<int FORM>() -> hipError_t {
                using NB = NbOf<FORM>;
                if constexpr (!P::F::shifted) {
                    if (kept) return step.template operator()<P, Kept<NB>, FORM>();
                }
                return step.template operator()<P, NB, FORM>();
            };
            hipError_t e = hipErrorInvalidValue;
            if (form == FORM_LANE) {
                e = by_form.template operator()<FORM_LANE>();
            } else if (form == FORM_ROW) {
                e = by_form.template operator()<FORM_ROW>();
            } else {
                e = by_form.template operator()<FORM_PACK>();
            }
            if (e == hipSuccess)
                e = launch_batch_nphi(storage, collision, kept, doms, tiles, ntiles, tbase, step_off, grid, stream);
            return e;
        }
    });
}

// flag |= 1 if the order parameter of the context's current level holds a
// non-finite value anywhere (grid-stride over the cells).
template <class P>
__global__ void __launch_bounds__(256) k_flag_nonfinite(const void *phi, long long n, int *flag)
{
    using T = typename P::T;
    bool bad = false;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        T v;
        if constexpr (P::F::shifted)
            v = rec_phi(gld(static_cast<const unsigned long long *>(phi), i));
        else
            v = gld(static_cast<const T *>(phi), i);
        bad = bad || !__builtin_isfinite(v);
    }
    if (bad) atomicOr(flag, 1);
}

hipError_t launch_flag_nonfinite(const Ctx &c, int *flag)
{
    const long long n = (long long)c.g.nx * c.g.ny * c.g.nz;
    const long long need = (n + 255) / 256;
    const int blocks = int(need < 1024 ? need : 1024);
    return dispatch(c, [&]<int D, class P>() {
        hipLaunchKernelGGL((k_flag_nonfinite<P>), dim3(blocks), dim3(256), 0, c.stream, c.p.phi, n,
                           flag);
        return hipGetLastError();
    });
}

hipError_t launch_set_i64(long long *ptr, long long v, hipStream_t stream)
{
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, stream, ptr, v);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int *ptr, int n, int v, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, stream, ptr, n, v);
    return hipGetLastError();
}


}  // namespace mplb
