// Host-side interface between the C ABI (api.cpp) and the kernel launchers
// (the k_*.hip files).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "lattice.hpp"

namespace mplb {

enum { ST_FP64 = 0, ST_FP32 = 1, ST_FP16S = 2, ST_FP16S_ALL = 3 };

// Physical parameters in the form the kernels use (double on the host,
// converted to the arithmetic type at launch).
struct PhysD {
    double rho_l, drho;    // rho = rho_l + drho phi
    double nu_l, dnu;      // nu = nu_l + dnu phi            (visc_interp 0)
    double rnu_l, drnu;    // nu = (rnu_l + drnu phi) / rho  (visc_interp 1)
    double beta, kappa;    // chemical potential coefficients
    double gx, gy, gz;     // body-force acceleration
    double inv_tpb;        // 1 / taubar_phi
    double src_pre;        // 1 - 1/(2 taubar_phi)
    double four_W;         // 4 / W
    double scl_l, dscl;    // FP16 flow codes' scale rho cs^2 = scl_l + dscl phi
    int visc_interp;
    int collision;         // 0 cumulant, 1 SRT
    int cac_edf;           // phase-field equilibrium: 0 second-order, 1 first-order + correction
};

// Device buffers one launch works on.  "in" buffers hold the post-collision
// state of the previous step (pre-collision values are pulled from them);
// "out" buffers receive the new post-collision state.
struct Ptrs {
    const void *Fin;
    void *Fout;
    const void *Gin;
    void *Gout;
    // order parameter of the current time level: [np] in the arithmetic
    // type; FP16 formats: [np] 8-byte records (phi, packed references of the
    // values the cell wrote a step earlier), see device.hpp "FP16 storage"
    void *phi;
    // FP16 formats: the packed references the update writes for the values
    // it stores ([np]), and the rest-direction values of the FP16 sets in
    // FP32 ([np] each, null for a set in plain storage)
    unsigned *ref;
    const float *frest_in, *grest_in;
    float *frest_out, *grest_out;
    // first-order phase-field equilibrium: (phi u) per cell, [3][np], of the
    // previous step (valid when have_prev) and of this step
    const void *phiu_in;
    void *phiu_out;
    int have_prev;
    // FP16 formats: the references of the values the cells wrote a step
    // earlier (ref itself, read by the phi stage before the update writes it;
    // another array where the step is one launch)
    const unsigned *ref_in;
};

struct Ctx {
    int dim;
    int storage;
    Geom g;
    PhysD ph;
    dim3 block;
    hipStream_t stream;
    Ptrs p;
};

hipError_t launch_phi(const Ctx &c);
hipError_t launch_collide(const Ctx &c);
// The whole step of a 2-D lattice in one launch: each block sums phi for its
// tile and the ring of cells around it into LDS, then updates its cells; the
// phi array is not written.  Its tiles (step2d_tiles of them) do not depend on
// the context's block.
int step2d_tiles(const Geom &g, int storage);
hipError_t launch_step2d(const Ctx &c);
// Several steps of a small such lattice in plain storage in one launch, from the Fin/Gin to the
// Fout/Gout buffers: the number of steps multi2d_steps gives (1: none; single
// steps instead).
int multi2d_steps(const Ctx &c);
hipError_t launch_multi2d(const Ctx &c, int steps);
// Partial sums of the next order parameter, written by launch_collide_nphi
// for launch_phi_merge of the following step: part [3][np], edge
// [2][3][ny / by][nz][nx] in the arithmetic type; by = tile rows,
// nphi_rows(nx, ny, storage format).
struct NextPhi {
    void *part;
    void *edge;
    int by;
};
// The update kernel that also sums the next order parameter from the values
// it stores, tile by tile (3-D, x periodic, nx as nphi_width_ok, y and z
// periodic or walls); nphi_ok tells whether it
// applies.  Its tiles are whole rows by nphi_rows rows, whatever
// the block shape of the other kernels.
bool nphi_ok(const Ctx &c);
int nphi_rows(int nx, int ny, int storage);
// Row lengths the phi-summing update takes: multiples of 64 up to 256, and
// 512 with FP32 arithmetic (one row per 512-thread tile).
bool nphi_width_ok(int nx, int storage);
// Groups of the batched phi-summing update by row length 64, 128, 192, 256, 512.
constexpr int NPHI_GROUPS = 5;
constexpr int nphi_group_width(int k) { return k < 4 ? 64 * (k + 1) : 512; }
constexpr int nphi_group(int nx) { return nx == 512 ? 4 : nx / 64 - 1; }
hipError_t launch_collide_nphi(const Ctx &c, const NextPhi &q);
// phi of the current level from the partial sums of the previous update.
hipError_t launch_phi_merge(const Ctx &c, const NextPhi &q);
// Equilibrium initial state from device FP64 fields (phi[N], u[dim][N], p[N])
// written into the Fout/Gout buffers in pull layout.
hipError_t launch_init(const Ctx &c, const double *phi, const double *u, const double *pr);
// Pre-collision populations a0..a1-1 of set `which` (0 f', 1 g) from the
// Fin/Gin buffers into dst[(a-a0)][N] (FP64).
hipError_t launch_get_pop(const Ctx &c, int which, int a0, int a1, double *dst);
// The inverse: src[(a-a0)][N] into the Fout/Gout buffers in pull layout.
hipError_t launch_set_pop(const Ctx &c, int which, int a0, int a1, const double *src);
// References of the FP16 formats (the ref array) for an initial state, from
// FP64 order-parameter and pressure fields.
hipError_t launch_set_refs(const Ctx &c, const double *phi, const double *pr);
// One macroscopic field of the state held in Fin/Gin (the phi array may be
// rewritten on the way).
hipError_t launch_field(const Ctx &c, int field, double *dst);
// Deterministic FP64 reduction: partials (at least reduce_blocks() x 8
// doubles), out[8] = {sum phi, sum rho ux, uy, uz, max|u|, nonfinite count}.
hipError_t launch_reduce(const Ctx &c, double *partials, double *out);
int reduce_blocks(const Ctx &c);
// launch_reduce with the partials and the result in the library's static
// device scratch (of the current device); *result receives the device
// address of the 8 results.  hipErrorInvalidValue if the reduction needs
// more partial blocks than the scratch holds (reduce_scratch_max_blocks).
hipError_t launch_reduce_static(const Ctx &c, double **result);
int reduce_scratch_max_blocks();

// One domain of a batch, as the batched kernels read it from device memory.
struct BatchDom {
    Geom g;
    PhysD ph;
    void *F[2], *G[2], *phi;
    unsigned *ref[2];
    float *frest[2], *grest[2];
    void *phiu[2];
    long long first, last;  // active for batch steps first <= t < last
    long long hist_from;    // (phi u) of the previous step valid for t >= hist_from
    // phi-summing update (see NextPhi): tile rows, 0 if the domain's update
    // does not sum phi; the partial sums; the phi stage of steps t >=
    // nphi_from merges them (earlier ones sum the pulled populations)
    int nphi_by;
    void *npart, *nedge;
    long long nphi_from;
};

// A tile of a batch: domain index, origin cell (x0, y0, z0) and width w: w
// cells in x by (threads per block) / w rows, one plane; w = 0: consecutive cells of plane z0 from in-plane index x0 (see
// NbPack).
struct BatchTile {
    int dom, x0, y0, z0, w;
};

// The domains that share launches are advanced in cache groups: a group's
// populations fit the Infinity Cache together (kept), and it takes a chunk of
// steps before the next group does.  At most BATCH_GROUPS groups.
constexpr int BATCH_GROUPS = 32;

// One step of a group of 2-D domains in one launch.  table: two ints per group (first position and number of domains),
// then the domains by position, then per group its running tile counts
// (step2d_tiles; number of domains + 1 entries, so position + group is their
// start).  Blocks beyond the last count exit.  status as for launch_batch_step.
hipError_t launch_batch_step2d(int storage, int collision, bool kept, const BatchDom *doms,
                               const int *table, int capacity, int group, const long long *tbase,
                               int step_off, int grid, int *status, hipStream_t stream);
// Whether both levels of the populations of np cells stay in the Infinity
// Cache from one step to the next.
bool kept_in_cache(int dim, int storage, long long np);

// True when the row-form kernels apply: block a multiple of 64 wide in x,
// x periodic, population arrays of fewer than 2^31 elements.
bool row_form_ok(int dim, const Geom &g, dim3 block);
// Addressing of a launch: per lane, rows, or packed planes (3-D).
enum { FORM_LANE, FORM_ROW, FORM_PACK };
// One step of a group of 3-D domains over the tile list, batch step index *tbase +
// step_off.
// collision: operator code, bit 0 the flow collision, bit 1 the first-order
// phase-field equilibrium (shared by all domains).  form: FORM_ROW where
// every domain the block kernels update satisfies row_form_ok with its tile
// width, FORM_PACK where each is periodic in x and y and within 32-bit
// indices (tiles of w = 0).
// ntiles, GROUP_INTS of them: the group's first tile; the number of block
// tiles of the domains the block kernels update, which come first; that number
// with the block tiles of the phi-summing domains (their phi stage merges
// partial sums), which come next; then, per row length (nphi_group), start and
// number of the tiles of the phi-summing update (domains with nphi_by > 0:
// whole rows of one plane).  grid[0], grid[1]: blocks of the phi stage and the
// update, at least one per tile; grid[2 + k]: of row length k's update (0: not
// launched); 2 + NPHI_GROUPS entries.
// status[dom] is or-ed with 1 when the phi stage finds a non-finite order
// parameter in that domain.
constexpr int GROUP_INTS = 16;
hipError_t launch_batch_step(int storage, int collision, int form, bool kept,
                             const BatchDom *doms, const BatchTile *tiles, const int *ntiles,
                             const long long *tbase, int step_off, dim3 block, const int *grid,
                             int *status, hipStream_t stream);
// Its phi-summing updates (k_batch_nphi.hip).
hipError_t launch_batch_nphi(int storage, int collision, bool kept, const BatchDom *doms,
                             const BatchTile *tiles, const int *ntiles, const long long *tbase,
                             int step_off, const int *grid, hipStream_t stream);
hipError_t launch_set_i64(long long *ptr, long long v, hipStream_t stream);
// *flag |= 1 if the order parameter of the context's current level (phi
// array, as the phi stage left it) holds a non-finite value.
hipError_t launch_flag_nonfinite(const Ctx &c, int *flag);
// ptr[0 .. n) = v by a kernel (no memset node when captured into a graph).
hipError_t launch_fill_i32(int *ptr, int n, int v, hipStream_t stream);

}  // namespace mplb
