// The one-launch step of 2-D lattices: a block sums phi for
// its tile and the ring of cells around it into LDS, then updates its cells.
// A separate phi pass costs a launch (2.6 of the 7.0 us of a 64 x 256 FP64
// step) and reads the phase-field set twice (40 of 188 B/cell).  The sums, the
// stencil and the update are those of k_phi and k_collide in the same order,
// so the results are the same bits.
//
// Bound: launch and load latency up to about 10^5 cells (800 x 400 FP32 runs one
// round of blocks, 3.9 wavefronts a SIMD, the VALU 75 % busy), then instruction
// issue and the Infinity Cache together (1024 x 1024 FP32 90 % busy at 5.9 TB/s of
// its 144 B/cell, FP16S 90 %, FP16S_ALL 98 %), beyond the cache HBM.  Tiles of 256
// threads: 512 and 1024 sum fewer ring cells (148 and 164 a tile against 140, for
// two and four times the cells) but leave a small lattice fewer blocks: 4.9, 6.1
// and 8.8 us on 64 x 256 FP64, 24.9, 25.4 and 26+ us on 1024 x 1024 FP32.  Measured
// per step, before (two launches) and now: 64 x 256 FP64 7.0 -> 4.9 us, 128 x 512
// FP32 (single relaxation time) 7.2 -> 4.8, 800 x 400 FP32 between symmetry planes
// 18.0 -> 10.7, 1024 x 1024 FP32 38.8 -> 24.9, 4096 x 2048 FP32 272 -> 252 us.
#pragma once

#include "device.hpp"

namespace mplb {

// The nine values of a set that a cell pulls.  Row form (ROWU): y and the
// rules along it are wavefront-uniform (as NbRow), so each load is a scalar
// base plus one of three lane columns; on axes that are not periodic the
// first and last column's lanes then load what bounced back or was mirrored,
// behind one branch that the other wavefronts skip.  Lane form: the rules of
// both axes as per-lane selects.
template <bool ROWU>
struct Pull2d {
    int x, xm, xp;      // own, left and right column (the own one beyond a wall or symmetry plane)
    long long r[3];     // row offsets of y - 1, y, y + 1, likewise
    bool wy[3], sy[3];  // a wall or symmetry plane between y and y + k - 1
    bool wx, sx;        // the lattice has walls / symmetry planes in x
    bool lo, hi;        // first / last column of a lattice not periodic in x

    __device__ __forceinline__ Pull2d(const Geom &g, int x_, int y) : x(x_)
    {
        const bool per = g.bcx == BC_PER;
        wx = g.bcx == BC_WALL;
        sx = g.bcx == BC_SYM;
        lo = !per && x == 0;
        hi = !per && x == g.nx - 1;
        xm = x > 0 ? x - 1 : per ? g.nx - 1 : 0;
        xp = x < g.nx - 1 ? x + 1 : per ? 0 : x;
        for (int k = 0; k < 3; ++k) {
            const int yy = y + k - 1;
            const bool out = (unsigned)yy >= (unsigned)g.ny;
            r[k] = (long long)(!out ? yy : g.bcy == BC_PER ? yy - (k - 1) * g.ny : y) * g.nx;
            wy[k] = out && g.bcy == BC_WALL;
            sy[k] = out && g.bcy == BC_SYM;
        }
    }

    template <typename R>
    __device__ __forceinline__ R at(const R *base, long long off, int col) const
    {
        if constexpr (ROWU)
            return *lane_ptr(base, off, col);
        else
            return gld(base, off + col);
    }

    template <typename R>
    __device__ __forceinline__ void load(const R *base, long long np, R (&v)[9]) const
    {
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const int cx = cx_of(a), cy = cy_of(a), k = 1 - cy;
            const int xs = cx == 0 ? x : cx > 0 ? xm : xp;
            if constexpr (ROWU) {
                const int dir = wy[k] ? 8 - a : sy[k] ? a - 6 * cy : a;
                v[a] = at(base, dir * np + r[k], wy[k] ? x : xs);
            } else {
                const bool ex = cx > 0 ? lo : cx < 0 ? hi : false;
                const bool bb = wy[k] || (wx && ex);
                const int dir = bb ? 8 - a : a - (sy[k] ? 6 * cy : 0) - (sx && ex ? 2 * cx : 0);
                v[a] = at(base, dir * np + (bb ? r[1] : r[k]), bb ? x : xs);
            }
        }
        if constexpr (ROWU) {
            if ((wx || sx) && __any(lo || hi)) {
#pragma unroll
                for (int a = 0; a < 9; ++a) {
                    const int cx = cx_of(a), cy = cy_of(a), k = 1 - cy;
                    if (cx == 0) continue;
                    if (!(cx > 0 ? lo : hi)) continue;
                    const bool bb = wx || wy[k];
                    const int b = bb ? 8 - a : a - 2 * cx - (sy[k] ? 6 * cy : 0);
                    v[a] = at(base, b * np + (bb ? r[1] : r[k]), x);
                }
            }
        }
    }
};

// phi as k_phi sums it: the pulled values in direction order.
template <typename T>
__device__ __forceinline__ T phi_sum9(const T (&v)[9])
{
    T s = 0;
#pragma unroll
    for (int a = 0; a < 9; ++a) s += v[a];
    return s;
}

// Tile: 256 threads, 64 x 4 cells; narrower and taller on lattices of less than
// 64 columns (down to one); on long ones of few rows 256 x 1, 128 x 2 and, in
// plain storage, 32 x 8 (5 or 6 rows), so that few threads are without a cell.  With tiles of at least
// 8 columns and 4 rows, and with these, a step in us: 3 million cells in one
// column FP32 310 and 87, FP16S_ALL 546 and 91; 300 000 in one row 14.7 and 10.9,
// 17.8 and 12.7; 600 000 x 5 FP64 221 and 177.  Shorter rows leave CUs idle in any case and
// are faster as whole wavefronts (20 000 cells FP16S 5.3 and 5.7), as are 7 and 8
// rows (428 571 x 7 FP32 119 and 139) and the FP16 formats' row form (600 000 x 5
// FP16S_ALL 102 and 114).
constexpr int STEP2D_THREADS = 256;
__host__ __device__ inline int step2d_width(const Geom &g, bool fp16)
{
    if (g.nx > 65536) return g.ny == 1 ? 8 : g.ny == 2 ? 7 : (g.ny == 5 || g.ny == 6) && !fp16 ? 5 : 6;
    if (g.nx > 64) return 6;
    int l = 0;
    while ((1 << l) < g.nx) ++l;
    return l;
}
// Slots of a tile in LDS with the ring around it.
constexpr int step2d_slots(bool wide)
{
    int most = 0;
    for (int bx = wide ? 64 : 1; bx <= (wide ? 64 : 256); bx *= 2) {
        const int n = (bx + 2) * (STEP2D_THREADS / bx + 2);
        most = n > most ? n : most;
    }
    return most;
}

// The ring around a tile in the forms without whole wavefronts per row.  A tile
// that spans the lattice along an axis is its own neighbour there: the ring's
// cells are images of the tile's, written by the threads that hold those, and
// nothing is summed twice.
struct Ring2d {
    int w, h;
    bool whole_x, whole_y, px, py;
    __device__ __forceinline__ Ring2d(const Geom &g, int w_, int h_)
        : w(w_), h(h_), whole_x(w_ == g.nx), whole_y(h_ == g.ny), px(g.bcx == BC_PER), py(g.bcy == BC_PER)
    {
    }
    // cells of the ring to sum: the k-th in (i, j), false beyond the last
    __device__ __forceinline__ bool cell(int k, int &i, int &j) const
    {
        const int row = whole_x ? w : w + 2, rows = whole_y ? 0 : 2 * row;
        if (k < rows) {
            i = (k < row ? k : k - row) - (whole_x ? 0 : 1);
            j = k < row ? -1 : h;
            return true;
        }
        k -= rows;
        i = k < h ? -1 : w;
        j = k < h ? k : k - h;
        return !whole_x && k < 2 * h;
    }
    // stores v for cell (i, j) of the tile or its ring, and for its images
    template <class Slot, typename V>
    __device__ __forceinline__ void put(const Slot &slot, int i, int j, V v) const
    {
        const bool lo = whole_x && i == (px ? w - 1 : 0), hi = whole_x && i == (px ? 0 : w - 1);
        const bool bot = whole_y && j == (py ? h - 1 : 0), top = whole_y && j == (py ? 0 : h - 1);
        auto row = [&](int jj) {
            *slot(i, jj) = v;
            if (lo) *slot(-1, jj) = v;
            if (hi) *slot(w, jj) = v;
        };
        row(j);
        if (bot) row(-1);
        if (top) row(h);
    }
};

// The first half of a tile from (x0, y0), bx = 2^lbx threads wide (cols of them
// with cells), 256 / bx rows high: the thread's cell with its pulled populations, and phi of the tile and
// its ring in lphi.  False for threads without a cell.
// KEPT: the populations are stored to stay in the Infinity Cache (kept_in_cache).
// flag, if given: or-ed with 1 where phi is not finite.
// Every thread of the block calls it (it holds a barrier).  ROWU: bx = 64, a
// wavefront per row; the rows below and above the tile are summed by the
// first two wavefronts in row form, the columns beside it by the third.
template <class P, bool ROWU, bool KEPT>
__device__ __forceinline__ bool step2d_load(const Geom &g, const Ptrs &p, typename P::T *lphi, int lbx,
                                            int cols, int x0, int y0, int *flag, NbTile<typename P::T, KEPT> &nb)
{
    using T = typename P::T;
    const int bx = ROWU ? 64 : 1 << lbx, by = STEP2D_THREADS / bx, ls = bx + 2;
    const int tid = int(threadIdx.x);
    const int tx = tid & (bx - 1);
    const int ty = ROWU ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> lbx;
    const int w = min(cols, g.nx - x0), h = min(by, g.ny - y0);
    const T *F = static_cast<const T *>(p.Fin), *G = static_cast<const T *>(p.Gin);
    // slot (i, j) of the tile, i, j from -1
    auto slot = [&](int i, int j) { return lphi + (j + 1) * ls + i + 1; };
    const bool active = tx < w && ty < h;
    const int x = x0 + tx, y = y0 + ty;
    if (active) {
        const Pull2d<ROWU> c(g, x, y);
        c.load(G, g.np, nb.gp);
        c.load(F, g.np, nb.f);
    }
    // the ring: beyond walls and symmetry planes the mirrored cell's phi
    auto ring = [&](auto rowu, int i, int j) {
        T v[9];
        const Pull2d<decltype(rowu)::value> c(g, stencil_coord(x0 + i, g.nx, g.bcx),
                                              stencil_coord(y0 + j, g.ny, g.bcy));
        c.load(G, g.np, v);
        return phi_sum9(v);
    };
    const Ring2d rim(g, w, h);
    if constexpr (ROWU) {
        if (ty < 2) {
            if (tx < w) *slot(tx, ty == 0 ? -1 : h) = ring(std::true_type{}, tx, ty == 0 ? -1 : h);
        } else if (ty == 2) {
            const int n = h + 2, i = tx < n ? -1 : w, j = (tx < n ? tx : tx - n) - 1;
            if (tx < 2 * n) *slot(i, j) = ring(std::false_type{}, i, j);
        }
    } else {
        int i, j;
        if (rim.cell(tid, i, j)) rim.put(slot, i, j, ring(std::false_type{}, i, j));
    }
    if (active) {
        const T s = phi_sum9(nb.gp);
        if constexpr (ROWU)
            *slot(tx, ty) = s;
        else
            rim.put(slot, tx, ty, s);
        if (flag && !__builtin_isfinite(s)) atomicOr(flag, 1);
    }
    __syncthreads();
    nb.row = y * g.nx;
    nb.x = x;
    nb.lphi = slot(tx, ty);
    nb.ls = ls;
    return active;
}

// One tile of the step.
template <class P, int COLL, bool ROWU, bool KEPT>
__device__ __forceinline__ void step2d_tile(const Geom &g, const Phys<typename P::T> &ph, const Ptrs &p,
                                            typename P::T *lphi, int lbx, int cols, int x0, int y0,
                                            int *flag = nullptr)
{
    NbTile<typename P::T, KEPT> nb;
    if (step2d_load<P, ROWU, KEPT>(g, p, lphi, lbx, cols, x0, y0, flag, nb)) collide_body<2, P, COLL>(nb, g, ph, p);
}

// Lane form of the FP16 formats' pulls: the rules of both axes as per-lane selects
// (where y is wavefront-uniform, its part is scalar), against the branches of
// NbLane: 100 x 130 between symmetry planes FP16S 7.8 -> 5.3 us a step.
struct NbFlat {
    int x, row;
    int xs[3], r[3];  // columns and rows of the neighbours (the own one beyond a wall or symmetry plane)
    bool lo, hi, bot, top;  // at an end of an axis that is not periodic
    bool wx, wy;            // that end is a wall (else a symmetry plane)
};
__device__ __forceinline__ NbFlat make_nb(const Geom &g, int x, int y, int, NbFlat *)
{
    NbFlat n;
    const bool px = g.bcx == BC_PER, py = g.bcy == BC_PER;
    n.x = x;
    n.row = y * g.nx;
    n.lo = !px && x == 0;
    n.hi = !px && x == g.nx - 1;
    n.bot = !py && y == 0;
    n.top = !py && y == g.ny - 1;
    n.wx = g.bcx == BC_WALL;
    n.wy = g.bcy == BC_WALL;
    n.xs[0] = x > 0 ? x - 1 : px ? g.nx - 1 : x;
    n.xs[1] = x;
    n.xs[2] = x < g.nx - 1 ? x + 1 : px ? 0 : x;
    n.r[0] = (y > 0 ? y - 1 : py ? g.ny - 1 : y) * g.nx;
    n.r[1] = n.row;
    n.r[2] = (y < g.ny - 1 ? y + 1 : py ? 0 : y) * g.nx;
    return n;
}
template <int D>
__device__ __forceinline__ PullLoc pull_loc(const NbFlat &n, int a)
{
    static_assert(D == 2, "2-D only");
    const int cx = cx_of(a), cy = cy_of(a);
    const bool ex = cx > 0 ? n.lo : cx < 0 ? n.hi : false, ey = cy > 0 ? n.bot : cy < 0 ? n.top : false;
    PullLoc l;
    l.bb = (ex && n.wx) || (ey && n.wy);
    l.dir = l.bb ? 8 - a : a - (ex ? 2 * cx : 0) - (ey ? 6 * cy : 0);
    l.rs = l.bb ? n.row : n.r[1 - cy];
    l.xs = l.bb ? n.x : n.xs[1 - cx];
    return l;
}
template <bool NT = false, typename R>
__device__ __forceinline__ R load_loc(const NbFlat &, const R *base, long long plane, const PullLoc &l)
{
    if constexpr (NT)
        return __builtin_nontemporal_load(&((gptr<const R>)base)[plane + l.rs + l.xs]);
    else
        return gld(base, plane + l.rs + l.xs);
}
template <int D>
__device__ __forceinline__ bool wall_out(const NbFlat &n, int a)
{
    const int cx = cx_of(a), cy = cy_of(a);
    return (n.wx && (cx > 0 ? n.hi : cx < 0 ? n.lo : false)) || (n.wy && (cy > 0 ? n.top : cy < 0 ? n.bot : false));
}
template <typename R>
__device__ __forceinline__ R own_at(const NbFlat &n, const R *base)
{
    return gld(base, n.row + n.x);
}

// One tile of the step in the FP16 formats (NB: NbRow, bx = 64, or NbFlat).
// The references of the level are in p.ref_in, and the update writes the next
// level's to another array, since neighbouring blocks still read these.
template <class P, int COLL, class NB, bool KEPT, bool WIDE>
__device__ __forceinline__ void step2d_tile16(const Geom &g, const Phys<float> &ph, const Ptrs &p,
                                              unsigned long long *lrec, int lbx, int cols, int x0, int y0,
                                              int *flag = nullptr)
{
    const int bx = WIDE ? 64 : 1 << lbx, by = STEP2D_THREADS / bx, ls = bx + 2;
    const int tid = int(threadIdx.x);
    const int tx = tid & (bx - 1);
    const int ty = WIDE ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> lbx;
    const int w = min(cols, g.nx - x0), h = min(by, g.ny - y0);
    auto slot = [&](int i, int j) { return lrec + (j + 1) * ls + i + 1; };
    const Ring2d rim(g, w, h);
    auto record = [&](const auto &nb, int i, int j, unsigned long long *to) {
        const float s = phi_value<2, P>(nb, g.np, p);
        if constexpr (WIDE)
            *to = make_rec(s, own_at(nb, p.ref_in));
        else
            rim.put(slot, i, j, make_rec(s, own_at(nb, p.ref_in)));
        return s;
    };
    // the ring: beyond walls and symmetry planes the mirrored cell's record
    auto ring = [&](auto *form, int i, int j) {
        record(make_nb(g, stencil_coord(x0 + i, g.nx, g.bcx), stencil_coord(y0 + j, g.ny, g.bcy), 0, form), i,
               j, slot(i, j));
    };
    const bool active = tx < w && ty < h;
    NbTile16<NB, KEPT> nb;
    if (active) {
        static_cast<NB &>(nb) = make_nb(g, x0 + tx, y0 + ty, 0, (NB *)nullptr);
        nb.lrec = slot(tx, ty);
        nb.ls = ls;
        const float s = record(nb, tx, ty, slot(tx, ty));
        if (flag && !__builtin_isfinite(s)) atomicOr(flag, 1);
    }
    if constexpr (WIDE) {
        if (ty < 2) {
            if (tx < w) ring((Kept<NB> *)nullptr, tx, ty == 0 ? -1 : h);
        } else if (ty == 2) {
            const int n = h + 2;
            if (tx < 2 * n) ring((Kept<NbFlat> *)nullptr, tx < n ? -1 : w, (tx < n ? tx : tx - n) - 1);
        }
    } else {
        int i, j;
        if (rim.cell(tid, i, j)) ring((Kept<NbFlat> *)nullptr, i, j);
    }
    __syncthreads();
    if (active) collide_body<2, P, COLL>(nb, g, ph, p);
}

// One tile in any format.
enum { TILE_NARROW, TILE_WIDE, TILE_ROW, TILE_LANE };
template <class P, int COLL, bool KEPT, int TILE>
__device__ __forceinline__ void step2d_any(const Geom &g, const Phys<typename P::T> &ph, const Ptrs &p,
                                           void *lds, int lbx, int cols, int x0, int y0, int *flag)
{
    if constexpr (P::F::shifted) {
        using NB = typename std::conditional<TILE == TILE_ROW, NbRow,
                   typename std::conditional<TILE == TILE_LANE, NbLane, NbFlat>::type>::type;
        step2d_tile16<P, COLL, NB, KEPT, TILE == TILE_WIDE || TILE == TILE_ROW>(g, ph, p, static_cast<unsigned long long *>(lds),
                                                              lbx, cols, x0, y0, flag);
    } else {
        step2d_tile<P, COLL, TILE == TILE_WIDE, KEPT>(g, ph, p, static_cast<typename P::T *>(lds), lbx, cols, x0,
                                                        y0, flag);
    }
}
// Narrow tiles, tiles of whole wavefronts, and those whose pulls in the FP16
// formats take the 3-D kernels' row form (x periodic and 32-bit indices).
// (TILE_LANE: narrow, with the 3-D kernels' lane form.)
template <class P>
__host__ __device__ inline int step2d_form(const Geom &g, int lbx)
{
    if (lbx != 6) return TILE_NARROW;
    return P::F::shifted && g.bcx == BC_PER && 9 * g.np < (1ll << 31) ? TILE_ROW : TILE_WIDE;
}

}  // namespace mplb
