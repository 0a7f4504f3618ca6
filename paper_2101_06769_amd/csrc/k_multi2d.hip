// Several steps of a small 2-D lattice in plain storage per launch.
#include "device.hpp"

namespace mplb {

// A step of a lattice of some 10^4 cells is a launch, a round trip to memory
// and about 1.5 us of a wavefront's own chain of instructions.  This kernel pays
// the first two once for K steps (64 x 256 FP64 4.85 -> 3.26 us a step, 97 x 113
// FP32 4.44 -> 2.94), and is bound by the chain: two wavefronts a SIMD keep the VALU
// 38 % (64 x 256 FP64) to 41 % busy (128 x 512 FP32, single relaxation time); the
// rest is dependent instructions and barriers, more so as the region shrinks to a
// wavefront or two.  A block loads a tile of MULTI_EDGE^2 cells
// into LDS and steps it there, the region it can still compute shrinking by two
// cells a side and step (a cell's update reaches the phase-field values two
// cells away), and stores the MULTI_EDGE - 4 K cells square that are left.  The
// cells computed twice carry the same bits in every block, and the arithmetic
// is collide_body's, so the results are those of single steps.
constexpr int MULTI_THREADS = 512;  // phi of the first step: (MULTI_EDGE - 2)^2 = 484 cells

// coordinate v (any integer) on an axis of n cells; -1 outside one that is not periodic
__device__ __forceinline__ int multi_coord(int v, int n, int bc)
{
    if ((unsigned)v < (unsigned)n) return v;
    if (bc != BC_PER) return -1;
    v %= n;
    return v < 0 ? v + n : v;
}

template <class P, int COLL>
__global__ void __launch_bounds__(MULTI_THREADS) k_multi2d(Geom g, Phys<typename P::T> ph, Ptrs p, int K, int ntx)
{
    using T = typename P::T;
    extern __shared__ double multi_lds[];
    constexpr int E = MULTI_EDGE, C = MULTI_CELLS;
    T *pop = reinterpret_cast<T *>(multi_lds), *lphi = pop + 18 * C;
    const int tid = int(threadIdx.x);
    const int bid = tile_of<true>(int(blockIdx.x), int(gridDim.x));
    const int core = E - 4 * K;
    const int x0 = (bid % ntx) * core - 2 * K, y0 = (bid / ntx) * core - 2 * K;
    const T *F = static_cast<const T *>(p.Fin), *G = static_cast<const T *>(p.Gin);
    for (int e = tid; e < C; e += MULTI_THREADS) {
        const int x = multi_coord(x0 + e % E, g.nx, g.bcx), y = multi_coord(y0 + e / E, g.ny, g.bcy);
        if (x < 0 || y < 0) continue;
        const int cell = y * g.nx + x;
        T v[18];
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            v[a] = gld(F + a * g.np, cell);
            v[9 + a] = gld(G + a * g.np, cell);
        }
#pragma unroll
        for (int a = 0; a < 18; ++a) pop[a * C + e] = v[a];
    }
    __syncthreads();
    const bool nper_x = g.bcx != BC_PER, nper_y = g.bcy != BC_PER;
    for (int s = 0; s < K; ++s) {
        // phi on w x w cells from (1 + 2 s, 1 + 2 s), the update one cell
        // inside: the cells that update fill the first wavefronts, so that the
        // ring, which only sums phi, does not spread them over more
        const int w = E - 2 - 4 * s, in = w - 2;
        int li, lj;
        const bool updates = tid < in * in;
        if (updates) {
            lj = tid / in;
            li = tid - lj * in + 1;
            ++lj;
        } else {
            const int r = tid - in * in, q = r - 2 * w;  // two rows of w, then two columns of w - 2
            li = q < 0 ? (r < w ? r : r - w) : q < in ? 0 : w - 1;
            lj = q < 0 ? (r < w ? 0 : w - 1) : 1 + (q < in ? q : q - in);
        }
        const int i = li + 1 + 2 * s, j = lj + 1 + 2 * s, e = j * E + i;
        const int x = x0 + i, y = y0 + j;
        const bool here = tid < w * w && !(nper_x && (unsigned)x >= (unsigned)g.nx) &&
                          !(nper_y && (unsigned)y >= (unsigned)g.ny);
        NbMulti<T> nb;
        if (here) {
            const bool xl = nper_x && x == 0, xh = nper_x && x == g.nx - 1;
            const bool yl = nper_y && y == 0, yh = nper_y && y == g.ny - 1;
            if (__any(xl || xh || yl || yh)) {
                const bool wx = g.bcx == BC_WALL, wy = g.bcy == BC_WALL;
#pragma unroll
                for (int a = 0; a < 9; ++a) {
                    const int cx = cx_of(a), cy = cy_of(a);
                    const bool ex = cx > 0 ? xl : cx < 0 ? xh : false, ey = cy > 0 ? yl : cy < 0 ? yh : false;
                    const bool bb = (ex && wx) || (ey && wy);
                    const int dir = bb ? 8 - a : a - (ex ? 2 * cx : 0) - (ey ? 6 * cy : 0);
                    const int at = dir * C + (bb ? e : e - (ex ? 0 : cx) - (ey ? 0 : E * cy));
                    nb.f[a] = pop[at];
                    nb.gp[a] = pop[9 * C + at];
                }
            } else {
                const T *p0 = pop + e, *p1 = p0 + 9 * C;
#pragma unroll
                for (int a = 0; a < 9; ++a) {
                    nb.f[a] = p0[a * C - cx_of(a) - E * cy_of(a)];
                    nb.gp[a] = p1[a * C - cx_of(a) - E * cy_of(a)];
                }
            }
            T sum = 0;
#pragma unroll
            for (int a = 0; a < 9; ++a) sum += nb.gp[a];
            lphi[e] = sum;
            nb.pop = pop + e;
            nb.phi = lphi + e;
            nb.ox[0] = xl ? 0 : -1; nb.ox[1] = 0; nb.ox[2] = xh ? 0 : 1;
            nb.oy[0] = yl ? 0 : -E; nb.oy[1] = 0; nb.oy[2] = yh ? 0 : E;
        }
        __syncthreads();  // phi is complete, and every value of the level has been pulled
        if (here && updates) collide_body<2, P, COLL>(nb, g, ph, p);
        __syncthreads();
    }
    const int j = tid / core, i = tid - j * core;
    const int x = x0 + 2 * K + i, y = y0 + 2 * K + j;
    if (j < core && x < g.nx && y < g.ny) {
        const int e = (j + 2 * K) * E + i + 2 * K, cell = y * g.nx + x;
        T *Fo = static_cast<T *>(p.Fout), *Go = static_cast<T *>(p.Gout);
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            *lane_ptr(Fo, a * g.np, cell) = pop[a * C + e];
            *lane_ptr(Go, a * g.np, cell) = pop[(9 + a) * C + e];
        }
    }
}

static long long multi2d_tiles(const Geom &g, int steps)
{
    const int core = MULTI_EDGE - 4 * steps;
    return (long long)((g.nx + core - 1) / core) * ((g.ny + core - 1) / core);
}

// As many steps as leave every block a CU of its own (256): cells computed
// twice then cost idle units, not time.  Per step, single steps and 2, 3, 4 a
// launch: 64 x 256 FP64 (4) 4.85, 4.67, 3.86, 3.26 us; 128 x 256 FP32 (3) 4.87,
// 4.07, 3.47, 3.84; 256 x 256 FP32 (2) 4.80, 4.20, 4.48, 5.63, FP64 6.02, 5.54,
// 7.18, 10.95; 400 x 400 FP32 (1) 7.28, 7.10, 7.86, 11.22.
int multi2d_steps(const Ctx &c)
{
    // the first-order phase-field equilibrium keeps (phi u) of every step in memory
    if (c.dim != 2 || (c.storage != ST_FP64 && c.storage != ST_FP32) || c.ph.cac_edf) return 1;
    for (int steps = 4; steps > 1; --steps)
        if (multi2d_tiles(c.g, steps) <= 256) return steps;
    return 1;
}

hipError_t launch_multi2d(const Ctx &c, int steps)
{
    if (steps < 2 || steps != multi2d_steps(c)) return hipErrorInvalidValue;
    const int core = MULTI_EDGE - 4 * steps;
    const int ntx = (c.g.nx + core - 1) / core;
    return with_coll(coll_code(c.ph), [&](auto cc) -> hipError_t {
        constexpr int COLL = decltype(cc)::value;
        if constexpr ((COLL & 2) != 0) {
            return hipErrorInvalidValue;
        } else {
            auto go = [&]<class P>(P *) {
                using T = typename P::T;
                const size_t lds = size_t(19) * MULTI_CELLS * sizeof(T);
                hipLaunchKernelGGL((k_multi2d<P, COLL>), dim3(unsigned(multi2d_tiles(c.g, steps))), dim3(MULTI_THREADS), lds, c.stream,
                                   c.g, to_phys<T>(c.ph), c.p, steps, ntx);
                return hipGetLastError();
            };
            return c.storage == ST_FP64 ? go((P64 *)nullptr) : go((P32 *)nullptr);
        }
    });
}

}  // namespace mplb
