// Several steps of a small d2v9 box per launch, in LDS.
//
// A box of a few thousand to a few hundred thousand cells is bound by latency:
// one step per kernel pays a launch (2 to 5 us) per step, and the register
// pipeline of lbm_multi.hip runs H (ly + H - 1) dependent collisions per pass in
// each wavefront.  Here a workgroup holds a window of the box in LDS, one cell
// per thread, and advances it h steps in place (AA pattern) with one barrier per
// step; the launch is paid once per h steps and every SIMD works on a step at
// the same time.  The window is the workgroup's tile plus h cells on each side
// of an axis that is cut; an axis that fits whole is not cut and keeps its own
// periodicity or walls.  At a cut the window's edge reflects, and the wrong
// populations travel one cell per step, through the halo only.
//
// A thread's cell does not change, so the eight slots that its odd steps use are
// resolved once, walls, solid cells and wraps included: population q is written
// to slot q of the cell at x + e_q, or to the cell's own slot -q where that link
// is reflected, and read back for -q from the same place.  The state goes from
// one lattice in natural layout to the other.  Same collide() per cell as the
// single-step kernels: the same results bit for bit.
#include <hip/hip_runtime.h>

#include "lbm_collide.h"
#include "lbm_internal.h"
#include "lbm_multi.h"

namespace lbm {

namespace {

using Lat = D2Q9;
constexpr int Q = Lat::Q;
// cells of a window: the nine planes of float64 within the 65535 bytes of an LDS
// instruction's immediate offset
constexpr int PL = 1008;

struct TileArgs {
    int sx, sy, h;       // tile, steps
    int ntx, cx, cy;     // tiles along x; 1 = the axis is whole
};

template <typename T, bool O3, bool POROUS>
__global__ void __launch_bounds__(1024) k_tile(const T *__restrict__ src, T *__restrict__ dst,
                                               const uint32_t *__restrict__ lm, Box b, Coef<T> c, Force<T> F,
                                               TileArgs a) {
    __shared__ T lds[Q * PL];
    const int tx = blockIdx.x % a.ntx, ty = blockIdx.x / a.ntx;
    const int x0 = tx * a.sx, y0 = ty * a.sy;
    const int nsx = b.nx - x0 < a.sx ? b.nx - x0 : a.sx, nsy = b.ny - y0 < a.sy ? b.ny - y0 : a.sy;
    // halo columns and rows; none beyond a wall
    int hl = 0, hr = 0, hb = 0, ht = 0;
    if (!a.cx) {
        hl = b.bbx && x0 < a.h ? x0 : a.h;
        hr = b.bbx && b.nx - x0 - nsx < a.h ? b.nx - x0 - nsx : a.h;
    }
    if (!a.cy) {
        hb = b.bby && y0 < a.h ? y0 : a.h;
        ht = b.bby && b.ny - y0 - nsy < a.h ? b.ny - y0 - nsy : a.h;
    }
    const int W = nsx + hl + hr, H = nsy + hb + ht, cells = W * H;
    const int own = threadIdx.x;
    const bool live = own < cells;
    const int cx = own % W, cy = own / W;
    int x = x0 - hl + cx, y = y0 - hb + cy;  // periodic boxes: wrapped
    x = x < 0 ? x + b.nx : (x >= b.nx ? x - b.nx : x);
    y = y < 0 ? y + b.ny : (y >= b.ny ? y - b.ny : y);
    const int64_t cell = (int64_t)y * b.nx + x;
    const bool mine = live && cx >= hl && cx < hl + nsx && cy >= hb && cy < hb + nsy;
    const uint32_t m = POROUS && live ? lm[cell] : 0u;
    const bool solid = (m & kSolidBit) != 0;

    // Steps of one cell along an axis, as a change of index; `wall`: reflected there
    // (a wall of the box, or a cut, where any rule will do).
    const bool wrapx = a.cx && !b.bbx, wrapy = a.cy && !b.bby;
    const bool wl = cx == 0 && !wrapx, wr = cx == W - 1 && !wrapx;
    const bool wb = cy == 0 && !wrapy, wt = cy == H - 1 && !wrapy;
    const int dxm = cx == 0 ? W - 1 : -1, dxp = cx == W - 1 ? 1 - W : 1;
    const int dym = cy == 0 ? (H - 1) * W : -W, dyp = cy == H - 1 ? -(H - 1) * W : W;
    int slot[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int ex = Lat::e[q][0], ey = Lat::e[q][1];
        const bool bb = (ex < 0 && wl) || (ex > 0 && wr) || (ey < 0 && wb) || (ey > 0 && wt) || ((m >> q) & 1u);
        const int to = own + (ex < 0 ? dxm : ex > 0 ? dxp : 0) + (ey < 0 ? dym : ey > 0 ? dyp : 0);
        slot[q] = bb ? Lat::opp[q] * PL + own : q * PL + to;
    }

    T g[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) g[q] = T(0);
    if (live) {
#pragma unroll
        for (int q = 0; q < Q; ++q) g[q] = src[q * b.plane + cell];
    }
    const bool run = live && !solid;
    for (int s = 0; s < a.h; s += 2) {
        if (run) {
            if (s > 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q) g[q] = lds[q * PL + own];
            }
            collide<Lat, T, O3, POROUS>(g, c, F.F);
#pragma unroll
            for (int q = 0; q < Q; ++q) lds[Lat::opp[q] * PL + own] = g[q];
        }
        __syncthreads();
        if (s + 1 < a.h) {
            if (run) {
#pragma unroll
                for (int q = 0; q < Q; ++q) g[q] = lds[slot[Lat::opp[q]]];
                collide<Lat, T, O3, POROUS>(g, c, F.F);
#pragma unroll
                for (int q = 0; q < Q; ++q) lds[slot[q]] = g[q];
            }
            __syncthreads();
        }
    }
    if (!mine) return;
    if (a.h & 1) {
#pragma unroll
        for (int q = 0; q < Q; ++q) g[q] = lds[slot[Lat::opp[q]]];
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) g[q] = lds[q * PL + own];
    }
    if (solid) return;  // its slots are not written
#pragma unroll
    for (int q = 0; q < Q; ++q) dst[q * b.plane + cell] = g[q];
}

// Window of a tile along one axis at h steps.
int window(int n, int s, bool whole, bool walls, int h) {
    if (whole) return n;
    const int full = s + 2 * h;
    return walls && full > n ? n : full;
}

template <typename T>
hipError_t launch_t(const TilePlan &p, int h, const void *src, void *dst, const uint32_t *lm, const Box &b,
                    const Model &m, double tau, double rho_ref, const double *F, hipStream_t s) {
    const bool wx = p.sx >= b.nx, wy = p.sy >= b.ny;
    const int W = window(b.nx, p.sx, wx, b.bbx, h), H = window(b.ny, p.sy, wy, b.bby, h);
    // a periodic axis is wrapped once, so its window may reach one box beyond each end
    if ((int64_t)W * H > PL || h < 1 || (!wx && h > b.nx) || (!wy && h > b.ny)) return hipErrorInvalidValue;
    const Coef<T> c = make_coef<T>(m, tau, rho_ref);
    const Force<T> f{{T(F[0]), T(F[1]), T(F[2])}};
    const TileArgs a{p.sx, p.sy, h, (b.nx + p.sx - 1) / p.sx, wx ? 1 : 0, wy ? 1 : 0};
    const dim3 grid(a.ntx * ((b.ny + p.sy - 1) / p.sy)), blk((W * H + 63) / 64 * 64);
    const bool o3 = has_third_order(m);
    const T *in = (const T *)src;
    if (lm && o3) hipLaunchKernelGGL((k_tile<T, true, true>), grid, blk, 0, s, in, (T *)dst, lm, b, c, f, a);
    else if (lm) hipLaunchKernelGGL((k_tile<T, false, true>), grid, blk, 0, s, in, (T *)dst, lm, b, c, f, a);
    else if (o3) hipLaunchKernelGGL((k_tile<T, true, false>), grid, blk, 0, s, in, (T *)dst, lm, b, c, f, a);
    else hipLaunchKernelGGL((k_tile<T, false, false>), grid, blk, 0, s, in, (T *)dst, lm, b, c, f, a);
    return hipGetLastError();
}

}  // namespace

// Tile and steps per launch from the time of a launch of h steps, in microseconds:
// 2.2, the window's loads and the tile's stores at 19.5 KB per
// microsecond and compute unit (a fifth less where the tile's rows are not whole
// 64-byte runs), and h times a
// step, which takes `wave` per wavefront that shares a SIMD and at least `least`
// (the chain of one collision, its LDS reads and the barrier).
// Measured on MI355X, us per step at the best tile against one step per kernel
// and the register pipeline: 512 x 4 float64 with walls 0.49 (h = 24), 5.0, 1.9;
// 128 x 4 0.46, 4.0, 1.8; 256^2 1.48 (32 x 8, h = 6), 5.0, 2.1; 700 x 150 with
// solids and a force 2.35 to 2.4, 7.6, 2.9; 512^2 2.97, 7.8, 3.15.
// Calls of one or two steps come down to launches of one step (`one`): 3.7 and 0.40
// (0.46) per wavefront of a compute unit, against a single-step kernel that takes 4.6
// (4.0 up to 1024 cells), 2.2 ns per column of the row a workgroup runs through (3.2
// with solids; float64 2.6 and 4.0) and 10 ps per cell from 40 000 cells on (float64
// 22, 4 more with solids).  Single step against tile of one step, us: 32^2 4.2: 4.3,
// 128^2 4.9: 4.5, 160^2 5.0: 4.5, 200^2 5.1: 6.2, 300^2 6.3: 7.7, 512 x 64 5.5: 4.9,
// 2048 x 8 8.4: 4.6, 8192 x 8 23: 5.5; float64 256^2 6.3: 7.1, 700 x 150 8.2: 7.3.
TilePlan tile_plan(int nx, int ny, bool bbx, bool bby, bool porous, int fp64, int cus) {
    TilePlan best{};
    best.time = 1e300;
    if (cus <= 0) cus = 256;
    const double wave = fp64 ? 0.25 : porous ? 0.27 : 0.225, least = fp64 ? 0.44 : 0.41;
    const double cell_bytes = Q * (fp64 ? 8.0 : 4.0);
    const int xs[] = {nx, 64, 48, 32, 24, 16, 8}, ys[] = {ny, 64, 48, 40, 32, 28, 24, 20, 18, 16, 14, 12, 10, 8, 6, 4};
    for (int sy : ys) {
        if (sy > ny) continue;
        const bool wy = sy >= ny;
        for (int sx : xs) {
            if (sx > nx) continue;
            const bool wx = sx >= nx;
            const int64_t tiles = (int64_t)((nx + sx - 1) / sx) * ((ny + sy - 1) / sy);
            if (tiles > 4 * (int64_t)cus) break;  // smaller tiles only make more
            const int hmax = wx && wy ? kTileSteps : 32;
            for (int h = wx && wy ? kTileSteps : 1; h <= hmax; ++h) {
                if ((!wx && h > nx) || (!wy && h > ny)) break;
                const int64_t win = (int64_t)window(nx, sx, wx, bbx, h) * window(ny, sy, wy, bby, h);
                if (win > PL) break;
                const int64_t waves = (win + 63) / 64, per_cu = (tiles + cus - 1) / cus;
                const double load = (double)((waves * per_cu + 3) / 4) * wave;
                const double move = (double)per_cu * cell_bytes * (double)(win + (int64_t)sx * sy) / 19.5e3;
                const double t = (load > least ? load : least) + (2.2 + (sx % 16 && !wx ? 1.2 : 1.0) * move) / h;
                if (t < best.time) best = TilePlan{sx, sy, h, t};
            }
        }
    }
    if (best.h > 0) {
        const int64_t tiles = (int64_t)((nx + best.sx - 1) / best.sx) * ((ny + best.sy - 1) / best.sy);
        const int64_t win = (int64_t)window(nx, best.sx, best.sx >= nx, bbx, 1) * window(ny, best.sy, best.sy >= ny, bby, 1);
        const double waves = (double)((win + 63) / 64 * ((tiles + cus - 1) / cus)), cells = (double)nx * ny;
        const double column = (fp64 ? 2.6e-3 : 2.2e-3) + (porous ? (fp64 ? 1.4e-3 : 1.0e-3) : 0.0);
        const double cell = (fp64 ? 2.2e-5 : 1.0e-5) + (porous ? 0.4e-5 : 0.0);
        const double single = (cells <= 1024 && !porous ? 4.0 : 4.6) + column * nx + (cells > 4e4 ? cell * (cells - 4e4) : 0.0);
        best.one = 3.7 + (fp64 ? 0.46 : 0.40) * waves < single;
    }
    return best;
}

hipError_t launch_tile(int fp64, const TilePlan &p, int h, const void *src, void *dst, const uint32_t *lm,
                       const Box &b, const Model &m, double tau, double rho_ref, const double *F, hipStream_t s) {
    if (b.nz != 1 || p.sx < 1 || p.sy < 1) return hipErrorInvalidValue;
    if (fp64) return launch_t<double>(p, h, src, dst, lm, b, m, tau, rho_ref, F, s);
    return launch_t<float>(p, h, src, dst, lm, b, m, tau, rho_ref, F, s);
}

}  // namespace lbm
