// Two lattice BGK steps of a d3v19 box in one pass over memory.
//
// One step per kernel moves 152 B per update in float32 and is bound by that.
// Here a workgroup marches along z over a window of 64 columns (the lanes) and 16
// rows (8 in float64) and takes two steps on the way: it collides plane z of
// the state it loads and, once that plane's populations have moved to their
// cells, plane z - 1 for the second time, whose populations it streams into the
// other lattice like the push step.  A population that moves in x goes to the
// neighbouring lane by a DPP wave shift, one that moves in y to the next row: in
// registers or through LDS (two buffers, one barrier per plane); one that moves in
// z waits in a register.  The window's outermost lanes and rows and a segment's
// first and last plane lack neighbours and are only collided once: 62 columns
// and 14 rows are written (256 columns take five strips).  Reads and writes
// go from one lattice to another, so no workgroup reads what another one writes,
// and every cell update is the same collide() as in the single-step kernels: the
// same results bit for bit.
//
// Bound by memory where the box is large: the windows' edges are read again, from
// the L2 as long as neighbouring windows stay within a plane of each other.  There
// (PACED) a wavefront takes two rows and loads and stores them slot by slot, its
// lanes without an output store past the buffer's end instead of branching, and it
// waits for loads without waiting for stores.  256^3 float32: 414 -> 331 us per
// step, L2 misses per pass 3.4 -> 2.9 GB; with loads or stores row by row 371.  A
// plane on its own takes longer that way (4.6 us for 3.2), so a small box has a row
// per wavefront and a branch.  Loads forced ahead of the first collision 376,
// between the collisions 400, three steps per pass 346 (it needs more registers
// than there are and recomputes 4 of 16 rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lbm_collide.h"
#include "lbm_internal.h"
#include "lbm_multi.h"

namespace lbm {

namespace {

using Lat = D3Q19;
constexpr int Q = Lat::Q;

// value of the lane at x - ex (ex a compile-time constant after unrolling)
template <typename T>
__device__ __forceinline__ T from_x(T v, int ex) {
    return ex > 0 ? lane_shift<0x138>(v) : (ex < 0 ? lane_shift<0x130>(v) : v);  // wave_shr:1, wave_shl:1
}

// LDS slot of a population that moves in y (10 of them)
constexpr int yslot(int q) {
    int n = 0;
    for (int k = 0; k < q; ++k) n += Lat::e[k][1] != 0;
    return n;
}
constexpr int NYQ = yslot(Q);

// OPEN: a row per wavefront; PACED: rows in pairs and every store issued; WALLED: a
// row per wavefront and walls on any axis.
enum Kind3 { OPEN, PACED, WALLED };
// W wavefronts of R rows, B LDS buffers
template <typename T, Kind3 KIND>
struct Rows3 {
    static constexpr int W = KIND == PACED || sizeof(T) == 8 ? 8 : 16, R = KIND == PACED && sizeof(T) == 4 ? 2 : 1;
    static constexpr int n = W * R, B = KIND == WALLED ? 3 : 2;
    static constexpr size_t lds = sizeof(T) * B * NYQ * W * 64;
};

template <typename T, bool O3, Kind3 KIND>
__global__ void __launch_bounds__((64 * Rows3<T, KIND>::W)) k_multi3(const T *__restrict__ src,
                                                                            T *__restrict__ dst, Box b, Coef<T> c,
                                                                            int strips, int groups, int lz) {
    constexpr int W = Rows3<T, KIND>::W, R = Rows3<T, KIND>::R, NW = W * R;
    extern __shared__ unsigned char smem3[];
    T(*lds)[NYQ][W][64] = reinterpret_cast<T(*)[NYQ][W][64]>(smem3);
    // neighbouring windows share lines
    const int blk = block_in_xcd_order();
    const int strip = blk % strips, group = (blk / strips) % groups, seg = blk / (strips * groups);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nx = b.nx, ny = b.ny, nz = b.nz;
    const int z0 = seg * lz, z1 = z0 + lz < nz ? z0 + lz : nz;
    using off = uint32_t;
    const off es = sizeof(T);
    const off pl = off(b.plane) * es, rowb = off(nx) * es, planeb = off(nx) * off(ny) * es;
    const LatticeBuffer<T> in(src, off(Q) * pl), to(dst, off(Q) * pl);
    // columns and rows past the last that an output needs repeat that one
    const int xo = strip * 62 + lane - 1, xc = xo < nx ? xo : nx;
    const int x = xc < 0 ? xc + nx : (xc == nx ? 0 : xc);
    // byte offsets of the columns x - 1, x, x + 1 and of the rows y - 1, y, y + 1
    const off ox = off(x) * es, oxm = x == 0 ? rowb - es : ox - es, oxp = x == nx - 1 ? off(0) : ox + es;
    off oy[R], oym[R], oyp[R];
    bool out[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k = w * R + r, yo = group * (NW - 2) + k - 1, yc = yo < ny ? yo : ny;
        const int y = yc < 0 ? yc + ny : (yc == ny ? 0 : yc);
        oy[r] = off(y) * rowb;
        oym[r] = y == 0 ? off(ny - 1) * rowb : oy[r] - rowb;
        oyp[r] = y == ny - 1 ? off(0) : oy[r] + rowb;
        out[r] = k >= 1 && k < NW - 1 && yo < ny;
    }
    // WALLED: does link q of this lane's cell leave the box through a wall; zm, zp: its plane lies there
    const bool wxm = b.bbx && x == 0, wxp = b.bbx && x == nx - 1;
    const bool wym = b.bby && oy[0] == 0u, wyp = b.bby && oy[0] == off(ny - 1) * rowb;
    const bool anyxy = KIND == WALLED && (wym || wyp || __builtin_amdgcn_ballot_w64(wxm || wxp) != 0);
    auto leaves = [&](int q, bool zm, bool zp) {
        const int ex = Lat::e[q][0], ey = Lat::e[q][1], ez = Lat::e[q][2];
        return (ex < 0 && wxm) || (ex > 0 && wxp) || (ey < 0 && wym) || (ey > 0 && wyp) || (ez < 0 && zm) || (ez > 0 && zp);
    };
    const bool outx = lane >= 1 && lane < 63 && xo < nx;

    T a[R][Q], b1[R][Q];  // ez = 0 of plane z - 1; ez = 1 moved from planes z - 2 (a) and z - 1 (b1)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < Q; ++q) a[r][q] = b1[r][q] = T(0);
    T nxt[R][Q];
    auto fetch = [&](int z) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int r = 0; r < R; ++r) nxt[r][q] = in.load(off(q) * pl + (off(z) * planeb + oy[r]), ox);
    };
    int z = z0 == 0 ? nz - 1 : z0 - 1;  // the plane being loaded
    fetch(z);
    auto advance = [&](int i, auto full) {
        T g[R][Q];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < Q; ++q) g[r][q] = nxt[r][q];
        const int zi = z;
        z = z + 1 == nz ? 0 : z + 1;
        fetch(z);  // after the last plane: one that is not used
#pragma unroll
        for (int r = 0; r < R; ++r) collide<Lat, T, O3>(g[r], c);
        // move the plane's populations in x, and in y: between a wavefront's rows in its
        // registers, to its neighbours through LDS
        T(*buf)[W][64] = lds[KIND == WALLED ? i % 3 : i & 1];
#pragma unroll
        for (int q = 1; q < Q; ++q) {
#pragma unroll
            for (int r = 0; r < R; ++r) g[r][q] = from_x(g[r][q], Lat::e[q][0]);
            if (Lat::e[q][1] != 0) buf[yslot(q)][w][lane] = g[Lat::e[q][1] > 0 ? R - 1 : 0][q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const int ey = Lat::e[q][1];
            if (ey == 0) continue;
            const T v = buf[yslot(q)][(w - ey) & (W - 1)][lane];
            if (R > 1) g[ey > 0 ? R - 1 : 0][q] = g[ey > 0 ? 0 : R - 1][q];
            g[ey > 0 ? 0 : R - 1][q] = v;
        }
        if constexpr (KIND == WALLED) {
            // Populations that cannot arrive: the cell's own of the opposite link, as collided.
            // Those sit one lane off in a register, or in the cell's row of the LDS buffer of
            // its plane (the third buffer keeps the previous plane's until all have read it).
            const int zj = zi == 0 ? nz - 1 : zi - 1;
            const bool am = b.bbz && zi == 0, ap = b.bbz && zi == nz - 1, bm = b.bbz && zj == 0, bp = b.bbz && zj == nz - 1;
            if (anyxy || am || ap || bm || bp) {
                T(*old)[W][64] = lds[(i + 2) % 3];
                auto own = [&](int p, T moved, T(*rows)[W][64]) {
                    return Lat::e[p][1] != 0 ? rows[yslot(p)][w][(lane + Lat::e[p][0]) & 63] : from_x(moved, -Lat::e[p][0]);
                };
#pragma unroll
                for (int q = 1; q < Q; ++q) {
                    const int p = Lat::opp[q], ez = Lat::e[q][2];
                    if (ez > 0) {  // q enters plane zi from below, p plane zi - 1 from above
                        const T u = own(p, g[0][p], buf), v = own(q, b1[0][q], old);
                        if (leaves(q, bm, bp)) g[0][p] = v;
                        if (leaves(p, am, ap)) b1[0][q] = u;
                    } else if (ez == 0 && q < p) {
                        const T u = own(p, g[0][p], buf), v = own(q, g[0][q], buf);
                        if (leaves(p, am, ap)) g[0][q] = u;
                        if (leaves(q, am, ap)) g[0][p] = v;
                    }
                }
            }
        }
        // the previous plane is complete with the ez = -1 populations of this one
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int ez = Lat::e[q][2];
                const T v = g[r][q];
                if (ez >= 0) g[r][q] = a[r][q];
                if (ez > 0) {
                    a[r][q] = b1[r][q];
                    b1[r][q] = v;
                } else if (ez == 0) {
                    a[r][q] = v;
                }
            }
        if (!decltype(full)::value) return;
#pragma unroll
        for (int r = 0; r < R; ++r) collide<Lat, T, O3>(g[r], c);
        const int zc = z0 + i - 2;  // the plane that has taken two steps
        const off oz = off(zc) * planeb;
        const off ozm = zc == 0 ? off(nz - 1) * planeb : oz - planeb, ozp = zc == nz - 1 ? off(0) : oz + planeb;
        auto store = [&](int q, int r, off none) {
            const off xx = Lat::e[q][0] < 0 ? oxm : (Lat::e[q][0] > 0 ? oxp : ox);
            const off yy = Lat::e[q][1] < 0 ? oym[r] : (Lat::e[q][1] > 0 ? oyp[r] : oy[r]);
            const off zz = Lat::e[q][2] < 0 ? ozm : (Lat::e[q][2] > 0 ? ozp : oz);
            to.store(off(q) * pl + zz + yy, none | xx, g[r][q]);
        };
        const bool zm = b.bbz && zc == 0, zp = b.bbz && zc == nz - 1;
        if constexpr (KIND == PACED) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int r = 0; r < R; ++r) store(q, r, outx && out[r] ? 0u : kNoStore);
        } else if (KIND == WALLED && (anyxy || zm || zp)) {
            if (outx && out[0]) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const off xx = Lat::e[q][0] < 0 ? oxm : (Lat::e[q][0] > 0 ? oxp : ox);
                    const off yy = Lat::e[q][1] < 0 ? oym[0] : (Lat::e[q][1] > 0 ? oyp[0] : oy[0]);
                    const off zz = Lat::e[q][2] < 0 ? ozm : (Lat::e[q][2] > 0 ? ozp : oz);
                    to.store(0u, leaves(q, zm, zp) ? off(Lat::opp[q]) * pl + oz + oy[0] + ox : off(q) * pl + zz + yy + xx,
                             g[0][q]);
                }
            }
        } else if (outx && out[0]) {
#pragma unroll
            for (int q = 0; q < Q; ++q) store(q, 0, 0u);
        }
    };
    // the first two planes only fill the pipeline
#pragma unroll 1
    for (int i = 0; i < 2; ++i) advance(i, std::false_type{});
    wait_loads();
#pragma unroll 1
    for (int i = 2; i < z1 - z0 + 2; ++i) advance(i, std::true_type{});
}

template <typename T, bool O3, Kind3 KIND>
hipError_t launch_k(const void *src, void *dst, const Box &b, const Coef<T> &c, int lz, hipStream_t s) {
    using Rows = Rows3<T, KIND>;
    const int strips = (b.nx + 61) / 62, groups = (b.ny + Rows::n - 3) / (Rows::n - 2), segs = (b.nz + lz - 1) / lz;
    const int64_t blocks = (int64_t)strips * groups * segs;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    static LdsLimit limit;
    const hipError_t e = limit.raise((const void *)k_multi3<T, O3, KIND>, (int)Rows::lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_multi3<T, O3, KIND>), dim3((unsigned)blocks), dim3(64 * Rows::W), Rows::lds, s,
                       (const T *)src, (T *)dst, b, c, strips, groups, lz);
    return hipGetLastError();
}

// Boxes from 2 million float32 cells on (half as many in float64) are bound by memory.
bool paced(double size) { return size >= 2e6; }

template <typename T, bool O3>
hipError_t launch_t(const void *src, void *dst, const Box &b, const Coef<T> &c, int lz, hipStream_t s) {
    if (b.bbx || b.bby || b.bbz) return launch_k<T, O3, WALLED>(src, dst, b, c, lz, s);
    if (paced((double)b.nx * b.ny * b.nz * (sizeof(T) / 4))) return launch_k<T, O3, PACED>(src, dst, b, c, lz, s);
    return launch_k<T, O3, OPEN>(src, dst, b, c, lz, s);
}

}  // namespace

// Planes per segment, 0 where single steps are faster.  A compute unit takes one
// workgroup at a time, so the segment is the one whose rounds take the least time.
// A plane takes 3.1 us (two collisions of 16 rows: 540 vector instructions per
// lane, in float64 of 8 rows), up to 5.9 in larger boxes; in the memory-bound ones
// 5.8 (5.1) and 0.4 % more per plane of the segment, as neighbours drift apart.  A
// launch costs 4; a single step takes 5 us and 38 ns per thousand cells.
// Measured on MI355X, float32, us per step (one step per kernel first): 256^3 511:
// 331 (414 before, with branches and rows of their own), 256 x 256 x 60 115: 82 (95),
// 160^3 137: 79 (81), 200 x 100 x 150 102: 73 (78), 128^3 82: 49.5 (52), 64^3 22: 9.4
// (9.8), 40 x 40 x 200 37: 10.8 (11.1); float64 256^3 1018: 690 (707).
// With walls a wavefront that holds one reads its own populations back.  float64: a
// plane takes 3.6 us and 1.8 more in large boxes, a single step 8 us for a start;
// passes win at every size measured (30^3 9.4: 6.0, 64^3 18.4: 13.3, 128^3 116: 104,
// 200 x 100 x 150 191: 131, 256^3 1025: 700).  float32 (16 wavefronts of 128 registers,
// 20 of them spilled) is slower, most of all with walls in x, where every wavefront
// holds one in every plane: a plane takes 4.6 us there, 4.0 with walls in y, 3.5 in z,
// and in boxes from 3 million cells on 5.0, 4.4 and 4.0 more; a single step takes 6 us
// for a start, a seventh with a wavefront for every SIMD, 1.5 ns per wavefront, at least
// 2 ns per workgroup, and the lattice's traffic at 5.2 TB/s.  Single steps against the
// best pass measured, us per step, walls in x / y / z:
//   64^3               13.8: 15.5   13.8: 13.4   14.1: 11.5
//   100^3              39.5: 35.6   39.8: 27.1   41.0: 21.9
//   128^3              59.2: 75.7   59.7: 59.4   61.7: 59.1
//   160^3             124: 133     123: 98       125: 88
//   200 x 100 x 150    91: 103      92: 87        94: 78
//   256^3             491: 460     485: 419      488: 419
// (256^3 with walls in x keeps single steps: its passes gain 1 to 6 %).
int multi3_plan(int nx, int ny, int nz, int fp64, int walls, int cus) {
    if (cus <= 0) cus = 256;
    const int nw = fp64 ? 8 : 16;
    const double cells = (double)nx * ny * nz, size = cells * (fp64 ? 2 : 1);
    const bool pace = paced(size) && !walls;
    const double fill = size < 2e6 ? size / 2e6 : 1.0, wide = cells < 3e6 ? cells / 3e6 : 1.0;
    const double plane = pace ? (fp64 ? 5.1 : 5.8)
                         : !walls ? 3.1 + 2.8 * fill
                         : fp64   ? 3.6 + 1.8 * fill
                                  : (walls == 3 ? 4.6 + 5.0 * wide : walls == 2 ? 4.0 + 4.4 * wide : 3.5 + 4.0 * wide);
    const int64_t windows = (int64_t)((nx + 61) / 62) * ((ny + nw - 3) / (nw - 2));
    double least = 2.0 * (5.0 + 38e-6 * size);  // of two single steps
    if (walls && fp64) {
        least = 2.0 * (8.0 + 38e-6 * size) * (size > 1e6 ? 0.85 : 1.0);
    } else if (walls) {
        const int block = nx < 256 ? (nx + 63) / 64 * 64 : 256;
        const double blocks = (double)ny * nz * ((nx + block - 1) / block), waves = blocks * (block / 64);
        const double single[] = {6.0 + (waves < 1024 ? waves / 1024 : 1.0) + 1.5e-3 * waves, 6.0 + 2e-3 * blocks,
                                 cells * 152 / 5.2e6};
        least = 2.0 * std::max({single[0], single[1], single[2]}) * (walls == 3 ? 0.97 : 1.0);
    }
    int best = 0;
    for (int lz = 1; lz <= 64 && lz <= nz; ++lz) {
        const int64_t blocks = windows * ((nz + lz - 1) / lz), rounds = (blocks + cus - 1) / cus;
        const double t = 4.0 + (double)rounds * (lz + 2) * plane * (pace ? 1.0 + 0.004 * lz : 1.0);
        if (t < least) {
            least = t;
            best = lz;
        }
    }
    return best;
}

hipError_t launch_multi3(int fp64, const void *src, void *dst, const Box &b, const Model &m, double tau,
                         double rho_ref, int lz, hipStream_t s) {
    if (lz < 1) return hipErrorInvalidValue;
    if (fp64) {
        const Coef<double> c = make_coef<double>(m, tau, rho_ref);
        return has_third_order(m) ? launch_t<double, true>(src, dst, b, c, lz, s) : launch_t<double, false>(src, dst, b, c, lz, s);
    }
    const Coef<float> c = make_coef<float>(m, tau, rho_ref);
    return has_third_order(m) ? launch_t<float, true>(src, dst, b, c, lz, s) : launch_t<float, false>(src, dst, b, c, lz, s);
}

}  // namespace lbm
