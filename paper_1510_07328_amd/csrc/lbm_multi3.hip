// Two lattice BGK steps of a periodic d3v19 box in one pass over memory.
//
// One step per kernel moves 152 B per update in float32 and is bound by that.
// Here a workgroup marches along z over a window of 64 columns (the lanes) and NW
// rows (one per wavefront) and takes two steps on the way: it collides plane z of
// the state it loads and, once that plane's populations have moved to their
// cells, plane z - 1 for the second time, whose populations it streams into the
// other lattice like the push step.  A population that moves in x goes to the
// neighbouring lane by a DPP wave shift, one that moves in y to the neighbouring
// wavefront through LDS (two buffers, one barrier per plane), one that moves in z
// waits in a register.  The window's outermost lanes and rows and a segment's
// first and last plane lack neighbours and are only collided once: 62 columns
// and NW - 2 rows are written (256 columns take five strips).  Reads and writes
// go from one lattice to another, so no workgroup reads what another one writes,
// and every cell update is the same collide() as in the single-step kernels: the
// same results bit for bit.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm_collide.h"
#include "lbm_internal.h"
#include "lbm_multi.h"

namespace lbm {

namespace {

using Lat = D3Q19;
constexpr int Q = Lat::Q;

template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    typedef int int2_t __attribute__((ext_vector_type(2)));
    int2_t w = __builtin_bit_cast(int2_t, v);
    w.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, true);
    w.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, w);
}
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

template <typename T>
struct Rows3 { static constexpr int n = sizeof(T) == 8 ? 8 : 16; };

template <typename T, bool O3>
__global__ void __launch_bounds__(64 * Rows3<T>::n) k_multi3(const T *__restrict__ src, T *__restrict__ dst, Box b,
                                                             Coef<T> c, int strips, int groups, int lz) {
    constexpr int NW = Rows3<T>::n;
    extern __shared__ unsigned char smem3[];
    T(*lds)[NYQ][NW][64] = reinterpret_cast<T(*)[NYQ][NW][64]>(smem3);
    // neighbouring windows share lines: a contiguous run of them per XCD
    const int nb = gridDim.x, per = (nb + 7) >> 3, full = nb & 7;
    const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
    const int blk = full == 0 || xcd <= full ? xcd * per + place : full * per + (xcd - full) * (per - 1) + place;
    const int strip = blk % strips, group = (blk / strips) % groups, seg = blk / (strips * groups);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nx = b.nx, ny = b.ny, nz = b.nz;
    const int xo = strip * 62 + lane - 1, yo = group * (NW - 2) + w - 1;
    // lanes and rows past the last that an output needs repeat that one
    const int xc = xo < nx ? xo : nx, yc = yo < ny ? yo : ny;
    const int x = xc < 0 ? xc + nx : (xc == nx ? 0 : xc), y = yc < 0 ? yc + ny : (yc == ny ? 0 : yc);
    const int z0 = seg * lz, z1 = z0 + lz < nz ? z0 + lz : nz;
    const bool out = lane >= 1 && lane < 63 && xo < nx && w >= 1 && w < NW - 1 && yo < ny;
    using off = uint32_t;
    const off es = sizeof(T);
    const off pl = off(b.plane) * es, rowb = off(nx) * es, planeb = off(nx) * off(ny) * es;
    // slot at a wave-uniform offset (scalar registers) and a lane's
    auto at = [](const T *p, off u, off l) { return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + u + l); };
    auto put = [](T *p, off u, off l, T v) { *reinterpret_cast<T *>(reinterpret_cast<char *>(p) + u + l) = v; };
    // byte offsets of the columns x - 1, x, x + 1 and of the rows y - 1, y, y + 1
    const off ox = off(x) * es, oxm = x == 0 ? rowb - es : ox - es, oxp = x == nx - 1 ? off(0) : ox + es;
    const off oy = off(y) * rowb, oym = y == 0 ? off(ny - 1) * rowb : oy - rowb, oyp = y == ny - 1 ? off(0) : oy + rowb;

    T a[Q], b1[Q];  // ez = 0 of plane z - 1; ez = 1 moved from planes z - 2 (a) and z - 1 (b1)
#pragma unroll
    for (int q = 0; q < Q; ++q) a[q] = b1[q] = T(0);
    T nxt[Q];
    auto fetch = [&](int z) {
        const off o = off(z) * planeb + oy;
#pragma unroll
        for (int q = 0; q < Q; ++q) nxt[q] = at(src, off(q) * pl + o, ox);
    };
    int z = z0 == 0 ? nz - 1 : z0 - 1;  // the plane being loaded
    fetch(z);
    auto advance = [&](int i, auto full) {
        T g[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) g[q] = nxt[q];
        z = z + 1 == nz ? 0 : z + 1;
        fetch(z);  // after the last plane: one that is not used
        collide<Lat, T, O3>(g, c);
        // move the plane's populations in x, and through LDS in y
        T(*buf)[NW][64] = lds[i & 1];
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            g[q] = from_x(g[q], Lat::e[q][0]);
            if (Lat::e[q][1] != 0) buf[yslot(q)][w][lane] = g[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 1; q < Q; ++q)
            if (Lat::e[q][1] != 0) g[q] = buf[yslot(q)][(w - Lat::e[q][1]) & (NW - 1)][lane];
        // the previous plane is complete with the ez = -1 populations of this one
        T f[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int ez = Lat::e[q][2];
            f[q] = ez < 0 ? g[q] : a[q];
            if (ez > 0) {
                a[q] = b1[q];
                b1[q] = g[q];
            } else if (ez == 0) {
                a[q] = g[q];
            }
        }
        if (!decltype(full)::value) return;
        collide<Lat, T, O3>(f, c);
        const int zc = z0 + i - 2;  // its plane
        if (out) {
            const off oz = off(zc) * planeb;
            const off ozm = zc == 0 ? off(nz - 1) * planeb : oz - planeb, ozp = zc == nz - 1 ? off(0) : oz + planeb;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const off xx = Lat::e[q][0] < 0 ? oxm : (Lat::e[q][0] > 0 ? oxp : ox);
                const off yy = Lat::e[q][1] < 0 ? oym : (Lat::e[q][1] > 0 ? oyp : oy);
                const off zz = Lat::e[q][2] < 0 ? ozm : (Lat::e[q][2] > 0 ? ozp : oz);
                put(dst, off(q) * pl + zz + yy, xx, f[q]);
            }
        }
    };
    // the first two planes only fill the pipeline
    advance(0, std::false_type{});
    advance(1, std::false_type{});
    for (int i = 2; i < z1 - z0 + 2; ++i) advance(i, std::true_type{});
}

template <typename T, bool O3>
hipError_t launch_t(const void *src, void *dst, const Box &b, const Coef<T> &c, int lz, hipStream_t s) {
    constexpr int NW = Rows3<T>::n;
    const int strips = (b.nx + 61) / 62, groups = (b.ny + NW - 3) / (NW - 2), segs = (b.nz + lz - 1) / lz;
    const int64_t blocks = (int64_t)strips * groups * segs;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    constexpr size_t lds = sizeof(T) * 2 * NYQ * NW * 64;
    static LdsLimit limit;
    const hipError_t e = limit.raise((const void *)k_multi3<T, O3>, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_multi3<T, O3>), dim3((unsigned)blocks), dim3(64 * NW), lds, s, (const T *)src, (T *)dst, b, c,
                       strips, groups, lz);
    return hipGetLastError();
}

}  // namespace

// Planes per segment, 0 where single steps are faster.  A compute unit takes one
// workgroup at a time; a plane takes about 3.2 us (two collisions of 16 rows: 540
// vector instructions per lane) to 5.9 once the box fills the chip and memory, so
// the segment is the one with the fewest planes in all rounds, and a launch costs
// 4; a single step takes 5 us and 38 ns per thousand cells.
// Measured on MI355X, float32, us per step (one step per kernel first): 256^3 511:
// 399 to 414 (segments of 8 to 32 planes), 128^3 82: 53.5, 200 x 100 x 150 102: 79,
// 64^3 22: 11.4, 40 x 40 x 200 37: 12.8; float64 256^3 1018: 707.  At 256^3 the
// pass is bound by memory: counters give 2.09 GB read and 1.41 GB written for two
// steps (1.27 GB each at best), because the windows' edges are read again (62 of 64
// columns in rows that straddle cache lines, 14 of 16 rows); stores that bypass the
// L2 cost 20 %.
int multi3_plan(int nx, int ny, int nz, int fp64, int cus) {
    if (cus <= 0) cus = 256;
    const int nw = fp64 ? 8 : 16;
    const double cells = (double)nx * ny * nz, size = cells * (fp64 ? 2 : 1);
    const double plane = 3.2 + 2.7 * (size < 2e6 ? size / 2e6 : 1.0);
    const int64_t windows = (int64_t)((nx + 61) / 62) * ((ny + nw - 3) / (nw - 2));
    int best = 0;
    double least = 2.0 * (5.0 + 38e-6 * size);
    for (int lz = 1; lz <= 64 && lz <= nz; ++lz) {
        const int64_t blocks = windows * ((nz + lz - 1) / lz), rounds = (blocks + cus - 1) / cus;
        const double t = 4.0 + (double)rounds * (lz + 2) * plane;
        if (t < least) {
            least = t;
            best = lz;
        }
    }
    return best;
}

hipError_t launch_multi3(int fp64, const void *src, void *dst, const Box &b, const Model &m, double tau,
                         double rho_ref, int lz, hipStream_t s) {
    if (lz < 1 || b.bbx || b.bby || b.bbz) return hipErrorInvalidValue;
    if (fp64) {
        const Coef<double> c = make_coef<double>(m, tau, rho_ref);
        return has_third_order(m) ? launch_t<double, true>(src, dst, b, c, lz, s) : launch_t<double, false>(src, dst, b, c, lz, s);
    }
    const Coef<float> c = make_coef<float>(m, tau, rho_ref);
    return has_third_order(m) ? launch_t<float, true>(src, dst, b, c, lz, s) : launch_t<float, false>(src, dst, b, c, lz, s);
}

}  // namespace lbm
