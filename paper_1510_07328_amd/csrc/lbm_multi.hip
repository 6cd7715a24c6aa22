// Several lattice BGK steps of a d2v9 box in one pass over memory.
//
// One step per kernel reads and writes every population once (72 B per update
// in float32) and is bound by that traffic.  Here one wavefront marches down a
// strip of 64 columns and carries H steps at a time in registers: a lane is a
// column, a row enters the pipeline as it is loaded, level k + 1 collides row
// y - 1 once level k has collided row y, and row y - (H - 1) leaves after H
// steps.  A population that moves in y waits in a register for its row; one
// that moves in x goes to the neighbouring lane by a DPP wave shift.  There is
// no LDS and no barrier; traffic per update falls to (1 + reread) / H.
//
// The strip's outermost lanes and rows lack neighbours, so each level loses one
// column per side: of the 64 lanes, 64 - 2 (H - 1) columns are written, and a
// segment of `ly` rows is entered H - 1 rows early and left H - 1 rows late
// (recomputed by the neighbouring segment).  The state is read from one lattice
// in natural layout (populations at their own slots) and the last level streams
// into the other lattice like the push step, so no wavefront reads what another
// one writes.  Every cell update is the same collide() as the single-step
// kernels in the same order, so H steps here equal H single steps bit for bit.
//
// Walls and solid cells: a link that leaves the box or ends in a solid cell
// returns to its cell reversed.  Their modes keep the previous row's collided
// populations, and a wavefront row that holds such a link replaces the gathered
// values by the cell's own.  A solid cell's slots are neither written in dst nor used.
//
// Bound: vector issue for deep pipelines (102 instructions per update, 6 of them
// lane shifts; 256 CUs x 64 lanes), memory for H = 2 and 3; 2048^2 float32 47.9
// -> 17.7 us per step, 4096^2 262 -> 63, 2048^2 float64 115 -> 28.  Registers:
// 9 values per level and 9 of the next row; periodic float32 kernels are held to
// 128 VGPRs (4 wavefronts per SIMD; 168 at 6 steps), float64 to 256.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "lbm_collide.h"
#include "lbm_internal.h"
#include "lbm_multi.h"

namespace lbm {

namespace {

using Lat = D2Q9;
constexpr int Q = Lat::Q;
constexpr int kWaves = 4;  // wavefronts per workgroup, neighbouring strips of one segment

// the population q of the cell x, from the lane of x - e_qx
template <int EX, typename T>
__device__ __forceinline__ T from_x(T v) {
    if constexpr (EX > 0) return lane_shift<0x138>(v);  // wave_shr:1
    else if constexpr (EX < 0) return lane_shift<0x130>(v);  // wave_shl:1
    else return v;
}

// Bits q whose link leaves the box through a wall in -x, +x, -y, +y.
constexpr uint32_t link_bits(int d, int s) {
    uint32_t m = 0;
    for (int q = 0; q < Q; ++q)
        if (Lat::e[q][d] == s) m |= 1u << q;
    return m;
}

// Populations between two levels.  push() takes the collided row y of a level
// and returns in `in` the streamed row y - 1 for the next one.
//   OPEN (no reflected links): the row y - 1 so far and the e_y = 1 part of row y.
template <typename T>
struct Open {
    T a[6];  // row y - 1: q = 0, 1, 2, 3, 5, 6
    T b[3];  // row y: q = 2, 5, 6
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < 6; ++i) a[i] = T(0);
#pragma unroll
        for (int i = 0; i < 3; ++i) b[i] = T(0);
    }
    __device__ __forceinline__ void push(const T (&g)[Q], T (&in)[Q]) {
        in[0] = a[0]; in[1] = a[1]; in[2] = a[2]; in[3] = a[3]; in[5] = a[4]; in[6] = a[5];
        in[4] = g[4];
        in[7] = from_x<-1>(g[7]);
        in[8] = from_x<1>(g[8]);
        a[0] = g[0];
        a[1] = from_x<1>(g[1]);
        a[2] = b[0];
        a[3] = from_x<-1>(g[3]);
        a[4] = b[1];
        a[5] = b[2];
        b[0] = g[2];
        b[1] = from_x<1>(g[5]);
        b[2] = from_x<-1>(g[6]);
    }
};
//   CLOSED: the whole collided row y - 1 (p) and the e_y = 1 part of row y - 2 (s, moved in x).
//   m: bit a set when the link of the cell of row y - 1 along e_a is reflected.
template <typename T>
struct Closed {
    T p[Q];
    T s[3];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < Q; ++i) p[i] = T(0);
#pragma unroll
        for (int i = 0; i < 3; ++i) s[i] = T(0);
    }
    __device__ __forceinline__ void push(const T (&g)[Q], T (&in)[Q], uint32_t m, bool any) {
        in[0] = p[0];
        in[1] = from_x<1>(p[1]);
        in[2] = s[0];
        in[3] = from_x<-1>(p[3]);
        in[4] = g[4];
        in[5] = s[1];
        in[6] = s[2];
        in[7] = from_x<-1>(g[7]);
        in[8] = from_x<1>(g[8]);
        if (any) {
#pragma unroll
            for (int q = 1; q < Q; ++q)
                if ((m >> Lat::opp[q]) & 1u) in[q] = p[Lat::opp[q]];
        }
        s[0] = p[2];
        s[1] = from_x<1>(p[5]);
        s[2] = from_x<-1>(p[6]);
#pragma unroll
        for (int q = 0; q < Q; ++q) p[q] = g[q];
    }
};

// MODE 0: periodic box; 1: walls in x or y; 2: solid cells and a body force
// (and walls).  Grid: wavefront w takes strip w % strips of segment w / strips.
// BUF (the deepest float32 pipeline): the lattices as buffers and every store issued,
// the lanes without an output past the buffer's end, so that a row's loads are waited
// for without its stores; 3 wavefronts per SIMD instead of 4 and a spill: 2048^2 18.4
// -> 17.7 us per step, 4096^2 65 -> 63.3.  The other kernels have wavefronts enough to
// cover that wait, and the added stores of edge lanes cost them up to 5 %.
template <typename T, int H, int MODE>
constexpr bool kBuf = MODE == 0 && H == 6 && sizeof(T) == 4;

template <typename T, bool O3, int H, int MODE>
__global__ void __launch_bounds__(64 * kWaves, (MODE ? 1 : sizeof(T) == 8 ? 2 : kBuf<T, H, MODE> ? 3 : 4))
    k_multi(const T *__restrict__ src, T *__restrict__ dst, const uint32_t *__restrict__ lm, Box bx, Coef<T> c,
            Force<T> F, int strips, int ly, int nwaves) {
    constexpr int WO = 64 - 2 * (H - 1);  // columns a strip writes
    constexpr uint32_t XM = link_bits(0, -1), XP = link_bits(0, 1), YM = link_bits(1, -1), YP = link_bits(1, 1);
    // neighbouring strips and segments share the lines at their edges
    const int blk = block_in_xcd_order();
    const int wid = __builtin_amdgcn_readfirstlane(blk * kWaves + (int)(threadIdx.x >> 6));
    if (wid >= nwaves) return;
    const int strip = wid % strips, seg = wid / strips;
    const int lane = threadIdx.x & 63;
    const int nx = bx.nx, ny = bx.ny;
    const int xo = strip * WO + lane - (H - 1);
    int x = xo % nx;
    if (x < 0) x += nx;
    const bool outlane = lane >= H - 1 && lane < 64 - (H - 1) && xo < nx;
    using off = uint32_t;
    const off pl = off(bx.plane) * off(sizeof(T)), rowb = off(nx) * off(sizeof(T));
    const off ox = off(x) * off(sizeof(T));
    const off oxm = x == 0 ? rowb - off(sizeof(T)) : ox - off(sizeof(T));
    const off oxp = x == nx - 1 ? off(0) : ox + off(sizeof(T));
    auto at = [](const T *p, off o) { return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + o); };
    auto put = [](T *p, off o, T v) { *reinterpret_cast<T *>(reinterpret_cast<char *>(p) + o) = v; };
    constexpr bool BUF = kBuf<T, H, MODE>;
    const LatticeBuffer<T> from(src, off(Q) * pl), to(dst, off(Q) * pl);
    const int r0 = seg * ly, r1 = r0 + ly < ny ? r0 + ly : ny;
    const int iters = r1 - r0 + 2 * (H - 1);
    int row = (r0 - (H - 1)) % ny;  // the row being loaded, wrapped
    if (row < 0) row += ny;

    uint32_t mx = 0u;
    if (MODE >= 1 && bx.bbx) mx = (x == 0 ? XM : 0u) | (x == nx - 1 ? XP : 0u);
    const bool anyx = MODE >= 1 && __builtin_amdgcn_ballot_w64(mx != 0u) != 0;
    // links of row r reflected at the y walls
    auto ybits = [&](int r) { return MODE >= 1 && bx.bby ? (r == 0 ? YM : 0u) | (r == ny - 1 ? YP : 0u) : 0u; };

    std::conditional_t<MODE == 0, Open<T>, Closed<T>> lev[H - 1];
#pragma unroll
    for (int k = 0; k < H - 1; ++k) lev[k].clear();
    uint32_t mk[H];  // MODE 2: link masks of the rows in flight, newest first
#pragma unroll
    for (int k = 0; k < H; ++k) mk[k] = 0u;

    T nxt[Q];
    uint32_t mnxt = 0u;
    auto fetch = [&](int r) {
        const off o = off(r) * rowb;
#pragma unroll
        for (int q = 0; q < Q; ++q) nxt[q] = BUF ? from.load(off(q) * pl + o, ox) : at(src, off(q) * pl + o + ox);
        if (MODE == 2) mnxt = lm[(int64_t)r * nx + x];
    };
    fetch(row);
    // The first 2 (H - 1) rows fill the pipeline (a level starts once its first
    // row's neighbours are there); in a loop of its own, the full pipeline runs
    // without branches and their register copies.
    auto advance = [&](int i, auto full) {
        constexpr bool FULL = decltype(full)::value;
        T g[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) g[q] = nxt[q];
        if (MODE == 2) {
#pragma unroll
            for (int k = H - 1; k > 0; --k) mk[k] = mk[k - 1];
            mk[0] = mnxt;
        }
        const int r = row;
        row = row + 1 == ny ? 0 : row + 1;
        fetch(row);  // after the last row: one that is not used
        collide<Lat, T, O3, MODE == 2>(g, c, F.F);
        int rk = r;  // row of level k
#pragma unroll
        for (int k = 0; k < H - 1; ++k) {
            rk = rk == 0 ? ny - 1 : rk - 1;
            T in[Q];
            if constexpr (MODE == 0) {
                lev[k].push(g, in);
            } else {
                const uint32_t m = mx | ybits(rk) | (MODE == 2 ? mk[k + 1] : 0u);
                const bool any = MODE == 2 ? __builtin_amdgcn_ballot_w64(m != 0u) != 0 : anyx || ybits(rk) != 0u;
                lev[k].push(g, in, m, any);
            }
            if (!FULL && i < 2 * (k + 1)) return;
#pragma unroll
            for (int q = 0; q < Q; ++q) g[q] = in[q];
            collide<Lat, T, O3, MODE == 2>(g, c, F.F);
        }
        // row rk has taken H steps: stream it into dst
        const uint32_t m = MODE == 0 ? 0u : mx | ybits(rk) | (MODE == 2 ? mk[H - 1] : 0u);
        const off oz = off(rk) * rowb;
        const off om = rk == 0 ? off(ny - 1) * rowb : oz - rowb, op = rk == ny - 1 ? off(0) : oz + rowb;
        if constexpr (BUF) {
            const off none = outlane ? 0u : kNoStore;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const off ro = Lat::e[q][1] < 0 ? om : (Lat::e[q][1] > 0 ? op : oz);
                const off xx = Lat::e[q][0] < 0 ? oxm : (Lat::e[q][0] > 0 ? oxp : ox);
                to.store(off(q) * pl + ro, none | xx, g[q]);
            }
        } else if (outlane && !(MODE == 2 && (m & kSolidBit))) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const off ro = Lat::e[q][1] < 0 ? om : (Lat::e[q][1] > 0 ? op : oz);
                const off xx = Lat::e[q][0] < 0 ? oxm : (Lat::e[q][0] > 0 ? oxp : ox);
                if constexpr (MODE == 0) {
                    put(dst, off(q) * pl + ro + xx, g[q]);
                } else {
                    const bool bb = (m >> q) & 1u;
                    put(dst, bb ? off(Lat::opp[q]) * pl + oz + ox : off(q) * pl + ro + xx, g[q]);
                }
            }
        }
    };
    int i = 0;
    for (; i < 2 * (H - 1); ++i) advance(i, std::false_type{});
    if (BUF) wait_loads();
    for (; i < iters; ++i) advance(i, std::true_type{});
}

template <typename T, bool O3, int H>
hipError_t launch_h(int mode, const void *src, void *dst, const uint32_t *lm, const Box &b, const Coef<T> &c,
                    const Force<T> &F, int ly, hipStream_t s) {
    const int wo = 64 - 2 * (H - 1);
    const int strips = (b.nx + wo - 1) / wo, segs = (b.ny + ly - 1) / ly;
    const int64_t waves = (int64_t)strips * segs;
    if (waves > 0x7fffff00) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((waves + kWaves - 1) / kWaves)), blk(64 * kWaves);
    const T *a = (const T *)src;
    if (mode == 0)
        hipLaunchKernelGGL((k_multi<T, O3, H, 0>), grid, blk, 0, s, a, (T *)dst, lm, b, c, F, strips, ly, (int)waves);
    else if (mode == 1)
        hipLaunchKernelGGL((k_multi<T, O3, H, 1>), grid, blk, 0, s, a, (T *)dst, lm, b, c, F, strips, ly, (int)waves);
    else
        hipLaunchKernelGGL((k_multi<T, O3, H, 2>), grid, blk, 0, s, a, (T *)dst, lm, b, c, F, strips, ly, (int)waves);
    return hipGetLastError();
}

template <typename T, bool O3>
hipError_t launch_o(int H, int mode, const void *src, void *dst, const uint32_t *lm, const Box &b, const Coef<T> &c,
                    const Force<T> &F, int ly, hipStream_t s) {
    switch (H) {
    case 2: return launch_h<T, O3, 2>(mode, src, dst, lm, b, c, F, ly, s);
    case 3: return launch_h<T, O3, 3>(mode, src, dst, lm, b, c, F, ly, s);
    case 4: return launch_h<T, O3, 4>(mode, src, dst, lm, b, c, F, ly, s);
    case 6: return launch_h<T, O3, 6>(mode, src, dst, lm, b, c, F, ly, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_t(int H, const void *src, void *dst, const uint32_t *lm, const Box &b, const Model &m, double tau,
                    double rho_ref, const double *F, int ly, hipStream_t s) {
    const Coef<T> c = make_coef<T>(m, tau, rho_ref);
    const Force<T> f{{T(F[0]), T(F[1]), T(F[2])}};
    const int mode = lm ? 2 : (b.bbx || b.bby ? 1 : 0);
    return has_third_order(m) ? launch_o<T, true>(H, mode, src, dst, lm, b, c, f, ly, s)
                              : launch_o<T, false>(H, mode, src, dst, lm, b, c, f, ly, s);
}

constexpr int kDepths[] = {2, 3, 4, 6};

}  // namespace

bool multi_eligible(int lattice, bool local, bool porous, int64_t plane, size_t elt) {
    // 32-bit byte offsets from the lattice base, as in the single-step kernels
    const int q = lattice == LBM_D2V9 ? D2Q9::Q : D3Q19::Q;
    return !local && (lattice == LBM_D2V9 || (lattice == LBM_D3V19 && !porous)) &&
           (uint64_t)q * (uint64_t)plane * elt < (uint64_t(1) << 32);
}

int multi_depth(const MultiPlan &p, int64_t n, int odd) {
    return n > kMultiTail ? p.best : p.next[n][odd];
}

// Depth and segment length from the time of a step, in microseconds:
//   issue: a SIMD runs w wavefronts, each H (ly + H - 1) rows of collisions of
//     `row` (fitted: 0.20 in float32, 0.25 with walls or solids, 0.30 in float64;
//     one or two wavefronts leave gaps: f[w]);
//   memory: the lattice written once and read once, with the recomputed columns
//     and rows, at 4.8 TB/s (7 when both lattices fit the 256 MB Infinity Cache);
//   the two overlap (a fourth-power mean), and a launch and the first rows'
//     latency take 4.
// Measured on MI355X, us per step, H = 2 / 3 / 4 / 6 at their best ly (one AA
// step per kernel first): 2048^2 float32 48: 32.2 / 22.9 / 19.3 / 17.7; 4096^2
// 262: 124 / 87 / 77 / 63; 1531 x 1019 with walls 21.6: 10.8 / 8.9 / 9.3 / 9.8;
// 2048^2 float64 115: 62 / 42 / 34 / 28.0; 256^2 4.7: 2.2 / 2.1 / 2.1 / 2.3;
// 700 x 150 with solids 7.7: 2.9 / 3.0 / 3.2 / 3.7.  Small boxes want short
// pipelines (their wavefronts run a few rows each), large ones deep (the traffic
// is divided by H, the issue of about 102 vector instructions per update is
// not: at 4096^2 and H = 6 it takes 55 of the 63 us).
// The rule takes 4 wavefronts per SIMD in float32 and 2 in float64; fewer fit the deep
// pipelines (float32 H = 6: 3, with links 2; float64 with walls H = 6 and with solids H = 4
// and 6: 1).  With links at the rule's choice and at the best depth and segment (one AA step
// per kernel): walls 1000^2 6.3, 6.3 (13.7), 2048^2 21.0, 19.4 (47.6), 4096^2 74, 70 (261),
// float64 8.8, 8.7 (24.5), 33.6, 31.9 (110), 122, 121 (486); solids 8.0, 7.8 (15.7), 26.6,
// 23.6 (52), 90, 88 (282), float64 12.5, 10.5 (26.2), 44, 42 (117), 160, 157 (513).
MultiPlan multi_plan(int nx, int ny, int fp64, bool links, bool single, int cus) {
    MultiPlan p{};
    const double row = fp64 ? 0.30 : links ? 0.25 : 0.20, bytes = 9.0 * (fp64 ? 8 : 4) * (double)nx * ny;
    const double rate = 2.0 * bytes <= 256e6 ? 7e6 : 4.8e6;  // bytes per microsecond
    const double f[] = {0, 1.45, 1.10, 1.0};
    const int simds = 4 * (cus > 0 ? cus : 256), wmax = fp64 ? 2 : 4;
    double best = 1e300, pass[8] = {};  // microseconds of a launch, by depth
    for (int H : kDepths) {
        const int wo = 64 - 2 * (H - 1), strips = (nx + wo - 1) / wo;
        double here = 1e300;
        for (int w = 1; w <= wmax; ++w) {
            int64_t segs = (int64_t)w * simds / strips;
            if (segs < 1) segs = 1;
            if (segs > ny) segs = ny;
            const int ly = (int)((ny + segs - 1) / segs);
            const int64_t waves = (int64_t)strips * ((ny + ly - 1) / ly);
            const int64_t rounds = (waves + simds - 1) / simds;
            const double issue = (double)rounds * (ly + H - 1) * row * f[rounds < 3 ? rounds : 3];
            const double mem = bytes * (64.0 / wo * (ly + 2.0 * (H - 1)) / ly + 1.0) / H / rate;
            const double t = std::pow(std::pow(issue, 4) + std::pow(mem, 4), 0.25) + 4.0 / H;
            if (t < here) {
                here = t;
                p.ly[H] = ly;
            }
        }
        pass[H] = here * H;
        if (here < best) {
            best = here;
            p.best = H;
        }
    }
    p.time = best;
    // The last steps: the cheapest launches that sum to n, by their count's parity
    // (the state has to end in the lattice that n single steps leave it in).
    pass[1] = 2.0 * bytes / 6e6 + 3.0;
    double cost[kMultiTail + 1][2];
    cost[0][0] = 0.0;
    cost[0][1] = 1e300;
    for (int n = 1; n <= kMultiTail; ++n)
        for (int odd = 0; odd < 2; ++odd) {
            cost[n][odd] = 1e300;
            for (int H : {1, 2, 3, 4, 6}) {
                if (H > n || (H == 1 && !single) || cost[n - H][odd ^ 1] >= 1e300) continue;
                const double t = pass[H] + cost[n - H][odd ^ 1];
                if (t < cost[n][odd]) {
                    cost[n][odd] = t;
                    p.next[n][odd] = (signed char)H;
                }
            }
        }
    return p;
}

hipError_t launch_multi(int fp64, int H, const void *src, void *dst, const uint32_t *lm, const Box &b, const Model &m,
                        double tau, double rho_ref, const double *F, int ly, hipStream_t s) {
    if (ly < 1 || b.nz != 1) return hipErrorInvalidValue;
    if (fp64) return launch_t<double>(H, src, dst, lm, b, m, tau, rho_ref, F, ly, s);
    return launch_t<float>(H, src, dst, lm, b, m, tau, rho_ref, F, ly, s);
}

}  // namespace lbm
