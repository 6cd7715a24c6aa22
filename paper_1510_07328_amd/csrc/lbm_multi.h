// Several steps of a d2v9 box per pass: in registers (lbm_multi.hip), which boxes,
// how deep and the launch; small boxes in LDS (lbm_tile.hip).
#pragma once

#include "lbm_internal.h"
#include "lds_limit.h"

namespace lbm {

// value of the lane to the left (x - 1) or to the right (x + 1); 0 at the strip's edge
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
// The workgroup's place in an order that gives each of the 8 XCDs, over which the
// hardware deals workgroups round robin, a contiguous run.
__device__ __forceinline__ int block_in_xcd_order() {
    const int nb = gridDim.x, per = (nb + 7) >> 3, full = nb & 7;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    return full == 0 || xcd <= full ? xcd * per + slot : full * per + (xcd - full) * (per - 1) + slot;
}

// One lattice as a buffer: a slot at a wave-uniform byte offset plus a lane's.  The
// hardware drops a store whose lane offset lies past the buffer, so a lane that has
// nothing to write takes kNoStore instead of a branch; behind a branch the compiler
// cannot count the stores in flight, and the wait for the next row's loads becomes
// one for every store.
constexpr uint32_t kNoStore = 0xffffffffu;
template <typename T>
struct LatticeBuffer {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ LatticeBuffer(const T *p, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, (int)bytes, 0x00020000)) {}
    __device__ __forceinline__ T load(uint32_t uniform, uint32_t lane) const {
        if constexpr (sizeof(T) == 8)
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane, (int)uniform, 0));
        else
            return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane, (int)uniform, 0));
    }
    __device__ __forceinline__ void store(uint32_t uniform, uint32_t lane, T v) const {
        if constexpr (sizeof(T) == 8) {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)lane, (int)uniform, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)lane, (int)uniform, 0);
        }
    }
};
// Waits for the loads in flight (vmcnt 0).  Before a loop that keeps stores in
// flight: else the waits at its head count as on entry, where no store follows the loads.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

constexpr int kMultiTail = 24;  // the last steps of a call, planned together

struct MultiPlan {
    int best = 0;     // steps per pass
    double time = 0;  // estimated microseconds per step
    int ly[8] = {};   // rows per segment, by depth
    // the next launch (1: a single step, 0: none fits) of n steps that are to take
    // an even (0) or odd (1) number of launches
    signed char next[kMultiTail + 1][2] = {};
};

// d2v9, or d3v19 without solids or a force; one weight for all cells, a lattice below 4 GiB
bool multi_eligible(int lattice, bool local, bool porous, int64_t plane, size_t elt);
// links: walls or solid cells; single: a single step may stand between passes (push; an AA step changes the layout)
MultiPlan multi_plan(int nx, int ny, int fp64, bool links, bool single, int cus);
// The next launch of n > 0 steps that are to take an even or odd number of launches.
int multi_depth(const MultiPlan &p, int64_t n, int odd);
// H steps from src into dst (another lattice), both in natural layout.
hipError_t launch_multi(int fp64, int H, const void *src, void *dst, const uint32_t *lm, const Box &b, const Model &m,
                        double tau, double rho_ref, const double *F, int ly, hipStream_t s);

// Two steps of a d3v19 box per pass (lbm_multi3.hip), segments of lz
// planes (multi3_plan: 0 where single steps are faster).
// walls: 0 none, 1 in z only, 2 in y (and z), 3 in x (and others)
int multi3_plan(int nx, int ny, int nz, int fp64, int walls, int cus);
hipError_t launch_multi3(int fp64, const void *src, void *dst, const Box &b, const Model &m, double tau,
                         double rho_ref, int lz, hipStream_t s);

// Small boxes: tiles in LDS (lbm_tile.hip).
constexpr int kTileSteps = 4096;  // most steps of one launch

struct TilePlan {
    int sx = 0, sy = 0;  // tile
    int h = 0;           // steps per launch
    double time = 0;     // estimated microseconds per step
    bool one = false;    // a launch of one step beats the single-step kernel
};
TilePlan tile_plan(int nx, int ny, bool bbx, bool bby, bool porous, int fp64, int cus);
// h <= p.h steps from src into dst, both in natural layout.
hipError_t launch_tile(int fp64, const TilePlan &p, int h, const void *src, void *dst, const uint32_t *lm,
                       const Box &b, const Model &m, double tau, double rho_ref, const double *F, hipStream_t s);

}  // namespace lbm
