// Several steps of a d2v9 box per pass (lbm_multi.hip): which boxes, how deep,
// and the launch.
#pragma once

#include "lbm_internal.h"

namespace lbm {

constexpr int kMultiTail = 24;  // the last steps of a call, planned together

struct MultiPlan {
    int best = 0;     // steps per pass
    int ly[8] = {};   // rows per segment, by depth
    // the next launch (1: a single step, 0: none fits) of n steps that are to take
    // an even (0) or odd (1) number of launches
    signed char next[kMultiTail + 1][2] = {};
};

// d2v9, one weight for all cells, a lattice below 4 GiB
bool multi_eligible(int lattice, bool local, int nx, int ny, int64_t plane, size_t elt);
// links: walls or solid cells; single: a single step may stand between passes (push; an AA step changes the layout)
MultiPlan multi_plan(int nx, int ny, int fp64, bool links, bool single, int cus);
// The next launch of n > 0 steps that are to take an even or odd number of launches.
int multi_depth(const MultiPlan &p, int64_t n, int odd);
// H steps from src into dst (another lattice), both in natural layout.
hipError_t launch_multi(int fp64, int H, const void *src, void *dst, const uint32_t *lm, const Box &b, const Model &m,
                        double tau, double rho_ref, const double *F, int ly, hipStream_t s);

}  // namespace lbm
