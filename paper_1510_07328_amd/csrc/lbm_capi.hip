// C ABI of liblbm: argument checking, workspace carving, launches and graph
// replay around the kernels of lbm_kernels.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "lbm_internal.h"
#include "lbm_multi.h"

namespace lbm {
hipError_t launch_step(int lattice, int fp64, int scheme, int parity, void *a, void *b, const Box &box, const Model &m,
                       double tau, double rho_ref, int block, const uint32_t *lm, const double *F, hipStream_t s);
hipError_t launch_init(int lattice, int fp64, void *lat, const double *n0, const double *u0, const Box &box,
                       const Model &m, double tau, double rho_ref, int block, hipStream_t s);
hipError_t launch_moments(int lattice, int fp64, const void *lat, double *n, double *u, const Box &box, double rho_ref,
                          int odd, int block, const uint32_t *lm, const double *F, int row0, int nrows,
                          int64_t ostride, hipStream_t s);
hipError_t launch_totals(int lattice, int fp64, const void *lat, double *part, double *out, const Box &box,
                         double rho_ref, int odd, int block, const uint32_t *lm, hipStream_t s);
hipError_t launch_link_mask(int D, const unsigned char *solid, uint32_t *lm, const Box &box, int block,
                            hipStream_t s);
}  // namespace lbm

namespace lbm {
namespace {
thread_local std::string g_err;
}  // namespace
void set_last_error(const std::string &msg) { g_err = msg; }
}  // namespace lbm

using namespace lbm;

namespace {

lbm_status fail(lbm_status s, const std::string &msg) {
    g_err = msg;
    return s;
}

lbm_status hip_fail(hipError_t e, const char *what) {
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return LBM_ERR_HIP;
}

constexpr size_t kAlign = 256;
constexpr size_t kPlanePadBytes = 33 * 256;
constexpr size_t kStageBytes = size_t(4) << 20;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    int64_t cells = 0, plane = 0;  // plane: elements between population planes
    int rows = 0;
    size_t elt = 0, lattice_bytes = 0, part_off = 0, out_off = 0, mask_off = 0, stage_off = 0, total = 0;
    size_t min_total = 0;  // without the second lattice of an AA box whose calls fuse steps
    bool multi = false;    // calls of several steps run as passes of several steps
    int stage_rows = 0;  // rows of moments staged per chunk of the host lbm_moments
    int nlat = 0;
    bool porous = false;  // obstacles or a body force: link mask in the workspace, porous kernels
};

constexpr int kCus = 256;  // compute units of an MI355X (the workspace does not depend on the device)

// d3v19: planes per segment of a pass, 0 for a box that runs single steps
int planes3(const lbm_config *cfg, int cus) {
    const int walls = cfg->bc[0] == LBM_BOUNCEBACK ? 3 : cfg->bc[1] == LBM_BOUNCEBACK ? 2 : cfg->bc[2] == LBM_BOUNCEBACK ? 1 : 0;
    return multi3_plan(cfg->nx, cfg->ny, cfg->nz, cfg->precision == LBM_FP64, walls, cus);
}

lbm_status check_config(const lbm_config *cfg, Model *m, Layout *lay) {
    std::string err;
    lbm_status s = build_model(cfg, m, &err);
    if (s != LBM_OK) return fail(s, err);
    if (cfg->nx < 1 || cfg->ny < 1 || cfg->nz < 1) return fail(LBM_ERR_ARG, "box sizes must be >= 1");
    if (m->D < 2 && cfg->ny != 1) return fail(LBM_ERR_ARG, "d1v3 needs ny = 1");
    if (m->D < 3 && cfg->nz != 1) return fail(LBM_ERR_ARG, "2D lattices need nz = 1");
    if (cfg->lattice == LBM_D2V41) {
        if (cfg->nx < 4 || cfg->ny < 4) return fail(LBM_ERR_ARG, "d2v41 needs nx, ny >= 4 (links of four cells)");
        if (cfg->block > D2Q41::MAXB) return fail(LBM_ERR_ARG, "d2v41 kernels take at most 512 threads per workgroup");
        if (cfg->bc[0] != LBM_PERIODIC || cfg->bc[1] != LBM_PERIODIC)
            return fail(LBM_ERR_UNSUPPORTED, "d2v41 runs on periodic boxes only");
        if (cfg->obstacles || cfg->force[0] != 0.0 || cfg->force[1] != 0.0 || cfg->force[2] != 0.0)
            return fail(LBM_ERR_UNSUPPORTED, "d2v41 has no obstacles or body force (41 links exceed the link mask)");
    }
    for (int d = 0; d < 3; ++d)
        if (cfg->bc[d] != LBM_PERIODIC && cfg->bc[d] != LBM_BOUNCEBACK) return fail(LBM_ERR_ARG, "bad bc");
    if (cfg->precision != LBM_FP32_DEV && cfg->precision != LBM_FP64) return fail(LBM_ERR_ARG, "bad precision");
    if (cfg->scheme != LBM_SCHEME_PUSH && cfg->scheme != LBM_SCHEME_AA) return fail(LBM_ERR_ARG, "bad scheme");
    if (cfg->block != 0 && (cfg->block < 64 || cfg->block > 1024 || cfg->block % 64))
        return fail(LBM_ERR_ARG, "block must be 0 or a multiple of 64 in [64, 1024]");
    if (cfg->graph_steps < 0 || cfg->graph_steps % 2) return fail(LBM_ERR_ARG, "graph_steps must be even, >= 0");
    if (cfg->obstacles != 0 && cfg->obstacles != 1) return fail(LBM_ERR_ARG, "obstacles must be 0 or 1");
    for (int d = 0; d < 3; ++d)
        if (!std::isfinite(cfg->force[d])) return fail(LBM_ERR_ARG, "force must be finite");
    const int64_t rows = (int64_t)cfg->ny * cfg->nz;
    const int64_t cells = rows * cfg->nx;
    if (rows > 0x7fffffff) return fail(LBM_ERR_ARG, "too many rows for one launch");
    lay->cells = cells;
    lay->rows = (int)rows;
    lay->elt = cfg->precision == LBM_FP64 ? sizeof(double) : sizeof(float);
    lay->nlat = cfg->scheme == LBM_SCHEME_AA ? 1 : 2;
    // population planes cells + pad apart: 33 x 256 B, so that the planes of a
    // power-of-two box do not all start on the same HBM channel
    lay->plane = cells + (int64_t)(kPlanePadBytes / lay->elt);
    lay->lattice_bytes = align_up((size_t)m->Q * (size_t)lay->plane * lay->elt);
    lay->part_off = lay->lattice_bytes * lay->nlat;
    lay->out_off = lay->part_off + align_up((size_t)rows * 5 * sizeof(double));
    lay->mask_off = lay->out_off + align_up(5 * sizeof(double));
    lay->porous = cfg->obstacles || cfg->force[0] != 0.0 || cfg->force[1] != 0.0 || cfg->force[2] != 0.0;
    lay->stage_off = lay->mask_off + (lay->porous ? align_up((size_t)cells * sizeof(uint32_t)) : 0);
    // staging of the host lbm_moments: whole rows of n and u0 (float64), about
    // kStageBytes at a time (at least one row)
    const size_t row_bytes = (size_t)(m->D + 1) * sizeof(double) * (size_t)cfg->nx;
    int64_t srows = (int64_t)(kStageBytes / row_bytes);
    if (srows < 1) srows = 1;
    if (srows > rows) srows = rows;
    lay->stage_rows = (int)srows;
    const size_t stage = align_up((size_t)srows * row_bytes);
    lay->min_total = lay->total = lay->stage_off + stage;
    lay->multi = multi_eligible(cfg->lattice, m->local != 0, lay->porous, lay->plane, lay->elt) &&
                 (m->D == 2 || planes3(cfg, kCus) > 0);
    // AA: the second lattice of the passes, which between calls is free for the staging
    if (lay->multi && lay->nlat == 1)
        lay->total = lay->stage_off + (lay->lattice_bytes > stage ? lay->lattice_bytes : stage);
    return LBM_OK;
}

int default_block(int nx) {
    int b = 256;
    if (nx < b) b = (nx + 63) / 64 * 64;
    return b < 64 ? 64 : b;
}

}  // namespace

struct lbm_ctx_s {
    lbm_config cfg{};
    Model model{};
    Layout lay{};
    Box box{};
    char *ws = nullptr;
    void *lat[2] = {nullptr, nullptr};
    double *part = nullptr, *out = nullptr;
    uint32_t *lm = nullptr;  // link mask (porous runs only)
    double F[3] = {0.0, 0.0, 0.0};
    int cur = 0;          // index of the lattice holding the state
    int64_t steps = 0;    // steps done
    int block = 256;
    int fp64 = 0;
    double rho_ref = 1.0;
    hipStream_t stream = nullptr;
    hipStream_t cap = nullptr;  // private stream for graph capture
    bool multi = false;   // calls of several steps run as passes between the two lattices
    MultiPlan plan{};
    TilePlan tile{};      // small boxes (h > 0): tiles in LDS instead
    int lz = 0;           // d3v19: planes per segment of a pass of two steps (0: single steps)
    hipGraphExec_t graph[2] = {nullptr, nullptr};  // by starting parity / lattice index
};

namespace {

// AA: parity of the steps done (0: natural layout)
int parity(const lbm_ctx_s *c) { return c->cfg.scheme == LBM_SCHEME_AA ? (int)(c->steps & 1) : 0; }

hipError_t one_step(lbm_ctx_s *c, hipStream_t s) {
    const bool push = c->cfg.scheme == LBM_SCHEME_PUSH;
    hipError_t e = launch_step(c->model.lattice, c->fp64, c->cfg.scheme, parity(c), c->lat[c->cur],
                               push ? c->lat[1 - c->cur] : nullptr, c->box, c->model, c->cfg.tau, c->rho_ref, c->block,
                               c->lm, c->F, s);
    if (e == hipSuccess) {
        if (push) c->cur = 1 - c->cur;
        c->steps++;
    }
    return e;
}

// n steps: launches of several steps where the box takes them, else one by one.
// Passes start and end in natural layout, so an AA run takes an odd step before
// and after on its own; after n steps the state is in the lattice that n single
// steps leave it in (a caller may capture the call and replay it).
// Solid cells: neither a pass nor a step writes their slots, so an AA run finds them
// in its first lattice as they were.  A push step leaves the previous step's state in
// the other lattice, and a cell that turns solid between calls keeps its slots of both;
// push runs with obstacles therefore end every call with a single step (`tail` = 1).
int tail_steps(const lbm_ctx_s *c) { return c->multi && c->cfg.scheme == LBM_SCHEME_PUSH && c->cfg.obstacles; }

hipError_t enqueue_steps(lbm_ctx_s *c, int64_t n, int tail, hipStream_t s) {
    const bool aa = c->cfg.scheme == LBM_SCHEME_AA;
    hipError_t e = hipSuccess;
    if (c->multi) {
        if (n > 0 && parity(c)) {
            e = one_step(c, s);
            --n;
        }
        int64_t m = aa ? n & ~int64_t(1) : n > tail ? n - tail : 0;
        n -= m;
        auto tile = [&](int h) {
            const hipError_t te = launch_tile(c->fp64, c->tile, h, c->lat[c->cur], c->lat[1 - c->cur], c->lm, c->box,
                                              c->model, c->cfg.tau, c->rho_ref, c->F, s);
            if (te == hipSuccess) {
                c->cur = 1 - c->cur;
                c->steps += h;
            }
            return te;
        };
        if (c->tile.h > 0) {
            // equal launches, as many as keep the parity of the launches that of the steps
            int64_t k = (m + c->tile.h - 1) / c->tile.h;
            if ((k ^ (aa ? 0 : m)) & 1) ++k;
            if (k == m && !c->tile.one) k = 0;  // one step each
            for (; e == hipSuccess && m > 0 && k > 0; --k) {
                const int h = (int)((m + k - 1) / k);
                e = tile(h);
                m -= h;
            }
            if (e != hipSuccess) return e;
            if (m == 0 && n == 1 && tail && c->tile.one) return tile(1);  // like a push step, leaves its source as it is
        }
        for (; c->lz > 0 && m >= 4 && e == hipSuccess; m -= 4) {  // in pairs: back to the same lattice
            for (int k = 0; k < 2 && e == hipSuccess; ++k) {
                e = launch_multi3(c->fp64, c->lat[c->cur], c->lat[1 - c->cur], c->box, c->model, c->cfg.tau, c->rho_ref,
                                  c->lz, s);
                if (e != hipSuccess) return e;
                c->cur = 1 - c->cur;
                c->steps += 2;
            }
        }
        for (int odd = aa ? 0 : (int)(m & 1); c->model.D == 2 && m > 0 && e == hipSuccess; odd ^= 1) {
            const int H = multi_depth(c->plan, m, odd);
            if (H < 2) {
                if (H == 0) break;
                e = one_step(c, s);
            } else {
                e = launch_multi(c->fp64, H, c->lat[c->cur], c->lat[1 - c->cur], c->lm, c->box, c->model, c->cfg.tau,
                                 c->rho_ref, c->F, c->plan.ly[H], s);
                if (e == hipSuccess) {
                    c->cur = 1 - c->cur;
                    c->steps += H;
                }
            }
            m -= H;
        }
        n += m;
    }
    for (; n > 0 && e == hipSuccess; --n) e = one_step(c, s);
    return e;
}

lbm_status build_graph(lbm_ctx_s *c, int ph) {
    hipError_t e;
    if (!c->cap) {
        e = hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking);
        if (e != hipSuccess) return hip_fail(e, "hipStreamCreateWithFlags");
    }
    const int save_cur = c->cur;
    const int64_t save_steps = c->steps;
    e = hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
    const hipError_t le = enqueue_steps(c, c->cfg.graph_steps, 0, c->cap);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(c->cap, &g);
    c->cur = save_cur;
    c->steps = save_steps;
    if (le != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return hip_fail(le, "kernel launch during capture");
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
    e = hipGraphInstantiate(&c->graph[ph], g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
    return LBM_OK;
}

}  // namespace

extern "C" {

const char *lbm_last_error(void) { return g_err.c_str(); }

lbm_status lbm_coefficients(const lbm_config *cfg, double *out, int cap, int *n_written) {
    if (!cfg || !out || !n_written) return fail(LBM_ERR_ARG, "null argument");
    Model m;
    std::string err;
    lbm_status s = build_model(cfg, &m, &err);
    if (s != LBM_OK) return fail(s, err);
    const bool o4 = cfg->lattice == LBM_D2V41;
    const int need = 6 * m.ncls + 4 + (o4 ? 3 * m.ncls + 1 : 0);
    if (cap < need) return fail(LBM_ERR_ARG, "output capacity too small");
    for (int k = 0; k < m.ncls; ++k) {
        const ClassCoef &cc = m.cls[k];
        const double v[6] = {cc.w, cc.l1, cc.q, cc.s, cc.c3, cc.k4};
        std::memcpy(out + 6 * k, v, sizeof v);
    }
    out[6 * m.ncls + 0] = m.J2;
    out[6 * m.ncls + 1] = m.J4;
    out[6 * m.ncls + 2] = m.d2sq;
    out[6 * m.ncls + 3] = m.d4sq;
    if (o4) {
        double *o = out + 6 * m.ncls + 4;
        for (int k = 0; k < m.ncls; ++k) {
            o[3 * k + 0] = m.cls[k].p4;
            o[3 * k + 1] = m.cls[k].r4;
            o[3 * k + 2] = m.cls[k].t4;
        }
        o[3 * m.ncls] = m.scale;
    }
    *n_written = need;
    return LBM_OK;
}

lbm_status lbm_workspace_bytes(const lbm_config *cfg, size_t *bytes) {
    if (!cfg || !bytes) return fail(LBM_ERR_ARG, "null argument");
    Model m;
    Layout lay;
    lbm_status s = check_config(cfg, &m, &lay);
    if (s != LBM_OK) return s;
    *bytes = lay.total;
    return LBM_OK;
}

lbm_status lbm_workspace_min_bytes(const lbm_config *cfg, size_t *bytes) {
    if (!cfg || !bytes) return fail(LBM_ERR_ARG, "null argument");
    Model m;
    Layout lay;
    lbm_status s = check_config(cfg, &m, &lay);
    if (s != LBM_OK) return s;
    *bytes = lay.min_total;
    return LBM_OK;
}

lbm_status lbm_init(const lbm_config *cfg, void *workspace, size_t bytes, void *stream, const double *n0_dev,
                    const double *u0_dev, lbm_ctx *out) {
    if (!cfg || !workspace || !n0_dev || !u0_dev || !out) return fail(LBM_ERR_ARG, "null argument");
    *out = nullptr;
    Model m;
    Layout lay;
    lbm_status s = check_config(cfg, &m, &lay);
    if (s != LBM_OK) return s;
    if (bytes < lay.min_total) return fail(LBM_ERR_ARG, "workspace smaller than lbm_workspace_min_bytes()");
    if ((uintptr_t)workspace % kAlign) return fail(LBM_ERR_ARG, "workspace must be 256-byte aligned");
    lbm_ctx_s *c = new (std::nothrow) lbm_ctx_s;
    if (!c) return fail(LBM_ERR_ARG, "out of host memory");
    c->cfg = *cfg;
    c->model = m;
    c->lay = lay;
    c->box = Box{cfg->nx, cfg->ny, cfg->nz, cfg->bc[0] == LBM_BOUNCEBACK, cfg->bc[1] == LBM_BOUNCEBACK,
                 cfg->bc[2] == LBM_BOUNCEBACK, lay.plane, lay.cells};
    c->ws = (char *)workspace;
    c->lat[0] = c->ws;
    c->lat[1] = lay.nlat == 2 ? c->ws + lay.lattice_bytes : (bytes >= lay.total && lay.multi ? c->ws + lay.stage_off : nullptr);
    c->part = (double *)(c->ws + lay.part_off);
    c->out = (double *)(c->ws + lay.out_off);
    c->block = cfg->block ? cfg->block : default_block(cfg->nx);
    c->fp64 = cfg->precision == LBM_FP64;
    c->rho_ref = cfg->rho_ref > 0 ? cfg->rho_ref : 1.0;
    c->stream = (hipStream_t)stream;
    if (lay.porous) {
        c->lm = (uint32_t *)(c->ws + lay.mask_off);
        for (int d = 0; d < 3; ++d) c->F[d] = cfg->force[d];
    }
    hipError_t e = hipSuccess;
    c->multi = lay.multi && c->lat[1];
    if (c->multi) {
        int dev = 0, cus = 0;
        e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        const bool links = lay.porous || c->box.bbx || c->box.bby;
        if (m.D == 3) {
            c->lz = planes3(cfg, cus);
        } else {
            c->plan = multi_plan(cfg->nx, cfg->ny, c->fp64, links, lay.nlat == 2, cus);
            c->tile = tile_plan(cfg->nx, cfg->ny, c->box.bbx, c->box.bby, lay.porous, c->fp64, cus);
            if (c->tile.time >= c->plan.time) c->tile.h = 0;
        }
    }
    if (e == hipSuccess && c->lm) e = hipMemsetAsync(c->lm, 0, (size_t)lay.cells * sizeof(uint32_t), c->stream);  // no solids yet
    if (e == hipSuccess)
        e = launch_init(m.lattice, c->fp64, c->lat[0], n0_dev, u0_dev, c->box, m, cfg->tau, c->rho_ref, c->block,
                        c->stream);
    // the slots of solid cells are never streamed into: both push lattices hold their initial values
    if (e == hipSuccess && c->lm && lay.nlat == 2)
        e = launch_init(m.lattice, c->fp64, c->lat[1], n0_dev, u0_dev, c->box, m, cfg->tau, c->rho_ref, c->block,
                        c->stream);
    if (e != hipSuccess) {
        delete c;
        return hip_fail(e, "init kernel launch");
    }
    *out = c;
    return LBM_OK;
}

lbm_status lbm_step(lbm_ctx c, int64_t nsteps) {
    if (!c) return fail(LBM_ERR_ARG, "null context");
    if (nsteps < 0) return fail(LBM_ERR_ARG, "nsteps < 0");
    const int G = c->cfg.graph_steps;
    const int tail = tail_steps(c);
    int64_t left = nsteps;
    while (G > 0 && left >= G + tail) {
        const int ph = c->cur | parity(c);  // AA: cur is 0 between calls
        if (!c->graph[ph]) {
            lbm_status s = build_graph(c, ph);
            if (s != LBM_OK) return s;
        }
        hipError_t e = hipGraphLaunch(c->graph[ph], c->stream);
        if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
        c->steps += G;  // G even: the lattice index and the AA parity are unchanged
        left -= G;
    }
    const hipError_t e = enqueue_steps(c, left, tail, c->stream);
    return e == hipSuccess ? LBM_OK : hip_fail(e, "step kernel launch");
}

lbm_status lbm_moments_device(lbm_ctx c, double *n_dev, double *u_dev) {
    if (!c || !n_dev || !u_dev) return fail(LBM_ERR_ARG, "null argument");
    const int odd = parity(c);
    const void *lat = c->lat[c->cur];
    hipError_t e = launch_moments(c->model.lattice, c->fp64, lat, n_dev, u_dev, c->box, c->rho_ref, odd, c->block,
                                  c->lm, c->F, 0, c->lay.rows, c->lay.cells, c->stream);
    if (e != hipSuccess) return hip_fail(e, "moments kernel launch");
    return LBM_OK;
}

lbm_status lbm_moments(lbm_ctx c, double *n_host, double *u_host) {
    if (!c || !n_host || !u_host) return fail(LBM_ERR_ARG, "null argument");
    const int odd = parity(c);
    const void *lat = c->lat[c->cur];
    const int D = c->model.D, nx = c->cfg.nx, rows = c->lay.rows, chunk = c->lay.stage_rows;
    const int64_t cells = c->lay.cells, cstride = (int64_t)chunk * nx;
    double *sn = (double *)(c->ws + c->lay.stage_off), *su = sn + cstride;
    // chunks of whole rows through the staging area, in stream order (a chunk's
    // kernel runs after the previous chunk's copy has drained the staging area)
    for (int r0 = 0; r0 < rows; r0 += chunk) {
        const int nr = rows - r0 < chunk ? rows - r0 : chunk;
        const int64_t off = (int64_t)r0 * nx, cnt = (int64_t)nr * nx;
        hipError_t e = launch_moments(c->model.lattice, c->fp64, lat, sn, su, c->box, c->rho_ref, odd, c->block, c->lm,
                                      c->F, r0, nr, cstride, c->stream);
        if (e != hipSuccess) return hip_fail(e, "moments kernel launch");
        e = hipMemcpyAsync(n_host + off, sn, cnt * sizeof(double), hipMemcpyDeviceToHost, c->stream);
        for (int d = 0; e == hipSuccess && d < D; ++d)
            e = hipMemcpyAsync(u_host + d * cells + off, su + d * cstride, cnt * sizeof(double),
                               hipMemcpyDeviceToHost, c->stream);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    }
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return LBM_OK;
}

lbm_status lbm_totals(lbm_ctx c, double *out_host) {
    if (!c || !out_host) return fail(LBM_ERR_ARG, "null argument");
    const int odd = parity(c);
    const void *lat = c->lat[c->cur];
    hipError_t e = launch_totals(c->model.lattice, c->fp64, lat, c->part, c->out, c->box, c->rho_ref, odd, c->block,
                                 c->lm, c->stream);
    if (e != hipSuccess) return hip_fail(e, "totals kernel launch");
    double tmp[5];
    e = hipMemcpyAsync(tmp, c->out, sizeof tmp, hipMemcpyDeviceToHost, c->stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    for (int d = 0; d <= c->model.D; ++d) out_host[d] = tmp[d];
    for (int d = 0; d <= c->model.D; ++d)
        if (!std::isfinite(tmp[d])) return fail(LBM_ERR_NUMERIC, "non-finite total");
    if (tmp[4] != 0.0) return fail(LBM_ERR_NUMERIC, "cells with non-positive or non-finite density");
    return LBM_OK;
}

lbm_status lbm_set_solid(lbm_ctx c, const unsigned char *solid_dev) {
    if (!c || !solid_dev) return fail(LBM_ERR_ARG, "null argument");
    if (!c->cfg.obstacles) return fail(LBM_ERR_STATE, "the context was created without obstacles");
    if (c->cfg.scheme == LBM_SCHEME_AA && (c->steps & 1))
        return fail(LBM_ERR_STATE, "solids can change only after an even number of AA steps");
    hipError_t e = launch_link_mask(c->model.D, solid_dev, c->lm, c->box, c->block, c->stream);
    if (e != hipSuccess) return hip_fail(e, "link mask kernel launch");
    return LBM_OK;
}

}  // extern "C"

namespace {

// Host-side permutation between the natural layout (g_a at its own cell) and
// the AA storage after an odd number of steps (g_a of cell x held in the slot
// of -a at x - e_a, or in slot a at x for a link that bounced at a wall or a
// solid cell; lm is the link mask of a run with solids, else null).
// `gather` maps storage -> natural; otherwise natural -> storage.
template <typename T>
void aa_odd_permute(const lbm_ctx_s *c, const T *in, T *out, bool gather, const uint32_t *lm) {
    const Box &b = c->box;
    const int64_t P = c->lay.cells;  // host copies hold the planes back to back
    const int Q = c->model.Q;
    const int(*e)[3] = D2Q9::e;
    const int *opp = D2Q9::opp;
    switch (c->model.lattice) {
    case LBM_D1V3: e = D1Q3::e; opp = D1Q3::opp; break;
    case LBM_D3V19: e = D3Q19::e; opp = D3Q19::opp; break;
    case LBM_D2V41: e = D2Q41::e; opp = D2Q41::opp; break;
    default: break;
    }
    const int dims[3] = {b.nx, b.ny, b.nz};
    const int bbs[3] = {b.bbx, b.bby, b.bbz};
    for (int z = 0; z < b.nz; ++z)
        for (int y = 0; y < b.ny; ++y)
            for (int x = 0; x < b.nx; ++x) {
                const int64_t cell = ((int64_t)z * b.ny + y) * b.nx + x;
                const int p[3] = {x, y, z};
                if (lm && (lm[cell] & kSolidBit)) {  // a solid cell owns only its own slots
                    if (gather)
                        for (int q = 0; q < Q; ++q) out[(int64_t)q * P + cell] = in[(int64_t)q * P + cell];
                    continue;
                }
                for (int q = 0; q < Q; ++q) {
                    int s[3];
                    bool bb = lm && opp[q] < 32 && ((lm[cell] >> opp[q]) & 1u);  // x - e_q is a solid cell
                    for (int d = 0; d < 3; ++d) {
                        s[d] = p[d] - e[q][d];
                        if (s[d] < 0 || s[d] >= dims[d]) {
                            if (bbs[d]) bb = true;
                            else s[d] = (s[d] + dims[d]) % dims[d];
                        }
                    }
                    const int64_t slot = bb ? (int64_t)q * P + cell
                                            : (int64_t)opp[q] * P + ((int64_t)s[2] * b.ny + s[1]) * b.nx + s[0];
                    const int64_t nat = (int64_t)q * P + cell;
                    if (gather) out[nat] = in[slot];
                    else out[slot] = in[nat];
                }
            }
}

}  // namespace

extern "C" {

lbm_status lbm_get_state(lbm_ctx c, void *host, size_t bytes) {
    if (!c || !host) return fail(LBM_ERR_ARG, "null argument");
    const size_t need = (size_t)c->model.Q * c->lay.cells * c->lay.elt;
    if (bytes != need) return fail(LBM_ERR_ARG, "state size mismatch");
    const void *lat = c->lat[c->cur];
    const bool odd = parity(c) != 0;
    std::vector<char> raw;
    void *dst = host;
    if (odd) {
        raw.resize(need);
        dst = raw.data();
    }
    std::vector<uint32_t> lm;
    const size_t row = (size_t)c->lay.cells * c->lay.elt, pitch = (size_t)c->lay.plane * c->lay.elt;
    hipError_t e = hipMemcpy2DAsync(dst, row, lat, pitch, row, c->model.Q, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && odd && c->lm) {
        lm.resize(c->lay.cells);
        e = hipMemcpyAsync(lm.data(), c->lm, lm.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, c->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(e, "state copy");
    if (odd) {
        const uint32_t *m = lm.empty() ? nullptr : lm.data();
        if (c->fp64) aa_odd_permute<double>(c, (const double *)raw.data(), (double *)host, true, m);
        else aa_odd_permute<float>(c, (const float *)raw.data(), (float *)host, true, m);
    }
    return LBM_OK;
}

lbm_status lbm_set_state(lbm_ctx c, const void *host, size_t bytes) {
    if (!c || !host) return fail(LBM_ERR_ARG, "null argument");
    const size_t need = (size_t)c->model.Q * c->lay.cells * c->lay.elt;
    if (bytes != need) return fail(LBM_ERR_ARG, "state size mismatch");
    void *lat = c->lat[c->cur];
    const bool odd = parity(c) != 0;
    std::vector<char> raw;
    const void *src = host;
    hipError_t e = hipSuccess;
    const size_t row = (size_t)c->lay.cells * c->lay.elt, pitch = (size_t)c->lay.plane * c->lay.elt;
    if (odd) {
        // the slots of the odd AA layout depend on the solids: read the stored
        // state first so that slots no cell owns (inside solids) keep their values
        std::vector<uint32_t> lm;
        raw.resize(need);
        e = hipMemcpy2DAsync(raw.data(), row, lat, pitch, row, c->model.Q, hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess && c->lm) {
            lm.resize(c->lay.cells);
            e = hipMemcpyAsync(lm.data(), c->lm, lm.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, c->stream);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return hip_fail(e, "state copy");
        const uint32_t *m = lm.empty() ? nullptr : lm.data();
        if (c->fp64) aa_odd_permute<double>(c, (const double *)host, (double *)raw.data(), false, m);
        else aa_odd_permute<float>(c, (const float *)host, (float *)raw.data(), false, m);
        src = raw.data();
    }
    e = hipMemcpy2DAsync(lat, pitch, src, row, row, c->model.Q, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return hip_fail(e, "state copy");
    return LBM_OK;
}

lbm_status lbm_steps_done(lbm_ctx c, int64_t *steps) {
    if (!c || !steps) return fail(LBM_ERR_ARG, "null argument");
    *steps = c->steps;
    return LBM_OK;
}

lbm_status lbm_info(lbm_ctx c, int64_t *cells, int *Q, int64_t *bytes_per_step) {
    if (!c || !cells || !Q || !bytes_per_step) return fail(LBM_ERR_ARG, "null argument");
    *cells = c->lay.cells;
    *Q = c->model.Q;
    *bytes_per_step = 2 * (int64_t)c->model.Q * c->lay.cells * (int64_t)c->lay.elt;
    return LBM_OK;
}

lbm_status lbm_velocities(int lattice, int *e_out, int cap, int *Q) {
    if (!e_out || !Q) return fail(LBM_ERR_ARG, "null argument");
    const int(*e)[3] = nullptr;
    int q = 0;
    if (lattice == LBM_D1V3) { e = D1Q3::e; q = D1Q3::Q; }
    else if (lattice == LBM_D2V9) { e = D2Q9::e; q = D2Q9::Q; }
    else if (lattice == LBM_D3V19) { e = D3Q19::e; q = D3Q19::Q; }
    else if (lattice == LBM_D2V41) { e = D2Q41::e; q = D2Q41::Q; }
    else return fail(LBM_ERR_ARG, "unknown lattice");
    if (cap < 3 * q) return fail(LBM_ERR_ARG, "output capacity too small");
    for (int a = 0; a < q; ++a)
        for (int d = 0; d < 3; ++d) e_out[3 * a + d] = e[a][d];
    *Q = q;
    return LBM_OK;
}

lbm_status lbm_free(lbm_ctx c) {
    if (!c) return LBM_OK;
    lbm_status st = LBM_OK;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) st = hip_fail(e, "hipStreamSynchronize");
    for (auto &g : c->graph)
        if (g) (void)hipGraphExecDestroy(g);
    if (c->cap) (void)hipStreamDestroy(c->cap);
    delete c;
    return st;
}

}  // extern "C"
