"""Calls of several steps on d2v9 boxes run as launches of several steps between two
lattices: small boxes as tiles in LDS (lbm_tile.hip), larger ones in registers
(lbm_multi.hip).  Every cell update is the same arithmetic in the same order as in
the single-step kernels, so one call of n steps must equal n calls of one step bit
for bit: over tiles, strips and segments that end inside a box, boxes smaller than
one, walls, solid cells with a force, both schemes and precisions, and the numbers
of steps around each depth."""
import numpy as np
import pytest
import torch

from paper_1510_07328_amd import inputs, lbm

pytestmark = pytest.mark.gpu

PUSH, AA = lbm.LBM_SCHEME_PUSH, lbm.LBM_SCHEME_AA


def make(shape, bc=(0, 0, 0), porous=False, **kw):
    nx, ny = shape
    force = (2e-5, -1e-5, 0.0) if porous else (0.0, 0.0, 0.0)
    cfg = lbm.make_config("d2v9", shape=(nx, ny, 1), bc=bc, tau=0.7, obstacles=int(porous), force=force, **kw)
    n0, u0 = inputs.perturbed_field((ny, nx), 0.02, 3.0, (0.01, -0.02), seed=nx)
    return cfg, n0, u0


def solid_of(shape):
    return inputs.porous_obstacles(shape, min(60, max(1, shape[0] * shape[1] // 300)), 2.0, seed=3)


def run(cfg, n0, u0, calls, solid=None):
    lat = lbm.Lattice.create(cfg, n0, u0)
    if solid is not None:
        lat.set_solid(solid)
    for n in calls:
        lat.step(n)
    out = lat.state(), lat.steps_done
    n, u = lat.moments()
    nh, uh = lat.moments_host()
    torch.cuda.synchronize()
    assert np.array_equal(nh, n.cpu().numpy()) and np.array_equal(uh, u.cpu().numpy())
    lat.free()
    return out


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64])
@pytest.mark.parametrize("shape,bc,porous,order", [
    ((200, 90), (0, 0, 0), False, 2),    # tiles cut in both axes, the last ones short
    ((61, 50), (0, 0, 0), False, 3),
    ((700, 7), (0, 0, 0), False, 2),     # one axis whole
    ((300, 4), (1, 0, 0), False, 2),
    ((5, 3), (0, 0, 0), False, 2),       # the whole box in one window
    ((1, 64), (0, 0, 0), False, 2),
    ((131, 1), (1, 0, 0), False, 2),
    ((131, 40), (1, 0, 0), False, 2),    # walls in x, in y, in both
    ((60, 33), (0, 1, 0), False, 2),
    ((58, 9), (1, 1, 0), False, 3),
    ((150, 70), (0, 0, 0), True, 2),     # solid cells and a force, without and with walls
    ((77, 41), (1, 1, 0), True, 3),
    ((23, 11), (1, 1, 0), True, 2),
])
def test_one_call_of_n_steps_equals_n_calls(gpu, shape, bc, porous, order, precision, scheme):
    cfg, n0, u0 = make(shape, bc, porous, order=order, precision=precision, scheme=scheme)
    solid = solid_of(shape) if porous else None
    for n in (2, 3, 4, 5, 6, 7, 8, 10, 13, 14, 25):
        one, s1 = run(cfg, n0, u0, [1] * n, solid)
        for calls in ([n], [1, n - 1], [n - 1, 1]):
            many, s2 = run(cfg, n0, u0, calls, solid)
            assert s1 == s2 == n
            assert np.array_equal(one, many), (n, calls, int((one != many).sum()))


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("shape,bc,porous,order,precision", [
    ((2111, 1537), (0, 0, 0), False, 2, lbm.LBM_FP32_DEV),   # the deepest pass
    ((1601, 1203), (0, 0, 0), False, 2, lbm.LBM_FP64),
    ((1030, 777), (1, 0, 0), False, 2, lbm.LBM_FP32_DEV),    # strips at walls in x
    ((1030, 777), (1, 1, 0), False, 3, lbm.LBM_FP64),
    ((901, 811), (0, 1, 0), False, 2, lbm.LBM_FP32_DEV),
    ((1000, 700), (0, 0, 0), True, 2, lbm.LBM_FP32_DEV),
    ((1000, 700), (1, 1, 0), True, 3, lbm.LBM_FP64),
    ((57, 20011), (0, 0, 0), False, 2, lbm.LBM_FP32_DEV),    # one strip and a part of one
])
def test_large_boxes(gpu, shape, bc, porous, order, precision, scheme):
    """Boxes beyond the LDS tiles: the register pipeline at the depths and segments of its plan."""
    cfg, n0, u0 = make(shape, bc, porous, order=order, precision=precision, scheme=scheme)
    solid = solid_of(shape) if porous else None
    for n in (5, 10, 26):
        one, _ = run(cfg, n0, u0, [1] * n, solid)
        many, _ = run(cfg, n0, u0, [n], solid)
        assert np.array_equal(one, many), (n, int((one != many).sum()))


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("shape,order,precision", [
    ((64, 64, 64), 2, lbm.LBM_FP32_DEV),     # strips of 62 columns and 14 rows, the last ones short
    ((62, 42, 100), 2, lbm.LBM_FP32_DEV),    # exact strips and groups
    ((130, 45, 61), 3, lbm.LBM_FP32_DEV),
    ((64, 31, 128), 2, lbm.LBM_FP64),        # groups of 6 rows
    ((33, 300, 21), 3, lbm.LBM_FP64),
])
def test_periodic_d3v19_boxes(gpu, shape, order, precision, scheme):
    """Two steps per pass in pairs of passes, and the steps left over."""
    nx, ny, nz = shape
    cfg = lbm.make_config("d3v19", shape=shape, order=order, tau=0.7, precision=precision, scheme=scheme)
    n0, u0 = inputs.perturbed_field((nz, ny, nx), 0.02, 3.0, (0.01, -0.02, 0.005), seed=1)
    for n in (4, 5, 7, 10):
        one, _ = run(cfg, n0, u0, [1] * n)
        for calls in ([n], [1, n - 1]):
            many, _ = run(cfg, n0, u0, calls)
            assert np.array_equal(one, many), (n, calls, int((one != many).sum()))


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("shape,order,precision", [
    ((130, 125, 128), 2, lbm.LBM_FP32_DEV),  # short last strip, group and segment
    ((186, 84, 131), 3, lbm.LBM_FP32_DEV),   # exact strips and groups
    ((63, 141, 114), 2, lbm.LBM_FP64),       # one column and three rows left over
    ((124, 60, 137), 3, lbm.LBM_FP64),
])
def test_large_periodic_d3v19_boxes(gpu, shape, order, precision, scheme):
    """Boxes of 2 million float32 cells (or as many bytes in float64): a wavefront's rows in pairs,
    lanes without an output store past the buffer's end."""
    nx, ny, nz = shape
    cfg = lbm.make_config("d3v19", shape=shape, order=order, tau=0.7, precision=precision, scheme=scheme)
    n0, u0 = inputs.perturbed_field((nz, ny, nx), 0.02, 3.0, (0.01, -0.02, 0.005), seed=2)
    for n in (4, 9):
        one, _ = run(cfg, n0, u0, [1] * n)
        many, _ = run(cfg, n0, u0, [n])
        assert np.array_equal(one, many), (n, int((one != many).sum()))


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64])
@pytest.mark.parametrize("shape,bc,order", [
    ((70, 45, 33), (1, 0, 0), 2),
    ((64, 31, 40), (0, 1, 0), 3),
    ((33, 60, 21), (0, 0, 1), 2),
    ((62, 42, 36), (1, 1, 1), 3),    # walls at the ends of exact strips and groups
    ((125, 16, 50), (1, 0, 1), 2),
    ((40, 3, 90), (0, 1, 1), 2),
])
def test_walled_d3v19_boxes(gpu, shape, bc, order, precision, scheme):
    """Two steps per pass with walls on one axis, on two and on all: links reflected on planes, edges and
    corners, in both steps of the pass and across segments."""
    nx, ny, nz = shape
    cfg = lbm.make_config("d3v19", shape=shape, bc=bc, order=order, tau=0.7, precision=precision, scheme=scheme)
    n0, u0 = inputs.perturbed_field((nz, ny, nx), 0.02, 3.0, (0.01, -0.02, 0.005), seed=3)
    for n in (4, 5, 7, 12):
        one, _ = run(cfg, n0, u0, [1] * n)
        for calls in ([n], [1, n - 1]):
            many, _ = run(cfg, n0, u0, calls)
            assert np.array_equal(one, many), (n, calls, int((one != many).sum()))


@pytest.mark.parametrize("lattice,shape,n", [("d3v19", (350, 353, 347), 4), ("d2v9", (9001, 9003, 1), 12)])
def test_lattices_between_2_and_4_gib(gpu, lattice, shape, n):
    """Byte offsets past 2^31 in the buffer accesses: 3.3 GB and 2.9 GB per lattice."""
    nx, ny, nz = shape
    dims = 3 if nz > 1 else 2
    g = torch.Generator(device="cuda").manual_seed(7)
    n0 = 1.0 + 0.01 * torch.rand(shape[::-1], generator=g, device="cuda", dtype=torch.float64)
    u0 = 0.01 * torch.rand((dims,) + shape[::-1], generator=g, device="cuda", dtype=torch.float64)
    cfg = lbm.make_config(lattice, shape=shape, order=2, tau=0.7, precision=lbm.LBM_FP32_DEV, scheme=AA)
    out = []
    for calls in ([1] * n, [n]):
        lat = lbm.Lattice.create(cfg, n0, u0)
        for k in calls:
            lat.step(k)
        m, u = lat.moments()
        torch.cuda.synchronize()
        lat.free()
        out.append((m, u))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_aa_runs_in_a_workspace_of_one_lattice(gpu):
    """A caller that gives an AA box no second lattice still gets its steps, in place."""
    cfg, n0, u0 = make((200, 90), order=2, scheme=AA)
    full = lbm.lbm_workspace_bytes(cfg)
    lattice = 9 * (200 * 90 + 8448 // 4) * 4
    stage = 3 * 8 * 200 * 90  # the whole box is staged at once by the host moments
    small = full - (lattice + 255) // 256 * 256 + (stage + 255) // 256 * 256
    assert small < full
    n = torch.as_tensor(n0).cuda()
    u = torch.as_tensor(u0).cuda().contiguous()
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    ctx = lbm.lbm_init(cfg, ws.data_ptr(), small, torch.cuda.current_stream().cuda_stream, n.data_ptr(), u.data_ptr())
    lbm.lbm_step(ctx, 13)
    got = np.empty((9, 200 * 90), dtype=np.float32)
    lbm.lbm_get_state(ctx, got.ctypes.data, got.nbytes)
    lbm.lbm_free(ctx)
    ref, _ = run(cfg, n0, u0, [1] * 13)
    assert np.array_equal(ref, got)
    with pytest.raises(lbm.LbmError):
        lbm.lbm_init(cfg, ws.data_ptr(), small - 256, torch.cuda.current_stream().cuda_stream, n.data_ptr(),
                     u.data_ptr())


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("n", [2, 6, 10])
def test_a_captured_call_can_be_replayed(gpu, scheme, n):
    """An even number of steps ends in the lattice it started from, so a caller's own graph of the
    call advances the state on every replay."""
    cfg, n0, u0 = make((150, 60), order=2, scheme=scheme)
    side = torch.cuda.Stream()
    lat = lbm.Lattice.create(cfg, n0, u0, stream=side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        lat.step(n)
    for k in range(1, 5):
        g.replay()
        torch.cuda.synchronize()
        got = lat.state()
        ref, _ = run(cfg, n0, u0, [1] * (n * k))
        assert np.array_equal(ref, got), k
    lat.free()
