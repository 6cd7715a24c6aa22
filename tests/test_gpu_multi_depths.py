"""The kernels of several steps per pass at the depths and segments that large boxes take,
with the library's plan asserted so that no case compares single steps with themselves:
the six-step d2v9 pipeline with reflected links in both precisions, and walled d3v19
passes over segments of several planes.  One call of n steps equals n calls of one step
bit for bit."""
import pytest
import torch

from paper_1510_07328_amd import lbm
from plans import depths, planes_per_segment

pytestmark = pytest.mark.gpu

PUSH, AA, F32, F64 = lbm.LBM_SCHEME_PUSH, lbm.LBM_SCHEME_AA, lbm.LBM_FP32_DEV, lbm.LBM_FP64


def equal_to_single_steps(cfg, n, solid=None):
    dims = 3 if cfg.nz > 1 else 2
    g = torch.Generator(device="cuda").manual_seed(11)
    shape = (cfg.nz, cfg.ny, cfg.nx)
    n0 = 1.0 + 0.01 * torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
    u0 = 0.02 * torch.rand((dims,) + shape, generator=g, device="cuda", dtype=torch.float64) - 0.01
    out = []
    for calls in ([1] * n, [n]):
        lat = lbm.Lattice.create(cfg, n0, u0)
        if solid is not None:
            lat.set_solid(solid)
        for k in calls:
            lat.step(k)
        out.append(torch.from_numpy(lat.state()))
        lat.free()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(*out), int((out[0] != out[1]).sum())


def squares(shape, count, side):
    """`count` solid squares at random places, some across the strips' and segments' edges."""
    nx, ny = shape
    solid = torch.zeros((ny, nx), dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    for x, y in torch.rand((count, 2), generator=g, device="cuda").tolist():
        solid[int(y * ny):int(y * ny) + side, int(x * nx):int(x * nx) + side] = 1
    return solid


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("shape,bc,porous,order,precision", [
    ((2300, 2100), (1, 1, 0), False, 2, F32),
    ((2300, 2100), (1, 0, 0), False, 3, F32),
    ((2300, 2100), (0, 1, 0), False, 2, F32),
    ((2300, 2100), (0, 0, 0), True, 2, F32),
    ((2300, 2100), (1, 1, 0), True, 3, F32),
    ((1801, 1703), (1, 1, 0), False, 2, F64),
    ((1801, 1703), (0, 0, 0), True, 3, F64),
    ((1801, 1703), (1, 1, 0), True, 2, F64),
])
def test_six_steps_per_pass_with_reflected_links(gpu, shape, bc, porous, order, precision, scheme):
    push, tail = scheme == PUSH, int(scheme == PUSH and porous)
    cfg = lbm.make_config("d2v9", shape=shape + (1,), bc=bc, order=order, tau=0.8, precision=precision, scheme=scheme,
                          obstacles=int(porous), force=(2e-6, -1e-6, 0.0) if porous else (0.0, 0.0, 0.0))
    solid = squares(shape, 600, 6) if porous else None
    for n, want in ((12, {6}), (10, {4, 6})):
        assert set(depths(shape, n, precision == F64, links=True, push=push)) == want
        equal_to_single_steps(cfg, n + tail, solid)  # a push run with obstacles ends with a single step


@pytest.mark.parametrize("scheme", [PUSH, AA])
@pytest.mark.parametrize("precision", [F32, F64])
@pytest.mark.parametrize("shape,bc,order", [
    ((100, 61, 97), (1, 0, 0), 2),    # segments of 4 planes, the last one of 1; of 9 and 7 in float64
    ((100, 61, 97), (1, 1, 1), 3),
    ((62, 56, 300), (0, 1, 0), 2),    # exact strips, groups and segments
    ((90, 100, 77), (0, 0, 1), 2),
    ((130, 125, 128), (1, 1, 1), 2),  # 15 planes
    ((24, 30, 256), (1, 0, 1), 3),
    ((60, 140, 140), (0, 1, 1), 2),
])
def test_walled_d3v19_segments_of_several_planes(gpu, shape, bc, order, precision, scheme):
    assert planes_per_segment(shape, bc, precision == F64) >= 4
    cfg = lbm.make_config("d3v19", shape=shape, bc=bc, order=order, tau=0.8, precision=precision, scheme=scheme)
    for n in (4, 9):
        equal_to_single_steps(cfg, n)
