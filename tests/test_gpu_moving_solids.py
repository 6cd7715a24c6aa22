"""Solids that change between calls of several steps.  A cell that turns solid keeps its
slots (in both lattices of a push run), so what a cell holds when it is opened again must
not depend on how the steps before and since were cut into calls: every state equals the
one of single steps bit for bit, slots of solid cells included, for boxes that run as LDS
tiles and as the register pipeline, with and without graphs."""
import numpy as np
import pytest
import torch

from paper_1510_07328_amd import inputs, lbm

pytestmark = pytest.mark.gpu

PUSH, AA = lbm.LBM_SCHEME_PUSH, lbm.LBM_SCHEME_AA


def states(cfg, n0, u0, plan, single):
    lat = lbm.Lattice.create(cfg, n0, u0)
    out = []
    for steps, solid in plan:
        if solid is not None:
            lat.set_solid(solid)
        for k in [1] * steps if single else [steps]:
            lat.step(k)
        out.append(lat.state())
    lat.free()
    return out


@pytest.mark.parametrize("graph_steps", [0, 4])
@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64])
@pytest.mark.parametrize("scheme,shape,bc", [
    (PUSH, (61, 50), (0, 0, 0)), (PUSH, (300, 90), (1, 1, 0)), (PUSH, (1000, 700), (0, 0, 0)),
    (PUSH, (901, 811), (0, 1, 0)), (AA, (61, 50), (1, 0, 0)), (AA, (1000, 700), (0, 0, 0)),
])
def test_solids_set_after_steps_and_cleared_later(gpu, scheme, shape, bc, precision, graph_steps):
    nx, ny = shape
    cfg = lbm.make_config("d2v9", shape=(nx, ny, 1), bc=bc, order=2, tau=0.7, obstacles=1, force=(2e-5, -1e-5, 0.0),
                          precision=precision, scheme=scheme, graph_steps=graph_steps)
    n0, u0 = inputs.perturbed_field((ny, nx), 0.02, 3.0, (0.01, -0.02), seed=nx)
    a = np.ascontiguousarray(inputs.porous_obstacles(shape, 40, 2.0, seed=3)).reshape(ny, nx) != 0
    b = np.ascontiguousarray(inputs.porous_obstacles(shape, 40, 2.0, seed=4)).reshape(ny, nx) != 0
    # AA takes new solids after an even number of steps only
    first = (5, 9, 13, 6, 7) if scheme == PUSH else (6, 8, 14, 6, 7)
    plan = list(zip(first, (None, a, a | b, b, np.zeros_like(a))))
    for k, (one, many) in enumerate(zip(states(cfg, n0, u0, plan, True), states(cfg, n0, u0, plan, False))):
        assert np.array_equal(one, many), (k, int((one != many).sum()))
