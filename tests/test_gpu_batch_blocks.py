"""Every window stride and workgroup of the batched round kernel against single
steps of the plain kernels, bit for bit: tubes whose ends fall on both sides of
wavefronts, tiles cut in the tube, odd and even rounds, tubes shorter than a
wavefront, and workgroup sizes that are rounded up to the compiled ones."""
import numpy as np
import pytest
import torch

from paper_1510_07328_amd import batch as B
from paper_1510_07328_amd import inputs, lbm

pytestmark = pytest.mark.gpu

NX = [2, 3, 63, 64, 65, 127, 129, 300, 511, 513, 1100]
TAU = [0.7, 0.6, 0.8, 0.55, 0.65, 0.9, 0.7, 0.6, 0.75, 0.8, 0.6]
STEPS = [9, 12, 41, 17, 50, 1, 2, 37, 64, 33, 21]


@pytest.fixture(scope="module")
def single_steps(gpu):
    ref = {}

    def get(precision, order):
        if (precision, order) not in ref:
            out = []
            for nx, tau, st in zip(NX, TAU, STEPS):
                cfg = lbm.make_config("d2v9", shape=(nx, 4, 1), bc=(1, 0, 0), order=order, tau=tau,
                                      precision=precision, scheme=lbm.LBM_SCHEME_PUSH)
                lat = lbm.Lattice.create(cfg, *inputs.riemann_step(nx, 4, 1.0, 0.85))
                for _ in range(st):
                    lat.step(1)
                n, u = lat.moments()
                out.append((n.cpu().numpy(), u.cpu().numpy()))
                lat.free()
            ref[precision, order] = out
        return ref[precision, order]

    return get


@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("precision", [lbm.LBM_FP32_DEV, lbm.LBM_FP64])
@pytest.mark.parametrize("shape", [(96, 16), (40, 7), (224, 16), (448, 32), (500, 6)])
@pytest.mark.parametrize("block", [64, 256, 320, 512, 1024])
def test_round_shapes_equal_single_steps(single_steps, shape, block, precision, order):
    tubes = B.make_tubes(np.array(NX), np.array(TAU), np.ones(len(NX)), np.full(len(NX), 0.85), np.array(STEPS))
    bt = B.Batch(tubes, B.make_options(order=order, precision=precision, tile_cols=shape[0], halo=shape[1], block=block))
    bt.run()
    n, u = bt.moments()
    torch.cuda.synchronize()
    n, u = n.cpu().numpy(), u.cpu().numpy()
    for t, (rn, ru) in enumerate(single_steps(precision, order)):
        bn, bu = bt.tube_fields(n, u, t)
        assert np.array_equal(bn.reshape(-1), rn) and np.array_equal(bu.reshape(2, -1), ru), (t, NX[t])
    bt.free()
