"""Edges of the surrogate's one-kernel forward when a profile is cut into segments
(fewer profiles than compute units), and of the fused backward kernels' tiles.

A segment's workgroup recomputes the reach of the layers' taps at its ends with
the same operations, so a profile's result does not depend on the batch it is
in: one profile alone (cut finely), in a batch of a few (cut coarsely) and in a
batch of more than there are compute units (not cut) must agree bit for bit,
with inference and with the pass that keeps the pre-activations."""
import numpy as np
import pytest
import torch

from oracle import conv
from paper_1510_07328_amd import surrogate as S

pytestmark = pytest.mark.gpu


def profiles(B, L, seed):
    rng = np.random.default_rng(seed)
    prof = np.stack([1 + 0.1 * rng.standard_normal((B, L)), 0.1 * rng.standard_normal((B, L))], 1).astype(np.float32)
    return torch.from_numpy(prof).cuda(), torch.from_numpy(rng.uniform(0.51, 1.0, B).astype(np.float32)).cuda()


@pytest.mark.parametrize("L", [128, 256, 384, 640, 1024, 4096])
def test_a_profile_does_not_depend_on_its_batch(gpu, L):
    params, _ = S.load_weights()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    x, tau = profiles(cus + 1, L, L)
    sur = S.Surrogate(cus + 1, L, params=params)
    whole = sur.infer(x, tau).clone()
    for B in (1, 3, cus // 2, cus - 1):
        a, t = x[:B].contiguous(), tau[:B].contiguous()
        assert torch.equal(sur.infer(a, t), whole[:B]), B
        assert torch.equal(sur.forward(a, t), whole[:B]), B
    sur.free()


@pytest.mark.parametrize("B,L", [(1, 128), (1, 384), (3, 1024), (300, 128), (2, 4224)])
def test_gradient_against_the_float64_network(gpu, B, L):
    """Tile counts below, at and above the workgroups of the backward kernels, segments in the
    forward pass, and the layer-by-layer forward (4224): the bars of the other gradient tests
    (bfloat16 roundings of the activations and of the back-propagated gradients, 2e-2 per tensor)."""
    params = S.init_params(5)
    x, tau = profiles(B, L, 7)
    rng = np.random.default_rng(9)
    dout = (rng.standard_normal((B, 2, L)) / (B * L)).astype(np.float32)
    sur = S.Surrogate(B, L, params=params)
    sur.forward(x, tau)
    g = sur.backward(torch.from_numpy(dout).cuda())
    g2 = sur.backward(torch.from_numpy(dout).cuda())
    assert torch.equal(g, g2)  # deterministic
    g = g.double().cpu().numpy()
    sur.free()
    xn = x.double().cpu().numpy()
    _, _, cache = conv.forward(params.astype(np.float64), xn[:, 0], xn[:, 1], tau.double().cpu().numpy(), quantize=True)
    ref = conv.backward(cache, dout[:, 0].astype(np.float64), dout[:, 1].astype(np.float64))
    ref = np.asarray(ref).reshape(-1)
    off = 0
    for n in (960, 64, 20480, 64, 20480, 64, 640, 2):
        a, r = g[off:off + n], ref[off:off + n]
        off += n
        err = np.linalg.norm(a - r) / np.linalg.norm(r)
        assert err < 2e-2, (off, n, err)
