"""An infinite output gradient in the surrogate's backward pass: the weight gradients of the
last layer are sums of products dy a, so one infinite dy makes its component's entries
infinite with the sign of the activation (where there is one), and leaves the other
component's finite."""
import numpy as np
import pytest
import torch

from oracle import conv
from paper_1510_07328_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("B,L,b,c,x0", [(1, 128, 0, 0, 60), (3, 384, 1, 1, 130), (2, 1024, 1, 0, 1023)])
def test_an_infinite_output_gradient(gpu, B, L, b, c, x0, sign):
    params = conv.init_params(3, scale_out=1.0).astype(np.float32)
    rng = np.random.default_rng(L)
    x = np.stack([1 + 0.1 * rng.standard_normal((B, L)), 0.1 * rng.standard_normal((B, L))], 1).astype(np.float32)
    tau = rng.uniform(0.51, 1.0, B).astype(np.float32)
    dout = (rng.standard_normal((B, 2, L)) / (B * L)).astype(np.float32)
    dout[b, c, x0] = sign * np.inf
    sur = S.Surrogate(B, L, params=params)
    prof, t = torch.from_numpy(x).cuda(), torch.from_numpy(tau).cuda()
    sur.forward(prof, t)
    g = sur.backward(torch.from_numpy(dout).cuda()).cpu().numpy()
    sur.free()
    _, _, cache = conv.forward(params.astype(np.float64), x[:, 0].astype(np.float64), x[:, 1].astype(np.float64),
                               tau.astype(np.float64), quantize=True)
    a3 = cache["a"][3]
    dw4, db4 = g[-642:-2].reshape(5, 2, 64), g[-2:]
    assert db4[c] == sign * np.inf and np.isfinite(db4[1 - c]) and np.isfinite(dw4[:, 1 - c]).all()
    for tap in range(5):
        y = x0 + (tap - 2) * 27
        if not 0 <= y < L:
            assert np.isfinite(dw4[tap, c]).all(), tap
            continue
        a = a3[b, :, y]
        clear = np.abs(a) > 1e-2  # far from a change of sign by the activations' rounding
        assert clear.sum() > 16
        assert (dw4[tap, c][clear] == sign * np.sign(a[clear]) * np.inf).all(), tap
