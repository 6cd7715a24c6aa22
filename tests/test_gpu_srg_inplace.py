"""srg_forward may write its output over its input profiles (out_dev == prof_dev) when
no gradient follows.  A profile that is cut into segments is staged by several
workgroups, so in place it must not be cut; the result equals the one out of place
bit for bit, for batches that would be cut, for one profile per workgroup, for two and
for lengths that run layer by layer."""
import numpy as np
import pytest
import torch

from paper_1510_07328_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L", [(1, 128), (1, 384), (1, 4096), (3, 1024), (40, 2048), (200, 384), (300, 1024),
                                 (2, 4224)])
def test_forward_in_place(gpu, B, L):
    params, _ = S.load_weights()
    rng = np.random.default_rng(L + B)
    x = np.stack([1 + 0.1 * rng.standard_normal((B, L)), 0.1 * rng.standard_normal((B, L))], 1).astype(np.float32)
    prof = torch.from_numpy(x).cuda()
    tau = torch.from_numpy(rng.uniform(0.51, 1.0, B).astype(np.float32)).cuda()
    sur = S.Surrogate(B, L, params=params)
    want = sur.forward(prof, tau)
    for _ in range(3):
        buf = prof.clone()
        assert sur.forward(buf, tau, out=buf) is buf
        torch.cuda.synchronize()
        assert torch.equal(buf, want)
    sur.free()
