"""Warm-start inference at the edges of its kernels' groups: one group of 16 samples, more groups
than resident blocks, and padding that must stay zero from sample to sample."""
import numpy as np
import pytest
import torch

from oracle import warm as owarm
from paper_2603_00145_amd import warmstart

pytestmark = pytest.mark.gpu
TOL = 2e-2 / 4      # BF16 weights and activations, FP32 accumulation: a few 1e-3 normwise


@pytest.mark.parametrize("n", [16, 528, 16 * 513])
def test_inference_matches_oracle(n):
    rng = np.random.default_rng(n)
    net = warmstart.WarmStartNet(seed=n % 7, zero_head=False)
    X = torch.rand((n, 3, 512), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    X[1::3] = 0.0                                   # empty patches between full ones
    Xb = X.to(torch.bfloat16).view(torch.int16)
    s0 = torch.from_numpy(rng.normal(-3.5, 0.1, (n, 3)).astype(np.float32)).cuda()
    l0 = torch.from_numpy(rng.normal(0, 0.5, n).astype(np.float32)).cuda()
    got = net.forward(Xb, s0, l0)
    pick = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(n - 16, n),
                                     rng.integers(0, n, 40)]))
    t = torch.from_numpy(pick).cuda()
    X0 = Xb[t].view(torch.bfloat16).double().cpu().numpy().reshape(pick.size, 3, 8, 8, 8)
    out, _, _ = owarm.forward(net.weights_host(), X0)
    zero = np.zeros((pick.size, 3)), np.zeros(pick.size)
    base = owarm.assemble(np.zeros_like(out), *zero)
    ref = owarm.assemble(out, *zero)
    for a, r, b0, start in zip(got, ref, base, (s0[t], None, l0[t])):
        a = a[t].double().cpu().numpy()
        if start is not None:
            a = a - start.double().cpu().numpy()
        # the network's own share of the output (what it adds to the initialisation)
        err = np.max(np.abs((a - b0) - (r - b0))) / np.max(np.abs(r - b0))
        assert err < TOL, err
    assert all(torch.equal(a, b) for a, b in zip(got, net.forward(Xb, s0, l0)))
