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


@pytest.mark.parametrize("n", [16, 1040])
def test_gradients_match_oracle(n):
    """One quad of samples per block (four blocks), and more quads than blocks; gradients add to
    what the buffers hold."""
    rng = np.random.default_rng(n)
    net = warmstart.WarmStartNet(seed=n % 5, zero_head=False)
    X = torch.rand((n, 3, 512), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    X[::5] = 0.0
    Xb = X.to(torch.bfloat16).view(torch.int16)
    s0, l0 = rng.normal(-3.5, 0.1, (n, 3)), rng.normal(0, 0.5, n)
    q_t = rng.normal(size=(n, 4))
    S = owarm.covariance(rng.normal(-3.5, 0.3, (n, 3)), q_t)
    sig6 = np.stack([S[:, 0, 0], S[:, 1, 1], S[:, 2, 2], S[:, 0, 1], S[:, 0, 2], S[:, 1, 2]], 1)
    lt = rng.normal(size=n)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    a = tuple(T(v) for v in (s0, l0, sig6, lt))
    loss = net.backward(Xb, *a)
    once = {k: v.clone() for k, v in net.g.items()}
    loss2 = net.backward(Xb, *a)
    assert float(loss) == float(loss2)
    assert all(torch.equal(net.g[k], once[k] * 2) for k in once)
    W = net.weights_host()
    out, _, _ = owarm.forward(W, X.to(torch.bfloat16).double().cpu().numpy().reshape(n, 3, 8, 8, 8))
    f32 = lambda v: np.asarray(v, np.float32).astype(np.float64)
    L, dout = owarm.loss_grad(out, f32(s0), f32(l0), S, f32(lt))
    assert float(loss) == pytest.approx(L, rel=TOL)
    ref = owarm.backward(W, X.to(torch.bfloat16).double().cpu().numpy().reshape(n, 3, 8, 8, 8), dout)
    got = {f"W{l + 1}": once[f"w{l}"].cpu().numpy()[:, :k] for l, k in enumerate(warmstart.KREAL)}
    got |= {f"b{l + 1}": once[f"b{l}"].cpu().numpy() for l in range(4)}
    got |= {"Wl": once["wl"].cpu().numpy(), "bl": once["bl"].cpu().numpy()}
    for k, v in got.items():
        r = np.asarray(ref[k]).reshape(v.shape)
        err = np.max(np.abs(v - r)) / np.max(np.abs(r))
        assert err < 2e-2, (k, err)      # as for every BF16 gradient of the network
    assert not bool(once["w0"][:, warmstart.KREAL[0]:].any())      # padded columns stay untouched
