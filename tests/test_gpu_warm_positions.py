"""A sample's results do not depend on where it stands in a batch: the first sample that a block
takes, staged right after the block has set up its LDS, is treated as every later one."""
import pytest
import torch

from paper_2603_00145_amd import warmstart

pytestmark = pytest.mark.gpu


def _batch(n, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    X = torch.rand((n, 3, 512), device="cuda", generator=gen).to(torch.bfloat16).view(torch.int16)
    return X, torch.randn((n, 3), device="cuda", generator=gen), torch.randn(n, device="cuda", generator=gen)


@pytest.mark.parametrize("n", [512, 16 * 33, 16 * 100])    # blocks of one sample, of one or two, of more
def test_inference_does_not_depend_on_the_place(n):
    """The same bits after the batch is turned by half the resident blocks and an odd number."""
    net = warmstart.WarmStartNet(seed=n % 7, zero_head=False)
    args = _batch(n, n)
    ref = net.forward(*args)
    for shift in (256, 37):
        got = net.forward(*(torch.roll(a, shift, 0) for a in args))
        assert all(torch.equal(torch.roll(r, shift, 0), g) for r, g in zip(ref, got))


@pytest.mark.parametrize("n", [1024, 2048])
def test_training_does_not_depend_on_the_place(n):
    """n copies of 16 samples: the loss of the 16, and their gradients up to the order of the FP32
    sums (means of the same values, scaled by powers of two: a rounding of 2^-24 for each of some
    tens of partial sums)."""
    net = warmstart.WarmStartNet(seed=3, zero_head=False)
    X, s0, l0 = _batch(16, 5)
    gen = torch.Generator("cuda").manual_seed(6)
    s_t = s0 + 0.2 * torch.randn((16, 3), device="cuda", generator=gen)
    q_t = torch.nn.functional.pad(0.2 * torch.randn((16, 3), device="cuda", generator=gen), (1, 0), value=1.0)
    args = (X, s0, l0, warmstart.sym6(s_t, q_t), l0 + 0.5)
    loss = float(net.backward(*args))
    ref = {k: v.clone() for k, v in net.g.items()}
    for v in net.g.values():
        v.zero_()
    many = tuple(a.repeat(n // 16, *[1] * (a.dim() - 1)) for a in args)
    assert float(net.backward(*many)) == pytest.approx(loss, rel=1e-6)
    for k, r in ref.items():
        assert float((net.g[k] - r).abs().max()) <= 1e-5 * float(r.abs().max()), k
