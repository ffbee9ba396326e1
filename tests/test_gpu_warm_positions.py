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
