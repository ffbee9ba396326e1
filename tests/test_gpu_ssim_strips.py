"""SSIM value and gradient at the edges of k_ssim's work split (strips of 54 columns, segments of
rows, cycles of 11 rows) against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import ssim as osim
from paper_2603_00145_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def api():
    from paper_2603_00145_amd import api as a
    a.load()
    return a


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 12, 54), (2, 13, 55), (3, 11, 108), (1, 200, 109),
                                   (160, 150, 60)])
def test_ssim_strip_and_segment_edges(api, shape):
    """Widths around a strip's 54 columns, heights around a segment and a cycle of 11 rows, and
    more strips than resident wavefronts."""
    rng = np.random.default_rng(shape[1])
    p, t = inputs.slice_pair(shape, rng)
    x, y = torch.from_numpy(p).cuda(), torch.from_numpy(t).cuda()
    start = torch.full_like(x, 0.25)
    dl = [start.clone()]
    loss = float(api.ssim_loss([x], [y], dl, 0.5))
    assert float(api.ssim_loss([x], [y], [torch.zeros_like(x)], 0.5)) == loss
    zs = [0, shape[0] // 2, shape[0] - 1]
    total = sum(1.0 - float(api.ssim_loss([x[z:z + 1].clone()], [y[z:z + 1].clone()],
                                            [torch.zeros_like(x[:1])], 0.0))
                for z in range(shape[0]))
    assert abs(loss - (1.0 - total / shape[0])) < 1e-6
    for z in zs:
        ssum, grad = osim.ssim_slice(p[z], t[z])
        ref = -0.5 * grad / p.size
        got = dl[0][z].cpu().numpy().astype(np.float64) - 0.25
        # the gradient adds onto 0.25: one rounding of it, 2^-26
        assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref)) + 2.0 ** -25
