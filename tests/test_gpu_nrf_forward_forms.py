"""The field's forward with the weights in registers and read from LDS (128 features, three layers on
more than 2^20 voxels or four): the bits of the field formed in the render's pass, whose empty tiles
leave nothing else, on grids on both sides of the change and ragged."""
import numpy as np
import pytest
import torch

from paper_2603_00145_amd import api, inputs, nrf

pytestmark = pytest.mark.gpu


def _grid(dims):
    A = np.zeros((3, 4))
    for k, m in enumerate(dims):
        A[k, k], A[k, 3] = m / 2.0, m / 2.0 - 0.5
    return inputs.Grid(*dims, A, 0.0)


@pytest.mark.parametrize("dims", [(1, 1, 1), (33, 17, 5), (128, 128, 64), (129, 128, 64)])
@pytest.mark.parametrize("n_freq,depth", [(10, 3), (16, 3), (10, 4), (16, 4), (6, 4)])
def test_forward_equals_the_fused_field(dims, n_freq, depth):
    grid = _grid(dims)
    net = nrf.NRF(n_freq=n_freq, depth=depth, seed=n_freq, zero_last=False)
    out = torch.zeros(grid.shape, device="cuda")
    net.forward_add(grid, out)
    # one Gaussian far outside: every tile's list is empty
    p = api.GaussParams.from_host(inputs.Gaussians(
        np.full((1, 3), 30.0, np.float32), np.array([[1, 0, 0, 0]], np.float32),
        np.full((1, 3), -4.0, np.float32), np.zeros(1, np.float32)))
    b = api.Bins(1, [grid])
    b.bin(p)
    assert b.n_pairs == 0
    assert torch.equal(out, api.render_volume(b, 0, nrf=net))
    assert bool(out.any())
    again = torch.zeros_like(out)
    net.forward_add(grid, again)
    assert torch.equal(again, out)


def test_four_layers_take_no_longer_than_a_register_wavefront():
    """128^3, 16 bands, four layers: 206 us; with the weights in registers at one wavefront a SIMD 272."""
    grid = inputs.volume_grid(128)
    net = nrf.NRF(n_freq=16, depth=4, seed=1, zero_last=False)
    out = torch.zeros(grid.shape, device="cuda")
    best = 1e9
    for _ in range(8):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s.record()
        for _ in range(10):
            net.forward_add(grid, out)
        e.record()
        e.synchronize()
        best = min(best, s.elapsed_time(e) * 1e2)
    assert best < 240, best
