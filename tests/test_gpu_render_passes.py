"""k_render's order of a batch's pieces and the passes that add two of them at once: footprints of
every class (up to 16, 32, 48 columns and more, and several passes' worth) in batches of one class
and mixed, pieces on top of each other, side by side and touching."""
import numpy as np
import pytest
import torch

from oracle import gauss
from paper_2603_00145_amd import api, inputs

pytestmark = pytest.mark.gpu

# half-widths (voxels) whose footprints fall in the classes: 3x3, 5x5, 6x7, 8x8, 14x14
SIZES = {"a": (0.4, 0.4), "b": (0.75, 0.75), "c": (0.95, 1.05), "d": (1.25, 1.25), "e": (2.4, 2.4)}


@pytest.mark.parametrize("place", ["same", "apart", "random"])
@pytest.mark.parametrize("classes", ["a", "b", "c", "d", "e", "ca", "cba", "abcde"])
@pytest.mark.parametrize("count", [1, 2, 31, 32, 33, 190])
def test_passes_against_oracle(classes, place, count):
    rng = np.random.default_rng(count + 7 * len(classes) + 100 * len(place))
    n = np.array([32, 16, 8], np.float64)
    size = np.array([SIZES[classes[i % len(classes)]] + (0.5,) for i in range(count)])
    c = np.array([8.0, 8.0, 2.0]) + rng.uniform(-0.3, 0.3, (count, 3))
    if place == "apart":        # left and right of the tile in turn: boxes that do not meet
        c[:, 0] += np.where(np.arange(count) % 2 == 0, -4.0, 4.0)
    elif place == "random":     # clipped by the tile's edges and by the grid's
        c = rng.uniform([0, 0, 0], n, (count, 3))
    A = np.zeros((3, 4))
    for k in range(3):
        A[k, k], A[k, 3] = n[k] / 2.0, n[k] / 2.0 - 0.5
    grid = inputs.Grid(32, 16, 8, A, 0.2)
    quat = np.zeros((count, 4), np.float32)
    quat[:, 0] = 1.0
    g = inputs.Gaussians(((2 * c + 1) / n - 1).astype(np.float32), quat,
                         np.log(2.0 * size / n).astype(np.float32),
                         rng.normal(0, 1, count).astype(np.float32))
    p = api.GaussParams.from_host(g)
    b = api.Bins(p.n, [grid])
    b.bin(p)
    out = api.render(b, [0])[0]
    (gt, lo, hi, ne, _), = gauss.prepare(g, [grid])
    ref = gauss.render_scatter(grid, gt, lo, hi, ne)
    err = np.linalg.norm(out.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err < 1e-5 / 4, err      # as the other parity tests of the render's sums
    assert torch.equal(out, api.render(b, [0])[0])
