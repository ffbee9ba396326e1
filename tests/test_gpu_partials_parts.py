"""k_partials at the edges of its work split: a tile's list in 1 to 16 parts, lists of no, one, few
and more than a window's Gaussians, boxes whose x passes, planes and rows run past the sort key's
caps, and few or many boxes past the staged region (the two lane widths of the global path)."""
import math

import numpy as np
import pytest
import torch

from oracle import gauss
from paper_2603_00145_amd import api, inputs

pytestmark = pytest.mark.gpu
TOL = 1e-5      # the bound of the ragged parity tests

# grid dims -> parts: 1, 64, 75, 256, 260, 512 and 513 or more tiles
DIMS = {"16 parts, one tile": (11, 16, 4), "16 parts, most tiles": (64, 64, 16),
        "8 parts": (80, 70, 12), "4 parts, most tiles": (128, 128, 15), "2 parts": (80, 200, 16),
        "2 parts, most tiles": (128, 128, 32), "1 part": (140, 141, 27)}


def _problem(dims, rng):
    n = np.array(dims, np.float64)
    ntx, nty = -(-dims[0] // 16), -(-dims[1] // 16)
    mean, ls = [], []

    def add(m, centre, spread, size, jitter):
        mean.append((2 * (np.asarray(centre) + rng.uniform(-1, 1, (m, 3)) * spread) + 1) / n - 1)
        ls.append(np.log(2.0 * np.asarray(size) / n) + rng.normal(0, jitter, (m, 3)))

    for t, m in enumerate([3, 1, 40, 15, 17, 300, 2600][:ntx * nty]):
        add(m, [16 * (t % ntx) + 8, min(16 * (t // ntx) + 8, n[1] / 2), 2], [4, 4, 1],
            [0.8, 0.8, 0.8], 0.3)
    add(6, n / 2, n / 4, [3.0, 2.5, 1.2], 0.1)          # past the caps, mostly inside a region
    add(12, n / 2, n / 4, [4.0, 4.5, 2.0], 0.1)         # past the region: few to a tile
    add(60, n / 2, [2, 2, 1], [3.5, 3.5, 1.0], 0.1)     # ... and many
    mean, ls = np.concatenate(mean).astype(np.float32), np.concatenate(ls).astype(np.float32)
    k = mean.shape[0]
    quat = np.concatenate([np.ones((k, 1)), rng.normal(0, 0.02, (k, 3))], 1).astype(np.float32)
    return inputs.Gaussians(mean, quat, ls, rng.normal(0, 1, k).astype(np.float32))


@pytest.mark.parametrize("name", DIMS)
def test_partials_against_oracle(name):
    rng = np.random.default_rng(len(name))
    dims = DIMS[name]
    A = np.zeros((3, 4))
    for k, m in enumerate(dims):
        A[k, k], A[k, 3] = m / 2.0, m / 2.0 - 0.5
    grid = inputs.Grid(*dims, A, 0.3)
    g = _problem(dims, rng)
    dl = rng.standard_normal((dims[2], dims[1], dims[0])).astype(np.float32)
    p = api.GaussParams.from_host(g)
    b = api.Bins(p.n, [grid], capacity=1 << 18)
    b.bin(p)
    d = [torch.from_numpy(dl).cuda()]
    api.grid_partials(p, b, [0], d)
    pg = b.grid_grads[0, :p.n].clone()
    (gt, lo, hi, ne, _), = gauss.prepare(g, [grid])
    d_amp, d_c, G_C = gauss.grid_partials(grid, gt, lo, hi, ne, dl)
    ref = np.concatenate([d_amp[:, None], d_c, np.stack(
        [G_C[:, 0, 0], G_C[:, 1, 1], G_C[:, 2, 2], G_C[:, 0, 1], G_C[:, 0, 2], G_C[:, 1, 2]], 1) /
        (-0.5 / math.log(2.0))], 1)
    got = pg.cpu().numpy().astype(np.float64)
    for part in (slice(0, 1), slice(1, 4), slice(4, 10)):
        err = np.max(np.abs(got[:, part] - ref[:, part])) / np.max(np.abs(ref[:, part]))
        assert err <= TOL, (part, err)
    for _ in range(3):
        b.grid_grads.fill_(7.0)
        b.bin(p)
        api.grid_partials(p, b, [0], d)
        assert torch.equal(b.grid_grads[0, :p.n], pg)
