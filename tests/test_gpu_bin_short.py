"""gm_bin's short paths (chunk totals in place of the scans, the radix pass that sums its own
counts) and the long ones at their borders: list for list what the oracle's boxes give."""
import numpy as np
import pytest
import torch

from oracle import recipe
from paper_2603_00145_amd import api, inputs

pytestmark = pytest.mark.gpu


def _grid(dims):
    A = np.zeros((3, 4))
    for k, n in enumerate(dims):
        A[k, k], A[k, 3] = n / 2.0, n / 2.0 - 0.5
    return inputs.Grid(*dims, A, 0.0)


def _gaussians(n, size, rng):
    quat = np.concatenate([np.ones((n, 1)), rng.normal(0, 0.05, (n, 3))], 1).astype(np.float32)
    return inputs.Gaussians(rng.uniform(-1.05, 1.05, (n, 3)).astype(np.float32), quat,
                            (np.log(size) + rng.normal(0, 0.3, (n, 3))).astype(np.float32),
                            rng.normal(0, 1, n).astype(np.float32))


# Gaussians, their size, grids: 1, 255 to 257 and 513 tiles (one and two radix passes); chunks
# around 2048 (524288 Gaussians on one grid, 65536 on eight); pairs around 192 blocks of 2048
CASES = [(1, 1e-4, [(256, 16, 4)]), (1, 1e-4, [(16, 16, 4)]), (255, 0.02, [(16, 16, 4)]),
         (256, 0.02, [(240, 16, 4)] * 8), (257, 0.05, [(240, 272, 4)]), (3000, 0.02, [(256, 256, 4)]),
         (3000, 0.02, [(257, 255, 4)]), (5000, 0.01, [(16 * 19, 16 * 27, 4)]),
         (524288, 0.001, [(64, 64, 16)]), (524289, 0.001, [(64, 64, 16)]),
         (65536, 0.002, [(40, 30, 8)] * 8), (65537, 0.002, [(40, 30, 8)] * 8),
         (393216, 1e-5, [(48, 48, 8)]), (393217, 1e-5, [(130, 90, 20)])]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_lists_match_boxes(case):
    n, size, dims = CASES[case]
    rng = np.random.default_rng(case)
    g = _gaussians(n, size, rng)
    grids = [_grid(d) for d in dims]
    p = api.GaussParams.from_host(g)
    b = api.Bins(n, grids)
    for _ in range(2):
        b.box_volume.fill_(-1)
        b.pair_gauss.fill_(-1)
        b.tile_start.fill_(-1)
        pairs = b.bin(p)
        keys, vals, vols, base = [], [], [], 0
        boxes = {}
        for k, gr in enumerate(grids):
            if dims[k] not in boxes:
                boxes[dims[k]] = recipe.boxes(g.mean, g.quat, g.log_scale, g.logit, gr)[:3]
            lo, hi, ne = boxes[dims[k]]
            ids = np.flatnonzero(ne)
            tlo, thi = lo[ids] // [16, 16, 4], hi[ids] // [16, 16, 4]
            nt = [-(-d // t) for d, t in zip(dims[k], (16, 16, 4))]
            w = thi - tlo + 1
            cnt = w.prod(1)
            rep = np.repeat(np.arange(len(ids)), cnt)
            j = np.arange(cnt.sum()) - np.repeat(np.cumsum(cnt) - cnt, cnt)
            x = tlo[rep, 0] + j % w[rep, 0]
            y = tlo[rep, 1] + j // w[rep, 0] % w[rep, 1]
            z = tlo[rep, 2] + j // (w[rep, 0] * w[rep, 1])
            keys.append(base + (z * nt[1] + y) * nt[0] + x)
            vals.append(ids[rep].astype(np.uint32) | np.where(j == 0, 1 << 31, 0).astype(np.uint32))
            vols.append(int((hi[ids] - lo[ids] + 1).prod(1).sum()))
            base += nt[0] * nt[1] * nt[2]
        keys, vals = np.concatenate(keys), np.concatenate(vals)
        order = np.argsort(keys, kind="stable")
        assert pairs == len(keys)
        assert b.box_pairs_host == vols
        assert b.box_volume[:len(grids)].tolist() == vols
        assert np.array_equal(b.tile_start.cpu().numpy(),
                              np.searchsorted(keys[order], np.arange(base + 1)))
        assert np.array_equal(b.pair_gauss[:pairs].cpu().numpy().view(np.uint32), vals[order])


def test_invalid_parameters_are_reported():
    for n in (100, 600000):
        g = _gaussians(n, 0.01, np.random.default_rng(n))
        p = api.GaussParams.from_host(g)
        b = api.Bins(n, [_grid((32, 32, 8))] * 2)
        b.bin(p)
        p.quat[n // 2] = 0.0
        with pytest.raises(api.GmError):
            b.bin(p)
        p.quat[n // 2, 0] = 1.0
        b.bin(p)
