"""The two ways a launch may take its tiles, a wavefront for each part of a list or one for all of
them (short lists on average), give a tile the same bits: the same Gaussians alone, and beside as many
others elsewhere as turn the launch to the other way."""
import numpy as np
import pytest
import torch

from oracle import gauss
from paper_2603_00145_amd import api, inputs

pytestmark = pytest.mark.gpu


def _cloud(rng, count, lo, hi, size):
    mean = rng.uniform(lo, hi, (count, 3))
    quat = rng.normal(size=(count, 4))
    return (mean, quat / np.linalg.norm(quat, axis=1, keepdims=True),
            np.log(size) + rng.normal(0, 0.3, (count, 3)), rng.normal(0, 1, count))


def _problem(n):
    """Few Gaussians in a corner, its tiles' lists of none to some hundred entries, and many elsewhere."""
    rng = np.random.default_rng(n)
    few = [_cloud(rng, 40, -0.95, -0.3, 6.0 / n), _cloud(rng, 100, -0.9, -0.4, 2.0 / n),
           _cloud(rng, 500, -0.72, -0.66, 1.0 / n)]
    many = [_cloud(rng, {128: 40000, 160: 60000, 272: 150000}[n], 0.1, 0.95, 10.0 / n)]
    cat = lambda parts: inputs.Gaussians(*(np.concatenate(v).astype(np.float32) for v in zip(*parts)))
    return cat(few), cat(few + many)


# parts of a tile's list: 8, 4 and 2
@pytest.mark.parametrize("n,grids", [(128, "stacks"), (160, "volume"), (272, "volume")])
def test_both_ways_give_the_same_bits(n, grids):
    grids = [inputs.volume_grid(n)] if grids == "volume" else \
        inputs.orthogonal_stacks(n, n // 4, 1.0, np.random.default_rng(1), 2.0, 1.0)
    ids = list(range(len(grids)))
    few, both = _problem(n)
    gen = torch.Generator("cuda").manual_seed(n)
    targets = [torch.rand(g.shape, device="cuda", generator=gen) for g in grids]
    got = []
    for g, short in ((few, True), (both, False)):
        p = api.GaussParams.from_host(g)
        b = api.Bins(p.n, grids)
        b.bin(p)
        mean = b.n_pairs // b.total_tiles
        assert mean < 15 if short else mean > 200, mean
        outs = api.render(b, ids)
        o2 = [torch.empty_like(t) for t in targets]
        dls = [torch.empty_like(t) for t in targets]
        loss, _ = api.render_loss(b, ids, targets, dls, outs=o2)
        assert all(torch.equal(x, y) for x, y in zip(outs, o2))
        again, _ = api.render_loss(b, ids, targets, [torch.empty_like(t) for t in targets])
        assert float(again) == float(loss)
        assert all(torch.equal(d, (o - t).clamp(-1, 1) * np.float32(1.0 / sum(g.n_voxels for g in grids)))
                   for d, o, t in zip(dls, outs, targets))
        got.append(outs)
    lit = 0
    for k, g in enumerate(grids):
        # voxels that no other Gaussian reaches: world x, y and z below 0
        w = torch.tensor(np.asarray(g.index_to_world()), dtype=torch.float64, device="cuda")
        z, y, x = torch.meshgrid(*(torch.arange(s, device="cuda", dtype=torch.float64) for s in g.shape),
                                 indexing="ij")
        low = ((torch.stack([x, y, z], -1) @ w[:, :3].T + w[:, 3]) < -0.25).all(-1)
        assert torch.equal(got[0][k][low], got[1][k][low])
        lit += int((got[0][k][low] > 0).sum())
    assert lit > 1000
    # and the value: sampled slices of the first grid against binary64
    ref = gauss.render_all(few, grids[:1])[0]
    err = np.max(np.abs(got[0][0].cpu().numpy() - ref)) / np.max(np.abs(ref))
    assert err <= 1e-5, err


def test_short_lists_take_a_wavefront_a_tile():
    """20000 Gaussians in 320^3: 37 us with a wavefront for each of its 32000 tiles, 71 with two."""
    rng = np.random.default_rng(2)
    g = inputs.Gaussians(*(v.astype(np.float32) for v in _cloud(rng, 20000, -1, 1, 2.0 / 320)))
    p = api.GaussParams.from_host(g)
    b = api.Bins(p.n, [inputs.volume_grid(320)])
    b.bin(p)
    out = torch.empty(b.grids[0].shape, device="cuda")
    best = 1e9
    for _ in range(10):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s.record()
        for _ in range(20):
            api.render(b, [0], [out])
        e.record()
        e.synchronize()
        best = min(best, s.elapsed_time(e) * 1e3 / 20)
    assert best < 52, best
