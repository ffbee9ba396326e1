"""The warm start's patch gather at the edges of its two forms: stacks one or two voxels thick along
each axis (a stack one voxel wide takes the general form), points exactly on the first and last
voxel, between and outside, against the oracle.  Positions are multiples of 1/2 and the data
positive, so only FP32 sums of positive terms and the rounding to BF16 (2^-9) separate the two:
bound 2^-8 of each value, zeros exact."""
import numpy as np
import pytest
import torch

from oracle import warm as owarm
from paper_2603_00145_amd import inputs

pytestmark = pytest.mark.gpu


def grid(nx, ny, nz):
    A = np.zeros((3, 4))
    A[:, :3] = np.eye(3)
    return inputs.Grid(nx=nx, ny=ny, nz=nz, world_to_index=A, psf_sigma_z=0.0, name="edge")


@pytest.mark.parametrize("dims", [
    ((9, 7, 5), (6, 1, 8), (7, 9, 1)),
    ((2, 2, 2), (2, 1, 1), (70, 3, 2)),
    ((1, 9, 7), (9, 7, 5), (2, 2, 2)),
    ((1, 1, 1), (1, 2, 1), (5, 1, 1)),
])
def test_gather_edges(dims):
    from paper_2603_00145_amd import warmstart as ws
    rng = np.random.default_rng(11)
    grids = [grid(*d) for d in dims]
    data = [rng.uniform(0.25, 1.0, g.shape).astype(np.float32) for g in grids]
    means = np.concatenate([
        0.25 + 0.5 * rng.integers(-4, 18, (40, 3)),
        np.repeat(0.25 + 0.5 * rng.integers(0, 4, (24, 1)), 3, 1)]).astype(np.float32)
    got = ws.WarmStartNet.gather(grids, [torch.from_numpy(d).cuda() for d in data],
                                 torch.from_numpy(means).cuda(), 0.5)
    got = got.cpu().view(torch.bfloat16).to(torch.float64).numpy().reshape(len(means), 3, 512)
    ref = owarm.gather(grids, data, means, 0.5).reshape(len(means), 3, 512)
    assert (np.abs(ref) > 0).any(axis=(0, 2)).all()
    assert (np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref)).all()
