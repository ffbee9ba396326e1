"""The two forms of the SSIM kernel, tiles of 32 x 32 where they are few and strips of 54 columns
elsewhere, at the edges of both (one more or less than a tile's or strip's columns, rows that end in a
segment) and with stacks of different sizes in one call, against the oracle; and the time of a call on
small stacks, which in strips is that of a wavefront's 33 dependent rows."""
import numpy as np
import pytest
import torch

from oracle import ssim as ossim
from paper_2603_00145_amd import api

pytestmark = pytest.mark.gpu

# (nz, ny, nx) of each stack, and the form that the call takes
SHAPES = {
    "tiles, one": [(1, 1, 1)], "tiles, 31": [(3, 31, 33)], "tiles, 32": [(4, 32, 32)],
    "tiles, 33": [(2, 33, 31)], "tiles, mixed": [(5, 64, 65), (1, 7, 200), (0, 9, 9), (9, 40, 12)],
    "tiles, a CU's second": [(70, 34, 33)], "tiles, a block's second": [(300, 64, 64)],
    "strips, 53": [(300, 33, 53)], "strips, 54": [(300, 40, 54)], "strips, 55": [(600, 65, 55)],
    "strips, 109": [(160, 43, 109)], "strips, mixed": [(240, 33, 40), (3, 90, 108), (200, 12, 54)],
    "strips, 5 pixels": [(900, 37, 5)], "strips, wide": [(12, 70, 640), (12, 69, 641)]}


KINDS = 7      # different slices of a stack, repeated along z
TOL = 1e-5     # the parity tests' bound


@pytest.mark.parametrize("name", SHAPES)
def test_both_forms_against_oracle(name):
    rng = np.random.default_rng(len(name))
    X, Y, refs, total = [], [], [], 0.0
    n = sum(a * b * c for a, b, c in SHAPES[name])
    for nz, ny, nx in SHAPES[name]:
        z = np.arange(nz) % KINDS
        x = rng.uniform(0, 1, (KINDS, ny, nx)).astype(np.float32)
        y = (0.7 * x + 0.3 * rng.uniform(0, 1, x.shape)).astype(np.float32)
        r = [ossim.ssim_slice(a, b) for a, b in zip(x, y)]
        total += sum(r[k][0] for k in z)
        refs.append((z, np.stack([-0.5 * g / n for _, g in r])))
        X.append(torch.from_numpy(x[z]).cuda())
        Y.append(torch.from_numpy(y[z]).cuda())
    d = [torch.full_like(a, 0.25) for a in X]
    loss = api.ssim_loss(X, Y, d, 0.5)
    assert float(loss) == pytest.approx(1.0 - total / n, abs=1e-6)
    top = max(np.abs(g).max() for _, g in refs)
    for got, (z, g) in zip(d, refs):
        if z.size:
            # the gradient adds onto 0.25: one rounding of it, 2^-26
            err = np.max(np.abs(got.cpu().numpy().astype(np.float64) - 0.25 - g[z]))
            assert err <= TOL * top + 2.0 ** -25
    again = [torch.full_like(a, 0.25) for a in X]
    assert float(api.ssim_loss(X, Y, again, 0.5)) == float(loss)
    assert all(torch.equal(a, b) for a, b in zip(d, again))


@pytest.mark.parametrize("shape", [(36, 64, 64), (18, 48, 33), (6, 128, 128)])
def test_small_stacks_take_the_time_of_a_tile(shape):
    """14 us in tiles, 26 to 28 in strips (the call's launches replayed from a graph)."""
    x = torch.rand(shape, device="cuda")
    y, d = torch.rand_like(x), torch.zeros_like(x)
    api.ssim_loss([x], [y], [d], 0.5)
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=s):
        for _ in range(20):
            api.ssim_loss([x], [y], [d], 0.5)
    best = 1e9
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 20)
    assert best < 20, best


def test_strips_do_not_depend_on_the_launch_before():
    """920 strips, fewer than the chip's 1024 SIMDs: one to a SIMD whatever ran before.  As blocks of one
    wavefront they shared SIMDs after a large launch, 56 us in place of 40."""
    x = [torch.rand((23, 74, 74), device="cuda") for _ in range(5)]
    y, d = [torch.rand_like(a) for a in x], [torch.zeros_like(a) for a in x]
    big = torch.zeros(40_000_000, device="cuda")

    def best(*calls):
        """us of the calls, replayed from a graph of ten times all of them."""
        for f in calls:
            f()
        torch.cuda.synchronize()
        g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(g, stream=st):
            for _ in range(10):
                for f in calls:
                    f()
        t = 1e9
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.replay()
            b.record()
            b.synchronize()
            t = min(t, a.elapsed_time(b) * 1e2)
        return t
    ssim, fill = lambda: api.ssim_loss(x, y, d, 0.5), lambda: big.fill_(1.0)
    alone = best(ssim)
    assert best(fill, ssim) - best(fill) <= 1.2 * alone, alone
