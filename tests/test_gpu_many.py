"""Adam, the BF16 copies and the clears of several tensors in one launch: the bits of the separate
calls, at sizes around a block's 1024 elements and lists longer than one launch takes."""
import ctypes

import pytest
import torch

from paper_2603_00145_amd import _lib, api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1,), (1023, 1024, 1025, 0, 70001), tuple(range(1, 18))])
def test_many_equal_separate_calls(sizes):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(sizes))
    p, g, m, v = ([torch.randn(n, device="cuda", generator=gen).abs() if k == 3 else
                   torch.randn(n, device="cuda", generator=gen) for n in sizes] for k in range(4))
    bf = [torch.empty(n, dtype=torch.int16, device="cuda") if i % 2 == 0 else None
          for i, n in enumerate(sizes)]
    ref = [[t.clone() for t in ts] for ts in (p, m, v)]
    for i, n in enumerate(sizes):
        if n:
            api.adam_step(ref[0][i], g[i], ref[1][i], ref[2][i], 1e-2, 3)
    api.adam_step_many(p, g, m, v, bf, 1e-2, 3)
    for a, b in zip((p, m, v), ref):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    for x, h in zip(p, bf):
        if h is not None and x.numel():
            out = torch.empty_like(h)
            _lib.check(_lib.load().gm_f32_to_bf16(ctypes.c_void_p(x.data_ptr()),
                                                  ctypes.c_void_p(out.data_ptr()), x.numel(),
                                                  api._stream()))
            assert torch.equal(out, h)
    guard = [torch.cat([t, torch.ones(5, device="cuda")]) for t in p]
    api.zero_many([t[:n] for t, n in zip(guard, sizes)])
    assert all(not t[:n].any() and bool((t[n:] == 1).all()) for t, n in zip(guard, sizes))


def test_clears_of_views_at_any_offset():
    """Gradients that are views into one buffer are cleared wherever they start, and nothing else."""
    flat = torch.ones(4096, device="cuda")
    spans = [(1, 5), (7, 1030), (1041, 1042), (2003, 4095)]
    api.zero_many([flat[a:b] for a, b in spans])
    ref = torch.ones(4096)
    for a, b in spans:
        ref[a:b] = 0
    assert torch.equal(flat.cpu(), ref)
