"""Channels-last sweeps at the edges of how they are cut: leftovers after whole chunks, narrow and wide rows.  Against the same sums and
values in float64, with the tolerances stated in gpu_harness.py."""

import numpy as np
import pytest
import torch

import gpu_harness as G
from paper_1711_07240_amd import cgbn as L

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
TOL = {"f32": 1e-4, "bf16": 2e-2}


def _draw(N, H, W, C, dtype, seed=3):
    gen = torch.Generator(device=G.DEV).manual_seed(seed)
    normal = lambda *s: torch.randn(*s, device=G.DEV, generator=gen)
    x = (normal(N, H, W, C) * (0.5 + torch.rand(C, device=G.DEV, generator=gen)) + normal(C)).to(TORCH[dtype])
    return x, normal(N, H, W, C).to(TORCH[dtype]), normal


def _workspace(N, C, H, W, dtype, K):
    return torch.empty(L.cgbn_workspace_bytes(N, C, H, W, "NHWC", dtype, K), dtype=torch.uint8, device=G.DEV)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# 64, 51, 16, 5 and 1 rows of threads; pixels of a shard: fewer than a chunk, whole chunks, each kind of leftover; value by value; two tiles
@pytest.mark.parametrize("shape", [(2, 16, 168, 16), (3, 33, 47, 40), (2, 61, 53, 128), (2, 9, 7, 408), (5, 3, 1, 2048), (3, 8, 8, 1024), (2, 7, 5, 33),
                                   (2, 7, 9, 2056)], ids=str)
def test_shard_sums(shape, dtype):
    N, H, W, C = shape
    print("[case] shard sums", shape, dtype, flush=True)
    x, dy, normal = _draw(N, H, W, C, dtype)
    ws = _workspace(N, C, H, W, dtype, N)
    mean = x.double().mean((0, 1, 2))
    hi = mean.float()
    lo, invstd = (mean - hi.double()).float(), (1 / x.double().std((0, 1, 2))).float()
    out = lambda: torch.empty(N, C, dtype=torch.float64, device=G.DEV)
    s, v, a, b = out(), out(), out(), out()
    L.cgbn_shard_sum(x, N, C, H, W, "NHWC", N, dtype, s, ws)
    L.cgbn_shard_sqdev(x, N, C, H, W, "NHWC", N, dtype, hi, lo, v, ws)
    L.cgbn_backward_shard_sums(dy, x, N, C, H, W, "NHWC", N, dtype, hi, lo, invstd, a, b, ws)
    torch.cuda.synchronize()
    d = x.double() - hi.double() - lo.double()
    g = dy.double()
    size = np.sqrt(H * W)          # what a shard's sum of unit values amounts to when nothing cancels
    for got, want, scale in ((s, x.double().sum((1, 2)), size), (v, (d * d).sum((1, 2)), H * W), (a, g.sum((1, 2)), size),
                             (b, (g * d * invstd.double()).sum((1, 2)), size)):
        assert float(((got - want).abs() / want.abs().clamp(min=scale)).max()) <= 1e-4
