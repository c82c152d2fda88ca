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


MAPS = [
    # value by value (pixels no whole number of groups): a row of threads, many, several tiles; chunks, leftovers, a piece of one pixel
    (3, 7, 9, 87), (1, 61, 53, 11), (1, 9, 37, 298), (1, 5, 33, 834), (1, 3, 1, 601), (1, 1, 17, 257),
    # rows of several tiles: pieces of a tile or of the row, ragged ones
    (2, 7, 11, 2560), (2, 33, 41, 1376), (1, 61, 53, 4104),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_map_pieces_value_by_value(dtype):
    for N, H, W, C in [m for m in MAPS if m[3] % 4]:
        get = lambda k: L.cgbn_plan_get(N, C, H, W, "NHWC", dtype, 1, k)
        assert get("vec") == 1 and get("may_group") == 1
        for pl, pp in (("PLm", "ppsm"), ("PLm2", "ppsm2")):
            PL, pps, rpp, spix = get(pl), get(pp), get("rpp"), N * H * W
            assert pps == -(-spix // PL) and (PL == spix or PL % (4 * rpp) == 0)
            assert PL <= 16 * rpp, "two chunks a thread at most"


@pytest.mark.parametrize("dtype,C", [("bf16", 2560), ("bf16", 4104), ("bf16", 4096), ("f32", 1376), ("f32", 2048), ("f32", 2052)])
def test_map_pieces_of_several_tiles(dtype, C):
    """32 KiB of the tile with one input, and with two of bfloat16, whose pieces are 96 if the last tile is shorter; of the row with two of
    float, or more than two tiles: in whole passes of four pixels a thread."""
    get = lambda k: L.cgbn_plan_get(64, C, 40, 50, "NHWC", dtype, 1, k)
    eb = 4 if dtype == "f32" else 2
    assert get("ctiles") > 1 and get("rpp") == 1
    tile, row = get("TW") * get("vec") * eb, C * eb
    whole = dtype == "f32" or get("cv") % get("TW") == 0
    by_row = max(4, 32768 // row // 4 * 4)
    assert get("PLm") == (by_row if dtype == "f32" and get("ctiles") > 2 else (32768 if whole else 98304) // tile // 4 * 4)
    assert get("PLm2") == (get("PLm") if dtype == "bf16" else by_row)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", MAPS + [(3, 37, 11, 64), (2, 25, 42, 1024), (2, 20, 40, 255), (4, 21, 30, 100)], ids=str)     # (whole vectors, and grouped)
def test_elementwise(shape, dtype):
    """Every elementwise sweep, per-channel vectors 4, 8 and 12 bytes off a 16-byte boundary: they need be no more than floats."""
    N, H, W, C = shape
    print("[case] elementwise", shape, dtype, flush=True)
    x, dy, normal = _draw(N, H, W, C, dtype)
    short = normal(N, H, W, C).to(TORCH[dtype])
    def vec(make, off):
        a = torch.empty(C + 4, device=G.DEV)
        assert a.data_ptr() % 16 == 0
        a[off:off + C] = make
        return a[off:off + C]
    rand = lambda: torch.rand(C, device=G.DEV)
    mean, lo, invstd, gamma, beta = vec(normal(C), 1), vec(1e-8 * normal(C), 2), vec(0.5 + rand(), 3), vec(0.5 + rand(), 1), vec(normal(C), 2)
    var, dgamma, dbeta = vec(0.25 + rand(), 3), vec(normal(C), 1), vec(normal(C), 2)
    x64, dy64, M = x.double(), dy.double(), N * H * W
    m, g = mean.double() + lo.double(), gamma.double()
    xhat = (x64 - m) * invstd.double()
    scale = g / torch.sqrt(var.double() + 1e-5)
    dims, y = (N, C, H, W, "NHWC"), torch.empty_like(x)
    def check(want):
        torch.cuda.synchronize()
        rms = want.square().mean().sqrt()
        assert float(((y.double() - want).abs() / want.abs().clamp(min=rms)).max()) <= TOL[dtype]
        y.zero_()
    L.cgbn_normalize(x, *dims, dtype, mean, lo, invstd, gamma, beta, y)
    check(xhat * g + beta.double())
    L.cgbn_backward_dx(dy, x, *dims, dtype, mean, lo, invstd, gamma, dgamma, dbeta, y)
    check(g * invstd.double() * (dy64 - dbeta.double() / M - xhat * dgamma.double() / M))
    L.cgbn_frozen_forward(x, *dims, dtype, mean, var, gamma, beta, 1e-5, y)
    check((x64 - mean.double()) * scale + beta.double())
    L.cgbn_frozen_backward(dy, *dims, dtype, var, gamma, 1e-5, y)
    check(dy64 * scale)
    # the sweeps with a shortcut and a mask: as the last ones of whole calls
    ws = _workspace(N, C, H, W, dtype, 1)
    y, dz, dx = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
    out = [vec(torch.zeros(C, device=G.DEV), o) for o in (1, 2, 3, 1, 3)]
    old = L.cgbn_get_tuning("fused")
    L.cgbn_set_tuning("fused", 0)
    try:
        L.cgbn_forward_relu(x, short, *dims, 1, gamma, beta, 1e-5, y, out[0], out[1], dtype, out[2], ws)
        m, i = out[0].double() + out[2].double(), out[1].double()
        want, stored = ((x64 - m) * i * g + beta.double() + short.double()).clamp(min=0), y.clone()
        check(want)
        L.cgbn_backward_relu(dy, stored, x, out[0], out[1], gamma, dx, dz, out[3], out[4], *dims, 1, dtype, out[2], ws)
        torch.cuda.synchronize()
        d = dy64 * (stored > 0)
        assert torch.equal(dz.double(), d)
        y.copy_(dx)
        check(g * i * (d - out[4].double() / M - (x64 - m) * i * out[3].double() / M))
    finally:
        L.cgbn_set_tuning("fused", old)


def test_map_pieces_of_vectors():
    """32 KiB, half of it with three float inputs; shorter where 512 workgroups (384 with two or three float inputs) do not come together."""
    get = lambda n, c, dtype, k: L.cgbn_plan_get(n, c, 28, 28, "NHWC", dtype, 1, k)
    for dtype, eb, grids in (("f32", 4, (512, 384, 384)), ("bf16", 2, (512, 512, 512))):
        for n, c in ((200, 64), (100, 128), (25, 512), (14, 1024)):
            for i, (suffix, grid) in enumerate(zip(("", "2", "3"), grids)):
                piece = get(n, c, dtype, "PLm" + suffix) * c * eb
                assert piece in ((16384, 8192) if i == 2 and dtype == "f32" else (32768, 16384)) and get(n, c, dtype, "gridm" + suffix) >= grid
    # 427 workgroups of 32 KiB: enough for two float inputs, too few for one
    assert get(35, 128, "f32", "PLm2") * 512 == 32768 and get(35, 128, "f32", "PLm") * 512 == 16384


def test_single_constants_rule():
    get = lambda n, c, dtype: L.cgbn_plan_get(n, c, 100, 168, "NHWC", dtype, 1, "single_consts")
    assert get(16, 256, "f32") == 1 and get(15, 256, "f32") == 0          # 275 and 258 MB
    assert get(8, 1024, "f32") == 1 and get(8, 1028, "f32") == 0          # one tile, two
    assert get(64, 256, "bf16") == 0 and get(400, 15, "f32") == 0


@pytest.mark.gpu
def test_single_constants():
    """Beyond 256 MiB: dx equals, bit by bit, dx of the two halves, each below (their sums and the count both halved, exactly); the forward with a
    shortcut against float64."""
    N, H, W, C = 18, 100, 168, 256
    assert L.cgbn_plan_get(N, C, H, W, "NHWC", "f32", 1, "single_consts") == 1
    x, dy, normal = _draw(N, H, W, C, "f32")
    print("[case] single constants", flush=True)
    mean, lo, invstd, gamma, beta, dgamma, dbeta = normal(C), 1e-8 * normal(C), 0.5 + torch.rand(C, device=G.DEV), 0.5 + torch.rand(C, device=G.DEV), normal(C), normal(C), normal(C)
    dx, parts = torch.empty_like(x), torch.empty_like(x)
    L.cgbn_backward_dx(dy, x, N, C, H, W, "NHWC", "f32", mean, lo, invstd, gamma, dgamma, dbeta, dx)
    for i in (slice(0, 9), slice(9, 18)):
        L.cgbn_backward_dx(dy[i], x[i], 9, C, H, W, "NHWC", "f32", mean, lo, invstd, gamma, dgamma / 2, dbeta / 2, parts[i])
    torch.cuda.synchronize()
    assert torch.equal(dx, parts)
    ws, y = _workspace(N, C, H, W, "f32", 2), parts
    old = L.cgbn_get_tuning("fused")
    L.cgbn_set_tuning("fused", 0)
    try:
        L.cgbn_forward_relu(x, dy, N, C, H, W, "NHWC", 2, gamma, beta, 1e-5, y, mean, invstd, "f32", lo, ws)
    finally:
        L.cgbn_set_tuning("fused", old)
    torch.cuda.synchronize()
    want = (x.double() - mean.double() - lo.double()) * (invstd.double() * gamma.double()) + beta.double() + dy.double()
    # a handful of roundings of values of up to ten times the standard deviation
    assert float((y.double() - want.clamp(min=0)).abs().max()) <= 1e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_launch_has_less_than_two_to_the_32_threads(dtype):
    """137 GB and more, value by value and in whole vectors: the pieces grow rather than the grid."""
    for N, C, H, W in ((1, 2047, 6401, 6400), (9, 127, 8001, 7999), (64, 2048, 800, 800)):
        get = lambda k: L.cgbn_plan_get(N, C, H, W, "NHWC", dtype, 1, k)
        for i in ("", "2", "3"):
            assert 0 < get("gridm" + i) * 256 < 2 ** 32 and get("ppsm" + i) == -(-N * H * W // get("PLm" + i))
