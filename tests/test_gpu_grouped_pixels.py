"""Channels-last tensors whose channel count is no multiple of a 16-byte vector: their sweeps take a group of pixels as one
pixel of whole vectors.  And the elementwise sweep's edges: pieces of fewer pixels than a chunk, constants formed once a workgroup
or by every thread.  Against the float64 oracles, with the tolerances stated in gpu_harness.py."""

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from oracle import cgbn_relu_oracle as R
from oracle import frozen_bn_oracle as F
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

# N, C, H, W, dtype, K, pixels a group (1: none)
CASES = [
    (3, 35, 41, 23, "f32", 3, 1),             # pixels not a multiple of 4: value by value
    (4, 35, 42, 22, "f32", 2, 4),
    (8, 35, 31, 23, "bf16", 8, 8),            # a shard of 713 pixels is no whole number of groups
    (2, 187, 30, 44, "bf16", 2, 8),
    (2, 255, 20, 40, "f32", 1, 4),            # 255 vectors: nearly a whole tile
    (4, 257, 20, 20, "bf16", 2, 1),           # 257: two tiles, value by value
    (4, 510, 12, 20, "bf16", 4, 4),           # 4 pixels, channels beyond the threads of a workgroup
    (4, 100, 21, 30, "bf16", 1, 2),
    (2, 2, 300, 300, "bf16", 2, 4),           # one vector a group
    (2, 6, 200, 211, "f32", 1, 2),
    (3, 50, 9, 8, "f32", 3, 1),               # a small tensor
    (15, 13, 32, 52, "bf16", 15, 8),          # few channels, many rows of threads: what is joined is most of a workgroup's work
    (16, 11, 60, 60, "f32", 4, 4),
    (24, 414, 8, 8, "bf16", 24, 4),           # the forward's sums value by value, the backward's grouped
    (16, 414, 4, 6, "bf16", 16, 4),           # both value by value, the elementwise sweeps grouped
    (32, 98, 14, 14, "f32", 32, 2),           # ragged last pass of grouped rows
    (200, 34, 5, 5, "bf16", 200, 4),          # shards of 25 pixels: pooled
    (4, 414, 50, 60, "f32", 4, 2),            # more channels than threads: constants in two rounds
    (2, 306, 24, 32, "f32", 2, 2),            # ... of a small tensor: with a second input value by value
]
# sums (of x alone, with dy) that group pixels, where pixels may be grouped at all
MAP2_ONE_BY_ONE = {(2, 306, 24, 32)}          # elementwise sweeps with a second input
ONE_BY_ONE = {(24, 414, 8, 8): (0, 1), (16, 414, 4, 6): (0, 0)}
FROZEN = CASES + [(2, 1024, 13, 9, "bf16", 1, 1), (1, 2048, 5, 7, "f32", 1, 1), (3, 64, 37, 11, "bf16", 1, 1), (2, 256, 3, 1, "f32", 1, 1)]


def _ids(c):
    return "%dx%dx%dx%d-%s" % (c[0], c[2], c[3], c[1], c[4])


def _draw(N, C, H, W, dtype, seed=5):
    r = np.random.default_rng(seed)
    mu, sg = r.uniform(-2, 2, C), r.uniform(0.5, 3, C)
    x = (r.standard_normal((N, H, W, C)) * sg + mu).astype(np.float32)
    dy = r.standard_normal((N, H, W, C)).astype(np.float32)
    if dtype == "bf16":
        x, dy = synth.f32_to_bf16_bits(x), synth.f32_to_bf16_bits(dy)
    gamma, beta = r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)
    return x, dy, gamma, beta, (mu + 0.1).astype(np.float32), (sg * sg).astype(np.float32)


@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_plan(case):
    """The pieces cover the tensor exactly and their rows fit the room there is for them."""
    N, C, H, W, dtype, K, group = case
    shape = (N, C, H, W, "NHWC", dtype, K)
    get = lambda k: L.cgbn_plan_get(*shape, k)
    assert get("may_group") == group
    assert (get("group_sums"), get("group_sums_dy")) == (ONE_BY_ONE.get((N, C, H, W), (1, 1)) if group > 1 else (0, 0))
    assert (get("group_map"), get("group_map2")) == ((1, (N, C, H, W) not in MAP2_ONE_BY_ONE) if group > 1 else (0, 0))
    if group > 1:
        g = lambda k: get("grouped_" + k)
        assert C * group % (16 // (4 if dtype == "f32" else 2)) == 0 and g("ctiles") == 1
        assert g("spix") * g("K") * group == N * H * W and g("K") in (1, K)
        assert (g("pps") - 1) * g("PL") < g("spix") <= g("pps") * g("PL") and g("rows") == g("pps") * g("K")
        assert g("rows") * C * 4 <= get("part_bytes")


@pytest.mark.gpu
@pytest.mark.parametrize("two_sweeps", [False, True])
@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_forward_backward(case, two_sweeps):
    N, C, H, W, dtype, K, _ = case
    print("[case] grouped", case, two_sweeps, flush=True)
    x, dy, gamma, beta, _, _ = _draw(N, C, H, W, dtype)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NHWC", dtype, K)
    L.cgbn_set_tuning("one_sweep_stats", 0 if two_sweeps else 1)
    try:
        p.forward()
        p.backward()
        torch.cuda.synchronize()
    finally:
        L.cgbn_set_tuning("one_sweep_stats", 1)
    ref = O.cgbn_forward_backward_ref(G.widen(x, dtype), G.widen(dy, dtype), gamma, beta, 1e-5, "NHWC")
    G.check_against_oracle(p.results(), ref, dtype, str(case))


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_shortcut_and_mask(case):
    """The sweeps with two and three inputs: equal to the plain ones followed, or preceded, by the elementwise part."""
    N, C, H, W, dtype, K, _ = case
    print("[case] grouped relu", case, flush=True)
    x, dy, gamma, beta, _, _ = _draw(N, C, H, W, dtype)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NHWC", dtype, K)
    short = synth.f32_to_bf16_bits(np.random.default_rng(9).standard_normal(x.shape).astype(np.float32)) if dtype == "bf16" else \
        np.random.default_rng(9).standard_normal(x.shape).astype(np.float32)
    sd, y, dz = G.to_dev(short), torch.empty_like(p.x), torch.empty_like(p.x)
    L.cgbn_forward_relu(p.x, sd, *p.shape_args, "NHWC", K, p.gamma, p.beta, 1e-5, y, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
    L.cgbn_backward_relu(p.dy, y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args, "NHWC", K, dtype,
                         p.mean_lo, p.ws)
    torch.cuda.synchronize()
    wx, wdy, wy = G.widen(x, dtype), G.widen(dy, dtype), G.to_host_f64(y, dtype)
    y_ref, mean, invstd = R.cgbn_relu_forward_ref(wx, gamma, beta, 1e-5, "NHWC", G.widen(short, dtype))[:3]
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert np.max(np.abs(wy - y_ref) / (1.0 if dtype == "f32" else np.maximum(np.abs(y_ref), G.rms(y_ref)))) <= tol
    # (the mask is read off the stored output, so the oracle is handed the same)
    ref = R.cgbn_relu_backward_ref(wdy, wy, wx, mean, invstd, gamma, "NHWC")
    assert np.array_equal(G.to_host_f64(dz, dtype), wdy * (wy > 0))
    for got, want in ((G.to_host_f64(p.dx, dtype), ref[0]), (p.dgamma.cpu().numpy(), ref[1]), (p.dbeta.cpu().numpy(), ref[2])):
        assert G.max_rel_err(got, want, G.rms(want)) <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("case", FROZEN, ids=_ids)
def test_frozen(case):
    N, C, H, W, dtype, _, _ = case
    print("[case] grouped frozen", case, flush=True)
    x, dy, gamma, beta, fm, fv = _draw(N, C, H, W, dtype)
    xd, dyd, gd, bd, md, vd = (G.to_dev(a) for a in (x, dy, gamma, beta, fm, fv))
    y, dx = torch.empty_like(xd), torch.empty_like(dyd)
    L.cgbn_frozen_forward(xd, N, C, H, W, "NHWC", dtype, md, vd, gd, bd, 1e-5, y)
    L.cgbn_frozen_backward(dyd, N, C, H, W, "NHWC", dtype, vd, gd, 1e-5, dx)
    torch.cuda.synchronize()
    y_ref = F.frozen_forward_ref(G.widen(x, dtype), fm, fv, gamma, beta, 1e-5, "NHWC")
    dx_ref = F.frozen_backward_ref(G.widen(dy, dtype), fv, gamma, 1e-5, "NHWC")
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert G.max_rel_err(G.to_host_f64(y, dtype), y_ref, G.rms(y_ref)) <= tol
    assert G.max_rel_err(G.to_host_f64(dx, dtype), dx_ref, G.rms(dx_ref)) <= tol
