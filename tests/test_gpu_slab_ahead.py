"""Column-slab backward over several rounds: with one slab in flight the next unit's first two passes are fetched ahead, with more
all the passes there is room for.  How far is fetched ahead changes no sum, so every launch gives the same bits."""

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype,C,N,H,W", [("bf16", 2048, 4, 50, 50), ("f32", 1024, 4, 50, 50), ("bf16", 2560, 4, 43, 50), ("f32", 1152, 4, 48, 51)])
def test_one_and_more_slabs_in_flight(dtype, C, N, H, W, masked):
    print("[case] slab ahead", dtype, C, N, H, W, masked, flush=True)
    r = np.random.default_rng(C + H)
    x = (r.standard_normal((N, H, W, C)) * r.uniform(0.5, 2, C) + r.uniform(-2, 2, C)).astype(np.float32)
    dy = r.standard_normal((N, H, W, C)).astype(np.float32)
    if dtype == "bf16":
        x, dy = synth.f32_to_bf16_bits(x), synth.f32_to_bf16_bits(dy)
    gamma, beta = r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NHWC", dtype, 1)
    plan = lambda k: L.cgbn_plan_get(N, C, H, W, "NHWC", dtype, 1, ("sbwdm_" if masked else "sbwd_") + k)
    U, slabs = plan("U"), plan("slabs")
    assert plan("ok") and U > 1 and slabs > 3 and plan("P") >= 14
    p.forward()
    y = torch.clone(p.y)                      # stored outputs of either sign: the mask
    ref = O.cgbn_forward_backward_ref(G.widen(x, dtype), G.widen(dy, dtype), gamma, beta, 1e-5, "NHWC")
    got = []
    try:
        for groups in (0, U, 2 * U, 3 * U):
            L.cgbn_set_tuning("fused_groups", groups)
            p.dx.zero_()
            if masked:
                L.cgbn_backward_relu(p.dy, y, p.x, p.mean, p.invstd, p.gamma, p.dx, None, p.dgamma, p.dbeta, *p.shape_args, "NHWC", 1, dtype,
                                     p.mean_lo, p.ws)
            else:
                p.backward()
            torch.cuda.synchronize()
            assert L.cgbn_get_tuning("last_backward_slab") == 1
            got.append([t.clone() for t in (p.dx, p.dgamma, p.dbeta)])
    finally:
        L.cgbn_set_tuning("fused_groups", 0)
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    if not masked:
        G.check_against_oracle(p.results(), ref, dtype, "%dx%dx%dx%d %s" % (N, H, W, C, dtype))
