"""Column-slab kernels in several rounds of slabs that share lines: which calls are planned so and how they are cut (CPU), and results against the
float64 oracles, with the tolerances stated in gpu_harness.py: a last slab of few vectors, a last round that is not full, a last unit that is short,
units that stop waiting."""

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from oracle import cgbn_relu_oracle as R
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

# N, H, W, C, dtype: (64 slabs of eight columns, the last of two vectors), ...
CASES = [(64, 8, 12, 2024, "f32"), (43, 12, 19, 2000, "f32"), (41, 17, 17, 1672, "f32"), (128, 6, 17, 1168, "f32"), (256, 12, 12, 680, "bf16"), (31, 25, 31, 936, "bf16"),
         (8, 32, 32, 1864, "f32"), (64, 13, 22, 1816, "bf16")]
# channels-last calls, N, H, W, C, that are faster as sweeps (measured, 1.04 to 1.2 times), and the directions in question
SLOWER = [((8, 56, 84, 2064, "f32"), "xfwd xbwd"), ((1, 195, 135, 2040, "f32"), "xfwd xbwd xbwdm"), ((36, 48, 26, 1016, "f32"), "xbwd"), ((2, 253, 143, 920, "f32"), "xbwd"), ((1, 118, 164, 2032, "bf16"), "xbwd"), ((36, 35, 35, 216, "f32"), "xbwd"),
          ((49, 32, 34, 168, "f32"), "xbwd"), ((9, 52, 92, 728, "f32"), "xfwd"), ((1, 179, 262, 840, "bf16"), "xfwd xbwd"), ((3, 146, 201, 880, "f32"), "xfwd")]
DIRECTIONS = ("xfwd", "xbwd", "xbwdm")
ID = lambda c: "%dx%dx%dx%d-%s" % c


def _get(case, key):
    N, H, W, C, dtype = case
    return L.cgbn_plan_get(N, C, H, W, "NHWC", dtype, 1, key)


def test_every_direction_is_run():
    for d in DIRECTIONS:
        assert sum(_get(c, d + "_ok") for c in CASES) >= 2, d
    assert all(_get(c, "xfwds_ok") == -1 for c in CASES)          # (no such plan for a forward with a shortcut)
    assert any(_get(c, "xbwd_cols") * _get(c, "xbwd_slabs") > _get(c, "xbwd_vecs") for c in CASES)


def test_calls_that_sweeps_are_faster_at_are_left_to_them():
    for case, directions in SLOWER:
        for d in directions.split():
            assert _get(case, d + "_ok") == 0, (case, d)


def test_plans():
    r = np.random.default_rng(12)
    taken = 0
    for _ in range(3000):
        dtype = "f32" if r.random() < 0.5 else "bf16"
        vec, C = (4 if dtype == "f32" else 8), 8 * int(np.exp(r.uniform(1, np.log(400))))
        N, H, W = int(2 ** r.integers(0, 9)), int(np.exp(r.uniform(1, 5.3))), int(np.exp(r.uniform(1, 5.3)))
        if N * C * H * W > 2 ** 30:
            continue
        shape = (N, C, H, W, "NHWC", dtype, 1)
        for d in DIRECTIONS:
            g = lambda k: L.cgbn_plan_get(*shape, d + "_" + k)
            if not g("ok"):
                continue
            taken += 1
            assert not L.cgbn_plan_get(*shape, "s" + d[1:] + "_ok")
            U, slabs, cols, vecs, rpu, Rows, nch = (g(k) for k in ("U", "slabs", "cols", "vecs", "rpu", "R", "nch"))
            assert cols == 8 and vecs * vec == C and vecs >= 24 and (slabs - 1) * cols < vecs <= slabs * cols and vecs * 16 % 128 != 0
            assert U % 8 == 0 and (U - 1) * rpu < Rows <= U * rpu and Rows == N * H * W
            assert rpu <= g("rpp") * g("P") and g("P") in ((6, 12, 18, 28, 36) if d == "xfwd" else (6, 9, 14, 18))
            flight = 256 // U                        # (the planning host's default)
            assert flight >= (6 if d == "xfwd" else 5 if dtype == "bf16" else 8 if d == "xbwdm" and vecs <= 256 else 4)
            assert slabs > flight and 10 * slabs >= 7 * -(-slabs // flight) * flight
            if vecs <= 256:                          # one tile of the sweeps: by how full the rounds are
                full = {"xfwd": 71 if flight >= 8 else 91, "xbwd": 81, "xbwdm": 78} if dtype == "bf16" else {"xfwd": 80, "xbwd": 84, "xbwdm": 0}
                assert 100 * slabs > full[d] * -(-slabs // flight) * flight
            assert slabs * nch * (U + 1) * 16 <= 2 * sum(L.cgbn_plan_get(*shape, k) for k in ("part_bytes", "shard_bytes"))
            assert slabs * -(-U // 32) <= C
    assert taken > 60


@pytest.mark.gpu
@pytest.mark.parametrize("spin_limit", [None, 0], ids=["", "units-that-stop-waiting"])
@pytest.mark.parametrize("case", CASES, ids=ID)
def test_against_the_oracle(case, spin_limit):
    N, H, W, C, dtype = case
    print("[case] shared lines", case, spin_limit, flush=True)
    r = np.random.default_rng(C)
    x = (r.standard_normal((N, H, W, C), dtype=np.float32) * r.uniform(0.5, 2, C) + r.uniform(-2, 2, C)).astype(np.float32)
    dy = r.standard_normal(x.shape, dtype=np.float32)
    if dtype == "bf16":
        x, dy = (synth.f32_to_bf16_bits(a) for a in (x, dy))
    gamma, beta = r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NHWC", dtype, 1)
    error = L.cgbn_workspace_error_offset(N, C, H, W, "NHWC", dtype, 1)
    old = L.cgbn_get_tuning("spin_limit")
    if spin_limit is not None:
        L.cgbn_set_tuning("spin_limit", spin_limit)
    try:
        p.forward()
        p.backward()
        torch.cuda.synchronize()
        for d, what in (("xfwd", "forward"), ("xbwd", "backward")):
            assert not _get(case, d + "_ok") or L.cgbn_get_tuning("last_%s_slab" % what) == 1
        assert int(p.ws[error:error + 4].view(torch.int32).item()) == 0
        wx, wdy = G.widen(x, dtype), G.widen(dy, dtype)
        scale = np.sqrt(N * H * W) * G.rms(wdy)       # a channel's sums of gradients: judged on the size they have when nothing cancels
        G.check_against_oracle(p.results(), O.cgbn_forward_backward_ref(wx, wdy, gamma, beta, 1e-5, "NHWC"), dtype, str(case), sum_scale=scale)
        L.cgbn_forward_relu(p.x, None, *p.shape_args, "NHWC", 1, p.gamma, p.beta, 1e-5, p.y, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
        L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, None, p.dgamma, p.dbeta, *p.shape_args, "NHWC", 1, dtype, p.mean_lo, p.ws)
        got = p.results()
        assert not _get(case, "xbwdm_ok") or L.cgbn_get_tuning("last_backward_slab") == 1
        assert int(p.ws[error:error + 4].view(torch.int32).item()) == 0
        y, mean, invstd = R.cgbn_relu_forward_ref(wx, gamma, beta, 1e-5, "NHWC")[:3]
        dx, dgamma, dbeta = R.cgbn_relu_backward_ref(wdy, got["y"], wx, mean, invstd, gamma, "NHWC")[:3]      # (masked by the stored output)
        G.check_against_oracle(got, dict(y=y, mean=mean, invstd=invstd, dx=dx, dgamma=dgamma, dbeta=dbeta), dtype, str(case), sum_scale=scale)
    finally:
        L.cgbn_set_tuning("spin_limit", old)
