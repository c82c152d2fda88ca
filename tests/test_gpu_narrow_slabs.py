"""Column-slab kernels with 8-byte vectors (NCHW, small planes): ragged slabs and passes, against the float64 oracles with
the tolerances stated in gpu_harness.py; and their plans, on the host alone.  Some of the shapes have such a plan but take the single-launch
kernels, which are faster there; every variant is run in test_gpu_slab_variants.py."""

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from oracle import cgbn_relu_oracle as R
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

# N, C, H, W, dtype, vectors a thread: forward, backward
CASES = [
    (5, 16, 5, 7, "bf16", 8, 8),
    (16, 256, 13, 21, "bf16", 16, 16),
    (24, 48, 9, 15, "bf16", 8, 8),
    (11, 64, 16, 31, "bf16", 12, 12),         # a row a pass, columns nearly as many as threads
    (9, 24, 1, 3, "bf16", 8, 8),              # several channels a vector column
    (81, 128, 3, 5, "bf16", 8, 8),
    (256, 1024, 7, 7, "bf16", 28, 28),        # instead of two units a slab
    (250, 1000, 7, 7, "bf16", 28, 28),
    (190, 40, 7, 7, "bf16", 20, 20),
    (113, 120, 7, 9, "f32", 16, 16),
    (91, 216, 7, 7, "f32", 12, 12),
    (19, 32, 10, 25, "f32", 12, 12),
    (53, 40, 6, 7, "f32", 8, 8),
]
THREADS = 512
ID = lambda c: "%dx%dx%dx%d-%s" % c[:5]


@pytest.mark.parametrize("case", CASES, ids=ID)
def test_plan(case):
    N, C, H, W, dtype, pf, pb = case
    vec = 2 if dtype == "f32" else 4
    for d, P in (("nfwd", pf), ("nbwd", pb), ("nfwds", pf), ("nbwdm", pb)):
        g = lambda k: L.cgbn_plan_get(N, C, H, W, "NCHW", dtype, 1, d + "_" + k)
        if d == "nbwdm" and dtype == "f32" and P > 8:
            assert g("ok") == 0                   # (16-byte vectors are faster)
            continue
        assert g("ok") == 1 and g("U") == 1 and g("P") == P
        cols, vecs, slabs, nch, rpp, tpc = (g(k) for k in ("cols", "vecs", "slabs", "nch", "rpp", "tpc"))
        assert vecs * vec == C * H * W and 1 <= cols <= THREADS and (slabs - 1) * cols < vecs <= slabs * cols and slabs <= C
        assert cols * vec == nch * H * W and nch & (nch - 1) == 0 and tpc & (tpc - 1) == 0 and tpc * nch <= THREADS and tpc <= 64
        assert rpp == THREADS // cols and N <= rpp * P


def _draw(N, C, H, W, dtype):
    r = np.random.default_rng(N * 1000 + C)
    x = (r.standard_normal((N, C, H, W)) * r.uniform(0.5, 2, C).reshape(1, -1, 1, 1) + r.uniform(-2, 2, C).reshape(1, -1, 1, 1)).astype(np.float32)
    dy, s = (r.standard_normal(x.shape).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        x, dy, s = (synth.f32_to_bf16_bits(a) for a in (x, dy, s))
    return x, dy, s, r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)


def _took(case, forward, backward):
    """The kernels with 8-byte vectors ran wherever their plan stands and does not come behind the single-launch kernels."""
    g = lambda k: L.cgbn_plan_get(*case[:4], "NCHW", case[4], 1, k)
    for way, d in (("forward", forward), ("backward", backward)):
        slab = g("s%s_first" % d) or not g(d[:3] + "_ok")
        assert L.cgbn_get_tuning("last_%s_slab_vector" % way) == (0 if not slab else 8 if g("n%s_ok" % d) else 16)


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=ID)
def test_forward_backward(case):
    N, C, H, W, dtype = case[:5]
    print("[case] narrow", case, flush=True)
    x, dy, s, gamma, beta = _draw(N, C, H, W, dtype)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NCHW", dtype, 1)
    p.forward()
    p.backward()
    _took(case, "fwd", "bwd")
    wx, wdy = G.widen(x, dtype), G.widen(dy, dtype)
    sums = dict(sum_scale=np.sqrt(N * H * W) * G.rms(wdy))
    G.check_against_oracle(p.results(), O.cgbn_forward_backward_ref(wx, wdy, gamma, beta, 1e-5, "NCHW"), dtype, str(case), **sums)
    sd, y, dz = G.to_dev(s), torch.empty_like(p.x), torch.empty_like(p.x)
    L.cgbn_forward_relu(p.x, sd, *p.shape_args, "NCHW", 1, p.gamma, p.beta, 1e-5, y, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
    L.cgbn_backward_relu(p.dy, y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args, "NCHW", 1, dtype,
                         p.mean_lo, p.ws)
    _took(case, "fwds", "bwdm")
    torch.cuda.synchronize()
    y_ref, mean, invstd = R.cgbn_relu_forward_ref(wx, gamma, beta, 1e-5, "NCHW", G.widen(s, dtype))
    wy = G.to_host_f64(y, dtype)
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert np.max(np.abs(wy - y_ref) / (1.0 if dtype == "f32" else np.maximum(np.abs(y_ref), G.rms(y_ref)))) <= tol
    # (the mask is read off the stored output, so the oracle is handed the same)
    dx, dgamma, dbeta, dz_ref = R.cgbn_relu_backward_ref(wdy, wy, wx, mean, invstd, gamma, "NCHW")
    assert np.array_equal(G.to_host_f64(dz, dtype), dz_ref)
    assert G.max_rel_err(G.to_host_f64(p.dx, dtype), dx, G.rms(dx)) <= tol
    for got, want in ((p.dgamma, dgamma), (p.dbeta, dbeta)):
        assert G.max_rel_err(got.cpu().numpy(), want, max(G.rms(want), sums["sum_scale"])) <= tol


@pytest.mark.gpu
def test_in_place():
    """y over x, dx over dy: a workgroup holds all it reads before it writes."""
    N, C, H, W, dtype = CASES[1][:5]
    x, dy, s, gamma, beta = _draw(N, C, H, W, dtype)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NCHW", dtype, 1)
    p.forward()
    p.backward()
    _took(CASES[1], "fwd", "bwd")
    y, dx = p.y.clone(), p.dx.clone()
    p.backward(dx=p.dy)
    p.forward(y=p.x)
    torch.cuda.synchronize()
    assert torch.equal(p.x, y) and torch.equal(p.dy, dx)
