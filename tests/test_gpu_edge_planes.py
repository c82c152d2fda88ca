"""The single-launch NCHW kernels with 16-byte loads on planes that are no multiple of 16 bytes: every count of slots a plane, tiles and planes
that share a workgroup, both element types, planes that start at every byte a plane can start at, with and without a second tensor, and results
written over the inputs.  The plan says whether a call takes them; results against the float64 oracles, with the tolerances stated in gpu_harness.py."""

import os
import re

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from oracle import cgbn_relu_oracle as R
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

# N, C, H, W, dtype, K
CASES = [
    # a plane a wavefront: 2 to 38 slots, one to many planes a wavefront, further planes in LDS (N just beyond the registers' share)
    (2, 128, 23, 23, "bf16", 2), (5, 48, 25, 43, "bf16", 5), (3, 64, 41, 45, "bf16", 1), (41, 48, 35, 37, "bf16", 1), (33, 64, 37, 55, "bf16", 3),
    (17, 48, 37, 53, "bf16", 17), (25, 48, 47, 53, "bf16", 5), (2, 64, 53, 57, "bf16", 2), (4, 48, 61, 65, "bf16", 4), (5, 56, 71, 71, "bf16", 1),
    (3, 48, 77, 79, "bf16", 3), (2, 64, 87, 89, "bf16", 1), (2, 48, 99, 119, "bf16", 2), (3, 48, 121, 131, "bf16", 1), (2, 48, 125, 151, "bf16", 2),
    (3, 48, 67, 67, "f32", 3), (9, 48, 33, 33, "f32", 3), (25, 48, 35, 35, "f32", 5), (3, 56, 47, 49, "f32", 1), (2, 48, 51, 57, "f32", 2),
    (4, 48, 53, 75, "f32", 2), (2, 48, 71, 85, "f32", 1), (2, 48, 89, 91, "f32", 2), (2, 48, 91, 103, "f32", 1), (33, 48, 23, 27, "f32", 3),
    (65, 48, 29, 27, "f32", 5),
    # planes that share a workgroup: four, three, two; not a whole number of them
    (6, 64, 141, 145, "bf16", 3), (7, 48, 101, 199, "bf16", 7), (5, 64, 73, 137, "bf16", 5), (6, 96, 100, 127, "bf16", 2), (4, 64, 99, 101, "f32", 2),
    (3, 64, 101, 115, "f32", 1), (2, 64, 131, 133, "f32", 2), (5, 64, 71, 73, "f32", 5), (5, 64, 77, 79, "f32", 1), (9, 64, 85, 85, "f32", 3),
    (16, 96, 131, 131, "f32", 4),
    # tiles: the last one shorter, a few values long; channels that are no whole vectors together
    (2, 128, 251, 241, "bf16", 2), (1, 130, 301, 303, "bf16", 1), (4, 65, 205, 201, "f32", 2), (2, 129, 149, 151, "f32", 1), (1, 131, 185, 249, "f32", 1),
    (2, 256, 1, 45061, "f32", 1), (8, 72, 201, 219, "f32", 8),
    # slot counts that calls of those shapes leave to other kernels
    (16, 64, 53, 47, "bf16", 4), (20, 64, 63, 33, "bf16", 5), (34, 104, 25, 41, "bf16", 2), (33, 16, 25, 41, "f32", 3), (4, 16, 25, 41, "f32", 2),
    (10, 16, 29, 53, "f32", 5), (6, 24, 49, 37, "f32", 3), (3, 16, 61, 70, "bf16", 1), (2, 16, 66, 79, "bf16", 2), (3, 16, 98, 63, "bf16", 3), (2, 16, 74, 111, "bf16", 1),
    (2, 20, 143, 86, "bf16", 2),
]
# forwards with a shortcut that take these kernels only from 100 MB on: planes that share a workgroup, tiles, a plane a wavefront with its last slots in LDS
LARGE = [(3, 728, 93, 129, "f32", 1), (2, 1040, 83, 145, "f32", 1), (1, 557, 171, 263, "f32", 1), (3, 1336, 75, 113, "f32", 1)]
ID = lambda c: "%dx%dx%dx%d-%s-k%d" % c
DIRECTIONS = {"fwd": "efwd_taken", "fwds": "efwd_taken2", "bwd": "ebwd_taken", "bwdm": "ebwd_taken2"}


def _variant(case, d):
    """(slots per plane, LDS split) of the kernel a call takes, None if it takes another."""
    g = lambda k: L.cgbn_plan_get(*case[:4], "NCHW", *case[4:], k)
    if not g(DIRECTIONS[d]) or (g("s%s_ok" % d) and g("s%s_first" % d)):
        return None
    return g("e%s_LPPC" % d[:3]), g("e%s_big" % d[:3])


def _built():
    text = open(os.path.join(os.path.dirname(L.__file__), "csrc", "cgbn_fused_list.h")).read().replace("\\\n", " ")
    bodies = dict(re.findall(r"#define CGBN_FUSED_EDGE_(\w+)\(X\)(.*)", text))

    def pairs(name):
        nested = re.findall(r"CGBN_FUSED_EDGE_(\w+)\(X\)", bodies[name])
        return {(int(a), int(b)) for a, b in re.findall(r"X\((-?\d+), (\d)\)", bodies[name])}.union(*map(pairs, nested))

    return {"fwd": pairs("FORWARD"), "fwds": pairs("SHORTCUT"), "bwd": pairs("BACKWARD"), "bwdm": pairs("BACKWARD")}


def test_every_layout_of_a_plane_is_run():
    """Each variant of each direction; with the ordinary LDS split large planes run again below."""
    for d in DIRECTIONS:
        run = {_variant(case, d) for case in CASES + LARGE + FAR[:1]} - {None}
        assert run | {(0, 0), (-2, 0)} == _built()[d], (d, _built()[d] ^ run)


# calls that were slower than through the kernels that took them before (measured, 1.04 to 2.1 times), and the directions in question
SLOWER = [((77, 8, 329, 399, "f32", 1), "fwd fwds bwd bwdm"), ((74, 19, 109, 195, "bf16", 1), "fwd"), ((65, 23, 195, 106, "bf16", 1), "fwd"), ((20, 148, 109, 103, "bf16", 1), "bwd"),
          ((70, 201, 85, 139, "bf16", 1), "bwd"), ((58, 416, 29, 45, "bf16", 1), "fwd"), ((5, 80, 211, 315, "f32", 1), "fwds"), ((42, 66, 166, 163, "bf16", 1), "fwds"),
          ((15, 312, 43, 69, "bf16", 1), "fwds"), ((87, 48, 27, 45, "f32", 1), "bwd bwdm"), ((79, 172, 53, 21, "f32", 1), "fwd fwds bwd"), ((115, 9, 67, 126, "f32", 1), "fwd"),
          ((101, 8, 150, 213, "f32", 1), "fwd"), ((2, 51, 202, 214, "bf16", 1), "bwd bwdm"), ((8, 121, 122, 86, "bf16", 1), "bwd bwdm"), ((68, 8, 68, 131, "bf16", 1), "bwd bwdm"),
          ((1, 3200, 19, 31, "f32", 1), "bwdm"), ((5, 1556, 61, 66, "bf16", 1), "fwd fwds bwd"), ((57, 160, 54, 75, "bf16", 1), "fwd fwds bwd")]


def test_calls_that_other_kernels_are_faster_at_are_left_to_them():
    for case, directions in SLOWER:
        for d in directions.split():
            assert _variant(case, d) is None, (case, d)


def _inputs(case):
    N, C, H, W, dtype, K = case
    r = np.random.default_rng(N * 1000 + C + H)
    per = lambda a: a.reshape(1, -1, 1, 1)
    x = (r.standard_normal((N, C, H, W), dtype=np.float32) * per(r.uniform(0.5, 2, C)) + per(r.uniform(-2, 2, C))).astype(np.float32)
    dy, s = (r.standard_normal(x.shape, dtype=np.float32) for _ in range(2))
    if dtype == "bf16":
        x, dy, s = (synth.f32_to_bf16_bits(a) for a in (x, dy, s))
    return x, dy, s, r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)


def _run(case):
    L.cgbn_set_tuning("flat", 0)          # (small ones: else the flat kernels come first)
    try:
        _run_here(case)
    finally:
        L.cgbn_set_tuning("flat", 1)


def _run_here(case):
    N, C, H, W, dtype, K = case
    print("[case] planes with edges", case, flush=True)
    x, dy, s, gamma, beta = _inputs(case)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NCHW", dtype, K)
    error = L.cgbn_workspace_error_offset(N, C, H, W, "NCHW", dtype, K)

    def took(*directions):
        torch.cuda.synchronize()
        assert int(p.ws[error:error + 4].view(torch.int32).item()) == 0
        for d in directions:
            what = "forward" if d[0] == "f" else "backward"
            assert L.cgbn_get_tuning("last_%s_edge" % what) == (_variant(case, d) is not None), d
            assert not _variant(case, d) or L.cgbn_get_tuning("last_%s_fused" % what) == 1, d

    p.forward()
    p.backward()
    took("fwd", "bwd")
    wx, wdy = G.widen(x, dtype), G.widen(dy, dtype)
    scale = np.sqrt(N * H * W) * G.rms(wdy)           # a channel's sums of gradients: judged on the size they have when nothing cancels
    plain = p.results()
    G.check_against_oracle(plain, O.cgbn_forward_backward_ref(wx, wdy, gamma, beta, 1e-5, "NCHW"), dtype, str(case), sum_scale=scale)
    sd, dz = G.to_dev(s), torch.empty_like(p.x)
    L.cgbn_forward_relu(p.x, sd, *p.shape_args, "NCHW", K, p.gamma, p.beta, 1e-5, p.y, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
    L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args, "NCHW", K, dtype, p.mean_lo, p.ws)
    took("fwds", "bwdm")
    got = p.results()
    y, mean, invstd = R.cgbn_relu_forward_ref(wx, gamma, beta, 1e-5, "NCHW", G.widen(s, dtype))[:3]
    dx, dgamma, dbeta, dzr = R.cgbn_relu_backward_ref(wdy, got["y"], wx, mean, invstd, gamma, "NCHW")[:4]      # (masked by the stored output)
    G.check_against_oracle(got, dict(y=y, mean=mean, invstd=invstd, dx=dx, dgamma=dgamma, dbeta=dbeta), dtype, str(case), sum_scale=scale)
    assert np.array_equal(G.to_host_f64(dz, dtype), dzr)
    # y over the shortcut, dx over the output it is masked by: the same bits
    kept = p.y.clone()
    L.cgbn_forward_relu(p.x, sd, *p.shape_args, "NCHW", K, p.gamma, p.beta, 1e-5, sd, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
    L.cgbn_backward_relu(p.dy, kept, p.x, p.mean, p.invstd, p.gamma, kept, dz, p.dgamma, p.dbeta, *p.shape_args, "NCHW", K, dtype, p.mean_lo, p.ws)
    torch.cuda.synchronize()
    assert torch.equal(sd, p.y) and torch.equal(kept, p.dx)
    # dx over dy, y over x
    p.forward()
    p.backward(dx=p.dy)
    p.forward(y=p.x)
    torch.cuda.synchronize()
    assert np.array_equal(G.to_host_f64(p.dy, dtype), plain["dx"]) and np.array_equal(G.to_host_f64(p.x, dtype), plain["y"])


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=ID)
def test_against_the_oracle(case):
    _run(case)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(6, 64, 141, 145, "bf16", 3), (2, 64, 131, 133, "f32", 2), (2, 128, 251, 241, "bf16", 2), (4, 65, 205, 201, "f32", 2)], ids=ID)
def test_with_the_ordinary_lds_split(case):
    L.cgbn_set_tuning("big_lds", 0)
    try:
        _run(case)
    finally:
        L.cgbn_set_tuning("big_lds", 1)


# images so large that a unit's planes lie further apart than 32 bits reach: planes that share a workgroup forward (four, three) and backward (three)
FAR = [(4, 40000, 99, 101, "f32", 1), (4, 40000, 141, 141, "bf16", 1), (3, 60000, 151, 151, "bf16", 1), (3, 80000, 81, 85, "f32", 1), (3, 80000, 117, 119, "bf16", 1)]


def test_planes_further_apart_than_32_bits():
    """Where a unit's last plane begins, formed as the kernels form it, is that many images on."""
    far = 0
    r = np.random.default_rng(5)
    cases = FAR + [(int(r.integers(2, 7)), int(r.integers(20000, 90000)), int(r.integers(60, 160)), int(r.integers(60, 160)), t, 1) for t in ("f32", "bf16") for _ in range(200)]
    for case in cases:
        N, C, H, W, dtype, _ = case
        image = C * H * W * (4 if dtype == "f32" else 2)
        for d in ("fwd", "bwd", "efwd", "ebwd"):
            g = lambda k: L.cgbn_plan_get(N, C, H, W, "NCHW", dtype, 1, d + "_" + k)
            if g("ok") == 1:
                planes = 1 if g("LPPC") == 0 else g("IPU") if g("LPPC") > 0 else -g("LPPC")
                assert g("last_plane") == (planes - 1) * image, (case, d)
                far += d[0] == "e" and g("last_plane") + image > 2 ** 32
                if g("LPPC") > 0:
                    assert planes * image < 2 ** 31
    assert far > 20 and all(any(_variant(c, d) for d in DIRECTIONS) for c in FAR)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [FAR[0], FAR[3]] + LARGE, ids=ID)
def test_planes_further_apart_than_32_bits_on_the_device(case):
    """(And large calls.)  Every value of every output against plain torch in float64, some channels at a time."""
    N, C, H, W, dtype, K = case
    print("[case] planes far apart", case, flush=True)
    gen = torch.Generator(device=G.DEV).manual_seed(9)
    x, dy, s = (torch.empty(N, C, H, W, device=G.DEV).normal_(generator=gen) for _ in range(3))
    per = lambda: torch.empty(C, device=G.DEV)
    gamma, beta = per().uniform_(0.5, 1.5, generator=gen), per().normal_(generator=gen)
    mean, invstd, mean_lo, dgamma, dbeta = (per() for _ in range(5))
    out, dz = torch.full_like(x, 7.0), torch.full_like(x, 7.0)
    ws = torch.empty(L.cgbn_workspace_bytes(N, C, H, W, "NCHW", dtype, K), dtype=torch.uint8, device=G.DEV)
    col = lambda t, c: t[c].double().view(1, -1, 1, 1)
    sums = lambda t: t.flatten(2).sum(2).sum(0)
    chunks = [slice(c, c + 1000) for c in range(0, C, 1000)]

    def worst(got, want):                       # (NaN: fails too)
        e = float((got.double() - want).abs().max())
        assert e <= 1e-4, (case, e)

    stats = {}
    for shortcut in (None, s):
        if shortcut is None:
            L.cgbn_forward(x, N, C, H, W, "NCHW", K, gamma, beta, 1e-5, out, mean, invstd, dtype, mean_lo, ws)
        else:
            L.cgbn_forward_relu(x, shortcut, N, C, H, W, "NCHW", K, gamma, beta, 1e-5, out, mean, invstd, dtype, mean_lo, ws)
        assert L.cgbn_get_tuning("last_forward_edge") == (_variant(case, "fwd" if shortcut is None else "fwds") is not None)
        for c in chunks:
            a = x[:, c].double()
            m = sums(a) / (N * H * W)
            a -= m.view(1, -1, 1, 1)
            i = 1 / torch.sqrt(sums(a * a) / (N * H * W) + 1e-5)
            worst(mean[c], m)
            worst(invstd[c], i)
            a = a * i.view(1, -1, 1, 1) * col(gamma, c) + col(beta, c)
            worst(out[:, c], a if shortcut is None else (a + shortcut[:, c].double()).clamp_(min=0))
            stats[c.start] = (m, i)
    y = out.clone()
    for masked in (False, True):
        out.fill_(7.0)
        if masked:
            L.cgbn_backward_relu(dy, y, x, mean, invstd, gamma, out, dz, dgamma, dbeta, N, C, H, W, "NCHW", K, dtype, mean_lo, ws)
        else:
            L.cgbn_backward(dy, x, mean, invstd, gamma, out, dgamma, dbeta, N, C, H, W, "NCHW", K, dtype, mean_lo, ws)
        assert L.cgbn_get_tuning("last_backward_edge") == (_variant(case, "bwdm" if masked else "bwd") is not None)
        for c in chunks:
            m, i = (v.view(1, -1, 1, 1) for v in stats[c.start])
            g, h = dy[:, c].double(), (x[:, c].double() - m) * i
            if masked:
                g *= y[:, c] > 0
                assert torch.equal(dz[:, c].double(), g)
            db, dg = sums(g), sums(g * h)
            root = (N * H * W) ** 0.5
            worst(dbeta[c] / root, db / root)
            worst(dgamma[c] / root, dg / root)
            worst(out[:, c], (g - (db / root ** 2).view(1, -1, 1, 1) - h * (dg / root ** 2).view(1, -1, 1, 1)) * i * col(gamma, c))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_the_plan_holds_every_plane(dtype):
    """Slots hold the whole vectors of a plane wherever it starts, the slots read without a look are full, rows fit what the workspace has, and the calls
    taken are no multiple of 16 bytes."""
    r = np.random.default_rng(3)
    eb, taken = (4 if dtype == "f32" else 2), 0
    for _ in range(4000):
        N, C = int(r.integers(1, 200)), int(r.choice([8, 16, 24, 48, 64, 100, 256, 1024, 1027]))
        H, W = int(np.exp(r.uniform(2.5, 6))), int(np.exp(r.uniform(2.5, 6)))
        K = int(r.choice([k for k in range(1, N + 1) if N % k == 0]))
        shape = (N, C, H, W, "NCHW", dtype, K)
        plane = H * W * eb
        for d, words in (("efwd", 128), ("ebwd", 64)):
            g = lambda k: L.cgbn_plan_get(*shape, d + "_" + k)
            if not g("ok"):
                assert not g("taken") and not g("taken2")
                continue
            assert plane % 16 != 0 and plane > 1024 and g("LB") == 16
            taken += g("taken") + g("taken2")
            lppc, big, regs = g("LPPC"), g("big"), words // 4
            lds = {0: 24, 1: 48, 2: 44}[big] * words // 128 // 4
            assert g("rows") * C * 4 <= L.cgbn_plan_get(*shape, "part_bytes")
            if lppc:
                assert C * plane % 16 == 0                               # a channel's planes start at the same byte of a vector
            # whole vectors in a plane, by where it starts; 16 k of it more than those need not be there
            most = max((plane - h) // 16 for h in range(0, 16, eb))
            least = min((plane - h) // 16 for h in range(0, 16, eb))
            if lppc > 0:
                full = 0 if lppc <= 2 else max(c for c in (2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32) if c < lppc)
                full = regs if lppc > regs else full if full * 16 >= regs else 0
                assert full * 64 <= least and most <= lppc * 64
                per_wave = 1 if lppc > regs else regs // lppc + (lds // lppc if big == 2 else 0)
                assert g("IPU") <= 4 * per_wave and g("U") * g("IPU") >= N > (g("U") - 1) * g("IPU")
                assert lppc <= regs + (lds if lppc > regs else 0)
            elif lppc < 0:
                assert most <= (regs + lds) // -lppc * 256 and g("U") == -(-N // -lppc)
            else:
                assert g("TL") * eb <= (regs + lds) * 4096 and g("tp") * g("TL") >= H * W > (g("tp") - 1) * g("TL") and g("U") == N * g("tp")
    assert taken > 1500


def errors(case, knob):
    """Root mean squares over channels and four inputs of how far mean (with its rest), dbeta and dgamma are from 64 bits, by (which, the knob's value)."""
    N, C, H, W, dtype, K = case
    gen = torch.Generator(device=G.DEV).manual_seed(31)
    T = torch.float32 if dtype == "f32" else torch.bfloat16
    per, col = lambda: torch.empty(C, device=G.DEV), lambda v: v.view(1, -1, 1, 1)
    ws = torch.empty(L.cgbn_workspace_bytes(N, C, H, W, "NCHW", dtype, K), dtype=torch.uint8, device=G.DEV)
    off = {}
    for _ in range(4):
        rnd = lambda: torch.empty(N, C, H, W, device=G.DEV).normal_(generator=gen)
        x = (rnd() * col(per().uniform_(0.5, 2, generator=gen)) + col(per().uniform_(-2, 2, generator=gen))).to(T)
        dy, out = rnd().to(T), torch.empty_like(x)
        gamma, beta, mean, invstd, mean_lo, dgamma, dbeta = (torch.ones(C, device=G.DEV) for _ in range(7))
        xd, gd = x.double(), dy.double()
        sums = lambda t: t.sum((0, 2, 3))
        m = sums(xd) / (N * H * W)
        sigma = torch.sqrt(sums((xd - col(m)) ** 2) / (N * H * W))
        h = gd * (xd - col(m)) * col(1 / torch.sqrt(sigma ** 2 + 1e-5))
        want = {"mean": (m, sigma), "dbeta": (sums(gd), torch.sqrt(sums(gd * gd))), "dgamma": (sums(h), torch.sqrt(sums(h * h)))}
        for value in (0, 1):
            L.cgbn_set_tuning(knob, value)
            try:
                L.cgbn_forward(x, N, C, H, W, "NCHW", K, gamma, beta, 1e-5, out, mean, invstd, dtype, mean_lo, ws)
                L.cgbn_backward(dy, x, mean, invstd, gamma, out, dgamma, dbeta, N, C, H, W, "NCHW", K, dtype, mean_lo, ws)
            finally:
                L.cgbn_set_tuning(knob, 1)
            for k, got in {"mean": mean.double() + mean_lo.double(), "dbeta": dbeta.double(), "dgamma": dgamma.double()}.items():
                off.setdefault((k, value), []).append((((got - want[k][0]) / want[k][1]) ** 2).mean())
    return {k: float(torch.stack(v).mean().sqrt()) for k, v in off.items()}


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2, 128, 251, 241, "bf16", 1), (6, 64, 141, 145, "bf16", 1), (8, 72, 201, 219, "f32", 1), (13, 88, 113, 149, "f32", 1)], ids=ID)
def test_no_further_from_64_bits_than_the_sweeps(case):
    """A row of these kernels is as long as several of the sweeps', so what is rounded once a row has to be formed more carefully.  (Measured with a first value as pivot and sums joined in float: mean 1.4 to
    2.0 times as far off as the sweeps, dbeta 1.1 to 1.2; now 0.3 to 0.7 and 0.6 to 0.8.  A ratio of two such root mean squares is good to 6 %.)"""
    print("[case] errors", case, flush=True)
    assert any(_variant(case, d) for d in ("fwd", "bwd"))
    rms = errors(case, "fused")
    for k in ("mean", "dbeta", "dgamma"):
        if _variant(case, "fwd" if k == "mean" else "bwd"):
            assert rms[k, 1] <= rms[k, 0], (case, k, rms)


@pytest.mark.gpu
def test_pivots_of_channels_without_a_finite_mean_or_near_the_largest_float():
    """The pivot is a mean over 16 values of the channel's first plane: infinities and NaN among them stay in their channel, where results are finite as the
    sweeps' are, and values near the largest float do not overflow it."""
    N, C, H, W = 8, 72, 201, 219
    r = np.random.default_rng(6)
    x = r.standard_normal((N, C, H, W), dtype=np.float32)
    at = 5 * H * W // 16                                  # one of the 16, not the first
    x[0, 3].flat[at], x[0, 4].flat[at], x[0, 5].flat[0], x[2, 6, 7, 8], x[:, 7] = np.inf, np.nan, -np.inf, np.inf, 3.3e38
    p = G.Problem(x, x, np.ones(C, np.float32), np.zeros(C, np.float32), 1e-5, "NCHW", "f32", 1)
    assert _variant((N, C, H, W, "f32", 1), "fwd")
    got = []
    for fused in (0, 1):
        L.cgbn_set_tuning("fused", fused)
        try:
            p.forward()
            got.append(p.results())
        finally:
            L.cgbn_set_tuning("fused", 1)
    sweeps, here = got
    assert here["mean"][3] == np.inf and np.isnan(here["mean"][4]) and np.isfinite(here["mean"][7]) and abs(here["mean"][7] / 3.3e38 - 1) < 1e-6
    for k in ("mean", "invstd"):
        assert np.array_equal(np.isfinite(here[k]), np.isfinite(sweeps[k])), k
    assert np.array_equal(np.isfinite(here["y"]).all((0, 2, 3)), np.isfinite(sweeps["y"]).all((0, 2, 3)))
    assert np.isfinite(here["y"]).all((0, 2, 3)).sum() == C - 4
