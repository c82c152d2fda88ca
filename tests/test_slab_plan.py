"""Host-side planning of the column-slab kernels without a GPU: for thousands of seeded shapes the numbers the kernels
index by cover the matrix exactly, fit the registers, the LDS and the workspace, and push no workspace over the static
scratch."""

import numpy as np
import pytest

from paper_1711_07240_amd import cgbn as L

THREADS = 512
VARIANTS = {("sfwd", True): (4, 8, 10, 12, 20), ("sfwd", False): (6, 12, 18, 28, 36),
            ("sbwd", True): (4, 6, 8, 10, 12, 20), ("sbwd", False): (6, 9, 14, 18)}
NARROW = (8, 12, 16, 20, 28)                        # ... of those with 8-byte vectors
MAX_CHANNELS = 128
STATIC_SCRATCH = 16 << 20


def _check(shape):
    N, C, H, W, layout, dtype, K = shape
    vec = 4 if dtype == "f32" else 8
    taken = 0
    for d in ("sfwd", "sfwds", "sbwd", "sbwdm"):
        g = lambda k: L.cgbn_plan_get(*shape, f"{d}_{k}")
        if not g("ok"):
            continue
        taken += 1
        cols, vecs, cpc, nch, rpp, tpc, slabs, U, rpu, P, R = (g(k) for k in (
            "cols", "vecs", "cpc", "nch", "rpp", "tpc", "slabs", "U", "rpu", "P", "R"))
        if layout == "NHWC":
            assert cpc == 1 and R == N * H * W and vecs * vec == C
        else:
            assert cpc == H * W and R == N and vecs * vec == C * H * W
        # slabs cover the vectors, units cover the rows, none of them empty
        assert 1 <= cols <= THREADS and (slabs - 1) * cols < vecs <= slabs * cols
        assert (U - 1) * rpu < R <= U * rpu
        # a slab is whole channels; the padded channel count is a power of two the threads divide into
        assert cols * vec % cpc == 0 and cols * vec // cpc <= nch <= MAX_CHANNELS and nch & (nch - 1) == 0
        assert tpc & (tpc - 1) == 0 and 1 <= tpc <= 64 and tpc * nch <= THREADS
        # registers: a kernel variant with room for the unit's passes
        assert rpp == THREADS // cols and rpu <= rpp * P and P in VARIANTS[d[:4], U == 1]
        assert rpp * (C * (H * W if layout == "NCHW" else 1)) * (16 // vec) + cols * 16 < 2 ** 31
        if U > 1:
            assert U <= 256                                     # (the compute units of the planning host's default)
            # rows of two doubles a unit and channel, two pairs of results: in the rows and shard sums of the other kernels
            assert slabs * nch * (U + 1) * 16 <= 2 * sum(L.cgbn_plan_get(*shape, k) for k in ("part_bytes", "shard_bytes"))
            assert slabs * -(-U // 32) <= C and slabs <= C      # counters and bitmaps inside the sync area
            if slabs * U > 256:                                 # several rounds: slabs end on lines, or are many lines wide
                assert cols >= 48 or (cols % 8 == 0 and vecs * 16 % 128 == 0)
            else:                                               # one round: no more units than their passes need, in whole eights
                fewest = -(-R // (-(-rpu // rpp) * rpp))
                assert U <= (fewest if fewest < 8 else -(-fewest // 8) * 8)
    # the rows need at most a MiB, or as much again as the other kernels' rows while everything fits the static scratch
    rows = max(L.cgbn_plan_get(*shape, "rows"), *(L.cgbn_plan_get(*shape, f"{d}_rows") for d in ("fwd", "bwd")))
    part, own = L.cgbn_plan_get(*shape, "part_bytes"), -(-C * rows * 4 // 256) * 256
    assert part <= max(2 * own, 512 << 10)
    if part > max(own, 512 << 10):
        assert L.cgbn_workspace_bytes(*shape) <= STATIC_SCRATCH
    return taken


def _check_narrow(shape):
    """The plans with 8-byte vectors that stand in for those: one workgroup a slab, NCHW, for the same matrix."""
    N, C, H, W, layout, dtype, K = shape
    vec = 2 if dtype == "f32" else 4
    taken = 0
    for d in ("fwd", "fwds", "bwd", "bwdm"):
        g, wide = (lambda k: L.cgbn_plan_get(*shape, f"n{d}_{k}")), (lambda k: L.cgbn_plan_get(*shape, f"s{d}_{k}"))
        if not g("ok"):
            continue
        taken += 1
        cols, vecs, cpc, nch, rpp, tpc, slabs, U, rpu, P, R = (g(k) for k in (
            "cols", "vecs", "cpc", "nch", "rpp", "tpc", "slabs", "U", "rpu", "P", "R"))
        assert layout == "NCHW" and wide("ok") and cpc == H * W and R == rpu == N and U == 1
        assert vecs * vec == C * H * W and 1 <= cols <= THREADS and (slabs - 1) * cols < vecs <= slabs * cols and slabs <= C
        assert cols * vec == nch * H * W and nch <= MAX_CHANNELS and nch & (nch - 1) == 0
        assert tpc & (tpc - 1) == 0 and 1 <= tpc <= 64 and tpc * nch <= THREADS
        assert rpp == THREADS // cols and N <= rpp * P and P in NARROW and (P == 8 or N > rpp * NARROW[NARROW.index(P) - 1])
        assert rpp * C * H * W * (8 // vec) + cols * 8 < 2 ** 31
        # no more than half the compute units (of the planning host's default) had a workgroup, or a slab was several units and each is now one
        assert 2 * wide("slabs") <= 256 if wide("U") == 1 else slabs <= 256
    return taken


def _shapes(count, seed, layout):
    r = np.random.default_rng(seed)
    for _ in range(count):
        dtype = "f32" if r.random() < 0.5 else "bf16"
        N = int(np.exp(r.uniform(0, np.log(512))))
        C = int(np.exp(r.uniform(np.log(4), np.log(4096))))
        C = max(8, C // 8 * 8) if r.random() < 0.9 else C
        H, W = int(np.exp(r.uniform(0, np.log(260)))), int(np.exp(r.uniform(0, np.log(400))))
        if N * C * H * W <= 2 ** 33:
            K = int(r.choice([k for k in range(1, N + 1) if N % k == 0]))
            yield (N, C, H, W, layout, dtype, K)


@pytest.mark.parametrize("layout", ["NHWC", "NCHW"])
@pytest.mark.parametrize("seed", [1, 2])
def test_random_shapes(seed, layout):
    taken = narrow = 0
    for shape in _shapes(1200, seed, layout):
        try:
            taken += _check(shape)
            narrow += _check_narrow(shape)
        except AssertionError as e:
            raise AssertionError(f"{shape}: {e}") from e
    assert taken > (2400 if layout == "NHWC" else 1500)          # (four plans a shape)
    assert narrow == 0 if layout == "NHWC" else narrow > 600


def test_detector_layers():
    one = (2, 512, 25, 42, "NHWC", "bf16", 2)
    assert L.cgbn_plan_get(*one, "sfwd_U") == 1 and L.cgbn_plan_get(*one, "sbwd_U") == 1 and _check(one) == 4
    many = (16, 256, 50, 84, "NHWC", "bf16", 8)
    assert L.cgbn_plan_get(*many, "sfwd_U") > 1 and _check(many) == 4
    small = (35, 16, 14, 16, "NHWC", "f32", 35)                 # 62 full passes: every further unit only costs
    for d in ("sfwd", "sbwd"):
        assert 1 < L.cgbn_plan_get(*small, f"{d}_U") <= 64
    # a second tensor: float shortcuts in several rounds go to the sweeps, masked backwards of this many pixels to several units
    large = (10, 192, 161, 189, "NHWC", "f32", 2)
    assert L.cgbn_plan_get(*large, "sfwd_ok") == 1 and L.cgbn_plan_get(*large, "sfwds_ok") == 0
    shared = (17, 80, 90, 135, "NHWC", "f32", 1)                # slabs that share lines, the longest units
    assert L.cgbn_plan_get(*shared, "sfwd_P") == 36 and L.cgbn_plan_get(*shared, "sfwds_ok") == 0
    head = (28, 32, 9, 12, "NHWC", "f32", 4)
    assert L.cgbn_plan_get(*head, "sfwd_U") == 1 and L.cgbn_plan_get(*head, "sbwdm_U") > 1
    # 2700 to 3072 pixels are one workgroup a slab where no number of units takes them (more slabs than compute units, sharing lines)
    wide = (15, 3304, 4, 51, "NHWC", "f32", 3)
    assert all(L.cgbn_plan_get(*wide, f"{d}_ok") == 1 for d in ("sfwd", "sfwds", "sbwd", "sbwdm"))
    odd = (16, 250, 50, 84, "NHWC", "bf16", 8)                  # channels that are no whole vectors
    assert L.cgbn_plan_get(*odd, "sfwd_ok") == 0 and L.cgbn_plan_get(*odd, "sbwd_ok") == 0
