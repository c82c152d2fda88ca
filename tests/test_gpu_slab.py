"""The column-slab kernels (one launch per direction, units of whole rows kept in registers) at the sizes where their cut
changes: remainders of rows, passes, slabs and vectors, the edges of the kernel variants, one and several units per slab,
several rounds of units, and units that stop waiting for their siblings.  Against the float64 oracle, with the tolerances of
gpu_harness.check_against_oracle (their derivation is there)."""

import dataclasses

import numpy as np
import pytest
import torch

import gpu_harness as G
from oracle import cgbn_oracle as O
from oracle import cgbn_relu_oracle as R
from paper_1711_07240_amd import cgbn as L
from paper_1711_07240_amd import synth

pytestmark = pytest.mark.gpu

BASE = synth.WORKLOADS["cfg1"]

# (what it is for, shape): N, C, H, W, K, layout, dtype; the units per slab of the plan with 16-byte vectors (1 or "several").  (NCHW with one unit:
# most of these take 8-byte vectors in its place; every variant of either is in test_gpu_slab_variants.py.)
SHAPES = [
    ("one-row", (1, 8, 1, 1, 1, "NHWC", "bf16"), 1),
    ("one-vector-ragged-pass", (1, 4, 5, 103, 1, "NHWC", "f32"), 1),
    ("4-passes-exactly", (4, 16, 16, 16, 2, "NHWC", "bf16"), 1),
    ("5-passes-ragged-slab", (5, 40, 15, 14, 5, "NHWC", "bf16"), 1),
    ("12-passes-exactly", (3, 24, 32, 32, 3, "NHWC", "f32"), 1),
    ("10-passes-exactly", (2, 16, 40, 32, 2, "NHWC", "bf16"), 1),
    ("slabs-of-two-vectors-ragged", (2, 1028, 20, 33, 2, "NHWC", "f32"), 1),
    ("most-rows-one-unit-forward", (2, 16, 40, 64, 1, "NHWC", "f32"), 1),
    ("first-rows-of-several-units", (1, 64, 53, 97, 1, "NHWC", "bf16"), "several"),
    ("narrow-c16", (7, 16, 45, 31, 7, "NHWC", "bf16"), "several"),
    ("5-vector-slab", (3, 40, 60, 70, 3, "NHWC", "bf16"), "several"),
    ("9-vector-slab", (2, 72, 75, 61, 2, "NHWC", "bf16"), "several"),
    ("two-uneven-slabs", (4, 68, 50, 41, 4, "NHWC", "f32"), "several"),
    ("ragged-last-slab-many-units", (2, 136, 110, 101, 1, "NHWC", "bf16"), "several"),
    ("full-lines-f32", (16, 64, 23, 29, 8, "NHWC", "f32"), "several"),
    ("longest-units", (1, 512, 100, 170, 1, "NHWC", "bf16"), "several"),
    ("planes-of-one", (64, 24, 1, 1, 8, "NCHW", "bf16"), 1),
    ("planes-of-two-vectors-of-channels", (40, 1024, 2, 1, 4, "NCHW", "f32"), 1),
    ("planes-of-9-doubled-slab", (30, 24, 3, 3, 3, "NCHW", "f32"), 1),
    ("planes-of-49-ragged-slab", (37, 40, 7, 7, 37, "NCHW", "bf16"), 1),
    ("planes-of-64-power-of-two", (27, 128, 8, 8, 3, "NCHW", "bf16"), 1),
    ("planes-of-273-one-row-a-pass", (16, 24, 13, 21, 8, "NCHW", "bf16"), 1),
    ("planes-of-512", (3, 1024, 16, 32, 3, "NCHW", "f32"), 1),
    ("planes-of-49-several-units", (300, 256, 7, 7, 5, "NCHW", "bf16"), "several"),
    ("planes-of-225-several-units", (60, 256, 15, 15, 4, "NCHW", "bf16"), "several"),
    ("planes-of-144-float-several-units", (100, 128, 12, 12, 4, "NCHW", "f32"), "several"),
    ("8x8-planes-channels-last-k1", (64, 128, 8, 13, 64, "NHWC", "bf16"), "several"),
]


def _problem(shape, base=BASE, change=None):
    n, c, h, w, k, layout, dtype = shape
    wl = dataclasses.replace(base, name="slab", N=n, C=c, H=h, W=w, K=k, layout=layout, dtype=dtype)
    d = synth.make_inputs(wl)
    if change is not None:
        x = G.widen(d["x"], dtype).astype(np.float32)
        change(x)
        d["x"] = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    return wl, d, G.Problem(d["x"], d["dy"], d["gamma"], d["beta"], wl.eps, layout, dtype, k)


def _reference(wl, d):
    return O.cgbn_forward_backward_ref(G.widen(d["x"], wl.dtype), G.widen(d["dy"], wl.dtype), d["gamma"].astype(np.float64),
                                       d["beta"].astype(np.float64), wl.eps, wl.layout)


def _ran_here(forward=True, backward=True):
    assert L.cgbn_get_tuning("last_forward_slab") == forward and L.cgbn_get_tuning("last_backward_slab") == backward


def _vectors_are(shape, forward, backward):
    """The bytes of the vectors of the kernels that ran: 8 where the plan has such a one in the other's place."""
    n, c, h, w, k, layout, dtype = shape
    for way, d in (("forward", forward), ("backward", backward)):
        want = 8 if L.cgbn_plan_get(n, c, h, w, layout, dtype, k, f"n{d}_ok") else 16
        assert layout == "NCHW" or want == 16
        assert L.cgbn_get_tuning(f"last_{way}_slab_vector") == want, way


def _outputs(p):
    return [t.clone() for t in (p.y, p.dx, p.mean, p.invstd, p.mean_lo, p.dgamma, p.dbeta)]


def _moved_on(p):
    """Some unit of the last launch has moved on."""
    return int(p.ws[8:12].view(torch.int32).item()) != 0


def _error_word(p):
    return int(p.ws[4:8].view(torch.int32).item())


class _Knobs:
    def __init__(self, **kw):
        self.kw = kw

    def __enter__(self):
        self.old = {k: L.cgbn_get_tuning(k) for k in self.kw}
        for k, v in self.kw.items():
            L.cgbn_set_tuning(k, v)

    def __exit__(self, *_):
        for k, v in self.old.items():
            L.cgbn_set_tuning(k, v)


@pytest.mark.parametrize("name,shape,units", SHAPES, ids=[s[0] for s in SHAPES])
def test_against_the_oracle(name, shape, units):
    print(f"[case] slab {name} {shape}", flush=True)
    wl, d, p = _problem(shape)
    n, c, h, w, k, layout, dtype = shape
    U = L.cgbn_plan_get(n, c, h, w, layout, dtype, k, "sfwd_U")
    assert (U == 1) if units == 1 else (U > 1)
    p.forward()
    p.backward()
    _ran_here()
    _vectors_are(shape, "fwd", "bwd")
    G.check_against_oracle(p.results(), _reference(wl, d), dtype, name)
    assert _error_word(p) == 0
    first = _outputs(p)
    p.ws.random_(0, 255)                    # whatever the workspace holds, the same bits come out
    p.forward()
    p.backward()
    torch.cuda.synchronize()
    for a, b in zip(first, _outputs(p)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("with_shortcut", [False, True], ids=["relu", "shortcut"])
@pytest.mark.parametrize("name,shape,units", SHAPES, ids=[s[0] for s in SHAPES])
def test_relu_against_the_oracle(name, shape, units, with_shortcut):
    print(f"[case] slab relu {name} {with_shortcut}", flush=True)
    wl, d, p = _problem(shape)
    gen = np.random.default_rng(5)
    sc_host = gen.standard_normal(d["x"].shape).astype(np.float32)
    if wl.dtype == "bf16":
        sc_host = synth.f32_to_bf16_bits(sc_host)
    sc = G.to_dev(sc_host) if with_shortcut else None
    dz = torch.empty_like(p.x) if with_shortcut else None

    def step():
        L.cgbn_forward_relu(p.x, sc, *p.shape_args, wl.layout, wl.K, p.gamma, p.beta, wl.eps, p.y, p.mean, p.invstd,
                            wl.dtype, p.mean_lo, p.ws)
        L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args,
                             wl.layout, wl.K, wl.dtype, p.mean_lo, p.ws)
        return p.results()

    got = step()
    _ran_here()
    _vectors_are(shape, "fwds" if with_shortcut else "fwd", "bwdm")
    x, dy = G.widen(d["x"], wl.dtype), G.widen(d["dy"], wl.dtype)
    g, b = d["gamma"].astype(np.float64), d["beta"].astype(np.float64)
    y, mean, invstd = R.cgbn_relu_forward_ref(x, g, b, wl.eps, wl.layout, G.widen(sc_host, wl.dtype) if with_shortcut else None)[:3]
    dx, dgamma, dbeta, dzr = R.cgbn_relu_backward_ref(dy, got["y"], x, mean, invstd, g, wl.layout)[:4]
    # a channel's sums of masked gradients: judged on the size they have when nothing cancels
    scale = np.sqrt(wl.M) * G.rms(dy)
    G.check_against_oracle(got, dict(y=y, mean=mean, invstd=invstd, dx=dx, dgamma=dgamma, dbeta=dbeta), wl.dtype, name,
                           sum_scale=scale)
    if with_shortcut:
        assert np.array_equal(G.to_host_f64(dz, wl.dtype), dzr)


MOVED_ON = [s for s in SHAPES if s[2] == "several"][:6] + [s for s in SHAPES if s[0] == "planes-of-49-several-units"]


@pytest.mark.parametrize("name,shape,units", MOVED_ON, ids=[s[0] for s in MOVED_ON])
def test_units_that_stop_waiting_are_finished_by_another(name, shape, units):
    """With no polls allowed every unit but the one that completes its slab's count moves on; that one reads the others'
    values again.  Same bits as ever, and no error: also in place, where the output overwrites what is read again."""
    wl, d, p = _problem(shape)
    p.forward()
    p.backward()
    torch.cuda.synchronize()
    want = _outputs(p)
    for t in (p.y, p.dx):
        t.zero_()
    moved = 0
    with _Knobs(spin_limit=0):
        for _ in range(20):                 # (units that all arrive at once may find the count complete: none moves on then)
            p.forward()
            moved += _moved_on(p)
            p.backward()
            moved += _moved_on(p)
            _ran_here()
            assert _error_word(p) == 0
            for a, b in zip(want, _outputs(p)):
                assert torch.equal(a, b)
        print(f"[moved on] {name}: in {moved} of 40 launches", flush=True)
        assert moved
        x, dy = p.x.clone(), p.dy.clone()
        L.cgbn_forward(x, *p.shape_args, wl.layout, wl.K, p.gamma, p.beta, wl.eps, x, p.mean, p.invstd, wl.dtype, p.mean_lo, p.ws)
        L.cgbn_backward(dy, p.x, p.mean, p.invstd, p.gamma, dy, p.dgamma, p.dbeta, *p.shape_args, wl.layout, wl.K, wl.dtype,
                        p.mean_lo, p.ws)
        torch.cuda.synchronize()
        assert torch.equal(x, want[0]) and torch.equal(dy, want[1])


@pytest.mark.parametrize("act", ["relu", "shortcut"])
def test_units_that_stop_waiting_relu(act):
    wl, d, p = _problem((3, 128, 60, 70, 3, "NHWC", "bf16"))
    sc = torch.randn(p.x.shape, device=G.DEV).to(torch.bfloat16).view(p.x.dtype) if act == "shortcut" else None
    dz = torch.empty_like(p.x) if act == "shortcut" else None

    def step():
        L.cgbn_forward_relu(p.x, sc, *p.shape_args, wl.layout, wl.K, p.gamma, p.beta, wl.eps, p.y, p.mean, p.invstd,
                            wl.dtype, p.mean_lo, p.ws)
        L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args,
                             wl.layout, wl.K, wl.dtype, p.mean_lo, p.ws)
        torch.cuda.synchronize()
        return _outputs(p) + ([dz.clone()] if dz is not None else [])

    want, moved = step(), 0
    with _Knobs(spin_limit=0):
        for _ in range(20):
            for t in (p.y, p.dx):
                t.zero_()
            assert all(torch.equal(a, b) for a, b in zip(want, step())) and _error_word(p) == 0
            moved += _moved_on(p)
    assert moved


@pytest.mark.parametrize("shape,direction,P", [((100, 688, 10, 12, 4, "NCHW", "f32"), "sfwd", 18), ((37, 1104, 19, 23, 1, "NCHW", "bf16"), "sfwd", 18),
                                               ((64, 528, 12, 12, 8, "NCHW", "f32"), "sbwd", 9), ((64, 1040, 12, 12, 8, "NCHW", "bf16"), "sbwd", 9)],
                         ids=["forward-f32", "forward-bf16", "backward-f32", "backward-bf16"])
def test_more_units_than_compute_units(shape, direction, P):
    """The variants built a second time with half the registers, for launches of 257 units and more."""
    print(f"[case] slab dense {shape}", flush=True)
    n, c, h, w, k, layout, dtype = shape
    get = lambda key: L.cgbn_plan_get(n, c, h, w, layout, dtype, k, f"{direction}_{key}")
    assert get("P") == P and get("U") > 1 and get("U") * get("slabs") > 256
    wl, d, p = _problem(shape)
    p.forward()
    p.backward()
    assert L.cgbn_get_tuning("last_forward_slab" if direction == "sfwd" else "last_backward_slab") == 1
    G.check_against_oracle(p.results(), _reference(wl, d), dtype, "dense")
    assert _error_word(p) == 0


@pytest.mark.parametrize("groups", [4, 23, 48])
def test_several_rounds_of_units(groups):
    """A small persistent grid: a workgroup walks units of many slabs, whose order is spread over the row (whole rounds
    and a ragged last one)."""
    wl, d, p = _problem((2, 512, 60, 50, 2, "NHWC", "f32"))
    p.forward()
    p.backward()
    _ran_here()
    torch.cuda.synchronize()
    want = _outputs(p)
    with _Knobs(fused_groups=groups):
        p.forward()
        p.backward()
        torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, _outputs(p)))
    G.check_against_oracle(p.results(), _reference(wl, d), wl.dtype, "rounds")


@pytest.mark.parametrize("shape", [(5, 128, 127, 126, 5, "NHWC", "f32"), (3, 192, 171, 200, 1, "NHWC", "bf16")], ids=["f32", "bf16"])
@pytest.mark.parametrize("slabs", [1, 2, 3])
def test_units_fetched_ahead(shape, slabs):
    """Long units in several rounds (one, two, three slabs in flight): a unit's first passes come out of LDS, where they were
    fetched while the one before waited.  The same bits as with the largest grid, also where every unit moves on."""
    wl, d, p = _problem(shape)
    n, c, h, w, k, layout, dtype = shape
    get = lambda key: L.cgbn_plan_get(n, c, h, w, layout, dtype, k, key)
    assert get("sfwd_P") >= 28 and get("sbwd_P") >= 14
    dz = torch.empty_like(p.x)

    def step():
        for t in (p.y, p.dx, dz):
            t.zero_()
        p.forward()
        p.backward()
        _ran_here()
        out = _outputs(p)
        L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz, p.dgamma, p.dbeta, *p.shape_args, wl.layout,
                             wl.K, wl.dtype, p.mean_lo, p.ws)
        torch.cuda.synchronize()
        assert _error_word(p) == 0
        return out + [p.dx.clone(), dz.clone(), p.dgamma.clone(), p.dbeta.clone()]

    want = step()
    if slabs == 1:
        p.forward()
        p.backward()
        G.check_against_oracle(p.results(), _reference(wl, d), dtype, "long units")
    for spin in (None, 0):
        with _Knobs(fused_groups=slabs * max(get("sfwd_U"), get("sbwd_U")), **({} if spin is None else {"spin_limit": spin})):
            assert all(torch.equal(a, b) for a, b in zip(want, step()))


@pytest.mark.parametrize("shape", [(2, 16, 30, 40, 2, "NHWC", "f32"), (4, 64, 40, 50, 4, "NHWC", "f32"),
                                   (4, 64, 40, 50, 4, "NHWC", "bf16")], ids=["one-unit", "several-f32", "several-bf16"])
@pytest.mark.parametrize("sigmas", [6.0, 12.0, 5000.0])
def test_first_value_far_from_the_mean(shape, sigmas):
    """The pass under the loads takes its squares about the threads' own means: the channel's first value, the pivot of the
    sums, may lie anywhere."""
    def outlier(x):
        for c in (1, 14):
            ch = x[..., c]
            ch[0, 0, 0] = np.float32(ch.mean() + sigmas * ch.std())
    wl, d, p = _problem(shape, change=outlier)
    p.forward()
    p.backward()
    _ran_here()
    got, ref = p.results(), _reference(wl, d)
    G.check_against_oracle(got, ref, wl.dtype, "far pivot")
    # float32 statistics: a few roundings of the stored value, whatever the pivot
    assert np.max(np.abs(got["invstd"] / ref["invstd"] - 1)) <= 1e-6


# one unit; several short and long ones; float and bf16; a plane's value per column and two units per slab
STATISTICS = [(2, 256, 25, 42, 2, "NHWC", "f32"), (2, 1024, 25, 42, 2, "NHWC", "bf16"), (4, 64, 40, 50, 4, "NHWC", "f32"),
              (1, 512, 100, 170, 1, "NHWC", "bf16"), (2, 128, 100, 168, 2, "NHWC", "f32"), (300, 256, 7, 7, 5, "NCHW", "bf16"),
              (37, 512, 7, 7, 37, "NCHW", "f32")]


def _skew(kind, layout):
    """Where a channel's first value lies: how many standard deviations off, or an activation among mostly zeros."""
    def change(x):
        v = x if layout == "NHWC" else x.transpose(0, 2, 3, 1)              # (a view: written through)
        if kind == "sparse":
            np.maximum(v - v.mean((0, 1, 2)) - 1.5 * v.std((0, 1, 2)), 0, out=v)
            v[0, 0, 0, :] = 4 * v.std((0, 1, 2))
        else:
            v[0, 0, 0, :] = v.mean((0, 1, 2)) + kind * v.std((0, 1, 2))
    return change


@pytest.mark.parametrize("kind", [0.0, 2.0, 4.0, 6.0, 7.9, 30.0, "sparse"])
@pytest.mark.parametrize("shape", STATISTICS, ids=lambda s: "x".join(map(str, s)))
def test_variance_keeps_its_accuracy_wherever_the_first_value_lies(shape, kind):
    """invstd of every channel to one unit in the last place, 2^-23 relative: half of one for the stored float; the sums of
    squared deviations are sums of positive terms, and a thread's 4 to 36 roundings (2^-25 of its sum on average each)
    count half in the root and average out over the hundreds of threads of a channel."""
    print(f"[case] variance {shape} {kind}", flush=True)
    wl, d, p = _problem(shape, change=_skew(kind, shape[5]))
    p.forward()
    torch.cuda.synchronize()
    assert L.cgbn_get_tuning("last_forward_slab") == 1
    x = G.widen(d["x"], wl.dtype)
    var = x.var((0, 1, 2) if wl.layout == "NHWC" else (0, 2, 3))
    err = np.abs(p.invstd.cpu().numpy().astype(np.float64) * np.sqrt(var + wl.eps) - 1)
    print(f"[error] {err.max():.2e}", flush=True)
    assert err.max() <= 2.0 ** -23


@pytest.mark.parametrize("kind", [1.0, 4.0, 30.0])
# (... and 8-byte vectors, 26 values a thread)
@pytest.mark.parametrize("shape", STATISTICS + [(256, 1024, 7, 7, 8, "NCHW", "bf16")], ids=lambda s: "x".join(map(str, s)))
def test_mean_keeps_its_accuracy(shape, kind):
    """mean + mean_lo in standard deviations, the first value (the pivot of all sums) `kind` of them off.  The only float
    sums are a thread's: of its n <= 36 values about its own first one (a rounding error of about 2^-25 sqrt(n) times a standard
    deviation per value), taken to the pivot by one more rounding (2^-25 kind per value); over the at least 256 threads
    of a channel they average out to an eighth at the worst of 1024 channels (4 of 16 standard errors)."""
    print(f"[case] mean {shape} {kind}", flush=True)
    wl, d, p = _problem(shape, change=_skew(kind, shape[5]))
    p.forward()
    torch.cuda.synchronize()
    assert L.cgbn_get_tuning("last_forward_slab") == 1
    axes = (0, 1, 2) if wl.layout == "NHWC" else (0, 2, 3)
    x = G.widen(d["x"], wl.dtype)
    err = np.abs(p.mean.cpu().numpy().astype(np.float64) + p.mean_lo.cpu().numpy() - x.mean(axes)) / x.std(axes)
    print(f"[mean error] {err.max():.2e}", flush=True)
    assert err.max() <= 2.0 ** -25 * (6 + kind) / 4


def test_offset_data_keeps_its_accuracy():
    """Normal(100, 0.01) in float32: |mean| is 10^4 standard deviations."""
    wl, d, p = _problem((4, 64, 40, 50, 4, "NHWC", "f32"), base=synth.WORKLOADS["cfg4b"])
    p.forward()
    p.backward()
    _ran_here()
    G.check_against_oracle(p.results(), _reference(wl, d), wl.dtype, "offset")


@pytest.mark.parametrize("shape", [(4, 256, 40, 50, 4, "NHWC", "f32"), (2, 256, 100, 150, 2, "NHWC", "f32"), (1, 512, 29, 51, 1, "NHWC", "f32"),
                                   (300, 256, 7, 7, 5, "NCHW", "f32")], ids=lambda s: "x".join(map(str, s)))
def test_gradients_with_a_mean(shape):
    """dy = 1 + noise: dx is what is left of dy when its mean has been taken off.  What a channel's constants leave of the mean, in
    units of it, root mean square over the channels: two roundings to float (dbeta and the constant), each uniform within
    2^-24 at the most."""
    print(f"[case] offset gradients {shape}", flush=True)
    wl, d, p = _problem(shape)
    axes = (0, 1, 2) if wl.layout == "NHWC" else (0, 2, 3)
    factor = np.random.default_rng(3).uniform(0.5, 1.5, wl.C).astype(np.float32)
    factor = factor if wl.layout == "NHWC" else factor[:, None, None]
    d["dy"] = ((1 + 1e-2 * d["dy"]) * factor).astype(np.float32)
    p.dy = G.to_dev(d["dy"])
    p.forward()
    p.backward()
    _ran_here()
    got, ref = p.results(), _reference(wl, d)
    left = (got["dx"] - ref["dx"]).mean(axes) / (d["gamma"] * ref["invstd"] * d["dy"].astype(np.float64).mean(axes))
    print(f"[left] {G.rms(left):.2e}", flush=True)
    assert G.rms(left) <= np.sqrt(2 / 3) * 2.0 ** -24


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("shape", [(2, 32, 30, 40, 2, "NHWC", "bf16"), (4, 64, 40, 50, 4, "NHWC", "f32")], ids=["one", "several"])
def test_a_bad_value_stays_in_its_channel(shape, bad):
    def poison(x):
        x[1, 3, 7, 5] = bad
        x[0, 0, 0, 9] = bad                 # the pivot of channel 9
    wl, d, p = _problem(shape, change=poison)
    p.forward()
    p.backward()
    _ran_here()
    got = p.results()
    clean = [c for c in range(wl.C) if c not in (5, 9)]
    for k in ("y", "dx"):
        assert np.isfinite(got[k][..., clean]).all() and np.isnan(got[k][..., [5, 9]]).any()
    for k in ("mean", "invstd", "dgamma", "dbeta"):
        assert np.isfinite(got[k][clean]).all()
    assert np.isnan(got["invstd"][[5, 9]]).all() and _error_word(p) == 0


def test_two_streams_need_no_cooperative_launch():
    """Layers on two streams at once: units may wait for siblings that have no room yet; they move on, and every result is
    the one of a run alone."""
    probs = [_problem((16, 256, 25, 42, 8, "NHWC", "bf16"))[2], _problem((16, 512, 25, 21, 8, "NHWC", "f32"))[2]]
    want = []
    for p in probs:
        p.forward()
        p.backward()
        _ran_here()
        torch.cuda.synchronize()
        want.append(_outputs(p))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(5):
        for p, s in zip(probs, streams):
            with torch.cuda.stream(s):
                p.forward()
                p.backward()
    torch.cuda.synchronize()
    for p, w in zip(probs, want):
        assert all(torch.equal(a, b) for a, b in zip(w, _outputs(p))) and _error_word(p) == 0


def test_captured_steps_replay():
    """Several units per slab inside a graph: the prepared rows are cleared by a kernel of the call."""
    _, _, p = _problem((4, 96, 50, 41, 2, "NHWC", "bf16"))
    p.forward()
    p.backward()
    _ran_here()
    torch.cuda.synchronize()
    want = _outputs(p)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        p.forward()
        p.backward()
    for _ in range(4):
        for t in (p.y, p.dx):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, _outputs(p)))
