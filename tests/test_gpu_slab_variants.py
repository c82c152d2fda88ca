"""Every one-workgroup-a-slab variant of the column-slab kernels on NCHW planes: vectors of 16 and of 8 bytes, every count of vectors a thread, both
element types, both directions, with and without a second tensor.  The plan says which variant a call takes, the library which one it took;
results against the float64 oracles, with the tolerances stated in gpu_harness.py."""

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

# N, C, H, W, dtype
CASES = [
    # 8 bytes: one slab or few, ragged last passes and slabs, several channels a column, one row a pass
    (16, 24, 2, 1, "bf16"), (523, 24, 1, 1, "bf16"), (524, 8, 2, 3, "bf16"), (679, 16, 3, 1, "bf16"), (986, 8, 7, 1, "bf16"), (190, 40, 7, 7, "bf16"),
    (280, 24, 1, 1, "f32"), (380, 8, 3, 1, "f32"), (776, 16, 2, 1, "f32"), (840, 8, 1, 5, "f32"), (978, 128, 3, 4, "f32"), (702, 72, 1, 3, "f32"),
    (600, 8, 3, 1, "f32"), (676, 8, 3, 1, "f32"),
    # 16 bytes: more slabs than half the compute units; float with few vectors a thread, or masked, whatever the slabs
    (9, 2064, 2, 2, "bf16"), (5, 1032, 1, 265, "bf16"), (7, 1112, 1, 263, "bf16"), (9, 1096, 3, 89, "bf16"), (11, 1048, 1, 277, "bf16"),
    (13, 1136, 7, 39, "bf16"),
    (16, 8, 2, 1, "f32"), (20, 2056, 1, 2, "f32"), (170, 1040, 1, 6, "f32"), (218, 1040, 1, 7, "f32"), (38, 520, 2, 26, "f32"), (291, 1040, 7, 1, "f32"),
    (18, 520, 1, 173, "f32"), (421, 2080, 3, 1, "f32"), (231, 536, 2, 13, "f32"), (25, 560, 21, 9, "f32"),
]
ID = lambda c: "%dx%dx%dx%d-%s" % c
# plan prefixes and, of the single-launch kernels that come before unless "first", theirs
DIRECTIONS = {"fwd": "fwd", "fwds": "fwd", "bwd": "bwd", "bwdm": "bwd"}


def _variant(case, d):
    """(bytes of a vector, vectors a thread) of the column-slab kernel that a call takes; None if a single-launch kernel is planned before it (a few
    masked float ones are not built: such a call does come here)."""
    g = lambda k: L.cgbn_plan_get(*case[:4], "NCHW", case[4], 1, k)
    if not g("s%s_ok" % d) or (g(DIRECTIONS[d] + "_ok") and not g("s%s_first" % d)):
        return None
    if g("n%s_ok" % d):
        return 8, g("n%s_P" % d)
    assert g("s%s_U" % d) == 1
    return 16, g("s%s_P" % d)


def _built():
    text = open(os.path.join(os.path.dirname(L.__file__), "csrc", "cgbn_slab.h")).read()
    counts = lambda name, solo: [int(v) for v in re.findall(r"X\((\d+)%s\)" % solo, re.search("#define %s\\(X\\) (.*)" % name, text).group(1))]
    wide = {"fwd": counts("CGBN_SLAB_FORWARD_P", ", true"), "bwd": counts("CGBN_SLAB_BACKWARD_P", ", true")}
    narrow = counts("CGBN_SLAB_NARROW_P", "")
    assert len(narrow) == 5 and len(wide["fwd"]) == 5 and len(wide["bwd"]) == 6
    return {(t, d, vb, P) for t in ("f32", "bf16") for d, way in DIRECTIONS.items() for vb, Ps in ((16, wide[way]), (8, narrow)) for P in Ps}


def test_every_variant_is_run():
    run = {(case[4], d) + _variant(case, d) for case in CASES for d in DIRECTIONS if _variant(case, d)}
    assert run == _built()


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=ID)
def test_against_the_oracle(case):
    N, C, H, W, dtype = case
    print("[case] slab variant", case, flush=True)
    r = np.random.default_rng(N * 1000 + C)
    per = lambda a: a.reshape(1, -1, 1, 1)
    x = (r.standard_normal((N, C, H, W)) * per(r.uniform(0.5, 2, C)) + per(r.uniform(-2, 2, C))).astype(np.float32)
    dy, s = (r.standard_normal(x.shape).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        x, dy, s = (synth.f32_to_bf16_bits(a) for a in (x, dy, s))
    gamma, beta = r.uniform(0.5, 1.5, C).astype(np.float32), r.normal(0, 0.1, C).astype(np.float32)
    p = G.Problem(x, dy, gamma, beta, 1e-5, "NCHW", dtype, 1)

    def took(*directions):
        torch.cuda.synchronize()
        for d in directions:
            v = _variant(case, d)
            assert v is None or L.cgbn_get_tuning("last_%s_slab_vector" % ("forward" if d[0] == "f" else "backward")) == v[0], d

    p.forward()
    p.backward()
    took("fwd", "bwd")
    wx, wdy = G.widen(x, dtype), G.widen(dy, dtype)
    # a channel's sums of gradients: judged on the size they have when nothing cancels
    scale = np.sqrt(N * H * W) * G.rms(wdy)
    G.check_against_oracle(p.results(), O.cgbn_forward_backward_ref(wx, wdy, gamma, beta, 1e-5, "NCHW"), dtype, str(case), sum_scale=scale)
    sd, dz = G.to_dev(s), torch.empty_like(p.x)
    for short in (None, sd):
        L.cgbn_forward_relu(p.x, short, *p.shape_args, "NCHW", 1, p.gamma, p.beta, 1e-5, p.y, p.mean, p.invstd, dtype, p.mean_lo, p.ws)
        L.cgbn_backward_relu(p.dy, p.y, p.x, p.mean, p.invstd, p.gamma, p.dx, dz if short is not None else None, p.dgamma, p.dbeta, *p.shape_args,
                             "NCHW", 1, dtype, p.mean_lo, p.ws)
        took("fwd" if short is None else "fwds", "bwdm")
        got = p.results()
        y, mean, invstd = R.cgbn_relu_forward_ref(wx, gamma, beta, 1e-5, "NCHW", None if short is None else G.widen(s, dtype))[:3]
        # (the mask is read off the stored output, so the oracle is handed the same)
        dx, dgamma, dbeta, dzr = R.cgbn_relu_backward_ref(wdy, got["y"], wx, mean, invstd, gamma, "NCHW")[:4]
        G.check_against_oracle(got, dict(y=y, mean=mean, invstd=invstd, dx=dx, dgamma=dgamma, dbeta=dbeta), dtype, str(case), sum_scale=scale)
        if short is not None:
            assert np.array_equal(G.to_host_f64(dz, dtype), dzr)
