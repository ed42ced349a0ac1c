"""Masks that remove pairs altogether (-inf, the lowest float) in the backward, with labels none of which is 0.  The rows
that pad a window to a multiple of 16 have no label of their own; if they were masked like label 0 they would see no key
at all, and what a softmax over nothing gives must not reach dK and dV, whose products run over the padded rows too.
One case per kernel and per form in which it takes the mask, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2501_06480_amd import synth
from gpu_util import TOL, check_bf16_output, f32_device, max_abs, to_device, to_f64

pytestmark = pytest.mark.gpu

# name, dtype, L, heads, d, N, nW, bias, dbias
CASES = [
    ("coop_kept", "bf16", 49, 3, 32, 12, 4, "f32", True),
    ("coop_kept_bf16_bias", "bf16", 50, 3, 32, 12, 4, "bf16", True),
    ("coop_kept_no_bias", "bf16", 33, 2, 32, 8, 4, None, False),
    ("coop_per_window", "bf16", 49, 3, 32, 300, 300, "f32", True),
    ("coop_per_window_bf16_bias", "bf16", 49, 3, 32, 300, 300, "bf16", False),
    ("wide", "bf16", 50, 2, 64, 8, 4, "f32", True),
    ("wide_half", "f16", 50, 2, 64, 8, 4, "f32", False),
    ("fp32", "f32", 49, 3, 32, 8, 4, "f32", False),
    ("fp32_wide", "f32", 37, 2, 64, 8, 4, None, False),
    ("large_kept", "bf16", 81, 3, 32, 16, 4, "f32", True),
    ("large_kept_bf16_bias", "bf16", 121, 2, 32, 16, 4, "bf16", True),
    ("large_labels", "bf16", 81, 24, 32, 100, 50, "f32", True),
    ("large_kept_pair", "bf16", 196, 4, 32, 96, 4, "f32", False),
    ("large_fused", "bf16", 81, 3, 32, 16, 4, "f32", False),
    ("large_fused_no_bias", "bf16", 196, 2, 32, 16, 4, None, False),
]


@pytest.mark.parametrize("value", [-np.inf, float(np.finfo(np.float32).min), 100.0], ids=["inf", "lowest", "positive"])
@pytest.mark.parametrize("name,dtype,L,heads,d,N,nW,bias_type,dbias", CASES, ids=[c[0] for c in CASES])
def test_backward(oracle, name, dtype, L, heads, d, N, nW, bias_type, dbias, value):
    import torch
    import paper_2501_06480_amd as fwa
    w = synth.Workload("padding_" + name, N, L, heads * d, heads, dtype, 9800 + L, 0, backward=True)
    x = synth.draw(w)
    bias = None if bias_type is None else synth.normal((heads, L, L), 9810 + L, 0.5)
    if bias_type == "bf16":
        bias = synth.bf16_round(bias.astype(np.float32))[0]
    labels = (1 + synth.rng(9820 + L).integers(0, 3, (nW, L))).astype(np.int32)
    mask = np.where(labels[:, :, None] == labels[:, None, :], np.float32(0.0), np.float32(value))
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask)
    q, k, v, g = (to_device(x, w, n) for n in ("q", "k", "v", "d_o"))
    bias_d = f32_device(bias) if bias_type != "bf16" else f32_device(bias).bfloat16()
    forms = [("labels", {"labels": torch.from_numpy(labels).cuda(), "mask_value": value})]
    if bias_type != "bf16":
        forms.append(("dense", {"mask": f32_device(mask)}))
    for form, kw in forms:
        print(f"{name} {form} {value}: {dtype} L={L} heads={heads} d={d} N={N} nW={nW} bias={bias_type} dbias={dbias}", flush=True)
        got = fwa.fwa_backward(q, k, v, g, heads, w.scale, bias_d, want_dbias=dbias, **kw)
        torch.cuda.synchronize()
        for what, a, b in zip(("dq", "dk", "dv"), got, ref):
            a = to_f64(a)
            assert np.isfinite(a).all(), (name, form, what)
            if dtype == "f32":
                # with the mask of 100, scores of 64 to 128 are rounded three times (product, sum, difference from the
                # maximum; half an ulp, 3.8e-6, each): P is off by at most 1.2e-5 of itself, and a gradient element sums
                # P |dP - delta| |K| scale to less than 8
                assert max_abs(a, b) <= (TOL["f32"] if value < 0 else 1e-4), (name, form, what)
            else:
                check_bf16_output(a, b, f"{name} {form} {what}")
        if dbias:
            assert max_abs(to_f64(got[3]), ref[3]) <= TOL["bf16"], (name, form)
