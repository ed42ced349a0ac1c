"""The forms in which the backward for windows of more than 64 tokens takes its additive term, each at the sizes
where the choice between them falls, against the fp64 oracle: kept in registers (the number of workgroups in flight
is a multiple of the mask period, or more workgroups than are resident are launched), the mask formed per window from
labels, and a dense mask read per window, both also where a multiple of the period would fit but leave much of the
device idle.  The block counts cover odd ones, whose last workgroup has idle waves."""
import numpy as np
import pytest

from paper_2501_06480_amd import synth
from gpu_util import TOL, check_bf16_output, f32_device, max_abs, to_device, to_f64

pytestmark = pytest.mark.gpu

# name, L, heads, N, nW, bias, dbias
CASES = [
    ("period_of_one", 65, 2, 70, 1, True, True),
    ("kept_idle_waves", 129, 3, 96, 8, True, True),
    ("kept_last_part_one_block", 193, 2, 64, 4, True, False),
    ("more_workgroups_than_resident", 65, 24, 960, 40, True, True),
    ("more_workgroups_than_resident_no_dbias", 65, 24, 960, 40, True, False),
    ("rounding_loses_labels", 256, 3, 100, 25, True, True),
    ("rounding_loses_labels_no_dbias", 241, 3, 150, 25, True, False),
    ("rounding_loses_dense", 193, 2, 288, 36, True, True),
    ("rounding_loses_dense_no_dbias", 193, 2, 288, 36, True, False),
    ("beyond_L65", 65, 24, 100, 50, True, True),
    ("beyond_L65_no_bias", 65, 24, 100, 50, False, True),
    ("beyond_L81_no_dbias", 81, 24, 100, 50, True, False),
    # block counts whose kernels state their waves per SIMD or take the tight form
    ("beyond_L80", 80, 24, 100, 50, True, True),
    ("beyond_L80_no_dbias", 80, 24, 100, 50, True, False),
    ("beyond_L96", 96, 24, 60, 60, True, True),
    ("beyond_L112", 112, 24, 44, 44, False, True),
    ("beyond_L144_no_dbias", 144, 16, 40, 40, True, False),
    ("beyond_L161", 161, 16, 36, 36, True, True),
    ("beyond_L176_no_dbias", 176, 16, 36, 36, True, False),
    ("beyond_L192", 192, 16, 36, 36, True, True),
    ("beyond_L177", 177, 16, 40, 40, True, True),
    ("beyond_L256", 256, 12, 24, 24, True, True),
    ("beyond_L256_mask_alone", 256, 12, 24, 24, False, False),
]


@pytest.mark.parametrize("name,L,heads,N,nW,use_bias,dbias", CASES, ids=[c[0] for c in CASES])
def test_large_window_backward(oracle, name, L, heads, N, nW, use_bias, dbias):
    import torch
    import paper_2501_06480_amd as fwa
    w = synth.Workload("forms_" + name, N, L, 32 * heads, heads, "bf16", 8100 + L, 0, backward=True)
    x = synth.draw(w)
    bias = synth.normal((heads, L, L), 8200 + L, 0.5) if use_bias else None
    labels = synth.rng(8300 + L).integers(0, 3, (nW, L)).astype(np.int32)
    mask = np.where(labels[:, :, None] == labels[:, None, :], 0.0, -3.0).astype(np.float32)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask)
    q, k, v, g = (to_device(x, w, n) for n in ("q", "k", "v", "d_o"))
    for form in ("dense", "labels"):
        print(f"{name} {form}: L={L} heads={heads} N={N} nW={nW} bias={use_bias} dbias={dbias}", flush=True)
        kw = {"mask": f32_device(mask)} if form == "dense" else {"labels": torch.from_numpy(labels).cuda(), "mask_value": -3.0}
        got = fwa.fwa_backward(q, k, v, g, heads, w.scale, f32_device(bias), want_dbias=dbias, **kw)
        torch.cuda.synchronize()
        for what, a, b in zip(("dq", "dk", "dv"), got, ref):
            check_bf16_output(to_f64(a), b, f"{name} {form} {what}")
        if dbias:
            assert max_abs(to_f64(got[3]), ref[3]) <= TOL["bf16"], (name, form)


# The backward for windows of up to 64 tokens with a mask period that no slot count is a multiple of: labels parked in
# LDS, or a dense tile fetched into LDS per window.  Tiles of less than, exactly and more than a 1 KB piece; 3 heads at
# L = 55 and 56 (with and without room for the padding of the slab rows) and 64; 1, 2 and 3 heads per workgroup (1 for
# dense tiles of L = 33 .. 48); row lengths whose tiles are stored turned (L = 16, 32, 64); several workgroups per CU
# (L <= 32), with one window and with many per workgroup; the trimmed last key block (L = 17, 33, 49).
# name, L, heads, N, nW, bias, dbias
SMALL = [
    ("L16", 16, 3, 600, 300, True, True),
    ("L17_pairs", 17, 4, 280, 140, True, False),
    ("L16_pairs", 16, 8, 1200, 600, True, True),
    ("L16_more_windows_than_workgroups", 16, 4, 1750, 875, False, False),
    ("L25_single_heads", 25, 7, 900, 450, True, True),
    ("L32_pairs", 32, 4, 560, 280, True, True),
    ("L32", 32, 3, 410, 410, True, False),
    ("L33_single_heads", 33, 24, 80, 40, True, True),
    ("L36", 36, 3, 520, 520, False, False),
    ("L48_pairs", 48, 2, 300, 300, True, True),
    ("L49", 49, 3, 600, 300, True, True),
    ("L49_mask_alone", 49, 2, 300, 300, False, True),
    ("L55", 55, 3, 300, 300, True, True),
    ("L56", 56, 3, 300, 300, True, True),
    ("L64", 64, 3, 300, 300, True, False),
    ("L64_pairs", 64, 8, 140, 70, True, True),
    ("L64_one_head", 64, 1, 800, 800, True, True),
]


@pytest.mark.parametrize("name,L,heads,N,nW,use_bias,dbias", SMALL, ids=[c[0] for c in SMALL])
def test_small_window_backward_long_periods(oracle, name, L, heads, N, nW, use_bias, dbias):
    test_large_window_backward(oracle, name, L, heads, N, nW, use_bias, dbias)


# The forward for windows of up to 64 tokens with such a period: the dense tile of every window in a second LDS buffer,
# with all heads of a window in one workgroup (3 heads; 4 heads, 16 waves, in the smaller calls) and with groups of 4 heads;
# beside them the calls next to the rule that read the mask per window (2 heads and groups of 2, row lengths that are
# multiples of 32 words, the smallest windows, too few windows, tiles that leave no room for two workgroups).  An odd number
# of windows per workgroup, and fewer windows than workgroups after the first round, end the walk at every stage of its
# prefetches.
# name, L, heads, N, nW, bias
FORWARD = [
    ("L16_pairs", 16, 2, 900, 300, True),
    ("L17", 17, 3, 600, 300, False),
    ("L33", 33, 3, 300, 300, True),
    ("L33_few_windows_more", 33, 3, 400, 400, True),
    ("L33_four_heads", 33, 4, 410, 410, False),
    ("L49", 49, 3, 1390, 695, True),
    ("L49_four_heads", 49, 4, 600, 300, True),
    ("L55_four_heads", 55, 4, 999, 333, True),
    ("L64", 64, 3, 600, 300, True),
    ("L49_groups_of_2", 49, 6, 1050, 350, True),
    ("L49_groups_of_4", 49, 8, 600, 300, True),
    ("L32_groups_of_4", 32, 12, 540, 270, False),
    ("L55_groups_of_4", 55, 8, 600, 300, True),
    ("L56_groups_of_4", 56, 8, 600, 300, True),
]


@pytest.mark.parametrize("name,L,heads,N,nW,use_bias", FORWARD, ids=[c[0] for c in FORWARD])
def test_small_window_forward_long_periods(oracle, name, L, heads, N, nW, use_bias):
    import torch
    import paper_2501_06480_amd as fwa
    from gpu_util import check_forward_arithmetic_bound
    w = synth.Workload("fforms_" + name, N, L, 32 * heads, heads, "bf16", 8500 + L, 0)
    x = synth.draw(w)
    bias = synth.normal((heads, L, L), 8600 + L, 0.5) if use_bias else None
    labels = synth.rng(8700 + L).integers(0, 3, (nW, L)).astype(np.int32)
    mask = np.where(labels[:, :, None] == labels[:, None, :], 0.0, -3.0).astype(np.float32)
    want = oracle.forward(x["q"], x["k"], x["v"], heads, w.scale, bias, mask)
    spread = oracle.forward(x["q"], x["k"], np.abs(x["v"]), heads, w.scale, bias, mask)
    q, k, v = (to_device(x, w, n) for n in ("q", "k", "v"))
    for form in ("dense", "labels"):
        print(f"{name} {form}: L={L} heads={heads} N={N} nW={nW} bias={use_bias}", flush=True)
        kw = {"mask": f32_device(mask)} if form == "dense" else {"labels": torch.from_numpy(labels).cuda(), "mask_value": -3.0}
        o = fwa.fwa_forward(q, k, v, heads, w.scale, f32_device(bias), **kw)
        torch.cuda.synchronize()
        check_forward_arithmetic_bound(to_f64(o), want, spread, f"{name} {form}")


# The backward for windows of up to 64 tokens with more groups of heads than the chip holds workgroups: one workgroup per
# group walks all windows.  The mask periods leave no other choice than a mask per window.
# heads, L, N, nW (0: no mask), bias type, dbias
MANY_HEADS = [(771, 9, 2, 0, "f32", True), (771, 9, 2, 0, "bf16", True), (1026, 5, 3, 3, "f32", True),
              (1026, 17, 2, 2, "f32", False), (773, 4, 4, 4, "bf16", True), (775, 33, 1, 1, "bf16", True)]


@pytest.mark.parametrize("heads,L,N,nW,bias_type,dbias", MANY_HEADS)
def test_more_head_groups_than_workgroups(oracle, heads, L, N, nW, bias_type, dbias):
    import torch
    import paper_2501_06480_amd as fwa
    w = synth.Workload(f"many_heads_{heads}_{L}", N, L, 32 * heads, heads, "bf16", 8900 + heads + L, 0, backward=True)
    x = synth.draw(w)
    bias = synth.normal((heads, L, L), 8950 + L, 0.5)
    if bias_type == "bf16":
        bias = synth.bf16_round(bias.astype(np.float32))[0]
    bias_d = f32_device(bias) if bias_type == "f32" else f32_device(bias).bfloat16()
    labels = synth.rng(8960 + L).integers(0, 3, (max(nW, 1), L)).astype(np.int32)
    mask = np.where(labels[:, :, None] == labels[:, None, :], 0.0, -3.0).astype(np.float32) if nW else None
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask)
    q, k, v, g = (to_device(x, w, n) for n in ("q", "k", "v", "d_o"))
    forms = [{}] if not nW else [{"labels": torch.from_numpy(labels).cuda(), "mask_value": -3.0}]
    if nW and bias_type == "f32":
        forms.append({"mask": f32_device(mask)})
    for kw in forms:
        print(f"heads={heads} L={L} N={N} nW={nW} bias={bias_type} dbias={dbias} {list(kw)}", flush=True)
        got = fwa.fwa_backward(q, k, v, g, heads, w.scale, bias_d, want_dbias=dbias, **kw)
        torch.cuda.synchronize()
        for what, a, b in zip(("dq", "dk", "dv"), got, ref):
            check_bf16_output(to_f64(a), b, f"{heads} heads {list(kw)} {what}")
        if dbias:
            assert max_abs(to_f64(got[3]), ref[3]) <= TOL["bf16"], list(kw)
