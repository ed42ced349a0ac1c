"""The backward without dBias for windows of more than 64 tokens, on both sides of the lines between the kernel that does
it in one launch and the pair that walks the windows: numbers of tiles below, in and beyond a round of resident
workgroups, for each class of block counts, with and without an additive term, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2501_06480_amd import synth
from gpu_util import check_bf16_output, f32_device, to_device, to_f64

pytestmark = pytest.mark.gpu

# L, heads, window counts, additive term
CASES = [
    (81, 4, (16, 390), "bias"), (96, 2, (770,), "labels"), (97, 4, (16, 520), "bias"), (128, 4, (513,), "labels"),
    (144, 4, (16, 128, 200), "bias"), (145, 3, (60, 300), "dense"), (160, 4, (40,), "none"),
    (161, 4, (64, 260), "bias"), (176, 2, (520,), "labels"), (177, 2, (30, 128, 200), "bias"),
    (193, 4, (64, 96), "labels"), (256, 4, (16, 64, 96), "bias"), (256, 4, (64,), "none"), (225, 4, (60,), "dense"),
]


@pytest.mark.parametrize("L,heads,counts,term", CASES, ids=[f"L{c[0]}_{c[3]}" for c in CASES])
def test_large_window_backward_without_dbias(oracle, L, heads, counts, term):
    import torch
    import paper_2501_06480_amd as fwa
    for N in counts:
        print(f"L={L} heads={heads} N={N} {term}", flush=True)
        w = synth.Workload("rounds", N, L, 32 * heads, heads, "bf16", 9100 + L, 0, backward=True)
        x = synth.draw(w)
        nW = N if term == "dense" else 1
        bias = synth.normal((heads, L, L), 9200 + L, 0.5) if term != "none" else None
        labels = synth.rng(9300 + L).integers(0, 3, (nW, L)).astype(np.int32)
        mask = np.where(labels[:, :, None] == labels[:, None, :], 0.0, -3.0).astype(np.float32)
        kw = {}
        if term == "dense":
            kw = {"mask": f32_device(mask)}
        elif term == "labels":
            kw = {"labels": torch.from_numpy(labels).cuda(), "mask_value": -3.0}
        ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask if kw else None)
        q, k, v, g = (to_device(x, w, n) for n in ("q", "k", "v", "d_o"))
        got = fwa.fwa_backward(q, k, v, g, heads, w.scale, f32_device(bias), want_dbias=False, **kw)
        torch.cuda.synchronize()
        for what, a, b in zip(("dq", "dk", "dv"), got, ref):
            check_bf16_output(to_f64(a), b, f"L={L} N={N} {term} {what}")
