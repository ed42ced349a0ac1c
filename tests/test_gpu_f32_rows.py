"""The fp32 forward for windows of more than 64 tokens: every choice of waves per workgroup (block counts 5 to 16, ragged
last blocks), with the query blocks of a tile in one workgroup and, for few tiles, spread over several."""
import numpy as np
import pytest

from paper_2501_06480_amd import synth
from gpu_util import TOL, f32_device, max_abs, to_device, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [65, 81, 112, 113, 144, 145, 176, 177, 193, 209, 225, 256])
@pytest.mark.parametrize("N,heads,form", [(1, 1, "none"), (2, 3, "dense"), (30, 5, "labels"), (2, 50, "bf16")])
def test_forward(oracle, L, N, heads, form):
    import torch
    import paper_2501_06480_amd as fwa
    w = synth.Workload(f"f32_rows_L{L}", N, L, 32 * heads, heads, "f32", 9100 + L, 0)
    x = synth.draw(w)
    nW = 2
    bias = None if form == "none" else synth.normal((heads, L, L), 9200 + L, 0.5)
    if form == "bf16":
        bias = synth.bf16_round(bias)[0]
    labels = synth.rng(9300 + L).integers(0, 3, (nW, L)).astype(np.int32)
    mask = np.where(labels[:, :, None] == labels[:, None, :], 0.0, -3.0).astype(np.float32) if form in ("dense", "labels") else None
    q, k, v = (to_device(x, w, n) for n in ("q", "k", "v"))
    b = f32_device(bias)
    print(f"L={L} N={N} heads={heads} {form}", flush=True)
    kw = {}
    if form == "dense":
        kw["mask"] = f32_device(mask)
    elif form == "labels":
        kw.update(labels=torch.from_numpy(labels).cuda(), mask_value=-3.0)
    o = fwa.fwa_forward(q, k, v, heads, w.scale, b.bfloat16() if form == "bf16" else b, **kw)
    torch.cuda.synchronize()
    want = oracle.forward(x["q"], x["k"], x["v"], heads, w.scale, bias, mask)
    assert max_abs(to_f64(o), want) <= TOL["f32"]


@pytest.mark.parametrize("L", [81, 96, 97, 112])
def test_both_sides_of_half_a_tile_per_cu(L):
    """6 and 7 blocks without a term split their values in one way up to half the 256 CUs and in another beyond: the same bits."""
    import torch
    import paper_2501_06480_amd as fwa
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn(129, L, 32, device="cuda", generator=g) for _ in range(3))
    many = fwa.fwa_forward(q, k, v, 1, 32 ** -0.5)
    few = fwa.fwa_forward(q[:128], k[:128], v[:128], 1, 32 ** -0.5)
    assert torch.equal(few, many[:128])


@pytest.mark.parametrize("L", [97, 100, 112])
@pytest.mark.parametrize("tiles", [128, 129, 256, 257])
@pytest.mark.parametrize("form", ["none", "bias"])
def test_about_one_tile_per_cu(oracle, L, tiles, form):
    """7 blocks: a wave per block from over half the 256 CUs to all of them, four waves per workgroup on either side."""
    import torch
    import paper_2501_06480_amd as fwa
    w = synth.Workload(f"f32_rows_tiles_L{L}", tiles, L, 32, 1, "f32", 9400 + L, 0)
    x = synth.draw(w)
    bias = None if form == "none" else synth.normal((1, L, L), 9500 + L, 0.5)
    q, k, v = (to_device(x, w, n) for n in ("q", "k", "v"))
    o = fwa.fwa_forward(q, k, v, 1, w.scale, f32_device(bias))
    torch.cuda.synchronize()
    assert max_abs(to_f64(o), oracle.forward(x["q"], x["k"], x["v"], 1, w.scale, bias, None)) <= TOL["f32"]
