"""The backward above 64 tokens at the edges of its score arithmetic.  One kernel takes the exponentials of the scores as they are
and makes a row again around its maximum where their sum leaves [2^-10, 2^40] or dQ is not finite; the other starts its products
from -M / scale.  A constant added to every score of a row changes nothing, which is the reference here; the scale may be zero or too
small to divide by."""
import numpy as np
import pytest

from paper_2501_06480_amd import synth
from gpu_util import check_bf16_output, f32_device, to_device, to_f64

pytestmark = pytest.mark.gpu

# L, heads, N, mask: block counts of each kind (whole and odd numbers of blocks, one and two parts), every source of the term
SHAPES = [(65, 2, 6, "none"), (100, 3, 9, "labels"), (177, 1, 5, "dense"), (193, 2, 6, "labels"), (256, 2, 300, "dense"), (250, 1, 4, "none")]


def _call(x, w, bias, mask, labels, scale, dbias, d_o=None):
    import torch
    import paper_2501_06480_amd as fwa
    q, k, v, g = (to_device(x, w, n) for n in ("q", "k", "v", "d_o"))
    if d_o is not None:
        g = d_o
    kw = {}
    if labels is not None:
        kw = {"labels": torch.from_numpy(labels).cuda(), "mask_value": -3.0}
    elif mask is not None:
        kw = {"mask": f32_device(mask)}
    got = fwa.fwa_backward(q, k, v, g, w.heads, scale, f32_device(bias), want_dbias=dbias, **kw)
    torch.cuda.synchronize()
    return [None if t is None else to_f64(t) for t in got]


def _draw(L, heads, N, kind):
    w = synth.Workload("scores", N, L, 32 * heads, heads, "bf16", 9400 + L, 0, backward=True)
    x = synth.draw(w)
    bias = synth.normal((heads, L, L), 9500 + L, 0.5).astype(np.float32)
    mask = labels = None
    if kind != "none":
        nW = 3 if kind == "labels" else min(N, 150)  # 150: a period that the resident workgroups cannot hold
        lab = synth.rng(9600 + L).integers(0, 3, (nW, L)).astype(np.int32)
        mask = np.where(lab[:, :, None] == lab[:, None, :], 0.0, -3.0).astype(np.float32)
        mask = mask[np.arange(N) % nW] if nW != N else mask
        labels = lab if kind == "labels" else None
        if kind == "dense":
            mask = mask[:nW]
    return w, x, bias, mask, labels


def _check(got, ref, what, unit=1.0):
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(a).all(), (what, name)
        check_bf16_output(a / unit, b, f"{what} {name}")


@pytest.mark.parametrize("dbias", [False, True])
@pytest.mark.parametrize("L,heads,N,kind", SHAPES, ids=[f"L{s[0]}_{s[3]}" for s in SHAPES])
def test_rows_far_from_zero(oracle, L, heads, N, kind, dbias):
    w, x, bias, mask, labels = _draw(L, heads, N, kind)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask, want_dbias=dbias)
    # rows of one block: both sides of the two limits (in units of ln 2), some blocks untouched
    shift = np.zeros((1, L, 1), np.float32)
    shift[0, :, 0] = np.resize(np.float32([0, 24, 40, 400, -14, -20, -300, 0]) * np.float32(0.6931472), L)
    shift[0, 32:64] = 0
    got = _call(x, w, bias + shift, mask, labels, w.scale, dbias)
    _check(got, ref, f"L={L} {kind}")
    if dbias:
        # scores of up to 300 are rounded to 2^-16 of themselves (15 bits behind a bias of 300), in N windows at random
        assert np.abs(got[3] - ref[3]).max() <= 2e-4 * max(1.0, np.sqrt(N))


@pytest.mark.parametrize("scale", [0.0, -0.25, 2.0 ** -103, 2.0 ** -83])
@pytest.mark.parametrize("L,heads,N,kind", [SHAPES[1], SHAPES[2], SHAPES[5]], ids=["L100", "L177", "L250"])
def test_scales(oracle, L, heads, N, kind, scale):
    w, x, bias, mask, labels = _draw(L, heads, N, kind)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, scale, bias, mask, want_dbias=True)
    got = _call(x, w, bias, mask, labels, scale, True)
    _check(got, ref, f"L={L} scale={scale}")
    if 0.0 < scale < 1e-20:  # dK and dQ are of the size of the scale
        for a, b in zip(got[:2], ref[:2]):
            check_bf16_output(a / scale, b / scale, f"L={L} scale={scale}")
    assert np.abs(got[3] - ref[3]).max() <= 2e-4


@pytest.mark.parametrize("L,heads,N,kind", [SHAPES[1], SHAPES[4]], ids=["L100", "L256"])
def test_gradients_of_any_size(oracle, L, heads, N, kind):
    """dO of 2^100 overflows beside exponentials of up to 2^40 (rows with a shift of 38), where it does not beside probabilities."""
    import torch
    w, x, bias, mask, labels = _draw(L, heads, N, kind)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask, want_dbias=False)
    shift = np.zeros((1, L, 1), np.float32)
    shift[0, 16:48] = np.float32(20.0)
    for power in (100, -90):
        g = to_device(x, w, "d_o") * torch.tensor(2.0 ** power, device="cuda").to(torch.bfloat16)
        got = _call(x, w, bias + shift, mask, labels, w.scale, False, g)
        _check(got, ref, f"L={L} dO 2^{power}", 2.0 ** power)


@pytest.mark.parametrize("value", [-1e4, -1e9, -1e38])
@pytest.mark.parametrize("L,heads,N,kind", [SHAPES[0], SHAPES[5]], ids=["L65", "L250"])
def test_rows_that_lost_every_key(oracle, L, heads, N, kind, value):
    """Finite whatever the mask's value; as without the mask while its rounding (2^-21 of it) is small."""
    w, x, bias, _, _ = _draw(L, heads, N, kind)
    bias = np.zeros_like(bias)
    mask = np.zeros((1, L, L), np.float32)
    mask[0, 5] = mask[0, 40:50] = value
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, None, want_dbias=False)
    got = _call(x, w, bias, mask, None, w.scale, True)
    assert all(np.isfinite(a).all() for a in got)
    if value == -1e4:  # 1.4e4 in units of log2, 2^-21 of that 0.7 %, of 11 rows' share
        for a, b in zip(got[:3], ref[:3]):
            assert np.abs(a - b).max() <= 0.02
