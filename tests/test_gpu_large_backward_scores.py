"""The backward above 64 tokens at the edges of its score arithmetic.  One kernel finds the maximum
and the sum of every row, the other makes the scores again and subtracts what the first found.  A constant added to every score of a row changes nothing, which is the reference here; the scale may
be zero."""
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


def _check(got, ref, what):
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(a).all(), (what, name)
        check_bf16_output(a, b, f"{what} {name}")


@pytest.mark.parametrize("dbias", [False, True])
@pytest.mark.parametrize("L,heads,N,kind", SHAPES, ids=[f"L{s[0]}_{s[3]}" for s in SHAPES])
def test_rows_far_from_zero(oracle, L, heads, N, kind, dbias):
    w, x, bias, mask, labels = _draw(L, heads, N, kind)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask, want_dbias=dbias)
    # rows of one block near zero and far from it on both sides (in units of ln 2), some blocks untouched
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


@pytest.mark.parametrize("dbias", [False, True])
@pytest.mark.parametrize("L,heads,N,kind", [SHAPES[1], SHAPES[3], SHAPES[4]], ids=["L100", "L193", "L256"])
def test_gradients_of_any_size(oracle, L, heads, N, kind, dbias):
    """dO of 2^100 and 2^-90, beside rows whose scores lie 20 (28.9 in units of ln 2) above the others': what a kernel keeps of a row
    before it divides by the row's sum may neither overflow nor vanish.  With dBias the pair of kernels takes every one of these calls."""
    import torch
    w, x, bias, mask, labels = _draw(L, heads, N, kind)
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, mask, want_dbias=dbias)
    shift = np.zeros((1, L, 1), np.float32)
    shift[0, 16:48] = np.float32(20.0)
    for power in (100, -90):
        g = to_device(x, w, "d_o") * torch.tensor(2.0 ** power, device="cuda").to(torch.bfloat16)
        got = _call(x, w, bias + shift, mask, labels, w.scale, dbias, g)
        _check([a / 2.0 ** power for a in got[:3]], ref, f"L={L} dO 2^{power}")
        if dbias:
            assert np.abs(got[3] / 2.0 ** power - ref[3]).max() <= 2e-4 * max(1.0, np.sqrt(N))


@pytest.mark.parametrize("value", [-1e4, -1e9, -1e38])
@pytest.mark.parametrize("L,heads,N,kind", [SHAPES[0], SHAPES[5]], ids=["L65", "L250"])
def test_rows_that_lost_every_key(oracle, L, heads, N, kind, value):
    """Finite whatever the mask's value; as without the mask while its rounding (2^-24 of it) is small."""
    w, x, bias, _, _ = _draw(L, heads, N, kind)
    bias = np.zeros_like(bias)
    mask = np.zeros((1, L, L), np.float32)
    mask[0, 5] = mask[0, 40:50] = value
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, None, want_dbias=False)
    got = _call(x, w, bias, mask, None, w.scale, True)
    assert all(np.isfinite(a).all() for a in got)
    if value == -1e4:  # 1.4e4 in units of log2: half an ulp is 2^-11, 0.03 % of a probability
        _check(got, ref, f"L={L} value={value}")


@pytest.mark.parametrize("dbias", [False, True])
@pytest.mark.parametrize("size", [8, 32, 128, 384, 1024])
@pytest.mark.parametrize("L,heads,N,kind", SHAPES, ids=[f"L{s[0]}_{s[3]}" for s in SHAPES])
def test_large_scores_of_q_and_k(oracle, L, heads, N, kind, size, dbias):
    """Channels of +-size: a row's two keys with its own signs score 32 size^2 scale (up to 8.6e6 in units of ln 2), every other key at
    least 2 size^2 scale less, and every sum of products is exact.  So both have a probability of 1/2 to within a rounding of the
    sums, in every unit of size: a score or a maximum that one kernel rounds and the other does not shows as a factor."""
    import torch
    w, x, _, mask, _ = _draw(L, heads, N, kind)
    r = synth.rng(9700 + L)
    pairs = (L + 1) // 2
    u = (r.integers(0, 2, (N, pairs, heads * 32)) * 2 - 1).astype(np.float32)
    row = np.arange(L) // 2
    x["q"], x["k"] = size * u[:, (row + 3) % pairs], size * u[:, row]
    for name in ("q", "k"):
        x[name + "_bits"] = torch.from_numpy(np.ascontiguousarray(x[name])).bfloat16().view(torch.int16).numpy().view(np.uint16)
    bias = mask = labels = None
    if kind != "none":  # an additive term that both keys of a pair share
        bias = np.zeros((heads, L, L), np.float32)
        nW = 3 if kind == "labels" else min(N, 150)
        lab = np.ascontiguousarray(r.integers(0, 3, (nW, pairs))[:, row].astype(np.int32))
        mask = np.where(lab[:, :, None] == lab[:, None, :], 0.0, -3.0).astype(np.float32)
        if kind == "labels":
            labels = lab
    full = None if mask is None else mask[np.arange(N) % mask.shape[0]]
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], heads, w.scale, bias, full, want_dbias=dbias)
    got = _call(x, w, bias, mask, labels, w.scale, dbias)
    unit = size * w.scale  # of dQ and dK
    # half an ulp of the output, and 2e-3 for what comes before it.  Without dBias the kernel that makes all in one launch may take the
    # call; it rounds score and maximum together in one fma: half an ulp of the maximum, in powers of two, on P and with it on dV and dK.
    top = 32 * size * size * w.scale * 1.4426951
    factor = 0.0 if dbias else 2.0 ** (0.5 * 2.0 ** (np.floor(np.log2(top)) - 23)) - 1.0
    for name, a, b, one in zip(("dq", "dk", "dv"), got, ref, (unit, unit, 1.0)):
        assert (np.abs(a - b) <= (2.0 ** -8 + factor) * np.abs(b) + (2e-3 + 8 * factor) * one).all(), (name, np.abs(a - b).max() / one)
    if dbias:
        assert np.abs(got[3] - ref[3]).max() <= 2e-4 * max(1.0, np.sqrt(N))


@pytest.mark.parametrize("dbias", [False, True])
@pytest.mark.parametrize("value", [-100.0, -6.5e4, -1e6, -1e7])
@pytest.mark.parametrize("L,heads,N,kind", SHAPES[:-1], ids=[f"L{s[0]}_{s[3]}" for s in SHAPES[:-1]])
def test_probabilities_sum_to_one(L, heads, N, kind, value, dbias):
    """dO = 1 makes the columns of dV the sums of the probabilities over the queries, and those of a window the number of its rows --
    also of rows that a finite mask has shut to every key, but for the rounding of M (half an ulp, a power of two) and of dV."""
    import torch
    w, x, _, _, _ = _draw(L, heads, N, kind)
    bias = np.zeros((heads, L, L), np.float32)
    bias[:, ::2] = value  # every second row
    mask = labels = None
    if kind == "labels":
        labels = np.zeros((3, L), np.int32)
    elif kind == "dense":
        mask = np.zeros((min(N, 150), L, L), np.float32)
    got = _call(x, w, bias, mask, labels, w.scale, dbias, torch.ones(N, L, 32 * heads, device="cuda", dtype=torch.bfloat16))
    ulp = 2.0 ** (np.floor(np.log2(abs(value) * 1.4426951 + 8)) - 23)
    total = got[2].sum(1) / L
    assert np.abs(np.log2(total)).max() <= 0.5 * ulp + 2.0 ** -8, (total.min(), total.max())
