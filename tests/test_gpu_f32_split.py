"""The fp32 forward for more than 64 tokens and the fp32 backward from 33 tokens on multiply in bf16 thirds: values over the
whole range of fp32, tiles that workgroups walk, and an error no larger than fp32 arithmetic has."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def tensors(N, L, heads, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((N, L, 32 * heads), generator=g) for _ in range(3)]


def reference(q, k, v, heads, scale):
    N, L, C = q.shape
    Q, K, V = (t.double().view(N, L, heads, 32).transpose(1, 2) for t in (q, k, v))
    P = torch.softmax(scale * Q @ K.transpose(2, 3).contiguous(), -1)
    return (P @ V).transpose(1, 2).reshape(N, L, C)


def forward(q, k, v, heads, scale):
    import paper_2501_06480_amd as fwa
    o = fwa.fwa_forward(q.cuda(), k.cuda(), v.cuda(), heads, scale).cpu().double()
    torch.cuda.synchronize()
    return o


# more tiles than workgroups are resident, for every count of waves; a sum of L products of 24-bit values, each rounded to
# 2^-24 of the largest partial sum, and the exponential: 2^-22 of the result's root mean square covers both
@pytest.mark.parametrize("L", [65, 96, 100, 128, 144, 160, 169, 196, 209, 225, 256])
def test_walked_tiles_and_error(L):
    heads, N = 3, 700 if L < 100 else 400
    q, k, v = tensors(N, L, heads, L)
    o, want = forward(q, k, v, heads, 32 ** -0.5), reference(q, k, v, heads, 32 ** -0.5)
    err = (o - want).norm() / want.norm()
    print(f"L={L} error {err:.2e}", flush=True)
    assert err < 2 ** -22


@pytest.mark.parametrize("L", [81, 144, 256])
def test_the_whole_range(L):
    heads, N = 2, 6
    q, k, v = tensors(N, L, heads, 7 + L)
    v[0] *= 1e-30                   # tiny values
    v[5] *= 1e-37
    v[1, :, :32] *= 1e32            # large ones, one of which rounds to infinity in bf16
    v[1, 3, 0] = 3.395e38
    q[1] *= 1e-3                    # (weights of 1 / L: nothing overflows)
    k[1, 3] = 0
    q[2, 5] *= 3e37                 # a query block beyond the split, with keys that bring its scores back
    k[2] *= 1e-37
    k[3, 2, 4] = float("inf")       # the key's scores are +-inf: rows that see +inf are NaN, the others drop the key
    v[4, 1, 9] = float("nan")       # one channel of one head
    q[4, 2, 40] = float("nan")      # one row of the other
    o, want = forward(q, k, v, heads, 0.2), reference(q, k, v, heads, 0.2)
    assert torch.equal(torch.isnan(o), torch.isnan(want)) and torch.equal(torch.isinf(o), torch.isinf(want))
    assert torch.isnan(want[3]).any() and not torch.isnan(want[3, :, 32:]).any() and not torch.isnan(want[3, :, :32]).all()
    for w in range(N):
        for h in range(heads):
            a, b = o[w, :, 32 * h:32 * h + 32], want[w, :, 32 * h:32 * h + 32]
            ok = torch.isfinite(b)
            # fp32 scores of up to 60 in the exponent: 2^-24 of them times log2(e) each way, and the sums
            assert (a - b)[ok].norm() <= 2 ** -18 * b[ok].norm(), (w, h)


def gradients(q, k, v, d_o, heads, scale):
    N, L, C = q.shape
    Q, K, V, G = (t.double().view(N, L, heads, C // heads).transpose(1, 2) for t in (q, k, v, d_o))
    P = torch.softmax(scale * Q @ K.transpose(2, 3).contiguous(), -1)
    S = G @ V.transpose(2, 3).contiguous()
    S = P * (S - (P * S).sum(-1, keepdim=True))
    out = scale * S @ K, scale * S.transpose(2, 3).contiguous() @ Q, P.transpose(2, 3).contiguous() @ G
    return [t.transpose(1, 2).reshape(N, L, C) for t in out]


# either side of the line between the two kernels, and the remainders above it
@pytest.mark.parametrize("L", [17, 32, 33, 48, 49, 63, 64])
@pytest.mark.parametrize("d", [32, 64, 128, 256])
def test_backward(L, d):
    import paper_2501_06480_amd as fwa
    heads, N = 2, 9
    g = torch.Generator().manual_seed(L + d)
    q, k, v, d_o = (torch.randn((N, L, d * heads), generator=g) for _ in range(4))
    d_o[0] *= 1e-30                 # tiny gradients
    v[1, :, :d] *= 1e-37
    d_o[1, :, :d] *= 1e30
    q[2, 5] *= 1e33                 # a row that fits the split in part, with keys that bring its scores back
    k[2] *= 1e-33
    d_o[3, 2, 4] = float("nan")     # one head of a window
    k[4, 3, d + 1] = float("inf")
    v[5, 1, 2] = 3.395e38           # rounds to infinity in bf16
    d_o[5, :, 2] = 0
    got = fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), heads, d ** -0.5)[:3]
    torch.cuda.synchronize()
    for a, b, name in zip(got, gradients(q, k, v, d_o, heads, d ** -0.5), ("dq", "dk", "dv")):
        a = a.cpu().double()
        for w in range(N):
            for h in range(heads):
                x, y = a[w, :, d * h:d * h + d], b[w, :, d * h:d * h + d]
                assert torch.equal(torch.isnan(x), torch.isnan(y)), (name, w, h)
                ok = torch.isfinite(y) & (y.abs() < 3e38)
                # sums of L and of d products in 2^-24 each, twice, and dP - delta cancels part of it
                assert (x - y)[ok].norm() <= 2 ** -19 * y[ok].norm(), (name, w, h)


def spoil(x, windows, what):
    """The same tensor with a value that the split does not take in one row of each of these windows."""
    x = x.clone()
    x[windows, 3, 5] = what
    return x


# Workgroups that walk several tiles, some of which leave for the fp32 instruction: one after the other, every other one and
# whole rounds of them, with bias and labels.  What a window gets does not depend on what the others hold.
@pytest.mark.parametrize("L,N,heads", [(81, 900, 3), (100, 700, 2), (144, 500, 3), (196, 400, 3), (256, 330, 3)])
@pytest.mark.parametrize("form", ["none", "labels", "dense", "bf16"])
def test_walked_tiles_of_both_kinds(L, N, heads, form):
    import paper_2501_06480_amd as fwa
    q, k, v = tensors(N, L, heads, 3 * L)
    g = torch.Generator().manual_seed(L)
    bias = torch.randn((heads, L, L), generator=g).bfloat16().float()
    labels = torch.randint(0, 3, (2, L), generator=g, dtype=torch.int32)
    mask = torch.where(labels[:, :, None] == labels[:, None, :], 0.0, -4.0)
    kw = {"none": {}, "labels": dict(labels=labels.cuda(), mask_value=-4.0), "dense": dict(mask=mask.cuda()), "bf16": {}}[form]
    b = None if form == "none" else (bias.cuda().bfloat16() if form == "bf16" else bias.cuda())

    def call(*x):
        return fwa.fwa_forward(*(t.cuda() for t in x), heads, 0.2, b, **kw).cpu()

    bad = torch.rand(N, generator=g) < 0.35
    bad[N // 2:N // 2 + 270 // heads] = True  # a round of all workgroups, about
    clean = call(q, k, v)
    for x in ((q, spoil(k, bad, 1e30), v), (q, k, spoil(v, bad, float("nan"))), (spoil(q, bad, 1e25), k, v)):
        o = call(*x)
        assert torch.equal(o[~bad], clean[~bad])
        some = torch.where(bad)[0][:: max(1, int(bad.sum()) // 40)]
        Q, K, V = (t[some].double().view(len(some), L, heads, 32).transpose(1, 2) for t in x)
        S = 0.2 * Q @ K.transpose(2, 3).contiguous()
        S += 0 if b is None else bias.double()
        S += mask.double()[some % 2][:, None] if kw else 0
        want = (torch.softmax(S, -1) @ V).transpose(1, 2).reshape(len(some), L, 32 * heads)
        got = o[some].double()
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        ok = torch.isfinite(want)
        assert (got - want)[ok].norm() <= 2 ** -18 * want[ok].norm()


# on both sides of the magnitudes from which on the fp32 instruction takes over, with a scale that brings the scores back (from
# 2^62 on the sums of 32 products are beyond fp32, whatever makes them: 32 * 2^124 > 2^128)
@pytest.mark.parametrize("L", [81, 256])
@pytest.mark.parametrize("power_qk,power_v", [(60, 86), (61, 0), (0, 87), (61, 100)])
def test_forward_about_the_limits(L, power_qk, power_v):
    g = torch.Generator().manual_seed(L)
    q, k, v = ((torch.rand((3, L, 64), generator=g) * 0.5 + 0.49) * torch.randn((3, L, 64), generator=g).sign() for _ in range(3))
    q, k, v = q * 2.0 ** power_qk, k * 2.0 ** power_qk, v * 2.0 ** power_v
    scale = 0.3 * 2.0 ** (-2 * power_qk)
    o, want = forward(q, k, v, 2, scale), reference(q, k, v, 2, scale)
    assert (o - want).norm() <= 2 ** -20 * want.norm()


def test_forward_with_a_large_scale():
    q, k, v = tensors(3, 144, 2, 12)
    q *= 2.0 ** -122
    o, want = forward(q, k, v, 2, 0.2 * 2.0 ** 122), reference(q, k, v, 2, 0.2 * 2.0 ** 122)
    assert (o - want).norm() <= 2 ** -20 * want.norm()


# tiles of both kinds in one call, with bias and mask; a value beyond the split in each input, and in dS alone
@pytest.mark.parametrize("L,d", [(33, 32), (49, 32), (64, 64), (49, 128), (64, 256)])
@pytest.mark.parametrize("form", ["labels", "dense"])
def test_backward_of_both_kinds(L, d, form):
    import paper_2501_06480_amd as fwa
    heads, N = 2, 24
    g = torch.Generator().manual_seed(L + d)
    x = [torch.randn((N, L, d * heads), generator=g) for _ in range(4)]
    bias = torch.randn((heads, L, L), generator=g)
    labels = torch.randint(0, 3, (2, L), generator=g, dtype=torch.int32)
    mask = torch.where(labels[:, :, None] == labels[:, None, :], 0.0, -4.0)
    kw = dict(labels=labels.cuda(), mask_value=-4.0) if form == "labels" else dict(mask=mask.cuda())

    def call(y):
        out = fwa.fwa_backward(*(t.cuda() for t in y), heads, d ** -0.5, bias.cuda(), **kw)[:3]
        return [t.cpu() for t in out]

    clean = call(x)
    for which in range(5):
        y, bad = [t.clone() for t in x], torch.rand(N, generator=g) < 0.4
        if which < 4:
            y[which][bad, 3, 5] = 2.0 ** 45  # a query's or key's own scores, V, or gradients
        else:
            y[2][bad] *= 2.0 ** 30
            y[3][bad] *= 2.0 ** 30
        got = call(y)
        Q, K, V, G = (t.double().view(N, L, heads, d).transpose(1, 2) for t in y)
        P = torch.softmax(d ** -0.5 * Q @ K.transpose(2, 3).contiguous() + bias.double() + mask.double()[torch.arange(N) % 2][:, None], -1)
        S = G @ V.transpose(2, 3).contiguous()
        S = P * (S - (P * S).sum(-1, keepdim=True))
        want = (d ** -0.5 * S @ K, d ** -0.5 * S.transpose(2, 3).contiguous() @ Q, P.transpose(2, 3).contiguous() @ G)
        for a, c, b in zip(got, clean, want):
            assert torch.equal(a[~bad], c[~bad])
            b = b.transpose(1, 2).reshape(N, L, d * heads)
            for w in torch.where(bad)[0]:
                # scores of 2^45 differ by far more than the exponent of a float: weights are 0 or 1, and dS of weight 1 is
                # dP - delta, the rounding of a sum of d products
                assert (a[w].double() - b[w]).norm() <= 2 ** -19 * b[w].norm() + 2 ** -20 * y[3][w].norm() * (y[2][w].norm() + y[1][w].norm()), which
