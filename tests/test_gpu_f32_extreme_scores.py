"""The fp32 forward with scores far from zero: rows whose keys are all masked by the type's lowest value or by -1e10, scores
of 1e10 and of the type's largest.  The largest score of a row has weight 1 whatever its size."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LOWEST = torch.finfo(torch.float32).min


def reference(q, k, v, heads, scale, term):
    """In 64 bits but for the scores, which are the fp32 values that the kernels compare (products in 64 bits)."""
    N, L, C = q.shape
    Q, K, V = (t.double().view(N, L, heads, 32).transpose(1, 2) for t in (q, k, v))
    S = (scale * Q @ K.transpose(2, 3).contiguous()).float() + term
    return (torch.softmax(S.double(), -1) @ V).transpose(1, 2).reshape(N, L, C)


# 49 is the kernel for short windows, the others one and several query blocks per wave of the one for long windows
@pytest.mark.parametrize("L", [49, 65, 81, 144, 256])
@pytest.mark.parametrize("form", ["lowest", "-1e10", "1e10", "largest", "labels"])
@pytest.mark.parametrize("split", [True, False])
def test_forward(L, form, split):
    import paper_2501_06480_amd as fwa
    heads, N = 2, 6
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn((N, L, 32 * heads), generator=g) for _ in range(3))
    if not split:
        v[:, :, 3] = 0.0
        v[:, 2, 3] = 1.8e38  # beyond what goes through the split products
    term, kw = torch.zeros(N, 1, L, L), {}
    if form == "labels":  # with a label of its own, a mask value of the lowest leaves a token its own key alone
        labels = torch.zeros((N, L), dtype=torch.int32)
        labels[:, ::5] = torch.arange(1, labels[:, ::5].shape[1] + 1, dtype=torch.int32)
        term = torch.where(labels[:, :, None] == labels[:, None, :], 0.0, LOWEST)[:, None]
        kw = dict(labels=labels.cuda(), mask_value=LOWEST)
    elif form in ("lowest", "-1e10"):  # padding tokens: rows without a key
        mask = torch.zeros(N, L, L)
        mask[:, 5::7] = LOWEST if form == "lowest" else -1e10
        mask[1:, :, 3::4] = -100.0
        mask[2, L - 1] = LOWEST
        term, kw = mask[:, None], dict(mask=mask.cuda())
    else:
        bias = torch.randn((heads, L, L), generator=g) * (1e10 if form == "1e10" else 1.0)
        if form == "largest":
            bias[:, :, ::9] = 3e38
            bias[:, 1::2, 4] = -3e38
        term, kw = bias[None], dict(bias=bias.cuda())
    o = fwa.fwa_forward(q.cuda(), k.cuda(), v.cuda(), heads, 32 ** -0.5, **kw).cpu().double()
    want = reference(q, k, v, heads, 32 ** -0.5, term)
    assert torch.isfinite(o).all()
    for c in range(32 * heads):  # per channel: one is far larger than the others
        # the scores' own rounding (2^-24 of up to 100 in the exponent) and the sums
        assert (o[:, :, c] - want[:, :, c]).norm() <= 2 ** -18 * want[:, :, c].norm(), c


# without an additive term the score is a bare product, whose rounding must not come back when the largest one is subtracted
@pytest.mark.parametrize("L", [49, 64, 65, 81, 112, 144, 256])
@pytest.mark.parametrize("size", [1e9, 1.3e15, 1e29, 1e36])
def test_forward_without_a_term(L, size):
    import paper_2501_06480_amd as fwa
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn((6, L, 64), generator=g) for _ in range(3))
    k[1::2] *= size  # every score of the window, one row's, one column's
    q[0, 5] *= size
    k[2, 7] *= size
    o = fwa.fwa_forward(q.cuda(), k.cuda(), v.cuda(), 2, 32 ** -0.5).cpu().double()
    # the two largest scores of a row lie far apart for some rows only: ties within fp32's rounding weigh what they like
    Q, K, V = (t.double().view(6, L, 2, 32).transpose(1, 2) for t in (q, k, v))
    S = 32 ** -0.5 * Q @ K.transpose(2, 3).contiguous()
    top = S.topk(2, -1).values
    sure = ((top[..., 0] - top[..., 1]) > 2 ** -20 * top.abs().amax(-1) + 30) | (S.abs().amax(-1) < 1e3)
    want = (torch.softmax(S, -1) @ V).transpose(1, 2).reshape(6, L, 2, 32)
    sure = sure.transpose(1, 2)
    assert torch.isfinite(o).all() and sure.float().mean() > 0.9
    assert (o.view(6, L, 2, 32) - want)[sure].norm() <= 2 ** -18 * want[sure].norm()


@pytest.mark.parametrize("L,d", [(25, 32), (49, 32), (64, 64), (49, 256)])
@pytest.mark.parametrize("size", [1e9, 1e12, 1e29])
def test_backward_without_a_term(L, d, size):
    import paper_2501_06480_amd as fwa
    g = torch.Generator().manual_seed(L)
    q, k, v, d_o = (torch.randn((4, L, 2 * d), generator=g) for _ in range(4))
    q[1::2] *= size
    got = [t.cpu().double() for t in fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, d ** -0.5)[:3]]
    assert all(torch.isfinite(t).all() for t in got)
    # weights of 0 and 1: dV gathers rows of dO
    Q, K, V, G = (t.double().view(4, L, 2, d).transpose(1, 2) for t in (q, k, v, d_o))
    P = torch.softmax(d ** -0.5 * Q @ K.transpose(2, 3).contiguous(), -1)
    want = (P.transpose(2, 3).contiguous() @ G).transpose(1, 2).reshape(4, L, 2 * d)
    assert (got[2] - want).norm() <= 2 ** -18 * want.norm()
