"""fp32 products in bf16 thirds keep the 24 bits of every value, however small: inputs, single channels and rows beside
ordinary ones, probabilities and dS, down to where fp32 itself runs out of bits."""
import pytest
import torch

from test_gpu_f32_split import forward, gradients, reference

pytestmark = pytest.mark.gpu


def tensors(n, N, L, C, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((N, L, C), generator=g) for _ in range(n)]


def columns_close(got, want, bound):
    err, size = (got - want).norm(dim=(0, 1)), want.norm(dim=(0, 1))
    worst = (err / size).max()
    print(f"worst channel {worst:.2e}", flush=True)
    assert (size > 0).all() and worst <= bound


# sums of up to 256 products, each rounded to 2^-24 of the largest partial sum, and the exponential
@pytest.mark.parametrize("L", [65, 144, 256])
@pytest.mark.parametrize("small", [1e-31, 1e-33, 1e-35, 1e-36])
def test_forward_channels(L, small):
    q, k, v = tensors(3, 3, L, 64, L)
    v[:, :, 1::4] *= small
    v[:, :, 40] = 0.0
    v[:, ::3, 40] = small
    columns_close(forward(q, k, v, 2, 0.2), reference(q, k, v, 2, 0.2), 2 ** -20)


# A key of weight 3e-34 to 1e-37 is all that a channel has.  fp32 knows a score of 85 to half of 2^-17, times log2(e) to half
# of 2^-17 once more.
@pytest.mark.parametrize("L", [65, 144, 256])
@pytest.mark.parametrize("depth", [77.0, 82.0, 85.0])
def test_forward_probabilities(L, depth):
    import paper_2501_06480_amd as fwa
    q, k, v = tensors(3, 2, L, 64, L + 1)
    q *= 0.1
    bias = torch.zeros(2, L, L)
    bias[:, :, 7] = -depth
    v[:, :, ::2] = 0.0
    v[:, 7, ::2] = torch.linspace(1.0, 3.0, 32)
    o = fwa.fwa_forward(q.cuda(), k.cuda(), v.cuda(), 2, 0.2, bias.cuda()).cpu().double()
    Q, K, V = (t.double().view(2, L, 2, 32).transpose(1, 2) for t in (q, k, v))
    want = (torch.softmax(0.2 * Q @ K.transpose(2, 3).contiguous() + bias.double(), -1) @ V).transpose(1, 2).reshape(2, L, 64)
    # 1e-37 has been divided by L: two more bits go where the result is below the smallest normal number
    columns_close(o, want, 2 ** -15)


# gradients whose dS, the product of P, dO and V, is far smaller than any input
@pytest.mark.parametrize("L", [33, 64])
@pytest.mark.parametrize("d", [32, 64, 256])
@pytest.mark.parametrize("small", [1e-15, 1e-16, 1e-17, 3e-18, 1e-18])
def test_backward_magnitudes(L, d, small):
    import paper_2501_06480_amd as fwa
    q, k, v, d_o = tensors(4, 3, L, 2 * d, L + d)
    v, d_o = v * small, d_o * small
    got = fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, d ** -0.5)[:3]
    for a, b, name in zip(got, gradients(q, k, v, d_o, 2, d ** -0.5), ("dq", "dk", "dv")):
        err = (a.cpu().double() - b).norm() / b.norm()
        print(f"L={L} d={d} {small:g} {name}: {err:.2e}", flush=True)
        # P dS is 1e-38 at 1e-18: fp32 has 18 bits of it
        assert err <= (2 ** -19 if small > 5e-18 else 2 ** -16), name


@pytest.mark.parametrize("L", [33, 49, 64])
@pytest.mark.parametrize("d", [32, 128])
@pytest.mark.parametrize("small", [1e-31, 1e-34, 1e-36])
def test_backward_channels_and_rows(L, d, small):
    import paper_2501_06480_amd as fwa
    q, k, v, d_o = tensors(4, 3, L, 2 * d, L + d + 1)
    q[:, :, 1::8] *= small
    k[:, :, 2::8] *= small
    d_o[:, :, 3::8] *= small
    v[:, :, 4::8] *= small
    got = [t.cpu().double() for t in fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, d ** -0.5)[:3]]
    for a, b in zip(got, gradients(q, k, v, d_o, 2, d ** -0.5)):
        columns_close(a, b, 2 ** -19)
    q, k, v, d_o = tensors(4, 3, L, 2 * d, L + d + 2)
    d_o[:, 1::5] *= small  # rows of dQ
    got = [t.cpu().double() for t in fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, d ** -0.5)[:3]]
    for a, b in zip(got, gradients(q, k, v, d_o, 2, d ** -0.5)):
        columns_close(a.transpose(1, 2), b.transpose(1, 2), 2 ** -17 if small < 1e-35 else 2 ** -19)


# dK and dV of a key that every query gives a weight of 1e-32 to 1e-36 (see test_forward_probabilities for the bound; the
# division by the row sum leaves P two bits fewer at the last)
@pytest.mark.parametrize("L", [33, 64])
@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("depth", [70.0, 76.0, 80.0])
def test_backward_probabilities(L, d, depth):
    import paper_2501_06480_amd as fwa
    q, k, v, d_o = tensors(4, 2, L, 2 * d, L + d + 3)
    q *= 0.1
    bias = torch.zeros(2, L, L)
    bias[:, :, 7] = -depth
    got = [t.cpu().double() for t in fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, d ** -0.5, bias.cuda())[:3]]
    Q, K, V, G = (t.double().view(2, L, 2, d).transpose(1, 2) for t in (q, k, v, d_o))
    P = torch.softmax(d ** -0.5 * Q @ K.transpose(2, 3).contiguous() + bias.double(), -1)
    S = G @ V.transpose(2, 3).contiguous()
    S = P * (S - (P * S).sum(-1, keepdim=True))
    for a, b in zip(got[1:], (d ** -0.5 * S.transpose(2, 3).contiguous() @ Q, P.transpose(2, 3).contiguous() @ G)):
        b = b.transpose(1, 2).reshape(2, L, 2 * d)
        err = (a[:, 7] - b[:, 7]).norm() / b[:, 7].norm()
        print(f"L={L} d={d} depth {depth}: {err:.2e}", flush=True)
        assert err <= 2 ** -15


# parts of a product that overflow with opposite signs: the score is -inf, and its key is dropped
def test_products_beyond_the_range():
    import paper_2501_06480_amd as fwa
    for L, d in ((81, 32), (256, 32), (49, 32), (64, 128)):
        q, k, v, d_o = tensors(4, 2, L, 2 * d, L)
        for x in (1.01e25, 1.003e25, 1.0e25):
            q[:, :, 3] = 0.0
            k[:, :, 3] = 0.0
            q[:, ::2, 3] = x
            k[:, 5, 3] = -1.007e20
            o = fwa.fwa_forward(q.cuda(), k.cuda(), v.cuda(), 2, 0.2).cpu().double()
            Q, K, V, G = (t.double().view(2, L, 2, d).transpose(1, 2) for t in (q, k, v, d_o))
            P = torch.softmax(0.2 * Q @ K.transpose(2, 3).contiguous(), -1)
            want = (P @ V).transpose(1, 2).reshape(2, L, 2 * d)
            assert (o - want).norm() <= 2 ** -20 * want.norm(), (L, d, x)
            if L <= 64:
                got = fwa.fwa_backward(q.cuda(), k.cuda(), v.cuda(), d_o.cuda(), 2, 0.2)[:3]
                for a, b in zip(got, gradients(q, k, v, d_o, 2, 0.2)):
                    a, ok = a.cpu().double(), b.abs() < 3e38
                    assert torch.isfinite(a[ok]).all() and (a - b)[ok].norm() <= 2 ** -19 * b[ok].norm(), (L, d, x)
