"""fp32 products in bf16 thirds keep the 24 bits of every value, however small: inputs, single channels and rows beside
ordinary ones, probabilities and dS, down to where fp32 itself runs out of bits."""
import pytest
import torch

from test_gpu_f32_split import gradients

pytestmark = pytest.mark.gpu


def tensors(n, N, L, C, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn((N, L, C), generator=g) for _ in range(n)]


def columns_close(got, want, bound):
    err, size = (got - want).norm(dim=(0, 1)), want.norm(dim=(0, 1))
    worst = (err / size).max()
    print(f"worst channel {worst:.2e}", flush=True)
    assert (size > 0).all() and worst <= bound


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


# dK and dV of a key that every query gives a weight of 1e-32 to 1e-36.  fp32 knows a score of 80 to half of 2^-17, times
# log2(e) to half of 2^-17 once more, and the division by the row sum leaves P two bits fewer at the last.
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
