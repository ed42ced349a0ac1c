"""The native autograd nodes do what the Python functions of the same calls do: outputs and gradients bit for bit, saved
tensors through hooks and version counters, errors as the same Python exceptions from either thread."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N, L, HEADS, D = 8, 49, 3, 32


def inputs(dtype=torch.bfloat16, bias=True):
    g = torch.Generator(device="cuda").manual_seed(5)
    qkv = torch.randn((N, L, 3, HEADS, D), device="cuda", generator=g).to(dtype).requires_grad_()
    d_o = torch.randn((N, L, HEADS * D), device="cuda", generator=g).to(dtype)
    b = torch.randn((HEADS, L, L), device="cuda", generator=g) if bias else None
    labels = torch.randint(0, 3, (4, L), device="cuda", generator=g, dtype=torch.int32)
    return qkv, d_o, b, labels


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("bias", ["none", "frozen", "learned"])
@pytest.mark.parametrize("labelled", [False, True])
def test_like_the_python_functions(fused, bias, labelled):
    from paper_2501_06480_amd import autograd
    qkv, d_o, b, labels = inputs(bias=bias != "none")
    labels = labels if labelled else None
    if bias == "learned":
        b.requires_grad_()
    wide = torch.zeros((N, L, 2, HEADS * D), dtype=d_o.dtype, device="cuda")
    wide[:, :, 0] = d_o
    if fused:
        x = (qkv,)
        native = autograd.window_attention_qkv(qkv, 0.2, b, labels=labels, mask_value=-3.0)
        plain = autograd._WindowAttentionQKV.apply(qkv, b, None, 0.2, labels, -3.0)
    else:
        x = tuple(qkv.detach()[:, :, t].reshape(N, L, -1).requires_grad_() for t in range(3))
        native = autograd.window_attention(*x, HEADS, 0.2, b, labels=labels, mask_value=-3.0)
        plain = autograd._WindowAttention.apply(*x, b, None, HEADS, 0.2, labels, -3.0)
    assert "autograd" not in type(native.grad_fn).__module__ and torch.equal(native, plain)
    x += (b,) if bias == "learned" else ()
    for got, want in zip(torch.autograd.grad(native, x, wide[:, :, 0]), torch.autograd.grad(plain, x, d_o)):
        assert torch.equal(got, want)


def test_without_grad_nothing_is_saved():
    from paper_2501_06480_amd import autograd
    qkv, _, b, _ = inputs()
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(t) or t, lambda t: t):
        with torch.no_grad():
            assert autograd.window_attention_qkv(qkv, 0.2, b).grad_fn is None
        assert not seen
        assert autograd.window_attention_qkv(qkv, 0.2, b).requires_grad and len(seen) == 2


def test_a_saved_tensor_that_was_written_to():
    from paper_2501_06480_amd import autograd
    qkv, d_o, b, _ = inputs()
    o = autograd.window_attention_qkv(qkv, 0.2, b)
    b.add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(o, qkv, d_o)


def test_errors_are_those_of_the_direct_calls():
    from paper_2501_06480_amd import autograd, binding
    qkv, d_o, b, labels = inputs()
    with pytest.raises(ValueError, match="bias must be"):
        autograd.window_attention_qkv(qkv, 0.2, b[:2])
    with pytest.raises(binding.FwaError, match="fwa_forward_labels"):
        autograd.window_attention_qkv(torch.zeros((2, 300, 3, 1, 32), dtype=torch.bfloat16, device="cuda"), 0.2,
                                      labels=torch.zeros((1, 300), dtype=torch.int32, device="cuda"))
    with pytest.raises(NotImplementedError, match="gradient of the bias"):
        autograd.window_attention_qkv(qkv.detach().float(), 0.2, b.clone().requires_grad_())
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t[:, :, :2] if t.dim() == 5 else t):
        o = autograd.window_attention_qkv(qkv, 0.2, b)
    with pytest.raises(ValueError, match="qkv must be"):
        o.backward(d_o)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: t.repeat(1, 7, 1, 1, 1) if t.dim() == 5 else t):
        o = autograd.window_attention_qkv(qkv, 0.2)
    with pytest.raises(ValueError, match="d_o must match"):
        o.backward(d_o)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: autograd.window_attention_qkv(t, 0.2).sum())(qkv.detach())


@pytest.mark.parametrize("reentrant", [False, True])
def test_checkpointed(reentrant):
    from torch.utils.checkpoint import checkpoint
    from paper_2501_06480_amd import autograd
    qkv, d_o, b, _ = inputs()
    b.requires_grad_()
    want = torch.autograd.grad(autograd.window_attention_qkv(qkv, 0.2, b), (qkv, b), d_o)
    checkpoint(lambda x, y: autograd.window_attention_qkv(x, 0.2, y), qkv, b, use_reentrant=reentrant).backward(d_o)
    assert torch.equal(qkv.grad, want[0]) and torch.equal(b.grad, want[1])


def test_on_a_stream_of_its_own():
    from paper_2501_06480_amd import autograd
    qkv, d_o, b, _ = inputs()
    want = torch.autograd.grad(autograd.window_attention_qkv(qkv, 0.2, b), qkv, d_o)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        o = autograd.window_attention_qkv(qkv, 0.2, b)
    got = torch.autograd.grad(o, qkv, d_o)  # the engine runs the node on the stream of its forward
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0])
