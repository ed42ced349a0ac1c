"""What cannot go through the native autograd nodes goes through the Python functions: calls that are being traced, tensor
subclasses in any place, forward mode."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N, L, HEADS, D = 4, 49, 3, 32


def fused(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((N, L, 3, HEADS, D), device="cuda", generator=g).bfloat16()


@pytest.mark.parametrize("grad", [False, True])
def test_traced(grad):
    """A traced call computes: its replay on other inputs is the call on those inputs."""
    from paper_2501_06480_amd import autograd
    bias = torch.randn((HEADS, L, L), device="cuda")

    def qkv_call(x):
        return autograd.window_attention_qkv(x, 0.2, bias)

    def three(q, k, v):
        return autograd.window_attention(q, k, v, HEADS, 0.2)

    a, b = (fused(s).requires_grad_(grad) for s in (1, 2))
    rows = [[t[:, :, i].reshape(N, L, -1).contiguous() for i in range(3)] for t in (a.detach(), b.detach())]
    assert torch.equal(torch.jit.trace(qkv_call, (a,), check_trace=False)(b), qkv_call(b))
    assert torch.equal(torch.jit.trace(three, tuple(rows[0]), check_trace=False)(*rows[1]), three(*rows[1]))


class Tagged(torch.Tensor):
    pass


@pytest.mark.parametrize("which", ["q", "k", "v", "bias", "mask", "labels"])
def test_subclasses(which):
    from paper_2501_06480_amd import autograd
    q, k, v = (fused(3)[:, :, i].reshape(N, L, -1).contiguous() for i in range(3))
    bias = torch.randn((HEADS, L, L), device="cuda")
    mask = torch.zeros((2, L, L), device="cuda")
    labels = torch.zeros((2, L), dtype=torch.int32, device="cuda")
    mask, labels = (None, labels) if which == "labels" else (mask, None)
    args = {"q": q, "k": k, "v": v, "bias": bias, "mask": mask, "labels": labels}
    args[which] = args[which].as_subclass(Tagged)
    q = args.pop("q").requires_grad_()
    o = autograd.window_attention(q, args.pop("k"), args.pop("v"), HEADS, 0.2, **args)
    assert "autograd" in type(o.grad_fn).__module__  # the Python function's


def test_forward_mode_is_refused_as_before():
    from paper_2501_06480_amd import autograd
    import torch.autograd.forward_ad as fwd
    x = fused(4)
    with fwd.dual_level():
        dual = fwd.make_dual(x, torch.ones_like(x))
        with pytest.raises(NotImplementedError):
            autograd.window_attention_qkv(dual, 0.2)
        rows = [dual[:, :, i].reshape(N, L, -1) for i in range(3)]
        with pytest.raises(NotImplementedError):
            autograd.window_attention(*rows, HEADS, 0.2)
