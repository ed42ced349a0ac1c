"""The fused-qkv calls read three slices of one tensor in place: only a contiguous [N, L, 3, heads, d] tensor may reach
them.  The checks stand in front of the one for a GPU tensor, so they are met without a GPU.  Between a forward and its
backward a saved-tensor hook may hand the tensor back in another layout; the gradients are those of its values."""
import pytest
import torch

from paper_2501_06480_amd import autograd, binding, synth

N, L, HEADS, D = 4, 9, 2, 32


def layouts():
    base = torch.zeros((N, L, 3, HEADS, D), dtype=torch.bfloat16)
    return {
        "two slices": base[:, :, :2].contiguous(),
        "one slice": base[:, :, :1].contiguous(),
        "four dimensions": torch.zeros((N, L, 3, HEADS * D), dtype=torch.bfloat16),
        "rows of a wider buffer": torch.zeros((N, L, 4, HEADS, D), dtype=torch.bfloat16)[:, :, :3],
        "heads in front of the slices": torch.zeros((N, L, HEADS, 3, D), dtype=torch.bfloat16).transpose(2, 3),
        "windows on the inside": torch.zeros((L, N, 3, HEADS, D), dtype=torch.bfloat16).transpose(0, 1),
    }


@pytest.mark.parametrize("name", list(layouts()))
def test_other_layouts_are_refused(name):
    qkv = layouts()[name]
    with pytest.raises(ValueError, match="qkv"):
        binding.fwa_forward_qkv(qkv, 0.1)
    with pytest.raises(ValueError, match="qkv"):
        binding.fwa_backward_qkv(qkv, torch.zeros((N, L, HEADS * D), dtype=torch.bfloat16), 0.1)


def test_the_right_layout_passes_on_to_the_next_check():
    qkv = torch.zeros((N, L, 3, HEADS, D), dtype=torch.bfloat16)
    with pytest.raises(TypeError, match="GPU"):
        binding.fwa_forward_qkv(qkv, 0.1)
    with pytest.raises(TypeError, match="GPU"):
        binding.fwa_backward_qkv(qkv, torch.zeros((N, L, HEADS * D), dtype=torch.bfloat16), 0.1)


def plain(qkv, scale):
    q, k, v = (qkv[:, :, t].transpose(1, 2) for t in range(3))
    return (torch.softmax(scale * q @ k.transpose(2, 3), -1) @ v).transpose(1, 2).flatten(2)


def repacked(t):
    """The values of t as a view of a wider buffer (the fused tensor alone; the others as they are)."""
    if t.dim() != 5:
        return t
    wide = torch.full((*t.shape[:2], 4, *t.shape[3:]), 7.0, dtype=t.dtype, device=t.device)
    wide[:, :, :3] = t
    return wide[:, :, :3]


def test_a_hook_that_repacks_the_saved_tensor_in_front_of_the_native_call(monkeypatch):
    """What the autograd function hands to the native backward, with the native calls stood in for on the CPU."""
    seen = []

    def backward_qkv(qkv, d_o, scale, *rest):
        seen.append(qkv)
        x = qkv.detach().requires_grad_()
        with torch.enable_grad():
            return torch.autograd.grad(plain(x, scale), x, d_o)[0].contiguous(), None

    monkeypatch.setattr(binding, "fwa_forward_qkv", lambda qkv, scale, *rest: plain(qkv, scale))
    monkeypatch.setattr(binding, "fwa_backward_qkv", backward_qkv)
    torch.manual_seed(3)
    qkv = torch.randn((N, L, 3, HEADS, D), requires_grad=True)
    g = torch.randn((N, L, HEADS * D))
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, repacked):
        autograd.window_attention_qkv(qkv, 0.2).backward(g)
    assert seen[0].is_contiguous() and torch.equal(seen[0], qkv)
    want, = torch.autograd.grad(plain(qkv, 0.2), qkv, g)
    assert torch.equal(qkv.grad, want)


@pytest.mark.gpu
@pytest.mark.parametrize("side", [7, 10])
def test_a_hook_that_repacks_the_saved_tensor(oracle, side):
    from gpu_util import TOL, check_bf16_output, f32_device, max_abs, to_device, to_f64
    w = synth.Workload(f"repacked_{side}", 24, side * side, 96, 3, "bf16", 9700 + side, 0, backward=True)
    x = synth.draw(w)
    bias_np = synth.normal((w.heads, w.L, w.L), 9710 + side, 0.5)
    qkv = torch.stack([to_device(x, w, n) for n in ("q", "k", "v")], 2).view(w.N, w.L, 3, w.heads, 32).requires_grad_()
    bias = f32_device(bias_np).requires_grad_()
    g = to_device(x, w, "d_o")
    plain_grads = torch.autograd.grad(autograd.window_attention_qkv(qkv, w.scale, bias), (qkv, bias), g)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, repacked):
        autograd.window_attention_qkv(qkv, w.scale, bias).backward(g)
    torch.cuda.synchronize()
    assert torch.equal(qkv.grad, plain_grads[0]) and torch.equal(bias.grad, plain_grads[1])
    ref = oracle.backward(x["q"], x["k"], x["v"], x["d_o"], w.heads, w.scale, bias_np, None)
    for t, (nme, want) in enumerate(zip(("dq", "dk", "dv"), ref)):
        check_bf16_output(to_f64(qkv.grad[:, :, t].reshape(w.N, w.L, w.C)), want, nme)
    assert max_abs(to_f64(bias.grad), ref[3]) <= TOL["bf16"]
