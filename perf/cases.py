"""The calls whose speed this library answers for, as data plus the code that makes one pass of each.

A case is one window-attention call as a Swin-style program makes it: ``batch`` images whose token map is cut into
``map_h`` x ``map_w`` windows of ``k`` x ``k`` tokens (N = batch * map_h * map_w windows, L = k * k tokens each),
``heads`` heads of width ``d``, the data type, the additive terms (relative-position bias; the shift mask as a dense
tensor or as region labels) and the direction:

  fwd    ``fwa_forward``: evaluation, or the forward half of a step
  bwd    ``fwa_backward``: the gradient call alone, with the bias gradient where ``dbias`` says so
  train  the attention of one training step through ``autograd.window_attention_qkv``: bias gathered from its table,
         forward and backward on the fused projection output, table gradient scattered

Inputs are what the path meets in training and evaluation: N(0, 1) projections and output gradients, bias tables of
standard deviation 0.02, the 0 / -100 mask of windows shifted by k // 2.
"""
import math

import numpy as np
import torch

import paper_2501_06480_amd as fwa
from paper_2501_06480_amd import autograd, synth

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODE = {"f32": 0, "bf16": 1, "f16": 2}
SIZE = {"f32": 4, "bf16": 2, "f16": 2}


def _case(direction, dtype, batch, map_h, map_w, k, heads, d=32, bias="none", mask="none", dbias=False, name=None):
    c = {"dir": direction, "dtype": dtype, "batch": batch, "map_h": map_h, "map_w": map_w, "k": k, "heads": heads, "d": d,
         "bias": bias, "mask": mask, "dbias": dbias}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one 56 x 56 map, one head, fp32: the smallest call, all launch and latency
        _case("fwd", "f32", 1, 8, 8, 7, 1, name="fwd_f32_one_map"),
        # Swin-T stage 1, batch 128: the workload of bench.py
        _case("fwd", "bf16", 128, 8, 8, 7, 3, name="fwd_stage1"),
        # Swin-T stage 3 (the stage with most blocks), batch 128, a shifted block
        _case("fwd", "bf16", 128, 2, 2, 7, 12, bias="f32", mask="dense", name="fwd_stage3_shift"),
        # Swin-T stage 1 in training, a shifted block: the gradient call with the bias gradient
        _case("bwd", "bf16", 128, 8, 8, 7, 3, bias="f32", mask="dense", dbias=True, name="bwd_stage1_shift"),
        # Swin-T stage 3 in training through autograd on the fused projection, mask as labels
        _case("train", "bf16", 128, 2, 2, 7, 12, bias="f32", mask="labels", dbias=True, name="train_stage3_qkv"),
        # detection: stage 1 of two 800 x 1333 images (200 x 334 tokens, padded to 29 x 48 windows), dense mask
        _case("bwd", "bf16", 2, 29, 48, 7, 3, bias="f32", mask="dense", dbias=True, name="bwd_detection_shift"),
        # 12 x 12 windows of 48 x 48 maps, batch 64, evaluation
        _case("fwd", "bf16", 64, 4, 4, 12, 4, bias="f32", name="fwd_window12"),
        # 16 x 16 windows of 64 x 64 maps, batch 64, a shifted block in training, mask as labels
        _case("bwd", "bf16", 64, 4, 4, 16, 4, bias="f32", mask="labels", dbias=True, name="bwd_window16_shift"),
        # the same windows evaluated in fp32
        _case("fwd", "f32", 16, 4, 4, 16, 4, bias="f32", name="fwd_f32_window16"),
        # ragged everything: 14 x 14 windows, 5 heads, a map of 3 x 5 windows, gradients of q, k, v
        _case("bwd", "bf16", 21, 3, 5, 14, 5, bias="f32", name="bwd_window14_odd"),
        # the kernel benchmark's shape (L = 64, 4 heads of width 64) in half precision, gradient call
        _case("bwd", "f16", 4096, 1, 1, 8, 4, d=64, name="bwd_f16_width64"),
        # the same in fp32
        _case("bwd", "f32", 2048, 1, 1, 8, 4, d=64, name="bwd_f32_width64"),
    ]


MOST_VALUES = 8192 * 49 * 96           # values of q at most (Swin-T stage 1, batch 128)
MOST_PRODUCTS = {"bf16": 1024 * 4 * 256 * 256 * 32, "f16": 1024 * 4 * 256 * 256 * 32, "f32": 2048 * 4 * 64 * 64 * 64}


def draw(rng):
    """Another call of the same ranges: window sides 4 to 16, 1 to 32 heads of width 32 or up to 8 wider ones, maps of one
    window to maps of detection size, from one image to a large batch."""
    while True:
        wide = rng.random() < 0.25
        if wide:
            d, k = rng.choice((64, 128, 256)), rng.randint(4, 8)
            heads = rng.randint(1, 8)
            dtype = rng.choice(("bf16", "f16", "f32"))
        else:
            d, k = 32, rng.choice((4, 5, 6, 7, 7, 7, 8, 8, 9, 10, 11, 12, 12, 13, 14, 15, 16, 16))
            heads = rng.choice((1, 2, 3, 3, 4, 5, 6, 6, 7, 8, 9, 11, 12, 12, 16, 24, 32))
            dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        direction = rng.choice(("fwd", "bwd", "train"))
        if dtype == "f32" and k > 8:
            direction = "fwd"          # the fp32 gradient is there for windows of up to 64 tokens
        side = rng.choice((1, 2, 3, 4, 5, 8, 8, 12))
        map_h, map_w = (rng.randint(20, 40), rng.randint(20, 48)) if rng.random() < 0.15 else (side, max(1, side + rng.choice((0, 0, 0, 1))))
        shifted = map_h > 1 and map_w > 1 and rng.random() < 0.5
        bias = "f32" if shifted or rng.random() < 0.7 else "none"
        mask = rng.choice(("dense", "labels")) if shifted else "none"
        if mask == "dense" and map_h * map_w * k ** 4 > 1 << 23:  # a dense mask of over 32 MB is not kept
            mask = "labels"
        if bias == "f32" and mask != "dense" and rng.random() < 0.15:
            bias = "bf16"
        dbias = direction == "train" or (direction == "bwd" and rng.random() < 0.6)
        dbias = dbias and bias == "f32" and dtype != "f32"
        window = k * k * heads * d
        most = min(MOST_VALUES / window, MOST_PRODUCTS[dtype] / (window * k * k)) / (map_h * map_w)
        if direction == "train":
            most /= 2
        if most < 1:
            continue
        batch = max(1, int(math.exp(rng.uniform(0.0, math.log(most)))))
        return _case(direction, dtype, batch, map_h, map_w, k, heads, d, bias, mask, dbias)


def _sizes(c):
    return c["batch"] * c["map_h"] * c["map_w"], c["k"] ** 2, c["heads"], c["d"]


def _table(c, seed):
    """The relative-position table of a case, [heads, (2k-1)^2] fp32 (numpy)."""
    return synth.bias_table(c["heads"], c["k"], seed * 16 + 8)


def _labels(c):
    return synth.shift_labels(c["map_h"] * c["k"], c["map_w"] * c["k"], c["k"], c["k"] // 2)


def _mask(c):
    return synth.shift_mask(c["map_h"] * c["k"], c["map_w"] * c["k"], c["k"], c["k"] // 2)


def _tensors(c, seed):
    """q, k, v [N, L, C] (train: one qkv [N, L, 3, heads, d]) and, with a gradient, dO."""
    N, L, heads, d = _sizes(c)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=g).to(TORCH[c["dtype"]])

    if c["dir"] == "train":
        return normal(N, L, 3, heads, d), normal(N, L, heads * d)
    return tuple(normal(N, L, heads * d) for _ in range(3 if c["dir"] == "fwd" else 4))


def prepare(case, seed):
    c = case
    N, L, heads, d = _sizes(c)
    s = {"case": c, "scale": float(d) ** -0.5, "bias": None, "mask": None, "labels": None, "workspace": None, "table": None}
    s["tensors"] = _tensors(c, seed)
    if c["bias"] != "none":
        s["table"] = torch.from_numpy(_table(c, seed)).cuda()
        if c["dir"] != "train" or not c["dbias"]:  # a training step gathers the bias itself
            s["bias"] = fwa.fwa_bias_gather(s["table"], c["k"]).to(TORCH[c["bias"]])
    if c["mask"] == "dense":
        s["mask"] = torch.from_numpy(_mask(c)).cuda()
    elif c["mask"] == "labels":
        s["labels"] = torch.from_numpy(_labels(c)).cuda()
    if c["dir"] == "train":
        s["tensors"][0].requires_grad_()
    elif c["dir"] == "bwd":
        need = fwa.fwa_backward_workspace_bytes(N, L, heads * d, heads, CODE[c["dtype"]], c["dbias"])
        s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s, c = state, state["case"]
    if c["dir"] == "fwd":
        q, k, v = s["tensors"]
        return fwa.fwa_forward(q, k, v, c["heads"], s["scale"], s["bias"], s["mask"], labels=s["labels"])
    if c["dir"] == "bwd":
        q, k, v, d_o = s["tensors"]
        dq, dk, dv, db = fwa.fwa_backward(q, k, v, d_o, c["heads"], s["scale"], s["bias"], s["mask"], want_dbias=c["dbias"],
                                          workspace=s["workspace"], labels=s["labels"])
        return {"dq": dq, "dk": dk, "dv": dv, "dbias": db}
    qkv, d_o = s["tensors"]
    bias = s["bias"]
    if c["dbias"]:
        bias = fwa.fwa_bias_gather(s["table"], c["k"]).requires_grad_()
    o = autograd.window_attention_qkv(qkv, s["scale"], bias, s["mask"], labels=s["labels"])
    if not c["dbias"]:
        dqkv, = torch.autograd.grad(o, (qkv,), d_o)
        return {"o": o, "dqkv": dqkv, "dtable": None}
    dqkv, db = torch.autograd.grad(o, (qkv, bias), d_o)
    return {"o": o, "dqkv": dqkv, "dtable": fwa.fwa_bias_scatter(db, c["k"])}


def work(case):
    """Each input once and each output once; the products of Algorithms 1 and 2 (two and five of L x L x d)."""
    c = case
    N, L, heads, d = _sizes(c)
    tile = N * L * heads * d * SIZE[c["dtype"]]
    products = 2 * N * heads * L * L * d
    tensors, matmuls = {"fwd": (4, 2), "bwd": (7, 5), "train": (11, 7)}[c["dir"]]
    extra = 0
    if c["bias"] != "none":
        extra += heads * L * L * (2 if c["bias"] == "bf16" else 4)
    if c["mask"] != "none":
        extra += c["map_h"] * c["map_w"] * L * (L if c["mask"] == "dense" else 1) * 4
    if c["dbias"]:
        extra += heads * L * L * 4
    return {"bytes": tensors * tile + extra, "flops": matmuls * products}


def tolerance(case):
    # Two correct implementations differ by their rounding of the results.  Against exact(), over the listed cases and
    # six drawn ones, the library measures: bf16 results 1.7e-3 to 2.2e-3, half results 2.6e-4 to 3.0e-4, fp32 results
    # 2.2e-7 to 4.7e-7.  About four times that; a single element may lie 40 times as far.
    return {"f32": {"rel": 2e-6, "max": 8e-5}, "f16": {"rel": 1.2e-3, "max": 5e-2}, "bf16": {"rel": 8e-3, "max": 1e-1}}[case["dtype"]]


def exact(case, seed):
    """The same call in 64 bits with plain torch, a few windows at a time."""
    c = case
    N, L, heads, d = _sizes(c)
    scale = float(d) ** -0.5
    dev = torch.device("cuda")
    bias = index = None
    if c["bias"] != "none":
        k = c["k"]
        at = np.stack([np.arange(L) // k, np.arange(L) % k])
        dy, dx = at[:, :, None] - at[:, None, :] + k - 1
        index = torch.from_numpy((dy * (2 * k - 1) + dx).reshape(-1)).to(dev)
        bias = torch.from_numpy(_table(c, seed)).to(dev)[:, index].reshape(heads, L, L)
        bias = bias.to(TORCH[c["bias"]]).double()
    mask = torch.from_numpy(_mask(c)).to(dev) if c["mask"] != "none" else None
    t = _tensors(c, seed)
    if c["dir"] == "train":
        q, k_, v = (t[0][:, :, i].reshape(N, L, heads * d) for i in range(3))
        d_o = t[1]
    else:
        q, k_, v = t[:3]
        d_o = t[3] if c["dir"] == "bwd" else None
    step = max(1, (1 << 26) // (heads * L * L))

    def part(x, a, b):
        return x[a:b].double().reshape(b - a, L, heads, d).transpose(1, 2).contiguous()

    def whole(x, b):
        return x.transpose(1, 2).reshape(b, L, heads * d)

    outs, grads, db = [], [], torch.zeros((heads, L, L), dtype=torch.float64, device=dev)
    for a in range(0, N, step):
        b = min(N, a + step)
        Q, K, V = part(q, a, b), part(k_, a, b), part(v, a, b)
        S = scale * torch.matmul(Q, K.transpose(2, 3).contiguous())
        if bias is not None:
            S += bias
        if mask is not None:
            S += mask[torch.arange(a, b, device=dev) % mask.shape[0]].double()[:, None]
        P = torch.softmax(S, -1)
        del S
        if c["dir"] != "bwd":
            outs.append(whole(torch.matmul(P, V), b - a))
        if d_o is None:
            continue
        G = part(d_o, a, b)
        dS = torch.matmul(G, V.transpose(2, 3).contiguous())
        dS = P * (dS - (P * dS).sum(-1, keepdim=True))
        if c["dbias"]:
            db += dS.sum(0)
        grads.append([whole(scale * torch.matmul(dS, K), b - a),
                      whole(scale * torch.matmul(dS.transpose(2, 3).contiguous(), Q), b - a),
                      whole(torch.matmul(P.transpose(2, 3).contiguous(), G), b - a)])
    if c["dir"] == "fwd":
        return torch.cat(outs)
    dq, dk, dv = (torch.cat([g[i] for g in grads]) for i in range(3))
    if c["dir"] == "bwd":
        return {"dq": dq, "dk": dk, "dv": dv, "dbias": db if c["dbias"] else None}
    dtable = None
    if c["dbias"]:
        dtable = torch.zeros((heads, (2 * c["k"] - 1) ** 2), dtype=torch.float64, device=dev)
        dtable.index_add_(1, index, db.reshape(heads, L * L))
    dqkv = torch.stack([dq, dk, dv], 2).reshape(N, L, 3, heads, d)
    return {"o": torch.cat(outs), "dqkv": dqkv, "dtable": dtable}
