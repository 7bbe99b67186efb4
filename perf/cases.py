"""The work this library is asked to do, as measurable cases.

A case is one layer of a convolutional network in the paper's notation (I is
i_n x i_h x i_w x i_c as stored, its zero ring included, K is k_h x k_w x i_c x
k_c) with the call a program makes on it:

  lowered  conv2d from a lowered copy of I; L stays in the caller's workspace
  fused    conv2d with no workspace
  dgrad    conv2d_dgrad, the input's gradient
  wgrad    conv2d_wgrad, the kernel's gradient
  train    one training step of a layer: the lowered forward pass, the kernel's
           gradient from the L it left, the input's gradient

Inference programs keep their weights, workspace and output buffer between
calls, and training programs their gradient buffers, so `prepare` makes them.
"""
import math

import torch

import paper_1706_06873_amd as mec


def _case(name, op, dtype, i_n, i_h, i_w, i_c, k_h, k_w, k_c, s, pad):
    return {"name": name, "op": op, "dtype": dtype, "i_n": i_n, "i_h": i_h, "i_w": i_w,
            "i_c": i_c, "k_h": k_h, "k_w": k_w, "k_c": k_c, "s_h": s, "s_w": s, "pad": pad}


def listed():
    return [
        # the smallest call: a 7x7 single-channel image, all latency and launches
        _case("tiny", "lowered", "f32", 1, 7, 7, 1, 3, 3, 1, 1, 0),
        # a deep layer of a residual network on one image: interactive inference
        _case("deep_one_image", "lowered", "f32", 1, 14, 14, 256, 3, 3, 256, 1, 0),
        # sizes that are multiples of nothing, a small batch
        _case("ragged", "fused", "f32", 9, 31, 43, 52, 3, 3, 75, 1, 1),
        # the large first layer (11x11 stride 4) at a full batch: the benchmark's headline
        _case("alexnet_conv1", "lowered", "f32", 128, 227, 227, 3, 11, 11, 96, 4, 0),
        # a 3x3 first layer: its output is twenty times its input
        _case("vgg_first", "fused", "f32", 16, 226, 226, 3, 3, 3, 64, 1, 1),
        # the middle of a residual network
        _case("resnet_mid", "fused", "f32", 32, 58, 58, 64, 3, 3, 64, 1, 1),
        # the same first layer in 16 bits: throughput inference
        _case("first_bf16", "lowered", "bf16", 32, 227, 227, 3, 11, 11, 96, 4, 0),
        # a large strided kernel over many channels in 16 bits
        _case("strided_bf16", "fused", "bf16", 32, 224, 224, 64, 7, 7, 64, 2, 0),
        # deep and narrow in 16 bits, the most arithmetic of all
        _case("deep_bf16", "lowered", "bf16", 256, 16, 16, 512, 3, 3, 512, 1, 1),
        # the gradients of middle layers
        _case("dgrad_mid", "dgrad", "f32", 32, 28, 28, 128, 3, 3, 128, 1, 0),
        _case("wgrad_mid", "wgrad", "f32", 32, 58, 58, 64, 3, 3, 64, 1, 1),
        # a training step of a layer that halves the image
        _case("train_stride2", "train", "f32", 16, 57, 57, 64, 3, 3, 128, 2, 1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A layer of a first, middle or deep part of a network, under any of the
    calls, with odd sizes among them."""
    op, dtype = rng.choice([("lowered", "f32"), ("fused", "f32"), ("lowered", "bf16"),
                            ("fused", "bf16"), ("dgrad", "f32"), ("wgrad", "f32"),
                            ("train", "f32")])
    first = op not in ("dgrad", "train") and rng.random() < 0.35  # no gradient of the image itself
    if first:
        k, s = rng.choice([(11, 4), (7, 2), (5, 2), (3, 1)])
        i_c = 3
        i_h = rng.randint(64, 231)
        k_c = rng.choice([32, 64, 96, rng.randint(24, 100)])
    else:
        k, s = rng.choice([(3, 1), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2), (1, 1)])
        i_h = _log_int(rng, max(7, k), 112)
        i_c, k_c = _log_int(rng, 16, 512), _log_int(rng, 16, 512)
        if rng.random() < 0.6:  # most networks round their channels
            i_c, k_c = (max(16, 16 * round(c / 16)) for c in (i_c, k_c))
    i_w = max(k, i_h + rng.choice([0, 0, 0, rng.randint(-5, 5)]))
    case = _case("", op, dtype, _log_int(rng, 1, 128), i_h, i_w, i_c, k, k, k_c, s, rng.choice([0, k // 2]))
    del case["name"]
    while case["i_n"] > 1:  # no dearer than the largest listed layer
        w = work(case)
        if w["flops"] <= (12e9 if dtype == "f32" else 60e9) and w["bytes"] <= 3e8:
            break
        case["i_n"] = (case["i_n"] + 1) // 2
    while work(case)["flops"] > (12e9 if dtype == "f32" else 60e9):
        case["k_c"] = (case["k_c"] + 1) // 2
    return case


def _out(case):
    return ((case["i_h"] - case["k_h"]) // case["s_h"] + 1,
            (case["i_w"] - case["k_w"]) // case["s_w"] + 1)


def _dims(case):
    return tuple(case[k] for k in ("i_n", "i_h", "i_w", "i_c", "k_h", "k_w", "k_c", "s_h", "s_w"))


def _inputs(case, seed):
    """I, K and the gradient of O: an image in [0, 1] for first layers, else
    what a ReLU leaves, inside its ring of zeros; weights of the usual scale."""
    i_n, i_h, i_w, i_c, k_h, k_w, k_c, _, _ = _dims(case)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (i_n, i_h, i_w, i_c)
    if i_c <= 3:
        I = torch.rand(shape, generator=gen, device="cuda")
    else:
        I = torch.randn(shape, generator=gen, device="cuda").relu_()
    p = case["pad"]
    if p:
        I[:, :p] = 0
        I[:, -p:] = 0
        I[:, :, :p] = 0
        I[:, :, -p:] = 0
    K = torch.randn((k_h, k_w, i_c, k_c), generator=gen, device="cuda") * math.sqrt(2.0 / (k_h * k_w * i_c))
    G = None
    if case["op"] in ("dgrad", "wgrad", "train"):
        G = torch.randn((i_n,) + _out(case) + (k_c,), generator=gen, device="cuda") * 0.01
    return I.to(dt), K.to(dt), G


def prepare(case, seed):
    d, op = _dims(case), case["op"]
    i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w = d
    o_h, o_w = _out(case)
    I, K, G = _inputs(case, seed)
    s = {"op": op, "s": (s_h, s_w), "size": (i_h, i_w), "k": (k_h, k_w), "K": K, "G": G}
    if op != "dgrad":
        s["I"] = I
    if op in ("lowered", "fused", "train"):
        s["O"] = torch.empty((i_n, o_h, o_w, k_c), device="cuda")
    if op in ("lowered", "train"):
        s["L"] = torch.empty((i_n, o_w, i_h, k_w, i_c), dtype=I.dtype, device="cuda")
    if op in ("dgrad", "train"):
        s["dI"] = torch.empty((i_n, i_h, i_w, i_c), device="cuda")
        need = mec.grad_workspace_bytes(*d, grad_pass=mec.GRAD_INPUT)
        s["dI_ws"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    if op in ("wgrad", "train"):
        s["dK"] = torch.empty((k_h, k_w, i_c, k_c), device="cuda")
        need = mec.grad_workspace_bytes(
            *d, grad_pass=mec.GRAD_KERNEL if op == "wgrad" else mec.GRAD_KERNEL_FROM_L)
        s["dK_ws"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    op, (s_h, s_w), (i_h, i_w) = s["op"], s["s"], s["size"]
    got = {}
    if op == "fused":
        got["O"] = mec.conv2d(s["I"], s["K"], s_h, s_w, algo="fused", O=s["O"])
    if op in ("lowered", "train"):
        got["O"] = mec.conv2d(s["I"], s["K"], s_h, s_w, workspace=s["L"], O=s["O"])
        got["L"] = s["L"]
    if op == "wgrad":
        got["dK"] = mec.conv2d_wgrad(s["I"], s["G"], *s["k"], s_h, s_w, dK=s["dK"],
                                     workspace=s["dK_ws"])
    if op == "train":
        got["dK"] = mec.wgrad_gemm(s["L"], s["G"], s["k"][0], i_w, s_h, s_w, dK=s["dK"],
                                   workspace=s["dK_ws"])
    if op in ("dgrad", "train"):
        got["dI"] = mec.conv2d_dgrad(s["G"], s["K"], i_h, i_w, s_h, s_w, dI=s["dI"],
                                     workspace=s["dI_ws"])
    return got


def work(case):
    i_n, i_h, i_w, i_c, k_h, k_w, k_c, _, _ = _dims(case)
    o_h, o_w = _out(case)
    op, es = case["op"], 4 if case["dtype"] == "f32" else 2
    I, K, O = i_n * i_h * i_w * i_c, k_h * k_w * i_c * k_c, i_n * o_h * o_w * k_c
    L = i_n * o_w * i_h * k_w * i_c
    passes = 3 if op == "train" else 1
    flops = 2.0 * passes * O * k_h * k_w * i_c
    moved = {"lowered": es * (I + K + L) + 4 * O, "fused": es * (I + K) + 4 * O,
             "dgrad": 4 * (O + K + I), "wgrad": 4 * (I + O + K),
             # I, K and G read, O, L, dK and dI written
             "train": 4 * (I + K + O + O + L + K + I)}[op]
    return {"bytes": float(moved), "flops": flops}


def tolerance(case):
    # Inputs of either type are multiplied exactly or to 32 bits and summed in
    # 32 bits, so one bound serves both: four times what a change of summation
    # order shows on the longest reductions (the kernel's gradient, some 1e5
    # terms, and the 7x7 kernels over hundreds of channels: 1e-6). L is a copy.
    return {"rel": 4e-6, "max": 2e-4}


def exact(case, seed):
    """The same outputs from products of float64 matrices, one kernel tap at a time."""
    i_n, i_h, i_w, i_c, k_h, k_w, k_c, s_h, s_w = _dims(case)
    o_h, o_w = _out(case)
    op = case["op"]
    I, K, G = _inputs(case, seed)
    I, K = I.double(), K.double()
    G = None if G is None else G.double().reshape(-1, k_c)
    got = {}

    def patch(t, a, b):  # the pixels that kernel tap (a, b) meets
        return t[:, a:a + s_h * (o_h - 1) + 1:s_h, b:b + s_w * (o_w - 1) + 1:s_w, :]

    taps = [(a, b) for a in range(k_h) for b in range(k_w)]
    if op in ("lowered", "fused", "train"):
        O = torch.zeros((i_n * o_h * o_w, k_c), dtype=torch.float64, device="cuda")
        for a, b in taps:
            O.addmm_(patch(I, a, b).reshape(-1, i_c), K[a, b])
        got["O"] = O.reshape(i_n, o_h, o_w, k_c)
    if op in ("lowered", "train"):
        L = torch.empty((i_n, o_w, i_h, k_w, i_c), dtype=torch.float64, device="cuda")
        for b in range(k_w):
            L[:, :, :, b] = I[:, :, b:b + s_w * (o_w - 1) + 1:s_w].transpose(1, 2)
        got["L"] = L
    if op in ("wgrad", "train"):
        dK = torch.empty((k_h, k_w, i_c, k_c), dtype=torch.float64, device="cuda")
        for a, b in taps:
            dK[a, b] = patch(I, a, b).reshape(-1, i_c).t().contiguous() @ G
        got["dK"] = dK
    if op in ("dgrad", "train"):
        dI = torch.zeros((i_n, i_h, i_w, i_c), dtype=torch.float64, device="cuda")
        for a, b in taps:
            patch(dI, a, b).add_((G @ K[a, b].t().contiguous()).reshape(i_n, o_h, o_w, i_c))
        got["dI"] = dI
    return got
