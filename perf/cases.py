"""The work that this library's performance is measured on.

Every case is one pass through the public entry points of
paper_2006_12645_amd.gba, as a program that uses the library calls them.  Two
kinds of case:

  "call"   one fused request, C = act(pro(A).B +/- pro(P).Q +/- bias), called
           eagerly: gemm_bias_act where that entry point can express it, else
           fused_gemm.  Layouts are two letters, A's then B's: R row-major,
           C column-major.  With weights stored (out, in), a linear layer's
           forward pass is RC, the gradient of its input RR and the gradient
           of its weights CR.
  "stack"  a feed-forward stack at inference: `blocks` pairs of width ->
           hidden (bias and ReLU) and hidden -> width (bias) layers over a
           few rows, captured once in a HIP graph that a pass replays.
"""
import math

import torch

from paper_2006_12645_amd import gba

# Products of a pass (2MNK) that no drawn case exceeds: the 4095^3 case's.
MOST_FLOPS = 2 * 4095 ** 3


def _call(layout, M, N, K, **more):
    case = {"kind": "call", "layout": layout, "M": M, "N": N, "K": K, "accum": "f32", "act": "relu",
            "bias": "row", "bias_op": "add", "prologue": "none", "second": "none", "K2": 0}
    case.update(more)
    return case


def _stack(M, width, hidden, blocks, accum="f32"):
    return {"kind": "stack", "M": M, "width": width, "hidden": hidden, "blocks": blocks, "accum": accum}


def listed():
    cases = [
        # the smallest call: latency of the entry point and of one launch
        ("tiny_128", _call("RC", 128, 128, 128)),
        # decoding a handful of sequences through four feed-forward blocks
        ("decode_stack_m4", _stack(4, 1024, 4096, 4)),
        # the same network on a batch of 32
        ("infer_stack_m32", _stack(32, 1024, 4096, 4)),
        # a small inference batch with fp16 accumulation
        ("infer_m128_acc16", _call("RC", 128, 4096, 1024, accum="f16")),
        # sizes that are no tile multiple, both operands stored transposed
        ("ragged_1000_cc", _call("CC", 1000, 1000, 1000)),
        # odd sizes and odd leading dimensions, so no row is 16-byte aligned
        ("odd_4095", _call("RC", 4095, 4095, 4095)),
        # training, feed-forward layer: forward (up), input gradient, weight gradient
        ("mlp_up_forward", _call("RC", 8192, 4096, 1024)),
        ("mlp_down_input_grad", _call("RR", 8192, 1024, 4096, act="none", bias="none")),
        ("mlp_weight_grad", _call("CR", 4096, 1024, 8192, act="none", bias="none")),
        # the large square product of the library's headline benchmark
        ("cube_4096", _call("RC", 4096, 4096, 4096)),
        # a gate: tanh of the difference of two products of rectified inputs and a full bias matrix
        ("gate_2048", _call("RC", 2048, 2048, 2048, act="tanh", bias="full", prologue="relu", second="sub", K2=1024)),
        # a long reduction over few outputs (split across workgroups)
        ("long_reduction", _call("RC", 64, 512, 32768)),
    ]
    return [dict(case, name=name) for name, case in cases]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, step):
    v = _spread(rng, lo, hi)
    return max(lo, min(hi, v // step * step)) if v >= step else v


def draw(rng):
    """One more case of the ranges above: stacks of 1 to 64 rows, requests of
    1 to 8192 rows and 32 to 8192 columns over reductions of 64 to 8192 (or
    few outputs over 16384 to 65536), a third of them of any size, the others
    multiples of 8 or 128, over every option."""
    if rng.random() < 0.2:
        width = 64 * _spread(rng, 8, 32)
        return _stack(_spread(rng, 1, 64), width, 4 * width, rng.randint(1, 4), rng.choice(["f32", "f32", "f32", "f16"]))
    step = rng.choice([1, 8, 128])
    if rng.random() < 0.12:
        M, N, K = _size(rng, 32, 512, step), _size(rng, 32, 512, step), _size(rng, 16384, 65536, step)
    else:
        while True:
            M, N, K = _size(rng, 1, 8192, step), _size(rng, 32, 8192, step), _size(rng, 64, 8192, step)
            if 4 * M * N * K <= MOST_FLOPS:
                break
    case = _call(rng.choice(["RC"] * 4 + ["RR"] * 2 + ["CR"] * 2 + ["CC"]), M, N, K,
                 act=rng.choice(["relu", "relu", "none", "sigmoid", "tanh"]),
                 bias=rng.choice(["row", "row", "row", "none", "full"]))
    if K <= 8192 and rng.random() < 0.15:
        case["accum"] = "f16"
    if rng.random() < 0.15:
        case["prologue"] = "relu"
    if K <= 8192 and rng.random() < 0.15:
        case["second"] = rng.choice(["add", "sub"])
        case["K2"] = max(64, min(K, _size(rng, 64, 8192, step)))
    if case["bias"] != "none" and rng.random() < 0.2:
        case["bias_op"] = "sub"
    return case


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))


def _uniform(g, *shape):
    return (torch.rand(shape, generator=g, device="cuda") * 2 - 1).half()


def _normal(g, std, *shape):
    return (torch.randn(shape, generator=g, device="cuda") * std).half()


def _inputs(case, seed):
    """The tensors of a case, all fp16: operands uniform in [-1, 1] for a
    call (those of a reduction above 4096 normal with the deviation that
    keeps outputs near 1), normal activations and weights for a stack."""
    g = _generator(seed)
    if case["kind"] == "stack":
        M, d, h = case["M"], case["width"], case["hidden"]
        x = _normal(g, 1.0, M, d)
        layers = []
        for _ in range(case["blocks"]):
            layers.append((_normal(g, d ** -0.5, h, d), _normal(g, 0.1, h), "relu"))
            layers.append((_normal(g, h ** -0.5, d, h), _normal(g, 0.1, d), "none"))
        return x, layers
    M, N, K, K2 = case["M"], case["N"], case["K"], case["K2"]
    ktot = K + K2

    def operand(rows, cols, layout):
        shape = (rows, cols) if layout == "R" else (cols, rows)
        # sigmoid and tanh: outputs spread over their range instead of saturating
        small = ktot > 4096 or case["act"] in ("sigmoid", "tanh")
        t = _normal(g, ktot ** -0.25, *shape) if small else _uniform(g, *shape)
        return t if layout == "R" else t.t()

    la, lb = case["layout"]
    t = {"A": operand(M, K, la), "B": operand(K, N, lb)}
    if case["second"] != "none":
        t["P"], t["Q"] = operand(M, K2, la), operand(K2, N, lb)
    if case["bias"] != "none":
        t["bias"] = _uniform(g, N) if case["bias"] == "row" else _uniform(g, M, N)
    return t


def prepare(case, seed):
    """Inputs on the GPU; for a stack also its output buffers and the
    captured graph, which a serving program makes once."""
    if case["kind"] == "call":
        return {"case": case, "t": _inputs(case, seed)}
    x, layers = _inputs(case, seed)
    outs = [torch.empty((case["M"], w.shape[0]), dtype=torch.float16, device="cuda") for w, _, _ in layers]

    def forward():
        h = x
        for (w, b, act), out in zip(layers, outs):
            h = gba.gemm_bias_act(h, w.t(), b, act=act, accum=case["accum"], out=out)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        forward()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        forward()
    return {"case": case, "graph": graph, "outs": outs, "x": x, "layers": layers}


def run(state):
    case = state["case"]
    if case["kind"] == "stack":
        state["graph"].replay()
        return state["outs"]
    t = state["t"]
    if case["prologue"] == "none" and case["second"] == "none" and case["bias"] != "full" and \
            case["bias_op"] == "add" and case["K"] < 16384:
        return gba.gemm_bias_act(t["A"], t["B"], t.get("bias"), act=case["act"], accum=case["accum"])
    return gba.fused_gemm(t["A"], t["B"], P=t.get("P"), Q=t.get("Q"),
                          second="add" if case["second"] == "none" else case["second"],
                          prologue=None if case["prologue"] == "none" else case["prologue"],
                          bias=t.get("bias"), bias_op=case["bias_op"], act=case["act"], accum=case["accum"])


def work(case):
    """Operands and bias read once and outputs written once, in fp16; 2MNK
    operations a product."""
    if case["kind"] == "stack":
        M, d, h, n = case["M"], case["width"], case["hidden"], case["blocks"]
        return {"bytes": 2 * n * (2 * d * h + d + h + 2 * M * (d + h)), "flops": 4 * n * M * d * h}
    M, N, k = case["M"], case["N"], case["K"] + case["K2"]
    bias = {"none": 0, "row": N, "full": M * N}[case["bias"]]
    return {"bytes": 2 * (M * k + k * N + M * N + bias), "flops": 2 * M * N * k}


def tolerance(case):
    """Results are rounded once to fp16 (half a unit in the last place is
    2^-11 of a value at most); another order of the fp32 sums moves some
    results to the neighbouring fp16 value.  Measured against exact(): 2.1e-4
    for one request, up to 5.2e-4 after eight layers, 0.9-1.9e-3 with fp16
    accumulation; about four times that is allowed.  With fp16 accumulation every
    32-deep group's sum is rounded, and a group on the other side of a tie
    moves by one fp16 step of the running sum."""
    if case["accum"] == "f16":
        return {"rel": 8e-3, "max": 6e-2}
    if case["kind"] == "stack":
        return {"rel": 2e-3, "max": 1e-2}
    return {"rel": 1e-3, "max": 4e-3}


def exact(case, seed):
    """The same function of the same inputs in 64 bits, without the
    intermediate roundings to fp16."""
    if case["kind"] == "stack":
        x, layers = _inputs(case, seed)
        h, outs = x.double(), []
        for w, b, act in layers:
            h = h @ w.double().t() + b.double()
            h = h.clamp_min(0) if act == "relu" else h
            outs.append(h)
        return outs
    t = {k: v.double() for k, v in _inputs(case, seed).items()}
    pro = (lambda x: x.clamp_min(0)) if case["prologue"] == "relu" else (lambda x: x)
    z = pro(t["A"]) @ t["B"]
    if case["second"] != "none":
        r = pro(t["P"]) @ t["Q"]
        z = z + r if case["second"] == "add" else z - r
    if "bias" in t:
        z = z + t["bias"] if case["bias_op"] == "add" else z - t["bias"]
    return {"none": lambda v: v, "relu": lambda v: v.clamp_min(0), "sigmoid": torch.sigmoid,
            "tanh": torch.tanh}[case["act"]](z)
