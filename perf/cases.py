"""Workloads of the sparse ternary linear layer as a program that uses it runs them, for timing and comparing builds.

A case is a dict of plain values.  Its "kind" says what one pass does; every pass goes through the public entry points of
the package.  The sizes are those of the repository's own benchmark (hidden 2560, FFN 6912, 4096 and 16384 tokens, decode
batches) and generic ones around them.

kind      one pass
layer     one forward call of one layer: sbn_sparse_ternary_linear
stack     one decode step of `blocks` transformer blocks: per block Q/K/V in one grouped call, O, up/gate in one grouped
          call, down; every projection has weights of its own, so a long stack streams them from memory
block     prefill of one block as Algorithm 1 writes it: Norm + quantizer, Q/K/V on the quantized rows, O, Norm +
          quantizer, up/gate on the quantized rows, down
prefill   one grouped forward call of an up and a square projection that share their input (the benchmark's step)
pack      the weight side of two training steps: quantize, mask and pack every matrix from its weights of the first
          step, then from those of the second (with the mask flips between the two, where asked for)
train     one training step of a block: remask of its seven matrices, forward that keeps the quantized rows, backward in
          four grouped calls
tune      gradient accumulation in one layer: remask, then forward and backward of two micro-batches, the second adding
          its weight gradient to the first's
"""
import math

import torch

import paper_2603_05168_amd as sbn

DEV = "cuda"


def listed():
    return [
        # the smallest call there is: one token through one square projection, latency and launches only
        {"name": "layer_1_token", "kind": "layer", "tokens": 1, "d_in": 2560, "d_out": 2560, "N": 2, "M": 4, "bias": False},
        # a decode step of a few sequences through a stack whose weights come from memory
        {"name": "stack_4_tokens", "kind": "stack", "blocks": 8, "tokens": 4, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4},
        # the same for a serving batch
        {"name": "stack_64_tokens", "kind": "stack", "blocks": 8, "tokens": 64, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4},
        # a layer whose sizes fit no tile, a short ragged prompt, with a bias
        {"name": "layer_ragged", "kind": "layer", "tokens": 50, "d_in": 1000, "d_out": 1500, "N": 2, "M": 4, "bias": True},
        # one prompt of an odd length through a block
        {"name": "block_777_tokens", "kind": "block", "tokens": 777, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4},
        # the paper's own pattern in serving: weights converted once to dense 2-bit codes
        {"name": "prefill_6of8_2048", "kind": "prefill", "tokens": 2048, "d_in": 2560, "wide": 6912, "square": 2560, "N": 6, "M": 8},
        # the benchmark's prefill step
        {"name": "prefill_4096", "kind": "prefill", "tokens": 4096, "d_in": 2560, "wide": 6912, "square": 2560, "N": 2, "M": 4},
        # a batch of long prompts through one wide layer
        {"name": "layer_32768_tokens", "kind": "layer", "tokens": 32768, "d_in": 2560, "d_out": 6912, "N": 2, "M": 4, "bias": False},
        # per-step remask of ten blocks with their mask flips
        {"name": "remask_10_blocks", "kind": "pack", "blocks": 10, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4, "dtype": "bf16", "flips": True},
        # remask of one block kept in fp32 master weights
        {"name": "remask_fp32_block", "kind": "pack", "blocks": 1, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4, "dtype": "fp32", "flips": False},
        # fine-tuning at the paper's own pattern, small micro-batches
        {"name": "tune_1024_tokens", "kind": "tune", "tokens": 1024, "d_in": 2560, "d_out": 6912, "N": 6, "M": 8},
        # the benchmark's training step of a block
        {"name": "train_16384_tokens", "kind": "train", "tokens": 16384, "hidden": 2560, "ffn": 6912, "N": 2, "M": 4},
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` between lo and hi, spread over its logarithm."""
    return max(step, int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) // step * step)


def draw(rng):
    kind = rng.choice(["layer", "layer", "stack", "stack", "block", "prefill", "pack", "train", "tune"])
    # 2:4 is the pattern with an instruction of its own; 6:8 the paper's; N = M plain ternary weights
    N, M = rng.choice([(2, 4), (2, 4), (2, 4), (6, 8), (4, 4), (1, 4), (2, 8)])
    if kind == "layer":
        # input dimensions: whole chunks of 128, halves of them, or any multiple of 8
        step = rng.choice([128, 128, 64, 8])
        return {"kind": kind, "tokens": _log(rng, 1, 16384), "d_in": _log(rng, 256, 8192, step), "d_out": _log(rng, 256, 8192),
                "N": N, "M": M, "bias": rng.random() < 0.3}
    hidden = _log(rng, 768, 4096, 128)
    ffn = int(hidden * rng.uniform(2.0, 4.0)) // 128 * 128
    if kind == "stack":
        N, M = rng.choice([(2, 4), (2, 4), (6, 8), (4, 4)])
        return {"kind": kind, "blocks": rng.randint(2, 8), "tokens": _log(rng, 1, 512), "hidden": hidden, "ffn": ffn, "N": N, "M": M}
    if kind == "block":
        N, M = rng.choice([(2, 4), (2, 4), (6, 8), (4, 4)])
        return {"kind": kind, "tokens": _log(rng, 32, 8192), "hidden": hidden, "ffn": ffn, "N": N, "M": M}
    if kind == "prefill":
        N, M = rng.choice([(2, 4), (2, 4), (6, 8), (4, 4)])
        return {"kind": kind, "tokens": _log(rng, 64, 32768), "d_in": hidden, "wide": ffn, "square": hidden, "N": N, "M": M}
    if kind == "pack":
        fast = (N, M) in ((2, 4), (1, 4), (2, 8))
        dtype = rng.choice(["bf16", "bf16", "fp32"])
        return {"kind": kind, "blocks": rng.randint(1, 6), "hidden": hidden, "ffn": ffn, "N": N, "M": M, "dtype": dtype,
                "flips": fast and dtype == "bf16" and rng.random() < 0.5}
    if kind == "train":
        return {"kind": kind, "tokens": _log(rng, 1024, 8192), "hidden": min(hidden, 2560), "ffn": min(ffn, 6912), "N": N, "M": M}
    return {"kind": kind, "tokens": _log(rng, 128, 8192), "d_in": hidden, "d_out": _log(rng, 768, 8192, 8), "N": N, "M": M}


# ---- what a program has in hand before the call ---------------------------------------------------------------------

class _Source:
    """Seeded tensors on the GPU: latent weights ~ N(0, 0.02^2), activations ~ N(0, 1), output gradients ~ N(0, 0.01^2)."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)

    def normal(self, shape, sigma, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=self.gen, device=DEV) * sigma).to(dtype)

    def weight(self, d_out, d_in, dtype=torch.bfloat16):
        return self.normal((d_out, d_in), 0.02, dtype)

    def rows(self, tokens, d_in):
        return self.normal((tokens, d_in), 1.0)


def _block_shapes(hidden, ffn):
    """(d_out, d_in) of Q, K, V, O, up, gate, down."""
    return [(hidden, hidden)] * 4 + [(ffn, hidden)] * 2 + [(hidden, ffn)]


def _workspace(nbytes):
    return sbn.new_workspace(nbytes, DEV)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _pack(W, N, M):
    d_out, d_in = W.shape
    packed = _empty(sbn.sbn_packed_bytes(d_out, d_in, N, M), torch.uint8)
    gamma = _empty(1, torch.float32)
    ws = _workspace(sbn.sbn_workspace_bytes(sbn.SBN_OP_QUANTIZE_MASK_PACK, 1, d_out, d_in, N, M))
    sbn.sbn_quantize_mask_pack(W, N, M, packed, gamma, ws)
    return packed, gamma


def _serving_weights(src, d_out, d_in, N, M):
    """Packed weights as a serving program keeps them: 6:8 converted once to dense 2-bit codes, the rest as packed."""
    packed, gamma = _pack(src.weight(d_out, d_in), N, M)
    if (N, M) == (6, 8):
        codes = _empty(sbn.sbn_packed_bytes(d_out, d_in, 8, 8), torch.uint8)
        sbn.sbn_convert_packed(packed, d_out, d_in, 6, 8, 8, 8, codes)
        packed = codes
    return packed, gamma


def _serving_pattern(N, M):
    return (8, 8) if (N, M) == (6, 8) else (N, M)


def _linear_ws(tokens, shapes, N, M):
    return _workspace(sum(sbn.sbn_workspace_bytes(sbn.SBN_OP_LINEAR, tokens, d_out, d_in, N, M) for d_out, d_in in shapes))


def prepare(case, seed):
    state = globals()["_prepare_" + case["kind"]](case, _Source(seed))
    state["kind"] = case["kind"]
    return state


def run(state):
    return globals()["_run_" + state["kind"]](state)


# ---- layer ------------------------------------------------------------------------------------------------------------

def _prepare_layer(c, src):
    T, K, O, N, M = c["tokens"], c["d_in"], c["d_out"], c["N"], c["M"]
    packed, gamma = _pack(src.weight(O, K), N, M)
    return {"X": src.rows(T, K), "packed": packed, "gamma": gamma, "Y": _empty((T, O), torch.float32), "N": N, "M": M,
            "bias": src.normal((O,), 0.1, torch.float32) if c["bias"] else None, "ws": _linear_ws(T, [(O, K)], N, M)}


def _run_layer(s):
    sbn.sbn_sparse_ternary_linear(s["X"], s["packed"], s["gamma"], s["Y"], s["N"], s["M"], s["ws"], bias=s["bias"])
    return s["Y"]


# ---- stack ------------------------------------------------------------------------------------------------------------

def _prepare_stack(c, src):
    T, H, F = c["tokens"], c["hidden"], c["ffn"]
    N, M = _serving_pattern(c["N"], c["M"])
    shapes = _block_shapes(H, F)
    ws = _linear_ws(T, shapes[:3] + shapes[4:6], N, M)      # one workspace for the whole chain of calls
    blocks, outputs = [], []
    for _ in range(c["blocks"]):
        w = [_serving_weights(src, o, k, c["N"], c["M"]) for o, k in shapes]
        X = [src.rows(T, H), src.rows(T, H), src.rows(T, H), src.rows(T, F)]   # inputs of Q/K/V, O, up/gate, down
        Y = [_empty((T, o), torch.float32) for o, _ in shapes]

        def group(ids, x):
            return sbn.LinearGroup([x] * len(ids), [w[i][0] for i in ids], [w[i][1] for i in ids], [Y[i] for i in ids], N, M, ws)
        blocks.append({"qkv": group([0, 1, 2], X[0]), "o": (X[1], w[3], Y[3]), "upgate": group([4, 5], X[2]), "down": (X[3], w[6], Y[6])})
        outputs += Y
    return {"blocks": blocks, "outputs": outputs, "N": N, "M": M, "ws": ws}


def _run_stack(s):
    N, M, ws = s["N"], s["M"], s["ws"]
    for b in s["blocks"]:
        b["qkv"].run()
        x, (packed, gamma), y = b["o"]
        sbn.sbn_sparse_ternary_linear(x, packed, gamma, y, N, M, ws)
        b["upgate"].run()
        x, (packed, gamma), y = b["down"]
        sbn.sbn_sparse_ternary_linear(x, packed, gamma, y, N, M, ws)
    return s["outputs"]


# ---- block ------------------------------------------------------------------------------------------------------------

def _prepare_block(c, src):
    T, H, F = c["tokens"], c["hidden"], c["ffn"]
    N, M = _serving_pattern(c["N"], c["M"])
    shapes = _block_shapes(H, F)
    return {"w": [_serving_weights(src, o, k, c["N"], c["M"]) for o, k in shapes],
            "X": [src.rows(T, H), src.rows(T, H), src.rows(T, H), src.rows(T, F)],
            "gain": [1.0 + src.normal((H,), 0.1, torch.float32) for _ in range(2)],
            "Y": [_empty((T, o), torch.float32) for o, _ in shapes],
            "xq": _empty((T, H), torch.int8), "sx": _empty(T, torch.float32), "xq2": _empty((T, H), torch.int8), "sx2": _empty(T, torch.float32),
            "ws": _workspace(max(sbn.sbn_workspace_bytes(sbn.SBN_OP_LINEAR, T, o, k, N, M) for o, k in shapes)), "N": N, "M": M}


def _run_block(s):
    w, X, Y, N, M, ws = s["w"], s["X"], s["Y"], s["N"], s["M"], s["ws"]
    sbn.sbn_rmsnorm_act_quant(X[0], s["xq"], s["sx"], s["gain"][0])
    for i in (0, 1, 2):
        sbn.sbn_sparse_ternary_linear(None, w[i][0], w[i][1], Y[i], N, M, ws, xq_out=s["xq"], sx_out=s["sx"])
    sbn.sbn_sparse_ternary_linear(X[1], w[3][0], w[3][1], Y[3], N, M, ws)
    sbn.sbn_rmsnorm_act_quant(X[2], s["xq2"], s["sx2"], s["gain"][1])
    for i in (4, 5):
        sbn.sbn_sparse_ternary_linear(None, w[i][0], w[i][1], Y[i], N, M, ws, xq_out=s["xq2"], sx_out=s["sx2"])
    sbn.sbn_sparse_ternary_linear(X[3], w[6][0], w[6][1], Y[6], N, M, ws)
    return Y + [s["xq"], s["sx"], s["xq2"], s["sx2"]]


# ---- prefill ----------------------------------------------------------------------------------------------------------

def _prepare_prefill(c, src):
    T, K = c["tokens"], c["d_in"]
    N, M = _serving_pattern(c["N"], c["M"])
    outs = [c["square"], c["wide"]]
    w = [_serving_weights(src, o, K, c["N"], c["M"]) for o in outs]
    X = src.rows(T, K)
    Y = [_empty((T, o), torch.float32) for o in outs]
    ws = _linear_ws(T, [(o, K) for o in outs], N, M)
    return {"group": sbn.LinearGroup([X, X], [p for p, _ in w], [g for _, g in w], Y, N, M, ws), "Y": Y}


def _run_prefill(s):
    s["group"].run()
    return s["Y"]


# ---- pack -------------------------------------------------------------------------------------------------------------

def _prepare_pack(c, src):
    N, M = c["N"], c["M"]
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    shapes = _block_shapes(c["hidden"], c["ffn"]) * c["blocks"]
    count = len(shapes)
    first = [src.weight(o, k, dtype) for o, k in shapes]
    # a step of the optimizer: every weight moves by about a tenth of its spread
    second = [(w + src.normal(w.shape, 0.002, dtype)).to(dtype) for w in first]
    # the model's packed weights lie in one buffer, its scales in another, a matrix is a view into them
    sizes = [sbn.sbn_packed_bytes(o, k, N, M) for o, k in shapes]
    places = [0]
    for n in sizes:
        places.append(places[-1] + (n + 255) // 256 * 256)
    flat = [torch.zeros(places[-1], dtype=torch.uint8, device=DEV) for _ in range(1 if c["flips"] else 2)]
    packed = [[buf[at:at + n] for at, n in zip(places, sizes)] for buf in flat]
    gammas = [_empty(count, torch.float32) for _ in range(2)]
    gamma = [[g[i:i + 1] for i in range(count)] for g in gammas]
    flips = [torch.zeros(count, dtype=torch.int64, device=DEV) for _ in range(2)] if c["flips"] else [None, None]
    ws = _workspace(sbn.sbn_workspace_bytes(sbn.SBN_OP_QUANTIZE_MASK_PACK, count, max(o for o, _ in shapes), max(k for _, k in shapes), N, M))
    steps = [sbn.PackBatch(W, N, M, packed[i % len(packed)], gamma[i], ws, flips[i]) for i, W in enumerate((first, second))]
    if c["flips"]:
        sbn.sbn_quantize_mask_pack_batched(second, N, M, packed[0], gamma[1], ws)   # the forms that the pass begins from
    return {"steps": steps, "out": flat + gammas + [f for f in flips if f is not None]}


def _run_pack(s):
    for step in s["steps"]:
        step.run()
    return s["out"]


# ---- train ------------------------------------------------------------------------------------------------------------

_TRAIN_GROUPS = ((6,), (4, 5), (3,), (0, 1, 2))      # layers whose output gradients arrive together, last first
_INPUT_OF = (0, 0, 0, 1, 2, 2, 3)                    # which of the block's four inputs a layer reads


def _prepare_train(c, src):
    T, H, F, N, M = c["tokens"], c["hidden"], c["ffn"], c["N"], c["M"]
    shapes = _block_shapes(H, F)
    W = [src.weight(o, k) for o, k in shapes]
    packed = [_empty(sbn.sbn_packed_bytes(o, k, N, M), torch.uint8) for o, k in shapes]
    gamma = [_empty(1, torch.float32) for _ in shapes]
    ws_pack = _workspace(sbn.sbn_workspace_bytes(sbn.SBN_OP_QUANTIZE_MASK_PACK, 7, max(H, F), max(H, F), N, M))
    widths = (H, H, H, F)
    X = [src.rows(T, k) for k in widths]
    xq = [_empty((T, k), torch.int8) for k in widths]
    sx = [_empty(T, torch.float32) for _ in widths]
    dY = [src.normal((T, o), 0.01) for o, _ in shapes]
    Y = [_empty((T, o), torch.float32) for o, _ in shapes]
    dX = [_empty((T, k), torch.bfloat16) for _, k in shapes]
    dW = [_empty((o, k), torch.bfloat16) for o, k in shapes]
    ws_bwd = _workspace(max(sum(sbn.sbn_workspace_bytes(sbn.SBN_OP_BACKWARD, T, *shapes[i], N, M) for i in ids) for ids in _TRAIN_GROUPS))
    groups = [sbn.BackwardGroup([dY[i] for i in ids], [packed[i] for i in ids], [gamma[i] for i in ids], [xq[_INPUT_OF[i]] for i in ids],
                                [sx[_INPUT_OF[i]] for i in ids], N, M, ws_bwd, [shapes[i][1] for i in ids], [dX[i] for i in ids],
                                [dW[i] for i in ids]) for ids in _TRAIN_GROUPS]
    return {"pack": sbn.PackBatch(W, N, M, packed, gamma, ws_pack), "X": X, "xq": xq, "sx": sx, "packed": packed, "gamma": gamma, "Y": Y,
            "dX": dX, "dW": dW, "groups": groups, "N": N, "M": M,
            "ws": _workspace(max(sbn.sbn_workspace_bytes(sbn.SBN_OP_LINEAR, T, o, k, N, M) for o, k in shapes))}


def _run_train(s):
    s["pack"].run()
    for x, xq, sx in zip(s["X"], s["xq"], s["sx"]):
        sbn.sbn_act_quant(x, xq, sx)
    for i, j in enumerate(_INPUT_OF):
        sbn.sbn_sparse_ternary_linear(None, s["packed"][i], s["gamma"][i], s["Y"][i], s["N"], s["M"], s["ws"], xq_out=s["xq"][j], sx_out=s["sx"][j])
    for g in s["groups"]:
        g.run()
    return {"packed": s["packed"], "gamma": s["gamma"], "xq": s["xq"], "sx": s["sx"], "Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}


# ---- tune -------------------------------------------------------------------------------------------------------------

def _prepare_tune(c, src):
    T, K, O, N, M = c["tokens"], c["d_in"], c["d_out"], c["N"], c["M"]
    return {"W": src.weight(O, K), "packed": _empty(sbn.sbn_packed_bytes(O, K, N, M), torch.uint8), "gamma": _empty(1, torch.float32),
            "X": [src.rows(T, K) for _ in range(2)], "dY": [src.normal((T, O), 0.01) for _ in range(2)],
            "Y": [_empty((T, O), torch.float32) for _ in range(2)], "dX": [_empty((T, K), torch.bfloat16) for _ in range(2)],
            "dW": _empty((O, K), torch.bfloat16), "xq": _empty((T, K), torch.int8), "sx": _empty(T, torch.float32), "N": N, "M": M,
            "ws": _workspace(max(sbn.sbn_workspace_bytes(op, T if op else 1, O, K, N, M)
                                 for op in (sbn.SBN_OP_QUANTIZE_MASK_PACK, sbn.SBN_OP_LINEAR, sbn.SBN_OP_BACKWARD)))}


def _run_tune(s):
    N, M, ws, K = s["N"], s["M"], s["ws"], s["W"].shape[1]
    sbn.sbn_quantize_mask_pack(s["W"], N, M, s["packed"], s["gamma"], ws)
    for i in range(2):
        sbn.sbn_sparse_ternary_linear(s["X"][i], s["packed"], s["gamma"], s["Y"][i], N, M, ws, xq_out=s["xq"], sx_out=s["sx"])
        sbn.sbn_sparse_ternary_linear_backward(s["dY"][i], s["packed"], s["gamma"], s["xq"], s["sx"], N, M, ws, K, dX=s["dX"][i], dW=s["dW"],
                                               accumulate=i > 0)
    return {"packed": s["packed"], "gamma": s["gamma"], "Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def _packed_bytes(o, k, N, M):
    b = 0 if N == M else {2: 1, 4: 2, 8: 3}[M]
    return o * ((k + 127) // 128) * (128 * N // M) * (2 + b) / 8


def _forward(T, o, k, N, M):
    """(bytes without the layer's input, operations) of one forward product: weights in, fp32 rows out."""
    return _packed_bytes(o, k, N, M) + 4 * T * o, 2.0 * T * o * k * N / M


def work(case):
    c, kind = case, case["kind"]
    N, M = (c["N"], c["M"]) if kind in ("layer", "pack", "train", "tune") else _serving_pattern(c["N"], c["M"])
    nbytes = flops = 0.0

    def add(T, o, k):
        nonlocal nbytes, flops
        b, f = _forward(T, o, k, N, M)
        nbytes += b
        flops += f
    if kind == "layer":
        add(c["tokens"], c["d_out"], c["d_in"])
        nbytes += 2 * c["tokens"] * c["d_in"]
    elif kind == "prefill":
        for o in (c["square"], c["wide"]):
            add(c["tokens"], o, c["d_in"])
        nbytes += 2 * c["tokens"] * c["d_in"]
    elif kind in ("stack", "block"):
        T, H, F = c["tokens"], c["hidden"], c["ffn"]
        for o, k in _block_shapes(H, F):
            add(T, o, k)
        nbytes += 2 * T * (3 * H + F)
        if kind == "block":
            nbytes += 2 * T * H      # the quantized rows that come back
        else:
            nbytes, flops = nbytes * c["blocks"], flops * c["blocks"]
    elif kind == "pack":
        size = 2 if c["dtype"] == "bf16" else 4
        for o, k in _block_shapes(c["hidden"], c["ffn"]):
            nbytes += 2 * c["blocks"] * (o * k * size + (2 if c["flips"] else 1) * _packed_bytes(o, k, N, M))
    elif kind == "train":
        T, H, F = c["tokens"], c["hidden"], c["ffn"]
        for o, k in _block_shapes(H, F):
            add(T, o, k)
            flops += 4.0 * T * o * k                                  # dX and dW on dense operands
            nbytes += 2 * o * k + 2 * T * o + 2 * T * k + 2 * o * k   # W, dY, dX, dW
        nbytes += 3 * T * (3 * H + F)                                 # inputs in, quantized rows out
    else:
        T, O, K = c["tokens"], c["d_out"], c["d_in"]
        for _ in range(2):
            add(T, O, K)
            flops += 4.0 * T * O * K
            nbytes += 2 * T * K + 2 * T * O + 2 * T * K
        nbytes += 2 * O * K + 2 * O * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return "exact"                  # packed bytes and flips are whole numbers, gamma is one rounding of a 64-bit sum
    if kind in ("train", "tune"):
        # bf16 gradients of operands that are themselves rounded to bf16 (dY / s_x).  Against the same products in 64 bits
        # dX is off by 1.7e-3 (at most 3.9e-3) and an accumulated dW, rounded twice, by 2.6e-3 (1.3e-2): about four times that
        return {"rel": 1e-2, "max": 0.05, "differ": 0.0}
    # the accumulators are exact: a division, a multiplication (and an addition of a bias) in fp32 per result.  Against
    # 64 bits: 4e-8, at most 1.6e-7
    return {"rel": 2e-7, "max": 1e-6, "differ": 0.0}
