"""What the library's performance is measured on.

Four kinds of pass, each a piece of what a program that uses the library has it do through the public
entry points of ``paper_2601_22716_amd``:

* ``linear``    one quantised linear layer, ``lords_matmul`` (or ``lords_matmul_repacked`` for weights kept in
                the slab-tile layout): one token and a handful (decode), hundreds and thousands (prefill);
* ``stack``     the seven linear layers of some transformer blocks as a serving loop calls them: q/k/v in one
                ``lords_matmul_batched``, the output projection, ``lords_gate_up``, the down projection;
* ``finetune``  one layer of a fine-tuning step of the scale factors: forward, gradient of the input, gradients
                of the factors;
* ``ptq``       quantising a layer after training: block-wise scales, codes under refined factors, and the
                dequantised weights that the refinement compares with the original ones.

Sizes are the layer shapes of the repository's configurations and benchmark, or generic ones around them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import lords_inputs
import paper_2601_22716_amd as L


def _linear(M, N, K, bits, r, factors="bf16", out="f32", layout="rows", signed=False, **kw):
    return dict(kw, kind="linear", M=M, N=N, K=K, bits=bits, r=r, factors=factors, out=out, layout=layout, signed=signed)


def _stack(M, blocks, hidden, kv, ffn, bits, r, **kw):
    return dict(kw, kind="stack", M=M, blocks=blocks, hidden=hidden, kv=kv, ffn=ffn, bits=bits, r=r)


def _finetune(M, N, K, bits, r, factors, **kw):
    return dict(kw, kind="finetune", M=M, N=N, K=K, bits=bits, r=r, factors=factors)


def _ptq(N, K, bits, group, r, factors, weights, **kw):
    return dict(kw, kind="ptq", N=N, K=K, bits=bits, group=group, r=r, factors=factors, weights=weights)


def listed():
    return [
        # The smallest call: a layer of half a megabit with fp32 factors, where a launch is all there is.
        _linear(4, 512, 256, 4, 4, factors="f32", name="tiny_f32_m4"),
        # One attention projection for one token: the shortest call of a decode step.
        _linear(1, 4096, 4096, 4, 32, name="decode_m1_qproj"),
        # One token through four blocks: what a decode step of a 4-bit model does, weights cold in the caches.
        _stack(1, 4, 4096, 1024, 14336, 4, 32, name="decode_m1_stack_4b"),
        # The same at 3 bits and the rank of the 3-bit layers.
        _stack(1, 3, 4096, 1024, 14336, 3, 48, name="decode_m1_stack_3b"),
        # Sixteen sequences decoded together.
        _stack(16, 4, 4096, 1024, 14336, 4, 32, name="decode_m16_stack_4b"),
        # A few sequences (an odd count) on one large 2-bit layer of high rank.
        _linear(5, 28672, 8192, 2, 64, name="decode_m5_28672x8192_2b"),
        # A prompt through one block.
        _stack(2048, 1, 4096, 1024, 14336, 4, 32, name="prefill_m2048_block_4b"),
        # A short prompt, or many sequences decoded together, on the large 2-bit layer.
        _linear(256, 28672, 8192, 2, 64, out="bf16", name="prefill_m256_28672x8192_2b"),
        # A prompt of odd length at 3 bits, on a layer whose rows do not fill the last tile.
        _linear(333, 11008, 4096, 3, 48, out="bf16", signed=True, name="prefill_m333_11008x4096_3b"),
        # A fine-tuning step of one gate/up layer with bf16 factors.
        _finetune(2048, 14336, 4096, 4, 32, "bf16", name="finetune_m2048_4b"),
        # A fine-tuning step on fp32 factors (as an optimiser keeps them), short batch.
        _finetune(500, 4096, 4096, 4, 16, "f32", name="finetune_m500_f32"),
        # Quantising one gate/up layer.
        _ptq(14336, 4096, 4, 128, 32, "bf16", "f32", name="ptq_14336x4096_4b"),
    ]


def _log(rng, lo, hi, step=1):
    """An integer in [lo, hi], spread over its logarithm, rounded down to a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v))) // step * step


# No drawn case needs more than the largest listed one (the prompt through one block).
_MOST_FLOPS = 8.9e11
_MOST_BYTES = 6e8


def draw(rng):
    while True:
        kind = rng.choice(["linear"] * 9 + ["stack"] * 5 + ["finetune"] * 3 + ["ptq"] * 3)
        bits = rng.choice([2, 3, 4, 4])
        if kind == "linear":
            M = _log(rng, 1, 16) if rng.random() < 0.5 else _log(rng, 17, 4096)
            N, K = _log(rng, 500, 28672), _log(rng, 256, 14336, 32)
            f32 = rng.random() < 0.15
            tiles = not f32 and rng.random() < 0.15
            # (the slab-tile layout is served up to rank 64 at any token count)
            r = _log(rng, 4, 64) if f32 or tiles else _log(rng, 4, 128)
            case = _linear(M, N, K, bits, r, factors="f32" if f32 else "bf16", out=rng.choice(["f32", "bf16"]),
                           layout="tiles" if tiles else "rows", signed=rng.random() < 0.5)
        elif kind == "stack":
            M = _log(rng, 1, 16) if rng.random() < 0.5 else _log(rng, 17, 2048)
            hidden = _log(rng, 512, 5120, 64)
            kv = hidden // rng.choice([1, 2, 4, 8])
            case = _stack(M, rng.choice([1, 2, 3]) if M <= 16 else 1, hidden, kv, int(hidden * rng.uniform(2.0, 4.0)) // 32 * 32,
                          bits, _log(rng, 8, 64))
        elif kind == "finetune":
            case = _finetune(_log(rng, 32, 4096), _log(rng, 512, 14336, 32), _log(rng, 512, 14336, 32), bits,
                             _log(rng, 4, 64), "f32" if rng.random() < 0.3 else "bf16")
        else:
            group = rng.choice([64, 128, 256])
            case = _ptq(_log(rng, 500, 14336), _log(rng, 512, 14336, group), bits, group, _log(rng, 4, 64),
                        rng.choice(["bf16", "f32"]), rng.choice(["bf16", "f32"]))
        w = work(case)
        if w["flops"] <= _MOST_FLOPS and w["bytes"] <= _MOST_BYTES:
            return case


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _dtype(name):
    return torch.float32 if name == "f32" else torch.bfloat16


def _normal(g, rows, cols, dtype=torch.bfloat16):
    return torch.randn((rows, cols), generator=g, device="cuda").to(dtype)


def _codes(g, N, K, bits):
    """Uniform packed codes: a row is a whole number of bytes, so uniform bytes are uniform codes."""
    return torch.randint(0, 256, (N, L.lords_row_bytes(K, bits)), generator=g, device="cuda", dtype=torch.uint8)


def _factors(g, N, K, r, dtype, signed=False):
    """Factors whose product is about 0.02 in every element, or signed ones as a singular value decomposition gives them."""
    if signed:
        B, A = torch.randn((N, r), generator=g, device="cuda"), torch.randn((r, K), generator=g, device="cuda")
        return (B * (0.02 / math.sqrt(r))).to(dtype), A.to(dtype)
    B = (torch.rand((N, r), generator=g, device="cuda") + 0.5) * (0.02 / r)
    A = torch.rand((r, K), generator=g, device="cuda") + 0.5
    return B.to(dtype), A.to(dtype)


def _codebook(bits):
    return torch.from_numpy(np.ascontiguousarray(lords_inputs.nf_codebook(bits))).cuda()


def _layer(g, N, K, bits, r, dtype=torch.bfloat16):
    return (_codes(g, N, K, bits),) + _factors(g, N, K, r, dtype)


def _empty(rows, cols, dtype):
    return torch.empty((rows, cols), dtype=dtype, device="cuda")


def prepare(case, seed):
    g = _gen(seed)
    c = dict(case)
    kind, bits, r = c["kind"], c["bits"], c["r"]
    s = {"case": c, "codebook": _codebook(bits)}
    if kind == "linear":
        M, N, K = c["M"], c["N"], c["K"]
        s["X"] = _normal(g, M, K)
        s["codes"] = _codes(g, N, K, bits)
        s["B"], s["A"] = _factors(g, N, K, r, _dtype(c["factors"]), c["signed"])
        if c["layout"] == "tiles":          # laid out once, when the model is loaded
            tiled = torch.empty(L.lords_repack_bytes(N, K, bits), dtype=torch.uint8, device="cuda")
            L.lords_repack(s["codes"], tiled, N, K, bits)
            s["codes"] = tiled
        s["Y"] = _empty(M, N, _dtype(c["out"]))
    elif kind == "stack":
        # Every block has weights of its own; the normalised residual stream and the attention output stand ready.
        M, hidden, kv, ffn = c["M"], c["hidden"], c["kv"], c["ffn"]
        s["blocks"] = []
        for _ in range(c["blocks"]):
            b = {"q": _layer(g, hidden, hidden, bits, r), "k": _layer(g, kv, hidden, bits, r), "v": _layer(g, kv, hidden, bits, r),
                 "o": _layer(g, hidden, hidden, bits, r), "gate": _layer(g, ffn, hidden, bits, r), "up": _layer(g, ffn, hidden, bits, r),
                 "down": _layer(g, hidden, ffn, bits, r),
                 "x_attn": _normal(g, M, hidden), "x_o": _normal(g, M, hidden), "x_mlp": _normal(g, M, hidden)}
            b["Y"] = [_empty(M, n, torch.bfloat16) for n in (hidden, kv, kv, hidden, ffn, hidden)]
            s["blocks"].append(b)
    elif kind == "finetune":
        M, N, K = c["M"], c["N"], c["K"]
        s["X"], s["dY"] = _normal(g, M, K), _normal(g, M, N)
        s["codes"], s["B"], s["A"] = _layer(g, N, K, bits, r, _dtype(c["factors"]))
        s["codes_t"] = torch.empty((K, L.lords_row_bytes(N, bits)), dtype=torch.uint8, device="cuda")
        L.lords_transpose_codes(s["codes"], s["codes_t"], N, K, bits)      # the codes are frozen: once per layer
        s["Y"], s["dX"] = _empty(M, N, torch.bfloat16), _empty(M, K, torch.bfloat16)
        s["dB"], s["dA"] = _empty(N, r, torch.float32), _empty(r, K, torch.float32)
    else:
        N, K = c["N"], c["K"]
        s["B"], s["A"] = _factors(g, N, K, r, _dtype(c["factors"]))
        # Weights of the spread that the factors stand for.
        s["W"] = (torch.randn((N, K), generator=g, device="cuda") * 0.008).to(_dtype(c["weights"]))
        rb = K // c["group"]
        s["B0"], s["A0"] = _empty(N, rb, _dtype(c["factors"])), _empty(rb, K, _dtype(c["factors"]))
        s["codes"] = torch.empty((N, L.lords_row_bytes(K, bits)), dtype=torch.uint8, device="cuda")
        s["W_hat"] = _empty(N, K, _dtype(c["weights"]))
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    c, cb = s["case"], s["codebook"]
    kind, bits, r = c["kind"], c["bits"], c["r"]
    if kind == "linear":
        f = L.lords_matmul_repacked if c["layout"] == "tiles" else L.lords_matmul
        f(s["X"], s["codes"], cb, s["B"], s["A"], s["Y"], c["M"], c["N"], c["K"], r, bits)
        return s["Y"]
    if kind == "stack":
        M, hidden, kv, ffn = c["M"], c["hidden"], c["kv"], c["ffn"]
        for b in s["blocks"]:
            q, k, v, o, gate, up, down = (b[n] for n in ("q", "k", "v", "o", "gate", "up", "down"))
            Yq, Yk, Yv, Yo, H, Yd = b["Y"]
            L.lords_matmul_batched(b["x_attn"], [q[0], k[0], v[0]], cb, [q[1], k[1], v[1]], [q[2], k[2], v[2]], [Yq, Yk, Yv],
                                   [hidden, kv, kv], M, hidden, r, bits)
            L.lords_matmul(b["x_o"], o[0], cb, o[1], o[2], Yo, M, hidden, hidden, r, bits)
            L.lords_gate_up(b["x_mlp"], gate[0], gate[1], gate[2], up[0], up[1], up[2], cb, H, M, ffn, hidden, r, bits)
            L.lords_matmul(H, down[0], cb, down[1], down[2], Yd, M, hidden, ffn, r, bits)
        return [b["Y"] for b in s["blocks"]]
    N, K = c["N"], c["K"]
    if kind == "finetune":
        M = c["M"]
        L.lords_matmul(s["X"], s["codes"], cb, s["B"], s["A"], s["Y"], M, N, K, r, bits)
        L.lords_backward_input(s["dY"], s["codes_t"], cb, s["B"], s["A"], s["dX"], M, N, K, r, bits)
        L.lords_backward_factors(s["dY"], s["X"], s["codes"], cb, s["B"], s["A"], s["dB"], s["dA"], M, N, K, r, bits)
        return {"Y": s["Y"], "dX": s["dX"], "dB": s["dB"], "dA": s["dA"]}
    L.lords_block_init(s["W"], cb, s["B0"], s["A0"], N, K, K // c["group"], bits)
    L.lords_quantize(s["W"], cb, s["B"], s["A"], s["codes"], N, K, r, bits)
    L.lords_dequant(s["codes"], cb, s["B"], s["A"], s["W_hat"], N, K, r, bits)
    return {"B0": s["B0"], "A0": s["A0"], "codes": s["codes"], "W_hat": s["W_hat"]}


# ---------------------------------------------------------------- what a pass cannot do without
def _size(name):
    return 4 if name == "f32" else 2


def _matmul_work(M, N, K, bits, r, fsize=2, osize=2):
    return N * K * bits // 8 + (N * r + r * K) * fsize + M * K * 2 + M * N * osize, 2 * M * N * K + 2 * r * N * K


def work(case):
    c = case
    kind, bits, r = c["kind"], c["bits"], c["r"]
    if kind == "linear":
        by, fl = _matmul_work(c["M"], c["N"], c["K"], bits, r, _size(c["factors"]), _size(c["out"]))
    elif kind == "stack":
        M, hidden, kv, ffn = c["M"], c["hidden"], c["kv"], c["ffn"]
        by = fl = 0
        for n, k in ((hidden, hidden), (kv, hidden), (kv, hidden), (hidden, hidden), (ffn, hidden), (ffn, hidden), (hidden, ffn)):
            b, f = _matmul_work(M, n, k, bits, r)
            by, fl = by + b, fl + f
        # q, k and v share their input, gate and up too, and of gate and up only one product is written
        by -= 3 * M * hidden * 2 + M * ffn * 2
        by, fl = by * c["blocks"], fl * c["blocks"]
    elif kind == "finetune":
        M, N, K = c["M"], c["N"], c["K"]
        # codes in both layouts, factors, X and dY once; Y, dX, dB and dA once; three products and the scales of each
        by = 2 * (N * K * bits // 8) + (N * r + r * K) * (_size(c["factors"]) + 4) + 2 * (M * K + M * N) * 2
        fl = 3 * 2 * M * N * K + 4 * 2 * r * N * K
    else:
        N, K = c["N"], c["K"]
        rb = K // c["group"]
        # W once, the codes and the dequantised weights once; both pairs of factors
        by = 2 * N * K * _size(c["weights"]) + N * K * bits // 8 + (N * (r + rb) + (r + rb) * K) * _size(c["factors"])
        fl = 2 * 2 * r * N * K
    return {"bytes": int(by), "flops": int(fl)}


# ---------------------------------------------------------------- how far another correct implementation may be off
def tolerance(case):
    kind = case["kind"]
    if kind == "ptq":
        # Scales by fp32 sums, one rounding on the way out; the codes' decision is fixed to the operation, so they are equal.
        return {"rel": 1e-5 if case["weights"] == "f32" and case["factors"] == "f32" else 4e-3}
    # bf16 operands on the matrix cores: the weight, or level and scaled activation, rounded to bf16 once, fp32 sums,
    # one rounding of the result.  Against the same products in float64 every call is off by 1.0e-3 .. 2.4e-3 (2-norm) and
    # by at most 1.1e-2 in one element; in a stack the down projection reads the rounded product of gate and up: 3.8e-3, and
    # an element of that product carries the errors of both its factors: 3.5e-2.  Four times these.
    if kind == "stack":
        return {"rel": 1.5e-2, "max": 0.15}
    return {"rel": 1e-2, "max": 0.045}
