"""Performance cases: the work a program does with this library, through its
public entry points, over the sizes it is used at.

Kinds of case
  linear    one ``W4A4Linear`` forward, called eagerly: fp16 activations in,
            fp16 out (activation quantizer + GEMM), weights quantized and laid
            out once beforehand.  ``scales`` "fp16" is the paper's method, "mx"
            the power-of-two scale variant.
  layer     the four linears of one decoder layer (qkv, output, gate + up,
            down) as a serving loop runs a decode step: captured once into a
            HIP graph, replayed for every token.
  gemm      ``apex4_w4a4_gemm_ws`` on codes that were quantized elsewhere, with
            the weights as the quantizer writes them (row-major) and a
            workspace the caller keeps.
  quantize  ``apex4_quantize_act`` alone: activations on their way to several
            GEMMs that share them, or weights being prepared.

``G`` is the quantization group along K; 0 stands for one group per row
(per-channel).  Activations are N(0, 1) with 1 % outlier channels at 20 times
that, weights N(0, 0.02); codes made elsewhere are uniform.
"""
from __future__ import annotations

import torch

import paper_2606_08761_amd as apex4


def listed():
    return [
        # one token through a key/value-sized projection, called eagerly: the
        # smallest call, launches and host time
        {"name": "linear_1row", "kind": "linear", "M": 1, "N": 1024, "K": 8192, "G": 128, "scales": "fp16"},
        # single-stream decode: one token through the linears of a
        # Llama-2-70B layer; streaming the weights
        {"name": "layer_decode_1", "kind": "layer", "M": 1, "H": 8192, "QKV": 10240, "I": 28672, "G": 128},
        # batched decode of the same layer
        {"name": "layer_decode_16", "kind": "layer", "M": 16, "H": 8192, "QKV": 10240, "I": 28672, "G": 128},
        # batched decode, a smaller model, a batch that is no power of two
        {"name": "layer_decode_27", "kind": "layer", "M": 27, "H": 5120, "QKV": 7168, "I": 13824, "G": 128},
        # a batch past the few-row sizes (large decode batch, short prompt)
        {"name": "linear_72rows", "kind": "linear", "M": 72, "N": 8192, "K": 8192, "G": 128, "scales": "fp16"},
        # a prompt chunk through the down projection
        {"name": "linear_256rows", "kind": "linear", "M": 256, "N": 8192, "K": 28672, "G": 128, "scales": "fp16"},
        # prefill at the shape the paper's sweeps use, codes from elsewhere
        {"name": "gemm_prefill", "kind": "gemm", "M": 2048, "N": 8192, "K": 8192, "G": 128},
        # a long prefill through gate + up, a prompt length that fits no tile: the largest call
        {"name": "linear_prefill_long", "kind": "linear", "M": 4001, "N": 57344, "K": 8192, "G": 128, "scales": "fp16"},
        # the paper's mixed configuration: down projection at G = 32, ...
        {"name": "linear_g32", "kind": "linear", "M": 1000, "N": 8192, "K": 28672, "G": 32, "scales": "fp16"},
        # ... and the other linears per channel
        {"name": "linear_channel", "kind": "linear", "M": 2048, "N": 10240, "K": 8192, "G": 0, "scales": "fp16"},
        # the power-of-two scale variant at prefill
        {"name": "linear_mx", "kind": "linear", "M": 2048, "N": 8192, "K": 8192, "G": 32, "scales": "mx"},
        # quantizing a prompt's activations once for the GEMMs that share them
        {"name": "quantize_prefill", "kind": "quantize", "M": 4096, "K": 8192, "G": 128},
    ]


MOST = 4001 * 57344 * 8192  # multiply-adds of the largest listed case


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    kind = rng.choices(["linear", "layer", "gemm", "quantize"], [6, 3, 2, 1])[0]
    if kind == "layer":
        H = 256 * round(_log(rng, 1024, 8192) / 256)
        return {"kind": kind, "M": round(_log(rng, 1, 32)), "H": H, "QKV": H + 256 * rng.randint(1, H // 256),
                "I": 256 * round(H * rng.uniform(2.5, 5.5) / 256), "G": 128}
    if kind == "quantize":
        G = rng.choice([128, 128, 32, 256, 0])
        K = 128 * round(_log(rng, 1024, 28672) / 128) if G in (32, 128, 0) else 256 * round(_log(rng, 1024, 28672) / 256)
        return {"kind": kind, "M": round(_log(rng, 16, 8192)), "K": K, "G": G}
    while True:
        scales = "mx" if kind == "linear" and rng.random() < 0.2 else "fp16"
        G = rng.choice([128, 128, 128, 128, 32, 64, 256, 512, 0]) if scales == "fp16" else rng.choice([32, 128])
        unit = max(G, 128) if scales == "mx" or G > 64 else 32
        M = round(_log(rng, 1, 4096))
        N = round(_log(rng, 512, 28672))
        if rng.random() < 0.8:
            N = 64 * max(1, round(N / 64))
        K = unit * max(1, round(_log(rng, 1024, 28672) / unit))
        if M * N * K <= MOST:
            break
    c = {"kind": kind, "M": M, "N": N, "K": K, "G": G}
    if kind == "linear":
        c["scales"] = scales
    return c


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _activations(M, K, g):
    x = torch.randn((M, K), device="cuda", generator=g, dtype=torch.float32)
    outliers = torch.randperm(K, device="cuda", generator=g)[: max(1, K // 100)]
    x[:, outliers] *= 20.0
    return x.to(torch.float16)


def _weights(N, K, g):
    return torch.empty((N, K), device="cuda", dtype=torch.float16).normal_(0.0, 0.02, generator=g)


def _codes(rows, K, G, g):
    q = torch.randint(0, 256, (rows, K // 2), device="cuda", generator=g, dtype=torch.uint8)
    s = (torch.rand((rows, K // G), device="cuda", generator=g) * 0.015 + 0.005).to(torch.float16)
    return q, s


def _group(case):
    return case["G"] or case["K"]


def _layer_shapes(case):
    H = case["H"]
    return [(case["QKV"], H), (H, H), (2 * case["I"], H), (H, case["I"])]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "linear":
        lin = apex4.W4A4Linear(_weights(case["N"], case["K"], g), G=case["G"], scales=case["scales"])
        return {"kind": kind, "lin": lin, "x": _activations(case["M"], case["K"], g)}
    if kind == "layer":
        lins, xs = [], []
        for N, K in _layer_shapes(case):
            lins.append(apex4.W4A4Linear(_weights(N, K, g), G=case["G"]))
            xs.append(_activations(case["M"], K, g))
        side = torch.cuda.Stream()  # one pass outside the capture, as torch's capture recipe has it
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for lin, x in zip(lins, xs):
                lin(x)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ys = [lin(x) for lin, x in zip(lins, xs)]
        return {"kind": kind, "lins": lins, "xs": xs, "graph": graph, "ys": ys}
    if kind == "gemm":
        M, N, K, G = case["M"], case["N"], case["K"], _group(case)
        A_q, s_a = _codes(M, K, G, g)
        W_q, s_w = _codes(N, K, G, g)
        need = apex4.apex4_w4a4_gemm_workspace_size(M, N, K, G)
        return {"kind": kind, "args": (A_q, s_a, W_q, s_w, G),
                "ws": torch.empty((max(need, 16),), dtype=torch.uint8, device="cuda"),
                "Y": torch.empty((M, N), dtype=torch.float16, device="cuda")}
    return {"kind": kind, "x": _activations(case["M"], case["K"], g), "G": _group(case)}


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return state["lin"](state["x"])
    if kind == "layer":
        state["graph"].replay()
        return state["ys"]
    if kind == "gemm":
        return apex4.apex4_w4a4_gemm_ws(*state["args"], workspace=state["ws"], Y=state["Y"])
    return apex4.apex4_quantize_act(state["x"], state["G"])


def work(case):
    kind, M = case["kind"], case["M"]
    if kind == "layer":
        each = [work({"kind": "linear", "M": M, "N": N, "K": K, "G": case["G"], "scales": "fp16"})
                for N, K in _layer_shapes(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    K, G = case["K"], _group(case)
    if kind == "quantize":
        return {"bytes": 2.5 * M * K + 2 * M * (K // G), "flops": 0}
    N = case["N"]
    if kind == "gemm":
        return {"bytes": (M + N) * (K / 2 + 2 * (K // G)) + 2 * M * N, "flops": 2.0 * M * N * K}
    weights = N * (0.75 * K + K // G) if case["scales"] == "mx" else N * (K / 2 + 2 * (K // G))
    return {"bytes": 2 * M * K + weights + 2 * M * N, "flops": 2.0 * M * N * K}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    # one rounding to binary16 at the end (2^-11 of a value at most, 1.7e-4 in
    # the 2-norm); 32-bit sums in another order move some values across a
    # rounding boundary, by one step of binary16 (2^-10 of the value)
    return {"rel": 4e-4, "max": 4e-3}


def _quantize64(x, G):
    """Codes (float64) and scales (float64, binary16 values) of SymQuant."""
    rows, K = x.shape
    v = x.double().view(rows, K // G, G)
    s = (v.abs().amax(dim=2) / 7.0).to(torch.float16).double()
    q = torch.where(s[:, :, None] > 0, v / s[:, :, None], torch.zeros_like(v))
    return q.round_().clamp_(-8, 7), s


def _dequantized64(x, G):
    q, s = _quantize64(x, G)
    return (q * s[:, :, None]).view(x.shape)


def _dequantized_mx64(x, G):
    """Scale 2^E with E = min{e : max|X_g| <= 7 2^e} (E = 0 for a zero group)."""
    rows, K = x.shape
    v = x.double().view(rows, K // G, G)
    f, k = torch.frexp(v.abs().amax(dim=2))
    E = torch.where(f == 0, torch.zeros_like(k), torch.where(f <= 0.875, k - 3, k - 2))
    s = torch.ldexp(torch.ones_like(f), E)[:, :, None]
    return ((v / s).round_().clamp_(-8, 7) * s).view(x.shape)


def _unpacked64(q, s, G):
    rows, K = q.shape[0], 2 * q.shape[1]
    n = torch.stack((q & 0xF, q >> 4), dim=2).view(rows, K).to(torch.int16)
    v = (n - 16 * (n > 7)).double()
    return (v.view(rows, K // G, G) * s.double()[:, :, None]).view(rows, K)


def _product64(a, rows, block, N):
    """a @ W^T with W's rows made block by block (rows(n0, n1), in 64 bits)."""
    y = torch.empty((a.shape[0], N), dtype=torch.float64, device=a.device)
    for n0 in range(0, N, block):
        n1 = min(n0 + block, N)
        y[:, n0:n1] = a @ rows(n0, n1).t()
    return y


def exact(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "linear":
        G, N = _group(case), case["N"]
        deq = _dequantized_mx64 if case["scales"] == "mx" else _dequantized64
        w = _weights(N, case["K"], g)
        x = _activations(case["M"], case["K"], g)
        return _product64(deq(x, G), lambda a, b: deq(w[a:b], G), 4096, N)
    if kind == "layer":
        out = []
        for N, K in _layer_shapes(case):
            w = _weights(N, K, g)
            x = _activations(case["M"], K, g)
            out.append(_product64(_dequantized64(x, case["G"]),
                                  lambda a, b: _dequantized64(w[a:b], case["G"]), 4096, N))  # noqa: B023
        return out
    if kind == "gemm":
        M, N, K, G = case["M"], case["N"], case["K"], _group(case)
        A_q, s_a = _codes(M, K, G, g)
        W_q, s_w = _codes(N, K, G, g)
        return _product64(_unpacked64(A_q, s_a, G), lambda a, b: _unpacked64(W_q[a:b], s_w[a:b], G), 4096, N)
    G = _group(case)
    q, s = _quantize64(_activations(case["M"], case["K"], g), G)
    n = (q.to(torch.int16) & 0xF).to(torch.uint8).view(case["M"], case["K"])
    return n[:, 0::2] | (n[:, 1::2] << 4), s
