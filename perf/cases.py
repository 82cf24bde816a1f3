"""The calls this library is used for, as timed cases.

A spiking decoder calls the library through `paper_2606_03026_amd._binding`:
single spike-gated projections, a decoder's stack of them (in stream order or
in one launch), a stream of independent tokens, the dense projections of its
continuous inputs, the exporter, and the verified output head.  `listed()`
holds one case for each, at the sizes of the 22-block, 1536-wide decoder that
`workloads.py` describes and at ragged ones; `draw(rng)` gives more of the
same ranges.  All inputs are seeded and made on the GPU.
"""
from __future__ import annotations

import math

import torch

from paper_2606_03026_amd import _binding as sp

WIDTH, HIDDEN, BLOCKS, VOCAB = 1536, 6144, 22, 57344

# a drawn case stays below the listed ones: multiply-adds of a dense call, of
# a matrix-core contraction, and of an active-column gather, and bytes of a
# weight stack and of an exported matrix
MAX_DENSE_MACS = 4.5e9
MAX_DENSE_MACS_UNALIGNED = 1e9
MAX_SPIKE_MACS = 2.3e10
MAX_GATHER_ADDS = 1e8
MAX_EXPORT = WIDTH * HIDDEN


def listed():
    return [
        # one token through one TCAM projection: the smallest call, all latency
        {"name": "tcam_b1", "kind": "proj", "K": WIDTH, "N": WIDTH, "B": 1, "p": 0.10},
        # one token through the decoder's 44 spike projections, in order
        {"name": "stack_b1", "kind": "stack", "width": WIDTH, "hidden": HIDDEN, "blocks": BLOCKS, "B": 1, "fused": False},
        # a small serving batch, all projections' spikes at hand (a ragged row count)
        {"name": "fused_b7", "kind": "stack", "width": WIDTH, "hidden": HIDDEN, "blocks": BLOCKS, "B": 7, "fused": True},
        # a full serving batch of 64 sequences
        {"name": "fused_b64", "kind": "stack", "width": WIDTH, "hidden": HIDDEN, "blocks": BLOCKS, "B": 64, "fused": True},
        # prefill of a 512-token prompt through an FFN down projection
        {"name": "prefill_512", "kind": "proj", "K": HIDDEN, "N": WIDTH, "B": 512, "p": 0.10},
        # prefill of a long prompt, a length that fills no tile
        {"name": "prefill_2500", "kind": "proj", "K": HIDDEN, "N": WIDTH, "B": 2500, "p": 0.10},
        # throughput mode: 250 independent tokens, the weights rotated over 4 copies
        {"name": "stream_250", "kind": "stream", "width": WIDTH, "hidden": HIDDEN, "blocks": BLOCKS, "tokens": 250, "sets": 4},
        # vocabulary logits of one token
        {"name": "head_b1", "kind": "dense", "K": WIDTH, "M": VOCAB, "B": 1},
        # vocabulary logits of the serving batch
        {"name": "head_b64", "kind": "dense", "K": WIDTH, "M": VOCAB, "B": 64},
        # FFN up projection of a prompt, a length that fills no tile
        {"name": "up_b500", "kind": "dense", "K": WIDTH, "M": HIDDEN, "B": 500},
        # export of an FFN down projection into the spike layout
        {"name": "export_down", "kind": "export", "M": WIDTH, "K": HIDDEN, "col": True},
        # output head with 64 candidates verified
        {"name": "verify_head", "kind": "verify", "K": WIDTH, "V": VOCAB, "top_k": 64, "threshold": 4.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["proj", "proj", "stack", "stream", "dense", "dense", "export", "verify"])
    if kind == "proj":
        K, N, B = _log_int(rng, 200, 8192), _log_int(rng, 200, 4096), _log_int(rng, 1, 2500)
        p = round(rng.uniform(0.02, 0.40), 3)
        if rng.random() < 0.7:  # model widths; else any N
            K, N = (K + 15) // 16 * 16, (N + 15) // 16 * 16
            B = max(1, min(B, int(MAX_SPIKE_MACS / (K * N))))
        else:
            B = max(1, min(B, int(MAX_GATHER_ADDS / (K * N * p))))
        return {"kind": kind, "K": K, "N": N, "B": B, "p": p}
    if kind == "stack":
        width = 16 * rng.randint(16, 96)
        fused = rng.random() < 0.6
        return {"kind": kind, "width": width, "hidden": 4 * width, "blocks": rng.randint(4, BLOCKS),
                "B": _log_int(rng, 1, 64) if fused else _log_int(rng, 1, 8), "fused": fused}
    if kind == "stream":
        width = 16 * rng.randint(16, 96)
        return {"kind": kind, "width": width, "hidden": 4 * width, "blocks": rng.randint(4, BLOCKS),
                "tokens": rng.randint(20, 200), "sets": rng.randint(1, 4)}
    if kind == "dense":
        K, M, B = _log_int(rng, 200, 4096), _log_int(rng, 200, VOCAB), _log_int(rng, 1, 500)
        if rng.random() < 0.75:
            K = (K + 15) // 16 * 16
            most = MAX_DENSE_MACS
        else:
            most = MAX_DENSE_MACS_UNALIGNED
        M = min(M, int(WIDTH * VOCAB / K))
        return {"kind": kind, "K": K, "M": M, "B": max(1, min(B, int(most / (K * M))))}
    if kind == "export":
        M, K = _log_int(rng, 200, 8192), _log_int(rng, 200, 8192)
        if rng.random() < 0.6:
            M, K = (M + 15) // 16 * 16, (K + 15) // 16 * 16
        M = min(M, MAX_EXPORT // K)
        return {"kind": kind, "M": M, "K": K, "col": rng.random() < 0.6}
    K = (_log_int(rng, 256, 4096) + 15) // 16 * 16
    V = min(_log_int(rng, 1000, VOCAB), int(WIDTH * VOCAB / K))
    return {"kind": kind, "K": K, "V": V, "top_k": rng.choice([16, 32, 64]), "threshold": rng.choice([0.0, 0.5, 4.0])}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _weights(g, rows, cols):
    """INT8 weights ~ N(0, 30), rounded and clipped."""
    w = torch.empty((rows, cols), dtype=torch.float32, device="cuda").normal_(0.0, 30.0, generator=g)
    return w.round_().clamp_(-127, 127).to(torch.int8)


def _scales(g, n):
    return torch.empty(n, dtype=torch.float32, device="cuda").uniform_(1e-3, 1e-2, generator=g)


def _bits(g, B, K, p):
    """Spikes of B rows, rate p."""
    return torch.rand((B, K), device="cuda", generator=g) < p


def _hot_bits(g, B, K):
    """Spikes of a serving batch: a hot twentieth of the columns fires with
    probability 0.9, the others at a rate of their row's own (mean 0.10)."""
    rate = torch.rand((B, 1), device="cuda", generator=g) * 0.16 + 0.02
    hot = torch.rand((1, K), device="cuda", generator=g) < 0.05
    return torch.rand((B, K), device="cuda", generator=g) < torch.where(hot, torch.full_like(rate, 0.9), rate)


def _pack(bits):
    """bool [B, K] -> int64 [B, ceil(K / 64)], bit k in bit k % 64 of word k // 64."""
    B, K = bits.shape
    words = (K + 63) // 64
    full = torch.zeros((B, words * 64), dtype=torch.int64, device=bits.device)
    full[:, :K] = bits
    place = torch.ones(64, dtype=torch.int64, device=bits.device) << torch.arange(64, device=bits.device)
    return (full.view(B, words, 64) * place).sum(dim=2)


def _shapes(case):
    """(K, N) of the projections of a decoder's stack: per block TCAM, then down."""
    return [(k, case["width"]) for _ in range(case["blocks"]) for k in (case["width"], case["hidden"])]


def _rates(case):
    """Spike rate of every projection: one per block, from 0.05 to 0.20."""
    n = case["blocks"]
    return [0.05 + 0.15 * (i % n) / max(1, n - 1) for i in range(n) for _ in (0, 1)]


def _inputs(case, seed):
    """The case's plain inputs, from the seed alone."""
    g = _generator(seed)
    kind = case["kind"]
    if kind == "proj":
        return {"W": _weights(g, case["K"], case["N"]), "scale": _scales(g, case["N"]),
                "bits": _bits(g, case["B"], case["K"], case["p"])}
    if kind == "stack":
        B = case["B"]
        return {"W": [_weights(g, K, N) for K, N in _shapes(case)], "scale": [_scales(g, N) for _, N in _shapes(case)],
                "bits": [_hot_bits(g, B, K) if B > 1 else _bits(g, B, K, p)
                         for (K, _), p in zip(_shapes(case), _rates(case))]}
    if kind == "stream":
        n = case["sets"]
        return {"W": [_weights(g, K, N) for _ in range(n) for K, N in _shapes(case)],
                "scale": [_scales(g, N) for _ in range(n) for _, N in _shapes(case)],
                "bits": [_bits(g, case["tokens"], K, p) for (K, _), p in zip(_shapes(case), _rates(case))]}
    if kind == "dense":
        return {"Q": _weights(g, case["M"], case["K"]), "scale": _scales(g, case["M"]),
                "x": torch.randn((case["B"], case["K"]), device="cuda", generator=g)}
    if kind == "export":
        return {"W": torch.randn((case["M"], case["K"]), device="cuda", generator=g) * 0.02}
    return {"Q": _weights(g, case["V"], case["K"]), "scale": _scales(g, case["V"]),
            "x": torch.randn(case["K"], device="cuda", generator=g)}


def prepare(case, seed):
    """Weights, handles, spikes or activations, and output buffers."""
    i = _inputs(case, seed)
    kind = case["kind"]
    new = lambda *shape, dtype=torch.float32: torch.zeros(shape, dtype=dtype, device="cuda")  # noqa: E731
    torch.cuda.synchronize()
    s = {"case": case}
    if kind == "proj":
        s["h"] = sp.spike_proj_create_reserved(i["W"], i["scale"], max(case["B"], 1))
        s["mask"], s["out"] = _pack(i["bits"]), new(case["B"], case["N"])
    elif kind == "stack":
        s["h"] = [sp.spike_proj_create_reserved(W, c, case["B"]) for W, c in zip(i["W"], i["scale"])]
        s["mask"] = torch.cat([_pack(b).reshape(-1) for b in i["bits"]])
        s["out"] = new(sum(case["B"] * N for _, N in _shapes(case)))
    elif kind == "stream":
        h = [sp.spike_proj_create_reserved(W, c, 1, gather_only=True) for W, c in zip(i["W"], i["scale"])]
        s["stream"] = sp.spike_stream_create(h, 2 * case["blocks"], case["sets"], case["tokens"])
        s["mask"] = torch.cat([_pack(b) for b in i["bits"]], dim=1).contiguous()
        s["out"] = new(case["tokens"], 2 * case["blocks"] * case["width"])
    elif kind == "dense":
        s.update(Q=i["Q"], scale=i["scale"], x=i["x"], y=new(case["B"], case["M"]))
    elif kind == "export":
        M, K = case["M"], case["K"]
        s.update(W=i["W"], Q=new(*((K, M) if case["col"] else (M, K)), dtype=torch.int8), scale=new(M),
                 layout=sp.SPIKE_LAYOUT_COL_MAJOR if case["col"] else sp.SPIKE_LAYOUT_ROW_MAJOR)
    else:
        k = case["top_k"]
        s.update(Q=i["Q"], scale=i["scale"], x=i["x"], logits=new(case["V"]), cand=new(k, dtype=torch.int32),
                 cand_logits=new(k), result=new(2, dtype=torch.int32), workspace=sp.head_verify_workspace())
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "proj":
        sp.spike_proj_forward(s["h"], s["mask"], case["B"], s["out"])
        return s["out"]
    if kind == "stack":
        (sp.spike_stack_forward_fused if case["fused"] else sp.spike_stack_forward)(s["h"], s["mask"], case["B"], s["out"])
        return s["out"]
    if kind == "stream":
        sp.spike_stream_forward(s["stream"], s["mask"], s["out"])
        return s["out"]
    if kind == "dense":
        sp.dense_proj_forward(s["Q"], s["scale"], s["x"], case["B"], s["y"])
        return s["y"]
    if kind == "export":
        sp.spike_quantize_int8(s["W"], s["layout"], s["Q"], s["scale"])
        return s["Q"], s["scale"]
    sp.head_verify_forward(s["Q"], s["scale"], s["x"], case["top_k"], case["threshold"], s["logits"], s["cand"],
                           s["cand_logits"], s["result"], workspace=s["workspace"])
    return s["logits"], s["cand"], s["cand_logits"], s["result"]


# ---------------------------------------------------------------------------
# What a pass cannot do without, how far results may differ, and the results
# ---------------------------------------------------------------------------

def _spike_work(K, N, B, p):
    """Bytes: the columns active in any row, scales, spikes, outputs; flops:
    one addition per active (row, column) pair and channel."""
    return K * (1 - (1 - p) ** B) * N + 4 * N + B * ((K + 63) // 64 * 8 + 4 * N), B * p * K * N


def work(case):
    kind = case["kind"]
    if kind == "proj":
        b, f = _spike_work(case["K"], case["N"], case["B"], case["p"])
    elif kind == "stack":
        B = case["B"]
        b = f = 0.0
        for (K, N), p in zip(_shapes(case), _rates(case)):
            if B == 1:
                wb, wf = _spike_work(K, N, 1, p)
            else:  # _hot_bits
                hb, hf = _spike_work(K, N, B, 0.9)
                cb, cf = _spike_work(K, N, B, 0.10)
                wb, wf = 0.05 * hb + 0.95 * cb, 0.05 * hf + 0.95 * cf
            b, f = b + wb, f + wf
    elif kind == "stream":
        b = f = 0.0
        for (K, N), p in zip(_shapes(case), _rates(case)):
            T, n = case["tokens"], case["sets"]
            wb, wf = _spike_work(K, N, T, p)
            # every weight copy's active columns are read
            each = K * N * (1 - (1 - p) ** (T / n))
            b, f = b + wb + n * each - K * N * (1 - (1 - p) ** T), f + wf
    elif kind == "dense":
        K, M, B = case["K"], case["M"], case["B"]
        b, f = M * K + 4 * M + 4 * B * (K + M), 2.0 * B * M * K
    elif kind == "export":
        M, K = case["M"], case["K"]
        b, f = 5 * M * K + 4 * M, 2.0 * M * K
    else:
        K, V = case["K"], case["V"]
        b, f = V * K + 4 * V + 4 * K + 4 * V, 2.0 * V * K
    return {"bytes": b, "flops": f}


def tolerance(case):
    # Spike projections: an integer sum, one conversion and one multiply, so
    # there is one correct bit pattern; the exporter's codes and scales are
    # defined in binary32 down to the bit.
    if case["kind"] not in ("dense", "verify"):
        return "exact"
    # Sums of up to 4096 FP32 products: four times what the same sums in
    # other orders differ by.  The head's approximate logits and candidates are exact.
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}


def _spike_exact(W, scale, bits):
    return (bits.double() @ W.double()) * scale.double()


def exact(case, seed):
    i = _inputs(case, seed)
    kind = case["kind"]
    if kind == "proj":
        return _spike_exact(i["W"], i["scale"], i["bits"])
    if kind == "stack":
        return torch.cat([_spike_exact(W, c, b).reshape(-1) for W, c, b in zip(i["W"], i["scale"], i["bits"])])
    if kind == "stream":
        n, n_proj = case["sets"], 2 * case["blocks"]
        out = torch.empty((case["tokens"], n_proj, case["width"]), dtype=torch.float64, device="cuda")
        for t in range(n):  # token t uses weight copy t mod n
            for j in range(n_proj):
                out[t::n, j] = _spike_exact(i["W"][t * n_proj + j], i["scale"][t * n_proj + j], i["bits"][j][t::n])
        return out.reshape(case["tokens"], -1)
    if kind == "dense":
        return (i["x"].double() @ i["Q"].double().t().contiguous()) * i["scale"].double()
    if kind == "export":
        # the scale; the codes are whole numbers
        return None, i["W"].abs().amax(dim=1).clamp_min(1e-8).double() / 127.0
    # the approximate logits from the quantized activations, the candidates'
    # logits from the FP32 ones where the gap asks for it
    Q, scale, x = i["Q"].double(), i["scale"], i["x"]
    s_x = x.abs().max().clamp_min(1e-8) / 127.0
    acc = Q @ (x / s_x).round().clamp_(-127, 127).double()
    logits = acc * (scale.double() * s_x.double())
    rounded = acc.float() * (scale * s_x)
    best = torch.sort(rounded, descending=True, stable=True)
    cand = best.indices[:case["top_k"]]
    verify = bool(best.values[0] - best.values[1] < case["threshold"])
    return logits, None, ((Q[cand] @ x.double()) * scale[cand].double()) if verify else logits[cand], None
