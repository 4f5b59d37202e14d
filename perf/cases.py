"""Workloads that stand for what a program built on this library has it do, timed and compared through the public entry
points of `paper_1805_12096_amd`.

Sizes are the repository's own: 512 / 2048 (base) and 1024 / 4096 (big) layer widths, a 36 000-word tied vocabulary,
batches of 384 and 8192 words, decode steps of 300 sentences with 25 source words each.  Values are Gaussian with the
deviations of `workloads.py` (activations 1, parameters 0.03 - 0.05, biases 0.1), made on the device from the seed.
Parameters are prepared and workspaces allocated once, as a program that translates more than one batch does it.
"""
import math

import torch

import paper_1805_12096_amd as mq

DEV = "cuda:0"

BASE = (512, 2048)
BIG = (1024, 4096)


def listed():
    return [
        # one 16-bit product of a CPU-sized batch of 384 words through a 512 x 512 parameter
        {"name": "linear_i16_384", "kind": "linear", "bits": 16, "M": 384, "K": 512, "N": 512, "relu": False, "fixed": False},
        # a projection over a ragged encoder batch of the big model, 8 bit
        {"name": "linear_i8_5003", "kind": "linear", "bits": 8, "M": 5003, "K": 1024, "N": 1024, "relu": False, "fixed": False},
        # base feed-forward block over a GPU-sized batch of 8192 words, on a workspace the program keeps
        {"name": "ffn_i8_8192", "kind": "ffn_i8", "M": 8192, "d": 512, "f": 2048, "prepared": True},
        # the same block over what is left of a stream of sentences, on a workspace shared with other calls
        {"name": "ffn_i8_1001", "kind": "ffn_i8", "M": 1001, "d": 512, "f": 2048, "prepared": False},
        # big feed-forward block, 16 bit, per-tensor multipliers, the largest batch
        {"name": "ffn_i16_8192", "kind": "ffn_i16", "M": 8192, "d": 1024, "f": 4096},
        # the same block with the fixed multiplier 2^10 over a ragged batch
        {"name": "ffn_i16_fixed_3001", "kind": "ffn_i16_fixed", "M": 3001, "d": 1024, "f": 4096},
        # one decoder layer at one position: a batch of 300 sentences, and one sentence alone (interactive use)
        {"name": "layer_300", "kind": "layer", "M": 300, "S": 25, "d": 512, "f": 2048, "aan": 2048, "t": 20},
        {"name": "layer_1", "kind": "layer", "M": 1, "S": 23, "d": 512, "f": 2048, "aan": 2048, "t": 7},
        # greedy output layer of a decode step over the whole vocabulary: base width, big width
        {"name": "greedy_300", "kind": "greedy", "M": 300, "V": 36000, "d": 512},
        {"name": "greedy_big_300", "kind": "greedy", "M": 300, "V": 36000, "d": 1024},
        # the same restricted to a batch's short list; few sentences left
        {"name": "shortlist_61", "kind": "shortlist", "M": 61, "V": 36000, "n": 1811, "d": 512},
        # beam search with four hypotheses for each of 300 sentences
        {"name": "beam_1200", "kind": "beam", "M": 1200, "V": 36000, "k": 4, "d": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "ffn_i8", "ffn_i16", "ffn_i16_fixed", "layer", "layer", "greedy", "shortlist", "beam"])
    d, f = rng.choice([BASE, BIG])
    if kind == "linear":
        if rng.random() < 0.3:           # widths of no particular model
            K, N = _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
        else:
            K, N = rng.choice([(d, d), (d, f), (f, d), (2 * d, 2 * d), (d, 3 * d)])
        return {"kind": kind, "bits": rng.choice([8, 16]), "M": _log_int(rng, 1, 8192), "K": K, "N": N,
                "relu": rng.random() < 0.4, "fixed": rng.random() < 0.3}
    if kind.startswith("ffn"):
        if rng.random() < 0.2:
            d, f = _log_int(rng, 128, 1024), _log_int(rng, 512, 4096)
        case = {"kind": kind, "M": _log_int(rng, 64, 8192), "d": d, "f": f}
        if kind == "ffn_i8":
            case["prepared"] = rng.random() < 0.5
        return case
    if kind == "layer":
        return {"kind": kind, "M": _log_int(rng, 1, 600), "S": _log_int(rng, 4, 60), "d": d, "f": f,
                "aan": rng.choice([d, f]), "t": _log_int(rng, 1, 80)}
    V = _log_int(rng, 8000, 50000)
    if kind == "greedy":
        return {"kind": kind, "M": _log_int(rng, 1, 600), "V": V, "d": d}
    if kind == "shortlist":
        return {"kind": kind, "M": _log_int(rng, 1, 600), "V": V, "n": _log_int(rng, 200, 7000), "d": 512}
    k = rng.choice([2, 3, 4])
    return {"kind": kind, "M": k * _log_int(rng, 1, 300), "V": V, "k": k, "d": 512}


class _Draw:
    """Gaussian tensors on the device from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def __call__(self, *shape, sigma=1.0, mean=0.0):
        x = torch.randn(*shape, dtype=torch.float32, device=DEV, generator=self.g)
        return x.mul_(sigma).add_(mean) if mean else x.mul_(sigma)


def _bytes(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device=DEV)


def _floats(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def prepare(case, seed):
    r = _Draw(seed)
    s = {"case": case}
    kind = case["kind"]
    M = case["M"]
    if kind == "linear":
        K, N, bits = case["K"], case["N"], case["bits"]
        s["A"] = r(M, K)
        # the paper's fixed multipliers: 2^10 in 16 bit, 127/2 in 8 bit
        mult = torch.full((1,), 1024.0 if bits == 16 else 63.5, dtype=torch.float32, device=DEV)
        s["sA"] = mult if case["fixed"] else None
        s["W"] = mq.prepare_weight(r(N, K, sigma=0.05), bits, scale=mult if case["fixed"] and bits == 16 else None)
        s["bias"] = r(N, sigma=0.1)
        s["Y"] = _floats(M, N)
        s["ws"] = _bytes(mq.mq_linear_ws_bytes(bits, M, K))
    elif kind.startswith("ffn"):
        d, f = case["d"], case["f"]
        bits = 8 if kind == "ffn_i8" else 16
        s["A"] = r(M, d)
        s["sc"] = torch.full((1,), 1024.0, dtype=torch.float32, device=DEV) if kind == "ffn_i16_fixed" else None
        sigma = 0.04 if bits == 8 else 0.03
        s["W1"] = mq.prepare_weight(r(f, d, sigma=sigma), bits, scale=s["sc"])
        s["W2"] = mq.prepare_weight(r(d, f, sigma=sigma), bits, scale=s["sc"])
        s["b1"], s["b2"] = r(f, sigma=0.1), r(d, sigma=0.1)
        s["Y"] = _floats(M, d)
        need = {"ffn_i8": mq.mq_ffn_ws_bytes, "ffn_i16": mq.mq_ffn_i16_ws_bytes, "ffn_i16_fixed": mq.mq_ffn_i16_fixed_ws_bytes}[kind]
        s["ws"] = _bytes(need(M, d, f))
        if case.get("prepared"):
            mq.mq_ffn_ws_prepare(s["ws"], s["ws"].numel(), M, d, f)
    elif kind == "layer":
        d, f, aan, S = case["d"], case["f"], case["aan"], case["S"]
        shapes = {"aan_ffn1": (aan, d), "aan_ffn2": (d, aan), "aan_gate": (2 * d, 2 * d), "ctx_q": (d, d), "ctx_o": (d, d),
                  "ffn1": (f, d), "ffn2": (d, f)}
        products = {n: (mq.prepare_weight(r(*shape, sigma=0.04), 8), r(shape[0], sigma=0.1)) for n, shape in shapes.items()}
        norms = {n: (r(d, sigma=0.1, mean=1.0), r(d, sigma=0.1)) for n in ("ln1", "ln2", "ln3")}
        s["layer"] = mq.aan_layer(products, norms, d, f, aan)
        s["x"] = r(M, d)
        s["g"] = r(M, d, sigma=1.0 / math.sqrt(max(case["t"] - 1, 1)))
        s["K"], s["V"] = r(M, S, d), r(M, S, d)
        s["y"], s["g_out"] = _floats(M, d), _floats(M, d)
        s["ws"] = _bytes(mq.mq_aan_layer_ws_bytes(M, d, f, aan))
    else:
        V, d = case["V"], case["d"]
        s["E"] = mq.prepare_weight(r(V, d, sigma=0.05), 8)
        s["Hd"] = r(M, d)
        s["sA"] = _floats(1)
        s["qws"] = _bytes(mq.mq_quantize_absmax_ws_bytes())
        mq.mq_quantize_absmax_ws_prepare(s["qws"], s["qws"].numel())
        k = case.get("k", 1)
        s["tok"] = torch.empty((M, k) if kind == "beam" else (M,), dtype=torch.int32, device=DEV)
        s["val"] = _floats(*s["tok"].shape)
        s["ws"] = _bytes(mq.mq_topk_ws_bytes(M, V, k) if kind == "beam" else mq.mq_argmax_ws_bytes(M, V))
        if d > 512:                      # the packed output layers serve widths up to 512
            s["q"] = torch.empty((M, d), dtype=torch.int8, device=DEV)
        else:
            s["q"] = _bytes(mq.mq_packed_bytes(8, M, d))
        if kind == "shortlist":
            s["list"] = torch.randperm(V, device=DEV, generator=r.g)[: case["n"]].sort().values.to(torch.int32)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    M = case["M"]
    ws = s["ws"]
    if kind == "linear":
        mq.mq_linear_f32(s["A"], M, case["K"], s["sA"], s["W"].packed, s["W"].scale, case["bits"], case["N"], s["bias"],
                         case["relu"], s["Y"], None, ws, ws.numel())
        return s["Y"]
    if kind.startswith("ffn"):
        d, f, W1, W2 = case["d"], case["f"], s["W1"], s["W2"]
        if kind == "ffn_i16_fixed":
            mq.mq_ffn_i16_fixed_f32(s["A"], M, d, f, s["sc"], W1.packed, W1.scale, s["b1"], s["sc"], W2.packed, W2.scale,
                                    s["b2"], s["Y"], ws, ws.numel())
        else:
            call = mq.mq_ffn_i16_f32 if kind == "ffn_i16" else mq.mq_ffn_i8_f32_prepared if case["prepared"] else mq.mq_ffn_i8_f32
            call(s["A"], M, d, f, W1.packed, W1.scale, s["b1"], W2.packed, W2.scale, s["b2"], s["Y"], ws, ws.numel())
        return s["Y"]
    if kind == "layer":
        mq.mq_aan_layer_f32(s["layer"], s["x"], s["g"], case["t"], s["K"], s["V"], M, case["S"], case["d"] // 64, True, True,
                            1e-6, s["y"], s["g_out"], ws, ws.numel())
        return s["y"], s["g_out"]
    V, d, E = case["V"], case["d"], s["E"]
    if d > 512:
        mq.mq_absmax_f32(s["Hd"], M * d, s["sA"])
        mq.mq_scale_from_amax(s["sA"], 8, s["sA"])
        mq.mq_quantize_f32(s["Hd"], M, d, 8, s["sA"], s["q"])
        mq.mq_gemm_argmax(s["q"], E.packed, M, V, d, s["sA"], E.scale, s["tok"], s["val"], ws, ws.numel())
        return s["tok"], s["val"]
    mq.mq_quantize_absmax_pack_f32_prepared(s["Hd"], M, d, 8, s["q"], s["sA"], s["qws"], s["qws"].numel())
    if kind == "greedy":
        mq.mq_gemm_argmax_packed(s["q"], E.packed, M, V, d, s["sA"], E.scale, s["tok"], s["val"], ws, ws.numel())
    elif kind == "shortlist":
        mq.mq_gemm_argmax_shortlist(s["q"], E.packed, s["list"], case["n"], M, V, d, s["sA"], E.scale, s["tok"], s["val"], ws,
                                    ws.numel())
    else:
        mq.mq_gemm_topk_packed(s["q"], E.packed, None, 0, M, V, d, s["sA"], E.scale, case["k"], s["tok"], s["val"], ws, ws.numel())
    return s["tok"], s["val"]


def work(case):
    """Inputs read once, outputs written once, parameters as the 8- or 16-bit integers they are kept as; two operations
    per multiplication of a product (a 16-bit one counted once, whatever the matrix units make of it)."""
    kind, M = case["kind"], case["M"]
    if kind == "linear":
        K, N, b = case["K"], case["N"], case["bits"] // 8
        return {"bytes": 4 * M * K + b * N * K + 4 * N + 4 * M * N, "flops": 2 * M * N * K}
    if kind.startswith("ffn"):
        d, f, b = case["d"], case["f"], 1 if kind == "ffn_i8" else 2
        return {"bytes": 4 * M * d + 2 * b * d * f + 4 * (d + f) + 4 * M * d, "flops": 4 * M * d * f}
    if kind == "layer":
        d, f, aan, S = case["d"], case["f"], case["aan"], case["S"]
        weights = 2 * d * aan + 4 * d * d + 2 * d * d + 2 * d * f
        return {"bytes": weights + 4 * (aan + f + 12 * d) + 8 * M * S * d + 16 * M * d, "flops": 2 * M * weights + 4 * M * S * d}
    rows = case["n"] if kind == "shortlist" else case["V"]
    k = case.get("k", 1)
    return {"bytes": rows * case["d"] + 4 * M * case["d"] + 8 * M * k + (4 * rows if kind == "shortlist" else 0),
            "flops": 2 * M * rows * case["d"]}


def tolerance(case):
    if case["kind"] == "layer":
        # A glue result (running average, attention, gate, normalisation) that differs in its last bit can round to the
        # neighbouring integer, which moves its row of the next products by about 1e-3 (by up to 6e-2 in single elements).
        # Against the layer with its glue in binary64 (nine shapes of this range, three seeds each): up to 1.8e-3 and 6.3e-2.
        return {"rel": 7e-3, "max": 0.25}
    if case["kind"] == "beam":
        # Tokens are chosen on integer sums; the log-probabilities carry a binary32 sum of V exponentials
        # (against binary64: 1.1e-7 and 2.6e-7).
        return {"rel": 5e-7, "max": 1e-6, "differ": 0.0}
    return "exact"                       # integer sums and one fused multiply-add per result
