"""The work that users of the quantized linears have them do, as measurable cases.

Serving walks the linears of a stack of transformer layers: per layer the qkv projection
(W1.58A4), the attention output projection (sparse W1.58A8), gate and up projection with the
squared-ReLU gate (W1.58A4, one entry point) and the down projection (sparse W1.58A8), at any
number of tokens from one (decode) to a few prompts at once (prefill).  What attention itself
would put between qkv and the output projection is an input of its own here.  Besides: the FP4
activation form, one training step of a linear, the low-bit attention states, and the smallest
call there is.  Widths are those of the paper's models (synth.SHAPES) in the listed cases.
"""
import math

import torch

from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import synth as S

BF16 = torch.bfloat16


# ---------------------------------------------------------------- the cases
def _layers(kind, model, m, layers):
    hidden, ffn = S.SHAPES[model]
    return {"kind": kind, "tokens": m, "hidden": hidden, "ffn": ffn, "layers": layers}


def listed():
    return [
        # two small linears on float32 rows, as a first program or a unit test calls them
        {"name": "pair_f32_16", "kind": "pair", "tokens": 16, "k": 256, "n": 512},
        # one sequence decoding: a token through eight 7B layers (405 MB of packed weights, so HBM serves them)
        dict(_layers("decode", "7B", 1, 8), name="decode_7b_1"),
        # a small batch decoding on a 3B model
        dict(_layers("decode", "3B", 8, 8), name="decode_3b_8"),
        # an ordinary serving batch
        dict(_layers("decode", "7B", 32, 8), name="decode_7b_32"),
        # a ragged batch near the top of the decode range, FFN width no multiple of 8
        dict(_layers("decode", "1.3B", 57, 8), name="decode_1b3_57"),
        # one short prompt
        dict(_layers("prefill", "3B", 200, 4), name="prefill_3b_200"),
        # a chunk of a chunked prefill, or one long prompt
        dict(_layers("prefill", "7B", 1000, 2), name="prefill_7b_1000"),
        # 2048 tokens on a 1.3B model
        dict(_layers("prefill", "1.3B", 2048, 2), name="prefill_1b3_2048"),
        # four sequences of 4096 tokens: the largest pass
        dict(_layers("prefill", "7B", 16384, 1), name="prefill_7b_16384"),
        # the FP4 activation form of the INT4 projections
        dict(_layers("fp4", "3B", 8192, 1), name="fp4_3b_8192"),
        # quantization-aware training of a 3B qkv projection: ternarize, forward, both gradients
        {"name": "train_3b_4096", "kind": "train", "tokens": 4096, "k": 3200, "n": 9600, "topk": 0},
        # a prompt's attention states: query codes, key and value appended to the cache and read back
        {"name": "states_7b_4096", "kind": "states", "tokens": 4096, "pos0": 0, "heads": 32, "dim": 128},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode"] * 4 + ["prefill"] * 4 + ["fp4", "train", "states", "pair"])
    if kind == "pair":
        return {"kind": kind, "tokens": rng.randint(1, 64), "k": rng.randrange(64, 1025, 4), "n": rng.randrange(64, 1025, 4)}
    if kind == "states":
        return {"kind": kind, "tokens": _log_int(rng, 1, 4096), "pos0": rng.randint(0, 4096), "heads": rng.randint(8, 32),
                "dim": rng.choice([64, 96, 128])}
    if kind == "train":
        k, n = rng.randrange(1024, 4097, 32), rng.randrange(1024, 9601, 32)
        return {"kind": kind, "tokens": _log_int(rng, 256, 4096), "k": k, "n": n, "topk": rng.choice([0, k // 2])}
    # layers: a model's own widths, or widths of another model's proportions
    if rng.random() < 0.5:
        hidden, ffn = S.SHAPES[rng.choice(sorted(S.SHAPES))]
    else:
        hidden = rng.randrange(1024, 4097, 64)
        ffn = int(hidden * rng.uniform(2.5, 2.7)) // 4 * 4
    if kind == "decode":
        return {"kind": kind, "tokens": _log_int(rng, 1, 64), "hidden": hidden, "ffn": ffn, "layers": 8}
    tokens = _log_int(rng, 65 if kind == "prefill" else 512, 16384 if kind == "prefill" else 8192)
    return {"kind": kind, "tokens": tokens, "hidden": hidden, "ffn": ffn,
            "layers": 4 if tokens < 512 else 2 if tokens < 4096 and kind == "prefill" else 1}


# ---------------------------------------------------------------- inputs
def _heavy(g, m, k):
    """bfloat16 N(0, 1) with about 0.5 % of the channels heavy-tailed (10 x Student-t, dof 2)."""
    x = torch.randn((m, k), generator=g, device="cuda", dtype=torch.float32)
    n_out = max(1, round(0.005 * k))
    ch = torch.randperm(k, generator=g, device="cuda")[:n_out]
    z = torch.randn((m, n_out), generator=g, device="cuda", dtype=torch.float32)
    e = torch.rand((m, n_out), generator=g, device="cuda", dtype=torch.float32).clamp_min(1e-6)
    x[:, ch] = 10.0 * z * torch.rsqrt((-torch.log(e)).clamp_min(1e-6))
    return x.to(BF16)


def _latent(g, n, k):
    return 0.02 * torch.randn((n, k), generator=g, device="cuda", dtype=torch.float32)


def _pack(g, n, k, layout):
    packed, alpha = B.pack_ternary(_latent(g, n, k), layout=layout)
    return {"w": packed, "alpha": alpha, "n": n, "layout": layout}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(20241104 + seed)
    kind, m = case["kind"], case["tokens"]
    dev = torch.device("cuda")

    if kind == "pair":
        k, n = case["k"], case["n"]
        x = torch.randn((m, k), generator=g, device=dev, dtype=torch.float32)
        x[:, torch.randperm(k, generator=g, device=dev)[:4]] *= 20.0
        return {"kind": kind, "x": x, "w1": _pack(g, n, k, B.BL_W_GEMM), "w2": _pack(g, k, n, B.BL_W_GEMM),
                "topk": n // 2}

    if kind == "train":
        k, n = case["k"], case["n"]
        return {"kind": kind, "m": m, "k": k, "n": n, "topk": case["topk"], "x": _heavy(g, m, k), "w": _latent(g, n, k),
                "dy": (1e-3 * torch.randn((m, n), generator=g, device=dev, dtype=torch.float32)).to(BF16)}

    if kind == "states":
        h, d, pos0 = case["heads"], case["dim"], case["pos0"]
        st = {"kind": kind, "pos0": pos0, "m": m, "h": h, "d": d}
        for name in ("k", "v"):
            st[name + "_cache"] = B.kv_cache_new(pos0 + m, h, d, dev)
            if pos0:
                past = torch.randn((pos0, h, d), generator=g, device=dev, dtype=torch.float32).to(BF16)
                B.kv_cache_append(past, 0, *st[name + "_cache"])
        for name in ("q", "k", "v"):
            st[name] = torch.randn((m, h, d), generator=g, device=dev, dtype=torch.float32).to(BF16)
        return st

    # stacks of layers.  Up to 64 tokens read the 2-bit tiles; more tokens the block-float form of the INT4
    # projections (2-bit codes; E2M1 nibbles for FP4 activations).  Workspaces and outputs are kept, as a
    # serving loop keeps them.
    hidden, ffn = case["hidden"], case["ffn"]
    a4 = {"decode": B.BL_W_GEMM, "prefill": B.BL_W_MX2, "fp4": B.BL_W_MX4}[kind]
    a4_mode = {"decode": B.BL_ACT_INT4_ABSMEAN, "prefill": B.BL_ACT_INT4_ABSMEAN_MX6, "fp4": B.BL_ACT_FP4_E2M1_B32_MX}[kind]
    layers = []
    for _ in range(case["layers"]):
        layers.append({
            "x": _heavy(g, m, hidden), "attn": _heavy(g, m, hidden), "x_ffn": _heavy(g, m, hidden),
            "qkv": _pack(g, 3 * hidden, hidden, a4), "o": _pack(g, hidden, hidden, B.BL_W_GEMM),
            "gate": _pack(g, ffn, hidden, a4), "up": _pack(g, ffn, hidden, a4), "down": _pack(g, hidden, ffn, B.BL_W_GEMM),
            "y_qkv": torch.empty((m, 3 * hidden), dtype=BF16, device=dev), "y_o": torch.empty((m, hidden), dtype=BF16, device=dev),
            "y_down": torch.empty((m, hidden), dtype=BF16, device=dev), "h": torch.empty((m, ffn), dtype=BF16, device=dev),
        })
    st = {"kind": kind, "m": m, "hidden": hidden, "ffn": ffn, "layers": layers,
          "ws_qkv": B.workspace(a4_mode, m, 3 * hidden, hidden, dev),
          "ws_o": B.workspace(B.BL_ACT_TOPK_INT8_ABSMAX, m, hidden, hidden, dev),
          "ws_down": B.workspace(B.BL_ACT_TOPK_INT8_ABSMAX, m, hidden, ffn, dev)}
    if kind == "fp4":
        st["ws_up"] = B.workspace(a4_mode, m, ffn, hidden, dev)
        st["gate"] = torch.empty((m, ffn), dtype=BF16, device=dev)
        st["up"] = torch.empty((m, ffn), dtype=BF16, device=dev)
    else:
        n = B.lib().bitlinear_gate_up_workspace_bytes(m, ffn, hidden, a4)
        st["ws_up"] = torch.empty(max(n, 16), dtype=torch.uint8, device=dev)
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    kind = st["kind"]
    if kind == "pair":
        y1 = B.bitlinear_a4(st["x"], st["w1"]["w"], st["w1"]["alpha"], st["w1"]["n"], y_dtype=torch.float32)
        y2 = B.bitlinear_a8_sparse(y1, st["topk"], st["w2"]["w"], st["w2"]["alpha"], st["w2"]["n"], y_dtype=torch.float32)
        return [y1, y2]

    if kind == "train":
        m, k, n, topk = st["m"], st["k"], st["n"], st["topk"]
        mode = B.BL_ACT_TOPK_INT8_ABSMAX if topk else B.BL_ACT_INT4_ABSMEAN
        wf, alpha = B.pack_ternary(st["w"], layout=B.BL_W_GEMM)
        wb, _ = B.pack_ternary(st["w"], layout=B.BL_W_KMAJOR)
        qa = B.quantize_act(st["x"], mode, topk=topk)
        y = B.bitlinear_gemm(qa["q"], qa["scale"], mode, m, k, wf, alpha, n)
        dx, dw = B.bitlinear_backward(st["dy"], qa["q"], qa["scale"], mode, k, wb, alpha)
        return {"y": y, "dx": dx, "dw": dw}

    if kind == "states":
        qc, qs = B.quantize_heads(st["q"], 4)
        out = [qc, qs]
        for name in ("k", "v"):
            cache, scales = st[name + "_cache"]
            B.kv_cache_append(st[name], st["pos0"], cache, scales)
            out += [cache, scales, B.kv_cache_read(cache, scales, 0, st["pos0"] + st["m"], st["h"], st["d"], BF16)]
        return out

    hidden, ffn, out = st["hidden"], st["ffn"], []
    for ly in st["layers"]:
        w = ly["qkv"]
        out.append(B.bitlinear_a4(ly["x"], w["w"], w["alpha"], w["n"], act_fp4=kind == "fp4", ws=st["ws_qkv"], out=ly["y_qkv"],
                                  layout=w["layout"]))
        w = ly["o"]
        out.append(B.bitlinear_a8_sparse(ly["attn"], hidden // 2, w["w"], w["alpha"], w["n"], ws=st["ws_o"], out=ly["y_o"]))
        g, u, d = ly["gate"], ly["up"], ly["down"]
        if kind == "fp4":
            B.bitlinear_a4(ly["x_ffn"], g["w"], g["alpha"], ffn, act_fp4=True, ws=st["ws_up"], out=st["gate"], layout=g["layout"])
            B.bitlinear_a4(ly["x_ffn"], u["w"], u["alpha"], ffn, act_fp4=True, ws=st["ws_up"], out=st["up"], layout=u["layout"])
            qa = B.quantize_act_glu(st["gate"], st["up"], ffn // 2)
            out += [st["gate"], st["up"],
                    B.bitlinear_gemm(qa["q"], qa["scale"], B.BL_ACT_TOPK_INT8_ABSMAX, st["m"], ffn, d["w"], d["alpha"], hidden,
                                     ws=st["ws_down"], out=ly["y_down"])]
        else:
            r = B.bitlinear_a4_gate_up(ly["x_ffn"], g["w"], g["alpha"], u["w"], u["alpha"], ffn, layout=g["layout"],
                                       want=("H",), ws=st["ws_up"], out={"H": ly["h"]})
            out += [r["H"], B.bitlinear_a8_sparse(r["H"], ffn // 2, d["w"], d["alpha"], hidden, ws=st["ws_down"],
                                                  out=ly["y_down"])]
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind, m = case["kind"], case["tokens"]
    if kind == "pair":
        k, n = case["k"], case["n"]
        return {"bytes": 4 * m * (2 * k + n) + 2 * n * k / 4, "flops": 4.0 * m * n * k}
    if kind == "train":
        # latent weights, X and dY read, Y, dX and dW written
        k, n = case["k"], case["n"]
        return {"bytes": 4 * n * k + 2 * m * k + 2 * m * n + 2 * m * n + 2 * m * k + 4 * n * k, "flops": 6.0 * m * n * k}
    if kind == "states":
        heads, d, end = case["heads"], case["dim"], case["pos0"] + m
        per = heads * d
        q = m * per * 2 + m * per / 2 + 4 * m * heads
        kv = m * per * 2 + m * (per * 3 / 8 + 4 * heads) + end * (per * 3 / 8 + 4 * heads + per * 2)
        return {"bytes": q + 2 * kv, "flops": 0}
    # layers: packed weights and token rows read, outputs written (H stays inside where the linears allow it)
    hidden, ffn = case["hidden"], case["ffn"]
    params = 4 * hidden * hidden + 3 * hidden * ffn
    rows = 3 * hidden + 3 * hidden + hidden + hidden
    rows += 2 * ffn if kind == "fp4" else ffn          # G and U, or H, are outputs
    return {"bytes": case["layers"] * (params / 4 + 2.0 * m * rows), "flops": case["layers"] * 2.0 * m * params}


def tolerance(case):
    # FP4: float32 sums inside the matrix instruction, then bfloat16 outputs (against sums in float64: rel 1.5e-3, the
    # output rounding).  Training: bfloat16(dY * scale) operands and bfloat16 dX (against float64: rel 1.7e-3 for
    # either gradient).  Everything else is integer sums and single float32 operations in a fixed order.
    return {"rel": 6e-3} if case["kind"] in ("fp4", "train") else "exact"
