"""Performance cases of the SharQ linear layer: the calls that a program which serves a model makes.

A case is one linear layer's work (or its preparation alone) through the public entry points of
`paper_2606_26587_amd.sharq`, on buffers that such a program holds: quantized weights, the prepared
activation's buffers and the output.  Shapes are the linears of Llama-3.1-8B, Qwen2.5-7B and Qwen3-30B-A3B
that the benchmark uses, at decode, chunk and prefill row counts, and generic ragged ones.
"""

import math

import torch

from paper_2606_26587_amd import sharq as S

EPS = 1e-5

# kind: "linear"   prepare (or prepare_residual / prepare_silu_mul, by `src`), then the two-path GEMM
#       "fused"    sharq_prepare_linear, the one-call form
#       "prepare"  the preparation alone
#       "moe"      prepare, then the grouped GEMM over the routed rows
# src:  "plain" | "norm" (RMSNorm) | "residual" (residual add and RMSNorm) | "silu" (SiLU.mul)
# backbone: "compressed" (the default form) | "dense" (the dense copy alone, which the benchmark uses)


def _case(name, kind, fmt, nm, src, M, K, N, backbone="dense", out="bf16", tokens=0, experts=0, topk=0):
    c = {"name": name, "kind": kind, "fmt": fmt, "nm": nm, "src": src, "M": M, "K": K, "N": N, "backbone": backbone,
         "out": out, "tokens": tokens, "experts": experts, "topk": topk}
    if not name:
        del c["name"]
    return c


def listed():
    return [
        # one token of one sequence: Llama-3.1-8B qkv, the smallest call
        _case("decode_qkv_m1_mx", "fused", "mx", "2:4", "norm", 1, 4096, 6144),
        # a decode batch of 16 on the widest Llama projection, the API's default storage
        _case("decode_gate_up_m16_mx", "linear", "mx", "2:4", "norm", 16, 4096, 28672, "compressed"),
        # a small decode batch in the paper's own setting (NVFP4, 4:8 in pairs), down projection behind SiLU.mul
        _case("decode_down_m4_nv_pairs", "linear", "nv", "4:8p", "silu", 4, 14336, 4096),
        # the preparation by itself: RMSNorm, mask and both quantizations of a prefill batch
        _case("prepare_m2048_mx", "prepare", "mx", "2:4", "norm", 2048, 4096, 0),
        # Llama prefill: residual add + RMSNorm into gate/up, and SiLU.mul into down
        _case("prefill_gate_up_mx", "linear", "mx", "2:4", "residual", 2048, 4096, 28672),
        _case("prefill_down_mx", "linear", "mx", "2:4", "silu", 2048, 14336, 4096),
        # Llama prefill qkv in the paper's own setting
        _case("prefill_qkv_nv_pairs", "linear", "nv", "4:8p", "norm", 2048, 4096, 6144),
        # Qwen2.5-7B prefill gate/up, NVFP4 2:4: the largest call
        _case("prefill_gate_up_qwen_nv", "linear", "nv", "2:4", "norm", 4096, 3584, 37888),
        # Qwen3-30B-A3B experts: gate/up of a prefill batch, and down of a decode batch
        _case("moe_gate_up_prefill_mx", "moe", "mx", "4:8", "norm", 4096, 2048, 1536, tokens=4096, experts=128,
              topk=8),
        _case("moe_down_decode_mx", "moe", "mx", "4:8", "plain", 512, 768, 2048, tokens=64, experts=128, topk=8),
        # HiF4, the accuracy format, on Llama qkv
        _case("prefill_qkv_hif4", "linear", "hif4", "2:4", "norm", 2048, 4096, 6144, "compressed"),
        # ragged rows, columns and K (no whole 128-wide panel at the end), fp32 output
        _case("ragged_m300_mx", "linear", "mx", "2:4", "plain", 300, 4000, 1000, "compressed", "f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fmt = rng.choice(["mx", "mx", "mx", "nv", "nv", "nv", "hif4"])
    kind = rng.choice(["linear", "linear", "linear", "fused", "prepare"] + (["moe"] if fmt == "mx" else []))
    nm = "2:4" if fmt == "hif4" else rng.choice(["2:4", "4:8", "4:8p"])
    out = rng.choice(["bf16", "bf16", "f32"])
    if kind == "moe":
        experts = rng.choice([8, 32, 64, 128])
        topk = rng.choice([2, 4, 8])
        tokens = _log_int(rng, 16, 4096)
        gather = rng.random() < 0.5
        return _case("", kind, fmt, nm, "norm" if gather else "plain", tokens if gather else tokens * topk,
                     128 * _log_int(rng, 6, 32), 8 * _log_int(rng, 64, 256), "dense", out, tokens, experts, topk)
    ragged = rng.random() < 0.2
    K = (64 if fmt == "hif4" else 32) * _log_int(rng, 32, 224) if ragged else 128 * _log_int(rng, 8, 148)
    src = rng.choice(["plain", "norm"] if kind == "fused" or fmt == "hif4" else ["plain", "norm", "residual", "silu"])
    if K > 16384 and src in ("norm", "residual"):
        src = "plain"
    M = _log_int(rng, 1, 64 if kind == "fused" else 4096)
    backbone = "compressed" if fmt == "hif4" or K % 128 else rng.choice(["dense", "compressed"])
    if kind == "prepare":
        return _case("", kind, fmt, nm, src, max(M, 16), K, 0, backbone)
    # the generic (ragged) and the 16-bit forms cost more per element
    most = 5.5e11 / (4 if fmt == "hif4" or K % 128 else 2 if backbone == "compressed" else 1)
    N = min(_log_int(rng, 256, 37888), int(most / (M * K)))
    if rng.random() < 0.7:
        N = max(64, N // 64 * 64)
    return _case("", kind, fmt, nm, src, M, K, max(N, 64), backbone, out)


# ---------------------------------------------------------------------------
# Inputs: normal activations with outlier channels and one massive token, normal weights
# ---------------------------------------------------------------------------

def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + stream)


def _acts(M, K, g):
    x = torch.randn((M, K), device="cuda", generator=g)
    ch = torch.randperm(K, device="cuda", generator=g)[:max(1, round(0.005 * K))]
    x[:, ch] *= torch.rand(ch.numel(), device="cuda", generator=g) * 80 + 20
    x[0, torch.randperm(K, device="cuda", generator=g)[:2]] *= 1000
    return x.to(torch.bfloat16)


def _inputs(case, seed):
    """x, the second operand (residual / up), gamma, W and the routing, as tensors on the GPU."""
    M, K, N, src = case["M"], case["K"], case["N"], case["src"]
    g = _gen(seed, 0)
    d = {"x": None, "x2": None, "gamma": None, "w": None, "rows": None, "offsets": None}
    if src == "silu":   # the two halves of a gate/up projection's output
        gu = torch.cat([torch.randn((M, K), device="cuda", generator=g) * 1.5, _acts(M, K, g).float() * 0.5], 1)
        gu = gu.to(torch.bfloat16)
        d["x"], d["x2"] = gu[:, :K], gu[:, K:]
    else:
        d["x"] = _acts(M, K, g)
    if src == "residual":
        d["x2"] = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
    if src in ("norm", "residual"):
        d["gamma"] = (1 + 0.1 * torch.randn(K, device="cuda", generator=_gen(seed, 1))).to(torch.bfloat16)
    E = case["experts"]
    if N:
        gw = _gen(seed, 2)
        n_w = max(E, 1)
        d["w"] = [(0.02 * torch.randn((N, K), device="cuda", generator=gw)).to(torch.bfloat16) for _ in range(n_w)]
    if E:
        T, k = case["tokens"], min(case["topk"], E)
        logits = torch.randn((T, E), device="cuda", generator=_gen(seed, 3))
        ex = logits.topk(k, dim=1).indices.reshape(-1)
        perm = torch.sort(ex, stable=True).indices
        off = torch.zeros(E + 1, dtype=torch.int64, device="cuda")
        off[1:] = torch.bincount(ex, minlength=E).cumsum(0)
        d["offsets"] = off.to(torch.int32)
        if src == "norm":   # gate/up gathers the tokens' rows; down's rows are in expert order already
            d["rows"] = (perm // k).to(torch.int32)
    return d


def _nm(case):
    n, m = (2, 4) if case["nm"] == "2:4" else (4, 8)
    return n, m, case["nm"] == "4:8p"


def prepare(case, seed):
    d = _inputs(case, seed)
    M, K, N, fmt = case["M"], case["K"], case["N"], case["fmt"]
    n, m, pairs = _nm(case)
    st = {"case": case, "x": d["x"], "x2": d["x2"], "gamma": d["gamma"], "rows": d["rows"], "offsets": d["offsets"],
          "act": S.alloc_act(M, K, n, m, fmt, "cuda", pairs, dense_only=case["backbone"] == "dense")}
    if case["src"] == "residual":
        st["h"] = torch.empty((M, K), dtype=torch.bfloat16, device="cuda")
    if N:
        ws = [S.sharq_quantize_weight(w, fmt) for w in d["w"]]
        st["w"] = S.stack_weights(ws) if case["experts"] else ws[0]
        total = case["tokens"] * min(case["topk"], case["experts"]) if case["experts"] else M
        dt = torch.float32 if case["out"] == "f32" else torch.bfloat16
        st["y"] = torch.empty((total, N), dtype=dt, device="cuda")
    torch.cuda.synchronize()
    return st


def run(state):
    case, act = state["case"], state["act"]
    fmt = case["fmt"]
    n, m, pairs = _nm(case)
    if case["kind"] == "fused":
        S.sharq_prepare_linear(state["x"], state["gamma"], state["w"], EPS, n, m, fmt, act=act, out=state["y"],
                               pairs=pairs)
        return {"y": state["y"]}
    got = {}
    if case["src"] == "residual":
        S.sharq_prepare_residual(state["x"], state["x2"], state["gamma"], EPS, n, m, fmt, h_out=state["h"], out=act,
                                 pairs=pairs)
        got["h"] = state["h"]
    elif case["src"] == "silu":
        S.sharq_prepare_silu_mul(state["x"], state["x2"], n, m, fmt, out=act, pairs=pairs)
    else:
        S.sharq_prepare(state["x"], state["gamma"], EPS, n, m, fmt, out=act, pairs=pairs)
    if case["kind"] == "prepare":
        got.update({k: getattr(act, k) for k in ("sp_codes", "sp_meta", "sp_dense", "sp_scale", "dn_codes",
                                                 "dn_scale", "tensor_scale")})
    elif case["kind"] == "moe":
        got["y"] = S.sharq_linear_grouped(act, state["rows"], state["offsets"], state["y"].shape[0], state["w"],
                                          out=state["y"])
    else:
        got["y"] = S.sharq_linear(act, state["w"], out=state["y"])
    return got


def work(case):
    M, K, N = case["M"], case["K"], case["N"]
    n, m, _ = _nm(case)
    wide = 2 if case["fmt"] != "mx" else 1          # scale bytes per 32 values of a dense path (HiF4: both paths)
    nbytes = 2 * M * K                              # x
    if case["src"] in ("silu", "residual"):
        nbytes += 2 * M * K                         # up, or the residual
    if case["src"] == "residual":
        nbytes += 2 * M * K                         # h
    if case["src"] in ("norm", "residual"):
        nbytes += 2 * K
    if case["kind"] == "prepare":
        sp = K // 2 if case["backbone"] == "dense" else K * n // m // 2 + K // 8
        sps = K // 16 if case["fmt"] == "hif4" else K // 32
        return {"bytes": nbytes + M * (sp + sps + K // 2 + K // 32 * wide), "flops": 0}
    E = case["experts"]
    rows = case["tokens"] * min(case["topk"], E) if E else M
    used = min(E, rows) if E else 1                 # experts whose weight has to be read
    per_w = N * K // 2 + N * K // (16 if case["fmt"] == "hif4" else 32)
    nbytes += used * per_w + rows * N * (4 if case["out"] == "f32" else 2)
    return {"bytes": nbytes, "flops": 2 * rows * N * K * (m + n) // m}


def tolerance(case):
    if case["kind"] == "prepare":
        return "exact"
    # measured against exact(): bf16 outputs 1.7e-3 (the rounding of the result itself), fp32 outputs below 1e-6
    # but for a handful of codes whose input lies on a rounding boundary of the 64-bit normalization
    if case["out"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 6.6e-3, "max": 1.6e-2}


# ---------------------------------------------------------------------------
# The same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------

_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _e2m1(v):
    """Nearest E2M1 value, ties to the even code, saturating at 6."""
    a = v.abs()
    q = torch.zeros_like(a)
    for i in range(7):   # from code i to i + 1 above their midpoint, and on it if i + 1 is even
        mid = (_E2M1[i] + _E2M1[i + 1]) / 2
        q = torch.where((a > mid) if i % 2 == 0 else (a >= mid), torch.full_like(a, _E2M1[i + 1]), q)
    return q * torch.sign(v)


def _mx(v):
    """MXFP4: blocks of 32, E8M0 = floor(log2 amax) - 2."""
    b = v.reshape(v.shape[0], -1, 32)
    e = torch.frexp(b.abs().amax(2, keepdim=True))[1].to(torch.float64) - 3
    s = torch.exp2(torch.clamp(e, min=-127.0))
    return (_e2m1(b / s) * s).reshape(v.shape)


def _nv_tensor_scale(v):
    top = v.abs().amax().to(torch.float32)
    return top / torch.full_like(top, 2688.0)   # a division: by a plain number, torch multiplies by its reciprocal


def _nv(v, ts, block):
    """NVFP4: one E4M3 scale a block, one 32-bit scale a tensor.  The format defines its scales, the quotients
    that become codes and the dequantized values as 32-bit numbers, so those steps run in 32 bits here."""
    b = v.to(torch.float32).reshape(v.shape[0], -1, block)
    d = torch.clamp(b.abs().amax(2, keepdim=True) / (ts * 6), max=448.0).to(torch.float8_e4m3fn).to(torch.float32)
    q = _e2m1(b / torch.where(d > 0, d * ts, torch.ones_like(d))) * (d > 0)
    return (q * d * ts).reshape(v.shape).double()


def _hif4(v):
    """HiF4: units of 64, an E6M2 scale, one-bit exponents for each 8 and each 4 values, quarters up to 1.75."""
    u = v.reshape(v.shape[0], -1, 64)
    v16 = u.abs().reshape(*u.shape[:2], 16, 4).amax(3)
    v8 = v16.reshape(*u.shape[:2], 8, 2).amax(3)
    seventh = torch.tensor(1 / 7, dtype=torch.bfloat16).item()
    sf = torch.clamp(v8.amax(2) * seventh, 2.0 ** -48, 1.5 * 2.0 ** 15)
    mant, ex = torch.frexp(sf)
    mant = torch.round(mant * 8) / 8 * 2                       # 1.00 .. 2.00 by quarters
    e6 = mant * torch.exp2(ex.to(torch.float64) - 1)
    mant, ex = torch.frexp(e6)
    rec = (1 / (mant * 2)).to(torch.bfloat16).to(torch.float64) * torch.exp2(1.0 - ex.to(torch.float64))
    s8 = (v8 * rec[..., None] >= 4).to(torch.float64)
    s16 = (v16 * rec[..., None] * torch.exp2(-s8.repeat_interleave(2, 2)) >= 2).to(torch.float64)
    sh = torch.exp2(s8.repeat_interleave(8, 2) + s16.repeat_interleave(4, 2))
    q = torch.clamp(torch.round(u * rec[..., None] / sh * 4) / 4, -1.75, 1.75)
    return (q * sh * e6[..., None]).reshape(v.shape)


def _keep(y, n, m, pairs):
    """The n largest magnitudes of every m, or the n/2 best pairs; of equal ones the lower index."""
    a = y.abs().reshape(y.shape[0], -1, m)
    if pairs:
        a = a.reshape(*a.shape[:2], m // 2, 2).amax(3)
    kept = torch.zeros_like(a, dtype=torch.bool)
    top = torch.sort(a, dim=2, descending=True, stable=True).indices[..., :n // 2 if pairs else n]
    kept.scatter_(2, top, True)
    if pairs:
        kept = kept.repeat_interleave(2, 2)
    return kept.reshape(y.shape)


def exact(case, seed):
    if case["kind"] == "prepare":
        return None
    d = _inputs(case, seed)
    fmt = case["fmt"]
    n, m, pairs = _nm(case)
    got = {}
    y = d["x"].double()
    if case["src"] == "residual":
        h = d["x"].double() + d["x2"].double()   # the sum of two bf16 values; stored as bf16
        got["h"] = h
        y = h.to(torch.float32).to(torch.bfloat16).double()
    elif case["src"] == "silu":
        y = (y / (1 + torch.exp(-y)) * d["x2"].double()).to(torch.float32).to(torch.bfloat16).double()
    if d["gamma"] is not None:
        y = y * torch.rsqrt(y.square().mean(1, keepdim=True) + EPS) * d["gamma"].double()
    keep = _keep(y, n, m, pairs)
    kept = torch.where(keep, y, torch.zeros_like(y))
    if fmt == "mx":
        sp = _mx(kept)
        a = sp + _mx(y - sp)
    elif fmt == "nv":
        ts = _nv_tensor_scale(y)
        y = y.to(torch.float32).double()
        kept = torch.where(keep, y, torch.zeros_like(y))
        sp = _nv(kept, ts, 32)
        a = sp + _nv(y - sp, ts, 16)
    else:
        sp = _hif4(kept)
        a = sp + _hif4(y - sp)

    def wq(w):
        w = w.double()
        return _mx(w) if fmt == "mx" else _hif4(w) if fmt == "hif4" else \
            _nv(w, _nv_tensor_scale(w), 32)

    if not case["experts"]:
        got["y"] = a @ wq(d["w"][0]).T
        return got
    off = d["offsets"].tolist()
    out = torch.zeros((off[-1], case["N"]), dtype=torch.float64, device="cuda")
    for e, w in enumerate(d["w"]):
        if off[e + 1] > off[e]:
            rows = slice(off[e], off[e + 1]) if d["rows"] is None else d["rows"][off[e]:off[e + 1]].long()
            out[off[e]:off[e + 1]] = a[rows] @ wq(w).T
    got["y"] = out
    return got
