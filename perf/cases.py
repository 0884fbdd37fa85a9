"""The work this library is asked to do, as cases that can be timed and compared.

Every case goes through the public entry points of `paper_2512_12131_amd.binding` the way a training or
serving program calls them: weights, checkpoints, gradient buffers and the block's workspace are held by
the caller; the layer-level calls return fresh outputs.  Kinds of cases:

  linear     one bottleneck layer, forward (also through the entry point that allocates nothing) or forward
             and backward, fp32 or bf16
  group      projections that share one input with RMSNorm folded in (Q/K/V, gate/up)
  block      the decoder block: forward alone (prefill) or forward and backward (a training step with rank-r
             checkpoints), with grouped key / value heads, rotary embedding, sigma = identity and LaX forms,
             fp32 or bf16 gradients
  attention  causal attention on its own, forward or forward and backward
  streams    the standalone memory-bound kernels: norm statistic, norm, its reverse, SwiGLU and its reverse

Sizes are those of the library's own benchmark workloads and tests (model shapes with rank d / 4, batch times
sequence up to 16384 tokens) and ragged relatives of them.
"""
import math

import torch

from paper_2512_12131_amd import binding as B

DEV = "cuda:0"
EPS = 1e-5
HD = 128
MAX_TOKENS = 16384


def listed():
    return [
        # the library's smallest configuration: one fp32 layer on 512 tokens, a training step of a small model or
        # of a numerical check; seven launches of next to no work each
        {"name": "linear_f32_step", "kind": "linear", "T": 512, "d_in": 256, "r": 64, "d_out": 256, "dtype": "f32",
         "act": "silu", "mode": "step"},
        # one 7B layer in a tight serving loop: a handful of tokens, no workspace, both weight matrices read once
        {"name": "linear_serve_16", "kind": "linear", "T": 16, "d_in": 4096, "r": 1024, "d_out": 4096,
         "dtype": "bf16", "act": "silu", "mode": "static"},
        # one layer of a mid-sized model on an odd number of tokens (packed, unpadded text), forward and backward
        {"name": "linear_ragged_step", "kind": "linear", "T": 1031, "d_in": 1024, "r": 256, "d_out": 768,
         "dtype": "bf16", "act": "silu", "mode": "step"},
        # grouped Q/K/V projections of the 1B shape with the norm folded in, forward and backward
        {"name": "group_qkv_1b_step", "kind": "group", "T": 16384, "d_in": 2048, "r": 512, "d_out": 2048, "G": 3,
         "norm": "online", "grad": "f32", "mode": "step"},
        # the smallest block the benchmark knows: unit tests, debugging runs and smoke training live here
        {"name": "block_tiny_step", "kind": "block", "batch": 2, "seq": 256, "heads": 2, "kv_heads": 2, "ffn": 344,
         "rank": 64, "variant": "silu", "rope": False, "chain": False, "grad": "f32", "mode": "step"},
        # the 1B block (d_ff 5461 is odd: padded to 5464)
        {"name": "block_1b_step", "kind": "block", "batch": 8, "seq": 2048, "heads": 16, "kv_heads": 16,
         "ffn": 5461, "rank": 512, "variant": "silu", "rope": False, "chain": False, "grad": "f32", "mode": "step"},
        # the headline workload: a middle block of a 7B stack, batch 4 x 4096 tokens
        {"name": "block_7b_step", "kind": "block", "batch": 4, "seq": 4096, "heads": 32, "kv_heads": 32,
         "ffn": 11008, "rank": 1024, "variant": "silu", "rope": False, "chain": True, "grad": "f32", "mode": "step"},
        # the same block with rank 128, pure bf16 training: most projections are bound by memory
        {"name": "block_7b_r128_step", "kind": "block", "batch": 4, "seq": 4096, "heads": 32, "kv_heads": 32,
         "ffn": 11008, "rank": 128, "variant": "silu", "rope": False, "chain": False, "grad": "bf16",
         "mode": "step"},
        # one rank's share of the 7B block under tensor parallelism of degree 8
        {"name": "block_7b_tp8_step", "kind": "block", "batch": 4, "seq": 4096, "heads": 4, "kv_heads": 4,
         "ffn": 1376, "rank": 1024, "variant": "silu", "rope": False, "chain": False, "grad": "f32", "mode": "step"},
        # prefill: the forward of a 7B block with grouped key / value heads and rotary embedding on one prompt
        # of odd length
        {"name": "block_7b_prefill_777", "kind": "block", "batch": 1, "seq": 777, "heads": 32, "kv_heads": 8,
         "ffn": 11008, "rank": 1024, "variant": "silu", "rope": True, "chain": False, "grad": "f32", "mode": "fwd"},
        # attention alone, grouped key / value heads, a sequence length that is a multiple of nothing
        {"name": "attention_gqa_ragged_step", "kind": "attention", "batch": 2, "seq": 2047, "heads": 32,
         "kv_heads": 8, "mode": "step"},
        # the standalone memory-bound kernels at the 7B widths
        {"name": "streams_7b", "kind": "streams", "T": 8192, "d": 4096, "f": 11008},
    ]


# ---- drawn cases -------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult8(v):
    return max(8, int(round(v / 8.0)) * 8)


def _tokens(rng, lo, hi):
    """Any number of tokens: half of the time whatever comes, else a multiple of 64."""
    t = int(_log(rng, lo, hi))
    return t if rng.random() < 0.5 or t < 64 else t // 64 * 64


def draw(rng):
    kind = rng.choice(["linear", "linear", "group", "block", "block", "block", "attention", "streams"])
    if kind == "linear":
        mode = rng.choice(["static", "fwd", "step"])
        if rng.random() < 0.25:       # the precision path, small models
            return {"kind": kind, "T": _tokens(rng, 1, 1024), "d_in": int(_log(rng, 40, 512)), "r": int(_log(rng, 12, 128)),
                    "d_out": int(_log(rng, 40, 512)), "dtype": "f32", "act": rng.choice(["silu", "identity"]), "mode": mode}
        d = _mult8(_log(rng, 256, 4096))
        r = _mult8(d / 4 if rng.random() < 0.7 else _log(rng, 64, d / 2))
        return {"kind": kind, "T": _tokens(rng, 4, 8192), "d_in": d, "r": min(r, 1024),
                "d_out": rng.choice([d, _mult8(d * rng.uniform(0.5, 3.0))]), "dtype": "bf16",
                "act": rng.choice(["silu", "silu", "identity"]), "mode": mode}
    if kind == "group":
        d = _mult8(_log(rng, 512, 4096))
        return {"kind": kind, "T": _tokens(rng, 256, MAX_TOKENS), "d_in": d, "r": _mult8(d / 4),
                "d_out": rng.choice([d, _mult8(d * 2.6875)]), "G": rng.choice([2, 3]),
                "norm": rng.choice(["online", "online", "two_pass", "none"]), "grad": rng.choice(["f32", "bf16"]),
                "mode": rng.choice(["fwd", "step"])}
    if kind == "block":
        heads = rng.choice([2, 4, 6, 8, 12, 16, 24, 32])
        kv = rng.choice([h for h in (heads, heads, heads // 2, heads // 4) if h >= 1 and heads % h == 0])
        d = heads * HD
        seq = _tokens(rng, 64, 4096)
        batch = rng.choice([b for b in (1, 2, 3, 4, 8) if b * seq <= MAX_TOKENS])
        ffn = int(d * rng.uniform(2.3, 3.0))
        rank = _mult8(d / 4) if rng.random() < 0.6 else _mult8(_log(rng, 64, 1024))
        return {"kind": kind, "batch": batch, "seq": seq, "heads": heads, "kv_heads": kv, "ffn": ffn, "rank": rank,
                "variant": rng.choice(["silu", "silu", "silu", "identity", "lax"]), "rope": rng.random() < 0.4,
                "chain": rng.random() < 0.5, "grad": rng.choice(["f32", "f32", "bf16"]),
                "mode": rng.choice(["fwd", "step", "step"])}
    if kind == "attention":
        heads = rng.choice([2, 4, 8, 16, 32])
        kv = rng.choice([h for h in (heads, heads, heads // 4) if h >= 1])
        seq = _tokens(rng, 64, 4096)
        batch = rng.choice([b for b in (1, 2, 4, 8) if b * seq <= MAX_TOKENS])
        return {"kind": kind, "batch": batch, "seq": seq, "heads": heads, "kv_heads": kv,
                "mode": rng.choice(["fwd", "step"])}
    d = _mult8(_log(rng, 256, 4096))
    return {"kind": kind, "T": _tokens(rng, 128, MAX_TOKENS), "d": d, "f": _mult8(d * rng.uniform(2.3, 3.0))}


# ---- inputs ------------------------------------------------------------------------------------------------
class _Source:
    """Gaussians on the GPU from one seed; drawn in fp32 and rounded to the storage type."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def __call__(self, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
        t = torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32)
        return t.mul_(std).add_(mean).to(dtype)


_ACTS = {"silu": B.LR_ACT_SILU, "identity": B.LR_ACT_IDENTITY}
_NORMS = {"online": B.LR_NORM_ONLINE, "two_pass": B.LR_NORM_TWO_PASS, "none": B.LR_NORM_NONE}
_GRADS = {"f32": B.LR_F32, "bf16": B.LR_BF16}
_LAX_WIDTHS = {"qkv": 3, "o": 1, "gu": 2, "d": 1}


def _prepare_linear(c, src):
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    s = {"x": src((c["T"], c["d_in"]), dtype=dt), "w_down": src((c["r"], c["d_in"]), c["d_in"] ** -0.5, dtype=dt),
         "w_up": src((c["d_out"], c["r"]), c["r"] ** -0.5, dtype=dt), "act": _ACTS[c["act"]]}
    if c["mode"] == "step":
        s["dy"] = src((c["T"], c["d_out"]), dtype=dt)
    if c["mode"] == "static":   # this entry point writes into the caller's tensors
        s["z"] = torch.empty((c["T"], c["r"]), dtype=dt, device=DEV)
        s["y"] = torch.empty((c["T"], c["d_out"]), dtype=dt, device=DEV)
    return s


def _run_linear(c, s):
    if c["mode"] == "static":
        return B.lr_linear_fwd_static(s["x"], s["w_down"], s["w_up"], s["z"], s["y"], s["act"])
    z, y = B.lr_linear_fwd(s["x"], s["w_down"], s["w_up"], s["act"])
    if c["mode"] == "fwd":
        return z, y
    return (z, y) + B.lr_linear_bwd(s["x"], s["w_down"], s["w_up"], z, s["dy"], s["act"])


def _prepare_group(c, src):
    T, d, r, n, G = c["T"], c["d_in"], c["r"], c["d_out"], c["G"]
    s = {"x": src((T, d)), "gamma": src((d,), 0.1, 1.0), "w_down": src((G * r, d), d ** -0.5),
         "w_up": src((G, n, r), r ** -0.5), "norm": _NORMS[c["norm"]], "grad": _GRADS[c["grad"]]}
    if c["mode"] == "step":
        s["dy"] = src((G, T, n))
    return s


def _run_group(c, s):
    z, stat, y = B.lr_group_fwd(s["x"], s["gamma"], EPS, s["norm"], s["w_down"], s["w_up"])
    normed = c["norm"] != "none"     # without a norm, stat and dgamma are not written
    out = (z, y) + ((stat,) if normed else ())
    if c["mode"] == "step":
        dx, dgamma, dwd, dwu = B.lr_group_bwd(s["x"], s["gamma"], EPS, s["norm"], s["w_down"], s["w_up"], z, stat,
                                              s["dy"], grad_dt=s["grad"])
        out += (dx, dwd, dwu) + ((dgamma,) if normed else ())
    return out


def _prepare_block(c, src):
    Bn, S, H, r, f = c["batch"], c["seq"], c["heads"], c["rank"], c["ffn"]
    T, d, dkv = Bn * S, H * HD, c["kv_heads"] * HD
    f_ld = (f + 7) // 8 * 8

    def rows(w):                     # zero pad rows of the ffn axis
        return torch.nn.functional.pad(w, (0, 0, 0, f_ld - f)).contiguous()

    p = {"gamma1": src((d,), 0.1, 1.0), "w_dn_qkv": src((3 * r, d), d ** -0.5),
         "w_up_qkv": src((d + 2 * dkv, r), r ** -0.5), "w_dn_o": src((r, d), d ** -0.5),
         "w_up_o": src((d, r), r ** -0.5), "gamma2": src((d,), 0.1, 1.0), "w_dn_gu": src((2 * r, d), d ** -0.5),
         "w_up_gu": torch.stack([rows(src((f, r), r ** -0.5)), rows(src((f, r), r ** -0.5))]),
         "w_dn_d": torch.nn.functional.pad(src((r, f), f ** -0.5), (0, f_ld - f)).contiguous(),
         "w_up_d": src((d, r), r ** -0.5)}
    if dkv == d:
        p["w_up_qkv"] = p["w_up_qkv"].view(3, d, r)
    rope = None
    if c["rope"]:
        ang = torch.arange(S, dtype=torch.float64)[:, None] * 10000.0 ** (-2.0 * torch.arange(64, dtype=torch.float64) / HD)
        rope = (torch.cos(ang).float().to(DEV), torch.sin(ang).float().to(DEV))
    sy = torch.empty((T,), dtype=torch.float32, device=DEV) if c["chain"] else None
    act = B.LR_ACT_SILU if c["variant"] == "silu" else B.LR_ACT_IDENTITY
    desc = B.make_block_desc(Bn, S, d, H, HD, f, f_ld, r, eps=EPS, act=act, rope=rope, stat_x_ready=c["chain"],
                             stat_y_out=sy, grad_dt=_GRADS[c["grad"]], n_kv_heads=c["kv_heads"])
    x = src((T, d))
    step = c["mode"] == "step"
    ck = B.alloc_block_ckpt(desc, DEV)
    if c["chain"]:                   # what the block below hands over
        ck["s1"].copy_(x.float().square_().sum(1))
    s = {"desc": desc, "params": p, "x": x, "ck": ck, "sy": sy, "y": torch.empty_like(x), "step": step,
         "ws": torch.empty(max(B.lr_block_workspace_bytes(desc, 0), B.lr_block_workspace_bytes(desc, 1) if step else 0),
                           dtype=torch.uint8, device=DEV)}
    if c["variant"] == "lax":        # a middle block of a stack: the rank-r activations of the block below arrive
        s["h_prev"] = {n: src((T, w * r), 0.5) for n, w in _LAX_WIDTHS.items()}
    if step:
        gt = torch.float32 if c["grad"] == "f32" else torch.bfloat16
        s["dy"], s["dx"] = src((T, d)), torch.empty_like(x)
        s["grads"] = {n: torch.zeros_like(p[n], dtype=gt) for n in B.PARAM_NAMES}
        if c["variant"] == "lax":
            s["dz_next"] = {n: src((T, w * r)) for n, w in _LAX_WIDTHS.items()}
    return s


def _run_block(c, s):
    lax = c["variant"] == "lax"
    if lax:
        B.lr_block_lax_fwd(s["desc"], s["params"], s["x"], h_prev=s["h_prev"], ckpt=s["ck"], ws=s["ws"], y=s["y"])
    else:
        B.lr_block_fwd(s["desc"], s["params"], s["x"], ckpt=s["ck"], ws=s["ws"], y=s["y"])
    out = {"y": s["y"], "ck": s["ck"]}
    if s["sy"] is not None:
        out["stat_y"] = s["sy"]
    if s["step"]:
        if lax:
            _, _, out["dh_prev"] = B.lr_block_lax_bwd(s["desc"], s["params"], s["x"], s["dy"], s["ck"],
                                                      h_prev=s["h_prev"], dz_next=s["dz_next"], grads=s["grads"],
                                                      ws=s["ws"], dx=s["dx"])
        else:
            B.lr_block_bwd(s["desc"], s["params"], s["x"], s["dy"], s["ck"], grads=s["grads"], ws=s["ws"], dx=s["dx"])
        out["dx"], out["grads"] = s["dx"], s["grads"]
    return out


def _prepare_attention(c, src):
    T, d, dkv = c["batch"] * c["seq"], c["heads"] * HD, c["kv_heads"] * HD
    s = {"q": src((T, d)), "k": src((T, dkv)), "v": src((T, dkv))}
    if c["mode"] == "step":
        s["do"] = src((T, d))
    return s


def _run_attention(c, s):
    shape = (c["batch"], c["seq"], c["heads"], c["kv_heads"], HD)
    o, lse = B.lr_attention_gqa_fwd(s["q"], s["k"], s["v"], *shape)
    if c["mode"] == "fwd":
        return o, lse
    return (o, lse) + B.lr_attention_gqa_bwd(s["q"], s["k"], s["v"], o, s["do"], lse, *shape)


def _prepare_streams(c, src):
    T, d, f = c["T"], c["d"], c["f"]
    return {"x": src((T, d)), "gamma": src((d,), 0.1, 1.0), "dxhat": src((T, d)), "dres": src((T, d)),
            "g": src((T, f)), "u": src((T, f)), "dm": src((T, f))}


def _run_streams(c, s):
    stat = B.lr_rms_stat(s["x"])
    xhat = B.lr_rmsnorm_apply(s["x"], s["gamma"], stat, EPS)
    dx, part = B.lr_rmsnorm_bwd(s["x"], s["gamma"], stat, EPS, s["dxhat"], s["dres"])
    dgamma = part.sum(0)             # the partial column sums are the caller's to add up
    m = B.lr_swiglu_fwd(s["g"], s["u"])
    dg, du = B.lr_swiglu_bwd(s["g"], s["u"], s["dm"])
    return stat, xhat, dx, dgamma, m, dg, du


_PREPARE = {"linear": _prepare_linear, "group": _prepare_group, "block": _prepare_block, "attention": _prepare_attention,
            "streams": _prepare_streams}
_RUN = {"linear": _run_linear, "group": _run_group, "block": _run_block, "attention": _run_attention,
        "streams": _run_streams}


def prepare(case, seed):
    return case, _PREPARE[case["kind"]](case, _Source(seed))


def run(state):
    case, s = state
    return _RUN[case["kind"]](case, s)


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def work(case):
    """FLOPs: 2MNK per product over the logical sizes, attention counted causal-halved; a block step counts the
    re-forward from the rank-r checkpoints, which is all the backward is handed.  Bytes: every input of a pass
    read once, every output written once, nothing in between."""
    c, k = case, case["kind"]
    if k == "linear":
        es = 4 if c["dtype"] == "f32" else 2
        T, d, r, n = c["T"], c["d_in"], c["r"], c["d_out"]
        fl, el = 2.0 * T * r * (d + n), T * (d + r + n) + r * (d + n)
        by = float(es) * el
        if c["mode"] == "step":      # dy in; dx, fp32 weight gradients out
            fl, by = 3 * fl, by + es * T * (d + n) + 4.0 * r * (d + n)
        return {"bytes": by, "flops": fl}
    if k == "group":
        T, d, r, n, G = c["T"], c["d_in"], c["r"], c["d_out"], c["G"]
        fl = 2.0 * T * G * r * (d + n)
        by = 2.0 * (T * (d + G * r + G * n) + G * r * (d + n))
        if c["mode"] == "step":
            fl, by = 3 * fl, by + 2.0 * T * (d + G * n) + (4.0 if c["grad"] == "f32" else 2.0) * G * r * (d + n)
        return {"bytes": by, "flops": fl}
    if k == "block":
        T, d, f, r = c["batch"] * c["seq"], c["heads"] * HD, c["ffn"], c["rank"]
        dkv = c["kv_heads"] * HD
        weights = r * (9.0 * d + 2 * dkv + 3 * f)
        lin = 2.0 * T * weights
        attn = 2.0 * c["batch"] * c["heads"] * float(c["seq"]) ** 2 * HD
        by = 2.0 * (2 * T * d + 7 * T * r + weights)
        if c["mode"] == "fwd":
            return {"bytes": by, "flops": lin + attn}
        again = 2.0 * T * r * (2 * d + 2 * dkv + 2 * f)      # six of the seven up-projections, and the attention
        by += 2.0 * 2 * T * d + (4.0 if c["grad"] == "f32" else 2.0) * weights
        if c["variant"] == "lax":
            by += 2.0 * 3 * 7 * T * r
        return {"bytes": by, "flops": 3 * lin + again + attn * 4.5}
    if k == "attention":
        T, d, dkv = c["batch"] * c["seq"], c["heads"] * HD, c["kv_heads"] * HD
        fl = 2.0 * c["batch"] * c["heads"] * float(c["seq"]) ** 2 * HD
        by = 2.0 * T * (2 * d + 2 * dkv)
        if c["mode"] == "step":
            fl, by = 3.5 * fl, by + 2.0 * T * (2 * d + 2 * dkv)
        return {"bytes": by, "flops": fl}
    T, d, f = c["T"], c["d"], c["f"]
    return {"bytes": 2.0 * T * (7 * d + 8 * f), "flops": 10.0 * T * (d + f)}


# Relative error in the 2-norm, the largest over a pass's outputs, measured against the same path in 64 bits: 5.4e-7
# (fp32 layer), 3.6e-3 (bf16 layers and groups), 3.0e-3 (attention), 1.7e-3 (streams: one rounding), 6.5e-3 (block:
# weight gradients behind a chain of about ten bf16 tensors).  The bounds are three to five times that, because two
# correct implementations each show it.
_REL = {"linear": 1e-2, "group": 1e-2, "attention": 1e-2, "streams": 5e-3, "block": 2e-2}


def tolerance(case):
    if case["kind"] == "linear" and case["dtype"] == "f32":
        return {"rel": 2.5e-6}
    return {"rel": _REL[case["kind"]]}
