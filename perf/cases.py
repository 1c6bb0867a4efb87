"""What a user of this library has it do: the prefill of a Finch / Finch-C2 layer over prompts of
every size, the token split for one long context, decode steps and short appends of a server, the
calls of a whole time-mix layer in a row, and the key compression behind the last layer.  Each case
goes through the public entry points on tensors that lie in HBM, as a serving program calls them.

Shapes are those of this repository's benchmark configurations and tests (head size 64; 12, 16, 32
and 64 heads: model widths 768, 1024, 2048 and 4096) with ragged batch and token counts between them.
Values follow the recipes of paper_2407_12077_amd/workloads.py, drawn on the device from the seed.
"""
import math

import torch

import paper_2407_12077_amd as wkv

N = 64                    # head size
INNER, RANK = 32, 64      # ranks of the two low-rank pairs of the decay path
HEADS = (12, 16, 32, 64)
PLACEMENT_ALIGN = 4096    # WKV6_PLACEMENT_ALIGN of the header


def listed():
    return [
        # one layer of a 1.6B model over a batch of eight full-context prompts: the headline workload, with
        # the tensors placed as the header recommends
        {"name": "prefill eight prompts", "kind": "prefill", "form": "finch", "B": 8, "T": 4096, "H": 32,
         "state": False, "out": "bf16", "placement": "arena"},
        # one user's prompt, one tensor per allocation: far fewer (batch, head) units than compute units
        {"name": "prefill one prompt", "kind": "prefill", "form": "finch_c2", "B": 1, "T": 4096, "H": 32,
         "state": False, "out": "bf16", "placement": "separate"},
        # a few prompts of an odd length in a small model, continued from a carried state, unrounded output
        {"name": "prefill ragged small model", "kind": "prefill", "form": "finch", "B": 5, "T": 1531, "H": 12,
         "state": True, "out": "f32", "placement": "separate"},
        # a large batch of short requests with a carried state each
        {"name": "prefill many requests", "kind": "prefill", "form": "finch_c2", "B": 256, "T": 512, "H": 32,
         "state": True, "out": "bf16", "placement": "separate"},
        # one long context: the token-split entry with the segment count the library recommends
        {"name": "split long context", "kind": "split", "form": "finch", "B": 1, "T": 131072, "H": 32,
         "state": False, "out": "bf16", "placement": "separate"},
        # a decode step of a full server, and of a single user: state updated in place
        {"name": "decode full server", "kind": "decode", "form": "finch", "B": 1024, "H": 32},
        {"name": "decode one user", "kind": "decode", "form": "finch_c2", "B": 1, "H": 32},
        # the next turn of a conversation for a group of users: a few tokens onto a carried state
        {"name": "append a turn", "kind": "append", "form": "finch_c2", "B": 32, "T": 24, "H": 32},
        # the calls of one Finch-C2 time-mix layer in a row, and the compression of its output: a prompt batch,
        # and the same calls for one new token per user
        {"name": "layer prompts", "kind": "layer", "B": 8, "T": 2048, "H": 32},
        {"name": "layer one token each", "kind": "layer", "B": 24, "T": 1, "H": 32},
        # the compressed key cache of a long prompt batch
        {"name": "key compression", "kind": "key_compress", "M": 131072, "D": 2048, "out": "bf16"},
        # the all-fp32 entry, as in a parity run of a small model
        {"name": "fp32 small model", "kind": "prefill_f32", "B": 2, "T": 512, "H": 16, "state": True},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "split", "decode", "append", "layer", "layer", "key_compress",
                       "key_compress", "prefill_f32"])
    form = rng.choice(["finch", "finch_c2"])
    H = rng.choice(HEADS)
    if kind == "prefill":
        B = _log(rng, 1, 256)
        T = _log(rng, 32, max(33, min(16384, 3_000_000 // (B * H))))
        return {"kind": kind, "form": form, "B": B, "T": T, "H": H, "state": rng.random() < 0.5,
                "out": rng.choice(["bf16", "bf16", "f32"]), "placement": rng.choice(["separate", "arena"])}
    if kind == "split":
        B = rng.choice([1, 1, 2])
        H = rng.choice((12, 16, 32))
        return {"kind": kind, "form": form, "B": B, "T": _log(rng, 4096, 3_500_000 // (B * H)), "H": H,
                "state": rng.random() < 0.5, "out": "bf16", "placement": "separate"}
    if kind == "decode":
        return {"kind": kind, "form": form, "B": _log(rng, 1, 32768 // H), "H": H}
    if kind == "append":
        return {"kind": kind, "form": form, "B": _log(rng, 1, 256), "T": _log(rng, 2, 64), "H": H}
    if kind == "layer":
        B = _log(rng, 1, 64)
        return {"kind": kind, "B": B, "T": _log(rng, 1, max(2, min(8192, 1_000_000 // (B * H)))), "H": H}
    if kind == "key_compress":
        D = rng.choice((768, 1024, 2048, 4096))
        return {"kind": kind, "M": _log(rng, 1, 131072 * 2048 // D), "D": D, "out": rng.choice(["bf16", "bf16", "f32"])}
    B = _log(rng, 1, 8)
    return {"kind": kind, "B": B, "T": _log(rng, 16, 1024), "H": H, "state": rng.random() < 0.5}


# ----------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, scale, dtype):
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(dtype)


def _uniform(g, shape, lo, hi, dtype):
    return (torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo).to(dtype)


def _time_mix(case, seed, dtype=torch.bfloat16):
    """Tensors of one time-mix call: projections ~ N(0, 1)/8, decay logits ~ U(-6, 1)."""
    g = _gen(seed)
    B, T, H = case["B"], case.get("T", 1), case["H"]
    t = {n: _normal(g, (B, T, H, N), 1 / 8, dtype) for n in ("r", "k", "v")}
    t["x"] = _uniform(g, (B, T, H, N), -6.0, 1.0, dtype)
    if case.get("form") == "finch_c2":
        t["uprime"] = _normal(g, (B, T, H, N), 1 / 8, dtype)
    else:
        t["u"] = _normal(g, (H, N), 0.5, torch.float32)
    t["state_in"] = None
    if case.get("state", True):
        t["state_in"] = _normal(g, (B, H, N, N), 0.1, torch.float32)
    return t


def _layer_inputs(case, seed):
    """Inputs of a Finch-C2 layer from its input x: weights as a trained layer scales them."""
    g = _gen(seed)
    B, T, H = case["B"], case["T"], case["H"]
    D, bf = H * N, torch.bfloat16
    t = {"x": _normal(g, (B, T, D), 1.0, bf), "x_prev": _normal(g, (B, D), 1.0, bf),
         "mu_x": _uniform(g, (D,), 0.0, 1.0, torch.float32), "lambda_d": _uniform(g, (D,), 0.0, 1.0, torch.float32),
         "a_d": _normal(g, (INNER, D), D ** -0.5, bf), "b_d": _normal(g, (D, INNER), 0.1, bf),
         "a_omega": _normal(g, (RANK, D), D ** -0.5, bf), "lambda": _uniform(g, (D,), -5.5, 0.5, torch.float32),
         "b_omega": _normal(g, (RANK, D), 0.2, bf)}
    for n in ("r", "k", "v", "uprime"):
        t[n] = _normal(g, (B, T, H, N), 1 / 8, bf)
    t["state_in"] = _normal(g, (B, H, N, N), 0.1, torch.float32)
    t["gamma"] = _uniform(g, (D,), 0.5, 1.5, torch.float32)
    t["beta"] = _normal(g, (D,), 0.1, torch.float32)
    t["w_kd"] = _normal(g, (D, D // 16), D ** -0.5, bf)
    return t


def _key_inputs(case, seed):
    g = _gen(seed)
    M, D = case["M"], case["D"]
    return {"x": _normal(g, (M, D), 1.0, torch.bfloat16), "w_kd": _normal(g, (D, D // 16), D ** -0.5, torch.bfloat16)}


def _in_arena(tensors):
    """The tensors inside one allocation, placed by the library's own layout helper."""
    sizes = [t.numel() * t.element_size() for t in tensors]
    total, offsets = wkv.wkv6_arena_layout(sizes)
    arena = torch.empty(total + PLACEMENT_ALIGN, dtype=torch.uint8, device="cuda")
    first = (-arena.data_ptr()) % PLACEMENT_ALIGN
    views = []
    for t, off, size in zip(tensors, offsets, sizes):
        view = arena[first + off:first + off + size].view(t.dtype).view(t.shape)
        view.copy_(t)
        views.append(view)
    return views


def prepare(case, seed):
    kind = case["kind"]
    empty = lambda shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    f32, bf = torch.float32, torch.bfloat16
    s = {"case": case}
    if kind == "key_compress":
        s.update(_key_inputs(case, seed))
        s["c"] = empty((case["M"], case["D"] // 16), bf if case["out"] == "bf16" else f32)
        return s
    B, T, H = case["B"], case.get("T", 1), case["H"]
    if kind == "layer":
        s.update(_layer_inputs(case, seed))
        D = H * N
        s.update(y=empty((B, T, RANK), bf), o=empty((B, T, H, N), bf), moments=empty((B, H, T, 2), f32),
                 state_out=empty((B, H, N, N), f32), mean_rstd=empty((B, T, 2), f32), normed=empty((B, T, D), bf),
                 c=empty((B * T, D // 16), bf))
        return s
    s.update(_time_mix(case, seed, f32 if kind == "prefill_f32" else bf))
    s["o"] = empty((B, T, H, N), f32 if kind == "prefill_f32" or case.get("out") == "f32" else bf)
    if kind == "decode":
        return s
    s["state_out"] = empty((B, H, N, N), f32)
    if case.get("placement") == "arena":
        names = [n for n in ("r", "k", "v", "x", "uprime", "o") if n in s]
        s.update(zip(names, _in_arena([s[n] for n in names])))
    if kind == "split":
        s["segments"] = wkv.wkv6_split_segments(B, T, H, N)
        s["workspace"] = empty((max(16, wkv.wkv6_split_workspace_bytes(B, T, H, N, s["segments"])),), torch.uint8)
    return s


# ----------------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    bf16 = wkv.WKV6_DTYPE_BF16
    if kind == "key_compress":
        wkv.wkv6_key_compress_bf16(case["M"], case["D"], s["x"], s["w_kd"], s["c"],
                                   bf16 if case["out"] == "bf16" else wkv.WKV6_DTYPE_F32)
        return s["c"]
    B, T, H = case["B"], case.get("T", 1), case["H"]
    if kind == "layer":
        D = H * N
        wkv.wkv6_decay_lora_input_bf16(B, T, D, INNER, RANK, s["x"], s["x_prev"], s["mu_x"], s["lambda_d"], s["a_d"],
                                       s["b_d"], s["a_omega"], s["y"], bf16)
        wkv.wkv6_finch_c2_prefill_lora_bf16(B, T, H, N, RANK, s["r"], s["k"], s["v"], s["y"], s["lambda"], s["b_omega"],
                                            s["uprime"], s["state_in"], s["o"], s["moments"], s["state_out"])
        wkv.wkv6_layernorm_finalize(B, T, H, N, s["moments"], 1e-5, s["mean_rstd"])
        wkv.wkv6_layernorm_apply_bf16(B, T, H, N, s["o"], s["mean_rstd"], s["gamma"], s["beta"], s["normed"], bf16)
        wkv.wkv6_key_compress_bf16(B * T, D, s["normed"], s["w_kd"], s["c"], bf16)
        return {n: s[n] for n in ("y", "o", "state_out", "mean_rstd", "normed", "c")}
    c2 = case.get("form") == "finch_c2"
    extra = s["uprime"] if c2 else s["u"]
    r, k, v, x, state_in, o = s["r"], s["k"], s["v"], s["x"], s["state_in"], s["o"]
    if kind == "decode":
        (wkv.wkv6_finch_c2_decode_bf16 if c2 else wkv.wkv6_decode_bf16)(B, H, N, r, k, v, x, extra, state_in, o)
        return o, state_in
    if kind == "split":
        fn = wkv.wkv6_finch_c2_prefill_bf16_split if c2 else wkv.wkv6_prefill_bf16_split
        ws = s["workspace"]
        fn(B, T, H, N, r, k, v, x, extra, state_in, o, s["state_out"], bf16, s["segments"], ws, ws.numel())
        return o, s["state_out"]
    if kind == "append":
        fn = wkv.wkv6_finch_c2_append_bf16 if c2 else wkv.wkv6_append_bf16
    elif kind == "prefill_f32":
        fn = wkv.wkv6_prefill_f32
    elif case["out"] == "f32":
        fn = wkv.wkv6_finch_c2_prefill_bf16_f32out if c2 else wkv.wkv6_prefill_bf16_f32out
    else:
        fn = wkv.wkv6_finch_c2_prefill_bf16 if c2 else wkv.wkv6_prefill_bf16
    fn(B, T, H, N, r, k, v, x, extra, state_in, o, s["state_out"])
    return o, s["state_out"]


# ----------------------------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "key_compress":
        M, D = case["M"], case["D"]
        C = D // 16
        return {"bytes": 2 * M * D + 2 * D * C + M * C * (2 if case["out"] == "bf16" else 4), "flops": 2 * M * D * C}
    B, T, H = case["B"], case.get("T", 1), case["H"]
    th, state = B * T * H, B * H * N * N * 4
    recurrence = 5 * N * N                                     # k v, w S + k v, r . S per token and head
    if kind == "layer":
        D = H * N
        C = D // 16
        M = B * T
        weights = (2 * INNER + 2 * RANK) * D * 2 + 5 * D * 4 + 2 * D * C
        front = 2 * M * D + 2 * B * D + 2 * M * RANK           # x and the row before it, y
        mix = th * N * 2 * 5 + 2 * state                       # r, k, v, u', o; state in and out
        norm = 8 * M + 2 * M * D                               # statistics, normalised rows
        return {"bytes": weights + front + mix + norm + 2 * M * C,
                "flops": 2 * M * D * (2 * INNER + 2 * RANK) + th * recurrence + 8 * M * D + 2 * M * D * C}
    item = 4 if kind == "prefill_f32" else 2
    out = 4 if kind == "prefill_f32" or case.get("out") == "f32" else 2
    streams = 5 if case.get("form") == "finch_c2" else 4
    carried = 2 if case.get("state", True) else 1
    return {"bytes": th * N * (streams * item + out) + carried * state + (0 if streams == 5 else H * N * 4),
            "flops": th * recurrence}


def tolerance(case):
    if case["kind"] == "prefill_f32":
        # fp32 throughout: 1.2e-7 to 2.5e-7 off 64 bits, sums in another order move it by as much
        return {"rel": 1e-6, "max": 1e-4}
    if case["kind"] == "key_compress" and case["out"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "layer":
        # five calls, each interface rounded to bf16 (1.7e-3 a rounding)
        return {"rel": 1e-2, "max": 0.2}
    # bf16 inputs; fp16 matrix-core operands (3e-4) and, for most outputs, one rounding to bf16 (1.7e-3)
    return {"rel": 7e-3, "max": 0.2}


# ----------------------------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------------------------
def _wkv64(r, k, v, x, u, uprime, state):
    """The recurrence in float64, 16 tokens at a time: decays between two tokens as exp of a difference of
    cumulated logarithms, which is never positive."""
    d = torch.float64
    B, T, H, _ = r.shape
    S = torch.zeros((B, H, N, N), dtype=d, device=r.device) if state is None else state.to(d)
    out = torch.empty((B, T, H, N), dtype=d, device=r.device)
    for t0 in range(0, T, 16):
        rc, kc, vc, xc = (a[:, t0:t0 + 16].to(d).transpose(1, 2).contiguous() for a in (r, k, v, x))     # [B,H,c,N]
        c = rc.shape[2]
        lw = -torch.exp(xc)
        if uprime is not None:
            kc = kc * -torch.expm1(lw)
        upto = torch.cumsum(lw, 2)                             # decays of tokens 0..t
        before = upto - lw                                     # decays of tokens 0..t-1
        causal = torch.ones((c, c), dtype=torch.bool, device=r.device).tril(-1)
        gap = (before[:, :, :, None] - upto[:, :, None]).masked_fill(~causal[None, None, :, :, None], -math.inf)
        scores = (rc[:, :, :, None] * kc[:, :, None] * torch.exp(gap)).sum(-1)
        o = torch.matmul(rc * torch.exp(before), S) + torch.matmul(scores, vc)
        if uprime is None:
            o = o + (rc * u.to(d)[None, :, None] * kc).sum(-1, keepdim=True) * vc
        out[:, t0:t0 + 16] = o.transpose(1, 2)
        last = upto[:, :, -1:]
        kt = (kc * torch.exp(last - upto)).transpose(2, 3).contiguous()
        S = torch.exp(last).transpose(2, 3) * S + torch.matmul(kt, vc)
    if uprime is not None:
        out += uprime.to(d)
    return out, S


def exact(case, seed):
    kind = case["kind"]
    d = torch.float64
    if kind == "key_compress":
        t = _key_inputs(case, seed)
        w = t["w_kd"].to(d)
        return torch.cat([torch.matmul(part.to(d), w) for part in t["x"].split(8192)])
    if kind != "layer":
        t = _time_mix(case, seed, torch.float32 if kind == "prefill_f32" else torch.bfloat16)
        return _wkv64(t["r"], t["k"], t["v"], t["x"], t.get("u"), t.get("uprime"), t["state_in"])
    # the layer: every call in 64 bits from what the call before it hands over, in the type that carries it
    t = _layer_inputs(case, seed)
    B, T, H = case["B"], case["T"], case["H"]
    D = H * N
    x = t["x"].to(d)
    step = torch.cat([t["x_prev"].to(d)[:, None], x[:, :-1]], 1) - x
    p = torch.tanh(torch.matmul(x + step * t["mu_x"].to(d), t["a_d"].to(d).t().contiguous()))
    z = x + step * (t["lambda_d"].to(d) + torch.matmul(p, t["b_d"].to(d).t().contiguous()))
    y = torch.tanh(torch.matmul(z, t["a_omega"].to(d).t().contiguous()))
    del x, step, p, z
    logits = t["lambda"].to(d) + torch.matmul(y.to(torch.bfloat16).to(d), t["b_omega"].to(d))
    o, state = _wkv64(t["r"], t["k"], t["v"], logits.view(B, T, H, N), None, t["uprime"], t["state_in"])
    rows = o.reshape(B, T, D)
    mean = rows.mean(-1, keepdim=True)
    rstd = 1 / torch.sqrt(((rows - mean) ** 2).mean(-1, keepdim=True) + 1e-5)
    normed = (rows.to(torch.bfloat16).to(d) - mean) * rstd * t["gamma"].to(d) + t["beta"].to(d)
    c = torch.matmul(normed.to(torch.bfloat16).to(d).reshape(B * T, D), t["w_kd"].to(d))
    return {"y": y, "o": o, "state_out": state, "mean_rstd": torch.cat([mean, rstd], -1), "normed": normed, "c": c}
