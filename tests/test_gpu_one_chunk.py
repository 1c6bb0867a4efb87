"""Sequences of at most 32 tokens, one chunk by four waves per unit: every entry point that takes them against the fp64 oracle at the
edges of the chunk, and bit for bit against the same tokens at the head of a longer sequence, which the kernel for several chunks takes."""
import numpy as np
import pytest
import torch

import paper_2407_12077_amd as wkv
from gpu_util import BF16_OUT_ROUNDING, TOL_BF16, max_norm_err
from oracle import finch_c2_oracle, wkv6_oracle

pytestmark = pytest.mark.gpu
LENGTHS = [1, 2, 3, 4, 5, 8, 15, 16, 17, 24, 31, 32]


def tensors(B, T, H, seed, state=True):
    g = torch.Generator().manual_seed(seed)
    bf = lambda *s: (torch.randn(s, generator=g) / 8).to(torch.bfloat16).cuda()  # noqa: E731
    t = {n: bf(B, T, H, 64) for n in ("r", "k", "v", "uprime")}
    t["x"] = (torch.rand((B, T, H, 64), generator=g) * 7 - 6).to(torch.bfloat16).cuda()
    t["u"] = (torch.randn((H, 64), generator=g) / 2).cuda()
    t["state_in"] = (torch.randn((B, H, 64, 64), generator=g) / 10).cuda() if state else None
    t["y"] = torch.tanh(torch.randn((B, T, 64), generator=g)).to(torch.bfloat16).cuda()
    t["lambda"] = (torch.rand((H * 64,), generator=g) * 6 - 5.5).cuda()
    t["b_omega"] = (torch.randn((64, H * 64), generator=g) / 5).to(torch.bfloat16).cuda()
    return t


def call(entry, t, B, T, H, out_dtype, moments=None, state_out=True):
    out = torch.full((B, T, H, 64), float("nan"), dtype=out_dtype, device="cuda")
    s = torch.full((B, H, 64, 64), float("nan"), device="cuda") if state_out else None
    rkv = t["r"], t["k"], t["v"]
    if "finch_c2_prefill_lora" in entry:
        getattr(wkv, entry)(B, T, H, 64, 64, *rkv, t["y"], t["lambda"], t["b_omega"], t["uprime"], t["state_in"], out, moments, s)
    elif "prefill_lora" in entry:
        getattr(wkv, entry)(B, T, H, 64, 64, *rkv, t["y"], t["lambda"], t["b_omega"], t["u"], t["state_in"], out, s)
    elif "moments" in entry:
        getattr(wkv, entry)(B, T, H, 64, *rkv, t["x"], t["uprime"], t["state_in"], out, moments, s)
    else:
        getattr(wkv, entry)(B, T, H, 64, *rkv, t["x"], t["uprime"] if "c2" in entry else t["u"], t["state_in"], out, s)
    torch.cuda.synchronize()
    return out, s


def host(a):
    return None if a is None else a.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("entry", ["wkv6_prefill_bf16", "wkv6_prefill_bf16_f32out", "wkv6_finch_c2_prefill_bf16", "wkv6_finch_c2_prefill_bf16_f32out"])
@pytest.mark.parametrize("T", LENGTHS)
@pytest.mark.parametrize("state", [True, False])
def test_edges_of_the_chunk(entry, T, state):
    B, H = 3, 5
    t = tensors(B, T, H, T, state)
    c2, f32 = "c2" in entry, "f32out" in entry
    out, s = call(entry, t, B, T, H, torch.float32 if f32 else torch.bfloat16)
    args = [host(t[n]) for n in ("r", "k", "v", "x")]
    o_ref, s_ref = finch_c2_oracle(*args, host(t["uprime"]), host(t["state_in"])) if c2 else wkv6_oracle(*args, host(t["u"]), host(t["state_in"]))
    assert max_norm_err(host(out), o_ref) <= TOL_BF16 + (0 if f32 else BF16_OUT_ROUNDING)
    assert max_norm_err(host(s), s_ref) <= TOL_BF16


ENTRIES = ["wkv6_prefill_bf16", "wkv6_prefill_bf16_f32out", "wkv6_finch_c2_prefill_bf16", "wkv6_finch_c2_prefill_bf16_f32out",
           "wkv6_finch_c2_prefill_bf16_moments", "wkv6_finch_c2_prefill_lora_bf16", "wkv6_prefill_lora_bf16"]


# (up to 2 to 4 tokens of a fused call are token by token); 2048 and 8192 units lie on both sides of the rows' cache policy
@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("B,T,H", [(1, 5, 1), (2, 7, 4), (3, 17, 8), (1, 31, 12), (2, 32, 3), (64, 20, 32), (256, 9, 32)])
def test_bits_are_those_of_the_head_of_a_longer_sequence(entry, B, T, H):
    compare_with_head_of_longer(entry, tensors(B, 33 + T % 3, H, 7 * T + H), B, T, H)


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("B,T,H", [(2, 7, 4), (3, 17, 8), (2, 32, 3)])
def test_bits_with_decays_of_nought_and_one_and_operands_beyond_fp16(entry, B, T, H):
    """Logits at both ends of their range (w = 0 and w = 1 exactly) and keys and values that are clamped to +-65504."""
    t = tensors(B, 33 + T % 3, H, T)
    g = torch.Generator().manual_seed(T)
    kind = torch.randint(0, 6, t["x"].shape, generator=g).cuda()
    big = torch.randint(0, 8, t["k"].shape, generator=g).cuda()
    column = torch.arange(H * 64, device="cuda") % 5
    for i, value in enumerate((float("inf"), float("-inf"), 10., -20.)):
        t["x"][kind == i] = value
        t["lambda"][column == i] = value
    for n, lo in (("k", 0), ("v", 2)):
        t[n][big == lo], t[n][big == lo + 1] = 1e5, -1e5
    o = compare_with_head_of_longer(entry, t, B, T, H)
    assert torch.isfinite(o).all() and o.float().abs().max() > 65504


def compare_with_head_of_longer(entry, t, B, T, H):
    longer = t["k"].shape[1]
    # the head of the longer sequence; its tail brings a state of its own, so the states are compared through tokens that change nothing
    for n in ("k", "v"):
        t[n][:, T:] = 0
    t["x"][:, T:] = float("-inf")
    short = {n: (a[:, :T].contiguous() if n in ("r", "k", "v", "x", "uprime", "y") else a) for n, a in t.items()}
    dtype = torch.float32 if "f32out" in entry else torch.bfloat16
    c2 = "moments" in entry or "c2_prefill_lora" in entry
    m_long, m_short = (torch.full((B, H, n, 2), float("nan"), device="cuda") if c2 else None for n in (longer, T))
    o_long, s_long = call(entry, t, B, longer, H, dtype, m_long)
    o_short, s_short = call(entry, short, B, T, H, dtype, m_short)
    assert torch.equal(o_long[:, :T], o_short)
    if c2:
        assert torch.equal(m_long[:, :, :T], m_short)
    if "lora" not in entry:                                   # (fused logits: the tail's decays are not 1)
        assert torch.equal(s_long, s_short)
    return o_short


def test_without_a_state_out_and_in_place():
    t = tensors(2, 20, 4, 5)
    o1, s1 = call("wkv6_finch_c2_append_bf16", t, 2, 20, 4, torch.bfloat16)
    o2, _ = call("wkv6_finch_c2_append_bf16", t, 2, 20, 4, torch.bfloat16, state_out=False)
    o3 = torch.empty_like(o1)
    state = t["state_in"].clone()
    wkv.wkv6_finch_c2_append_bf16(2, 20, 4, 64, t["r"], t["k"], t["v"], t["x"], t["uprime"], state, o3, state)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(o1, o3) and torch.equal(s1, state)


def test_strided_batches_of_one_chunk():
    B, T, H = 3, 19, 4
    t = tensors(B, 40, H, 6)                                  # batches lie 40 tokens apart, 19 of them are read
    short = {n: (a[:, :T].contiguous() if n in ("r", "k", "v", "x", "uprime") else a) for n, a in t.items()}
    want, s_want = call("wkv6_finch_c2_prefill_bf16", short, B, T, H, torch.bfloat16)
    out = torch.zeros((B, 40, H, 64), dtype=torch.bfloat16, device="cuda")
    s = torch.empty((B, H, 64, 64), device="cuda")
    wkv.wkv6_finch_c2_prefill_bf16_strided(B, T, H, 64, t["r"], t["k"], t["v"], t["x"], t["uprime"], t["state_in"], out, s, 40 * H * 64, wkv.WKV6_DTYPE_BF16)
    torch.cuda.synchronize()
    assert torch.equal(out[:, :T], want) and torch.equal(s, s_want) and not out[:, T:].any()


def test_more_units_than_a_launch_has_workgroups_for():
    """2^24 (batch, head) units of one token: the kernel for longer sequences, whose workgroups take several units, with the same bits."""
    B, T, H = 524288, 1, 32
    g = torch.Generator(device="cuda").manual_seed(1)
    r, k, v = (torch.randn((B, T, H, 64), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    x, u = r, torch.randn((H, 64), generator=g, device="cuda")
    out = torch.full((B, T, H, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    wkv.wkv6_prefill_bf16(B, T, H, 64, r, k, v, x, u, None, out, None)
    for b in (0, 131072, B - 3):                              # element offsets up to 2^30, bytes up to 2^31
        sl = slice(b, b + 3)
        few = torch.empty((3, T, H, 64), dtype=torch.bfloat16, device="cuda")
        wkv.wkv6_prefill_bf16(3, T, H, 64, r[sl], k[sl], v[sl], x[sl], u, None, few, None)
        torch.cuda.synchronize()
        assert torch.equal(few, out[sl]), b
