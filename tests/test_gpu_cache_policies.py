"""The chunked kernel's cache policies follow the bytes of a call: a batch on the far side of a line gives, sequence by sequence, the bits
of calls small enough for the first policy.  (The split entries with one segment: they never split by themselves.)"""
import pytest
import torch

import paper_2407_12077_amd as wkv

pytestmark = pytest.mark.gpu


# one unit a workgroup beyond 90 MiB; several units beyond 90 MiB and beyond a GiB
@pytest.mark.parametrize("c2", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,T,H", [(4, 1001, 64), (20, 300, 32), (40, 100, 32), (64, 800, 32)])
def test_bits_do_not_depend_on_the_size_of_the_batch(c2, dtype, B, T, H):
    g = torch.Generator(device="cuda").manual_seed(B * T)
    r, k, v, up = ((torch.randn((B, T, H, 64), generator=g, device="cuda") / 8).to(torch.bfloat16) for _ in range(4))
    x = (torch.rand((B, T, H, 64), generator=g, device="cuda") * 7 - 6).to(torch.bfloat16)
    extra = up if c2 else torch.randn((H, 64), generator=g, device="cuda") / 2
    state = torch.randn((B, H, 64, 64), generator=g, device="cuda") / 10
    entry = wkv.wkv6_finch_c2_prefill_bf16_split if c2 else wkv.wkv6_prefill_bf16_split
    out = torch.full((B, T, H, 64), float("nan"), dtype=dtype, device="cuda")
    s = torch.full_like(state, float("nan"))
    code = wkv.WKV6_DTYPE_F32 if dtype == torch.float32 else wkv.WKV6_DTYPE_BF16
    entry(B, T, H, 64, r, k, v, x, extra, state, out, s, code, 1, None, 0)
    one, s1 = torch.empty((1, T, H, 64), dtype=dtype, device="cuda"), torch.empty((1, H, 64, 64), device="cuda")
    for b in range(0, B, 7):
        sl = slice(b, b + 1)
        entry(1, T, H, 64, r[sl], k[sl], v[sl], x[sl], up[sl] if c2 else extra, state[sl], one, s1, code, 1, None, 0)
        torch.cuda.synchronize()
        assert torch.equal(one, out[sl]) and torch.equal(s1, s[sl]), b


@pytest.mark.parametrize("mode", ["moments", "lora", "lora_moments", "finch_lora"])
def test_bits_of_the_modes_inside_a_layer_do_not_depend_on_the_size_of_the_batch(mode):
    """140 MiB, several units a workgroup (a unit's logits are formed while the one before it is worked on), against calls of 28 MiB with
    one unit a workgroup.  128 units of 300 tokens are not split."""
    B, T, H, few = 20, 300, 32, 4
    g = torch.Generator(device="cuda").manual_seed(3)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    r, k, v, up = ((n(B, T, H, 64) / 8).to(torch.bfloat16) for _ in range(4))
    x = (torch.rand((B, T, H, 64), generator=g, device="cuda") * 7 - 6).to(torch.bfloat16)
    y, lam, b_omega = torch.tanh(n(B, T, 64)).to(torch.bfloat16), torch.rand((H * 64,), generator=g, device="cuda") * 6 - 5.5, (n(64, H * 64) / 5).to(torch.bfloat16)
    u, state = n(H, 64) / 2, n(B, H, 64, 64) / 10

    def call(sl):
        b = sl.stop - sl.start
        out = torch.full((b, T, H, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
        s, m = torch.full((b, H, 64, 64), float("nan"), device="cuda"), torch.full((b, H, T, 2), float("nan"), device="cuda")
        if mode == "moments":
            wkv.wkv6_finch_c2_prefill_bf16_moments(b, T, H, 64, r[sl], k[sl], v[sl], x[sl], up[sl], state[sl], out, m, s)
        elif mode == "finch_lora":
            wkv.wkv6_prefill_lora_bf16(b, T, H, 64, 64, r[sl], k[sl], v[sl], y[sl], lam, b_omega, u, state[sl], out, s)
        else:
            wkv.wkv6_finch_c2_prefill_lora_bf16(b, T, H, 64, 64, r[sl], k[sl], v[sl], y[sl], lam, b_omega, up[sl], state[sl], out,
                                                m if mode == "lora_moments" else None, s)
        torch.cuda.synchronize()
        return (out, s, m) if "moments" in mode else (out, s)

    whole = call(slice(0, B))
    for b in range(0, B, few):
        sl = slice(b, b + few)
        for got, part in zip(whole, call(sl)):
            assert torch.isfinite(part).all() and torch.equal(got[sl], part), b


@pytest.mark.parametrize("H,tokens,piece", [(12, 1400, 700), (12, 25000, 5000), (32, 17409, 4100), (4, 4097, 1026)])
def test_bits_of_normalised_rows_do_not_depend_on_the_number_of_tokens(H, tokens, piece):
    """Whole: rows written through (1400 and 4097 tokens) or streamed; in pieces the other way."""
    g = torch.Generator(device="cuda").manual_seed(tokens)
    o = torch.randn((tokens, H * 64), generator=g, device="cuda").to(torch.bfloat16)
    ms = torch.rand((tokens, 2), generator=g, device="cuda")
    gain, offset = (torch.randn((H * 64,), generator=g, device="cuda") for _ in range(2))
    whole, parts = torch.empty_like(o), torch.empty_like(o)
    wkv.wkv6_layernorm_apply_bf16(1, tokens, H, 64, o, ms, gain, offset, whole, wkv.WKV6_DTYPE_BF16)
    for t in range(0, tokens, piece):
        sl = slice(t, min(t + piece, tokens))
        wkv.wkv6_layernorm_apply_bf16(1, sl.stop - t, H, 64, o[sl], ms[sl], gain, offset, parts[sl], wkv.WKV6_DTYPE_BF16)
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)
    want = (o.double() - ms[:, :1]) * ms[:, 1:] * gain + offset      # fp32 arithmetic, one rounding to bf16
    assert ((whole.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all()
