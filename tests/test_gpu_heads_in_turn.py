"""Workgroups with several units whose head moves on from one unit to the next (large calls whose token rows are a multiple of
1 KiB): sequence by sequence the bits of calls with one unit a workgroup.  (The split entries with one segment: they never split by
themselves.)"""
import pytest
import torch

import launch_util as lu
import paper_2407_12077_amd as wkv


# several rounds, the last one short; units of two chunks, whose first three belong to two of them; workgroups of 8, 32, 240 and 192 of 256
# compute units' heads; a unit's heads past the last one
@pytest.mark.gpu
@pytest.mark.parametrize("c2", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,T,H", [(560, 65, 8), (90, 200, 24), (80, 161, 32), (58, 170, 40), (8, 300, 192), (95, 33, 64)])
def test_bits_of_units_with_the_heads_in_turn(c2, dtype, B, T, H):
    g = torch.Generator(device="cuda").manual_seed(B * T + H)
    r, k, v, up = ((torch.randn((B, T, H, 64), generator=g, device="cuda") / 8).to(torch.bfloat16) for _ in range(4))
    x = (torch.rand((B, T, H, 64), generator=g, device="cuda") * 7 - 6).to(torch.bfloat16)
    extra = up if c2 else torch.randn((H, 64), generator=g, device="cuda") / 2
    state = torch.randn((B, H, 64, 64), generator=g, device="cuda") / 10
    entry = wkv.wkv6_finch_c2_prefill_bf16_split if c2 else wkv.wkv6_prefill_bf16_split
    code = wkv.WKV6_DTYPE_F32 if dtype == torch.float32 else wkv.WKV6_DTYPE_BF16
    out = torch.full((B, T, H, 64), float("nan"), dtype=dtype, device="cuda")
    s = torch.full_like(state, float("nan"))
    entry(B, T, H, 64, r, k, v, x, extra, state, out, s, code, 1, None, 0)
    one, s1 = torch.empty((1, T, H, 64), dtype=dtype, device="cuda"), torch.empty((1, H, 64, 64), device="cuda")
    for b in sorted({*range(0, B, 7), B - 2, B - 1}):
        sl = slice(b, b + 1)
        entry(1, T, H, 64, r[sl], k[sl], v[sl], x[sl], up[sl] if c2 else extra, state[sl], one, s1, code, 1, None, 0)
        torch.cuda.synchronize()
        assert torch.equal(one, out[sl]) and torch.equal(s1, s[sl]), b


def _call(entry, B, T, H, shift):
    name, args = lu.time_mix(entry, B, T, H)
    args[10] += shift                                            # out
    return name, args


@pytest.mark.parametrize("entry,B,T,H,shift,turn", [
    ("wkv6_finch_c2_prefill_bf16", 256, 512, 32, 0, True), ("wkv6_finch_c2_prefill_bf16", 256, 512, 32, 1024, True),
    ("wkv6_finch_c2_prefill_bf16", 256, 512, 32, 128, False), ("wkv6_finch_c2_prefill_bf16", 16, 180, 32, 0, False),
    ("wkv6_finch_c2_prefill_bf16", 16, 270, 40, 0, False), ("wkv6_finch_c2_prefill_bf16", 16, 290, 40, 0, True),
    ("wkv6_finch_c2_prefill_bf16", 16, 800, 36, 0, False), ("wkv6_finch_c2_prefill_bf16", 8, 800, 32, 0, False), ("wkv6_finch_c2_prefill_bf16", 11, 800, 32, 0, False),
    ("wkv6_prefill_bf16", 16, 880, 32, 0, False), ("wkv6_prefill_bf16", 16, 930, 32, 0, True), ("wkv6_prefill_bf16", 256, 512, 32, 0, False),
    ("wkv6_prefill_bf16_f32out", 256, 512, 32, 128, True), ("wkv6_prefill_bf16", 3, 900, 192, 0, True), ("wkv6_prefill_bf16", 3, 900, 200, 0, False)])
def test_heads_in_turn_where_that_is_faster(tmp_path, entry, B, T, H, shift, turn):
    """Not where the streams start in different address classes, nor where the bonus of all heads does not fit the LDS."""
    fake = lu.build_fake(tmp_path)
    run = [e for e in lu.events(fake, [_call(entry, B, T, H, shift)])[0] if e.kind == "launch"][-1]
    assert run.kernel.split(", ")[2] == str(turn).lower(), run.kernel
    limits = {e.kernel: e.bytes for e in lu.events(fake, [_call(entry, B, T, H, shift)])[0] if e.kind == "attribute"}
    assert run.bytes <= limits[run.kernel] <= 160 * 1024


@pytest.mark.parametrize("entry,B,T,H,turn", [
    ("wkv6_finch_c2_prefill_bf16", 12, 900, 32, False), ("wkv6_finch_c2_prefill_bf16", 13, 2000, 32, False), ("wkv6_finch_c2_prefill_bf16", 14, 900, 32, True),
    ("wkv6_prefill_bf16", 13, 2000, 32, False), ("wkv6_prefill_bf16", 14, 2000, 32, True), ("wkv6_prefill_bf16", 10, 2000, 40, False),
    ("wkv6_prefill_bf16", 11, 2000, 40, True), ("wkv6_prefill_bf16_f32out", 11, 900, 32, False), ("wkv6_prefill_bf16_f32out", 12, 900, 32, True),
    ("wkv6_finch_c2_prefill_bf16_f32out", 12, 600, 32, True)])
def test_heads_in_turn_from_enough_rounds_on(tmp_path, entry, B, T, H, turn):
    """Finch-C2, 12 x 900 tokens x 32 heads, one and a half rounds of workgroups: 70.9 us, in turn 72.3."""
    [ev] = lu.events(lu.build_fake(tmp_path), [_call(entry, B, T, H, 0)])
    assert [e for e in ev if e.kind == "launch"][-1].kernel.split(", ")[2] == str(turn).lower()
