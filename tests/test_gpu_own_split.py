"""The token split that the prefill entry points make by themselves (few (batch, head) units, many tokens): the
segments' states pass through the segments' own rows of `out`.  Against the fp64 oracle at the stated bars, over the forms
that accept it, and against one another where they promise the same bits."""
import numpy as np
import pytest
import torch

import paper_2407_12077_amd as wkv
from oracle import decay_logits_numpy, finch_c2_oracle, wkv6_oracle
from paper_2407_12077_amd.workloads import CONFIGS, make_decay_lora_inputs, make_inputs, make_uprime, round_to_bf16, scaled

from gpu_util import BF16_OUT_ROUNDING, TOL_BF16, max_norm_err, to_dev
from split_shapes import SPLIT, WHOLE

pytestmark = pytest.mark.gpu

# both sides of the rule, with the plans that the CPU tests pin
SHAPES = list(SPLIT) + WHOLE


def inputs(B, T, H, state=True):
    cfg = scaled(CONFIGS[4 if state else 2], B=B, T=T, H=H)
    inp = make_inputs(cfg, seed=40 + T)
    inp["uprime"] = make_uprime(cfg, 40 + T)
    return cfg, inp


def run(entry, inp, out_dtype, in_place=False):
    B, T, H, N = inp["r"].shape
    r, k, v, x = (to_dev(inp[n], torch.bfloat16) for n in "rkvx")
    extra = to_dev(inp["uprime"], torch.bfloat16) if "finch_c2" in entry else to_dev(inp["u"], torch.float32)
    s_in = to_dev(inp["state_in"], torch.float32)
    s_out = s_in if in_place else torch.full((B, H, N, N), float("nan"), device="cuda")
    out = torch.full((B, T, H, N), float("nan"), dtype=out_dtype, device="cuda")
    getattr(wkv, entry)(B, T, H, N, r, k, v, x, extra, s_in, out, s_out)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), s_out.cpu().numpy()


@pytest.mark.parametrize("B,T,H", SHAPES)
def test_matches_oracle_and_output_types_agree(gpu_device, B, T, H):
    for state in (True, False):
        _, inp = inputs(B, T, H, state)
        refs = {"wkv6_prefill_bf16": wkv6_oracle(inp["r"], inp["k"], inp["v"], inp["x"], inp["u"], inp["state_in"]),
                "wkv6_finch_c2_prefill_bf16": finch_c2_oracle(inp["r"], inp["k"], inp["v"], inp["x"], inp["uprime"], inp["state_in"])}
        for entry, (o_ref, s_ref) in refs.items():
            o32, s32 = run(entry + "_f32out", inp, torch.float32)
            assert max_norm_err(o32, o_ref) <= TOL_BF16 and max_norm_err(s32, s_ref) <= TOL_BF16, entry
            o16, s16 = run(entry, inp, torch.bfloat16, in_place=state)
            assert np.array_equal(o16, round_to_bf16(o32)) and np.array_equal(s16, s32), entry


# the last three: a last segment of exactly the hand-over's tokens, and waves of the state pass with two or three (one or two)
# chunks each, whose loop carries the state, its decay and the next chunk's loads from one chunk to the next
@pytest.mark.parametrize("B,T,H", [(1, 1100, 4), (2, 1531, 12), (1, 898, 1), (1, 4200, 32), (2, 1300, 40)])
def test_fused_decay_path_and_moments(gpu_device, B, T, H):
    cfg, inp = inputs(B, T, H)
    lo = make_decay_lora_inputs(cfg, 5)
    logits = decay_logits_numpy(lo["y"], lo["lam"], lo["b_omega"], H, 64)
    r, k, v, up, y, bw = (to_dev(a, torch.bfloat16) for a in (inp["r"], inp["k"], inp["v"], inp["uprime"], lo["y"], lo["b_omega"]))
    u, lam, s_in = (to_dev(a, torch.float32) for a in (inp["u"], lo["lam"], inp["state_in"]))
    s_out = torch.empty((B, H, 64, 64), device="cuda")
    out = torch.empty((B, T, H, 64), dtype=torch.bfloat16, device="cuda")
    mom = torch.full((B, H, T, 2), float("nan"), device="cuda")
    bar = TOL_BF16 + BF16_OUT_ROUNDING
    wkv.wkv6_finch_c2_prefill_lora_bf16(B, T, H, 64, 64, r, k, v, y, lam, bw, up, s_in, out, mom, s_out)
    o_ref, s_ref = finch_c2_oracle(inp["r"], inp["k"], inp["v"], logits, inp["uprime"], inp["state_in"])
    assert max_norm_err(out.float().cpu().numpy(), o_ref) <= bar and max_norm_err(s_out.cpu().numpy(), s_ref) <= TOL_BF16
    # a sum of 64 values, each within the output's bar
    sums = o_ref.sum(-1).transpose(0, 2, 1)
    assert np.abs(mom[..., 0].cpu().numpy() - sums).max() <= 64 * TOL_BF16 * np.abs(o_ref).max()
    plain = out.clone()
    wkv.wkv6_finch_c2_prefill_lora_bf16(B, T, H, 64, 64, r, k, v, y, lam, bw, up, s_in, out, None, s_out)
    assert torch.equal(out, plain)
    wkv.wkv6_prefill_lora_bf16(B, T, H, 64, 64, r, k, v, y, lam, bw, u, s_in, out, s_out)
    o_ref, s_ref = wkv6_oracle(inp["r"], inp["k"], inp["v"], logits, inp["u"], inp["state_in"])
    assert max_norm_err(out.float().cpu().numpy(), o_ref) <= bar and max_norm_err(s_out.cpu().numpy(), s_ref) <= TOL_BF16
    # zero activations: the plain entry's bits
    y.zero_()
    lam = lam.bfloat16().float()
    x = lam.bfloat16().view(1, 1, H, 64).expand(B, T, H, 64).contiguous()
    wkv.wkv6_prefill_lora_bf16(B, T, H, 64, 64, r, k, v, y, lam, bw, u, s_in, out, s_out)
    out2, s2 = torch.empty_like(out), torch.empty_like(s_out)
    wkv.wkv6_prefill_bf16(B, T, H, 64, r, k, v, x, u, s_in, out2, s2)
    assert torch.equal(out, out2) and torch.equal(s_out, s2)


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_window_writes_only_its_own_rows(gpu_device, out_dtype):
    """A window of a larger buffer: the hand-over stays inside the window's rows of its own heads."""
    B, T_full, t0, T, H = 2, 1500, 130, 1201, 6
    _, inp = inputs(B, T_full, H)
    r, k, v, x = (to_dev(inp[n], torch.bfloat16) for n in "rkvx")
    u, s_in = to_dev(inp["u"], torch.float32), to_dev(inp["state_in"], torch.float32)
    out = torch.full((B, T_full, H, 64), 7.0, dtype=out_dtype, device="cuda")
    s_out = torch.empty((B, H, 64, 64), device="cuda")
    code = wkv.WKV6_DTYPE_BF16 if out_dtype == torch.bfloat16 else wkv.WKV6_DTYPE_F32
    win = [t[:, t0:] for t in (r, k, v, x, out)]
    wkv.wkv6_prefill_bf16_strided(B, T, H, 64, *win[:4], u, s_in, win[4], s_out, T_full * H * 64, code)
    torch.cuda.synchronize()
    assert bool((out[:, :t0] == 7.0).all()) and bool((out[:, t0 + T:] == 7.0).all())
    sl = {n: np.ascontiguousarray(inp[n][:, t0:t0 + T]) for n in "rkvx"}
    o_ref, s_ref = wkv6_oracle(sl["r"], sl["k"], sl["v"], sl["x"], inp["u"], inp["state_in"])
    bar = TOL_BF16 + (BF16_OUT_ROUNDING if out_dtype == torch.bfloat16 else 0.0)
    assert max_norm_err(out[:, t0:t0 + T].float().cpu().numpy(), o_ref) <= bar
    assert max_norm_err(s_out.cpu().numpy(), s_ref) <= TOL_BF16


@pytest.mark.parametrize("xval", [-np.inf, np.inf, 20.0, -30.0])
def test_extreme_decays(gpu_device, xval):
    _, inp = inputs(1, 1000, 4)
    inp["x"][:, :, :, ::2] = xval
    o_ref, s_ref = wkv6_oracle(inp["r"], inp["k"], inp["v"], inp["x"], inp["u"], inp["state_in"])
    o, s = run("wkv6_prefill_bf16_f32out", inp, torch.float32)
    assert max_norm_err(o, o_ref) <= TOL_BF16 and max_norm_err(s, s_ref) <= TOL_BF16


def test_replays_in_a_graph(gpu_device):
    """Captured, replayed several times with eager work between: every replay is the eager result."""
    _, inp = inputs(1, 1300, 8)
    r, k, v, x = (to_dev(inp[n], torch.bfloat16) for n in "rkvx")
    u, s_in = to_dev(inp["u"], torch.float32), to_dev(inp["state_in"], torch.float32)
    out, s_out = torch.empty_like(r), torch.empty_like(s_in)
    call = lambda: wkv.wkv6_prefill_bf16(1, 1300, 8, 64, r, k, v, x, u, s_in, out, s_out)  # noqa: E731
    call()
    torch.cuda.synchronize()
    want, s_want = out.clone(), s_out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(4):
        out.fill_(float("nan"))
        s_out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(s_out, s_want)


def test_moments_of_a_split_prefill_are_those_of_its_output(gpu_device):
    """The LayerNorm partials carry the sequence's token index, not the segment's: the plain entry's bits for out and state,
    and sums and squared deviations of the head's read-outs (fp32 out of the same split, so 64 fp32 sums: 1e-5)."""
    B, T, H = 2, 1531, 12
    _, inp = inputs(B, T, H)
    r, k, v, x, up = (to_dev(inp[n], torch.bfloat16) for n in ("r", "k", "v", "x", "uprime"))
    s_in = to_dev(inp["state_in"], torch.float32)
    out, s_out, mom = torch.empty_like(r), torch.empty_like(s_in), torch.full((B, H, T, 2), float("nan"), device="cuda")
    wkv.wkv6_finch_c2_prefill_bf16_moments(B, T, H, 64, r, k, v, x, up, s_in, out, mom, s_out)
    out0, s0 = torch.empty_like(r), torch.empty_like(s_in)
    wkv.wkv6_finch_c2_prefill_bf16(B, T, H, 64, r, k, v, x, up, s_in, out0, s0)
    assert torch.equal(out, out0) and torch.equal(s_out, s0)
    o32 = torch.empty((B, T, H, 64), device="cuda")
    wkv.wkv6_finch_c2_prefill_bf16_f32out(B, T, H, 64, r, k, v, x, up, s_in, o32, s0)
    o = o32.double().permute(0, 2, 1, 3)
    mean = o.mean(-1, keepdim=True)
    assert (mom[..., 0].double() - o.sum(-1)).abs().max() <= 1e-5 * o.abs().sum(-1).max()
    m2 = ((o - mean) ** 2).sum(-1)
    assert ((mom[..., 1].double() - m2).abs() <= 1e-5 * m2.max()).all()


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
def test_segments_beyond_four_gib(gpu_device, out_dtype):
    """85 heads and so many tokens that the third segment starts beyond 4 GiB in every tensor (fp32 out: beyond 8 GiB), which is
    where the hand-over then lies: two heads against the oracle over the last segment and some tokens in front of it, and
    the final state."""
    H, T = 85, 620_000
    seg_len = (T + 3 * 32 - 1) // (3 * 32) * 32
    assert 2 * seg_len * H * 64 * 2 > 1 << 32
    g = torch.Generator(device="cuda").manual_seed(77)
    make = lambda scale: torch.randn((1, T, H, 64), generator=g, device="cuda", dtype=torch.bfloat16).mul_(scale)  # noqa: E731
    r, k, v = make(0.125), make(0.125), make(0.125)
    x = make(1.0).sub_(3.0)
    u = torch.randn((H, 64), generator=g, device="cuda") * 0.5
    out = torch.full((1, T, H, 64), float("nan"), dtype=out_dtype, device="cuda")
    s_out = torch.full((1, H, 64, 64), float("nan"), device="cuda")
    entry = wkv.wkv6_prefill_bf16 if out_dtype == torch.bfloat16 else wkv.wkv6_prefill_bf16_f32out
    entry(1, T, H, 64, r, k, v, x, u, None, out, s_out)
    torch.cuda.synchronize()
    first = 2 * seg_len
    heads = [0, H - 1]
    # the decays forget (0.08 a token in the exponent on average): 20 000 tokens in front hold the segment's entering state
    lead = 20_000
    host = {n: np.ascontiguousarray(t[:, first - lead:, heads].float().cpu().numpy()) for n, t in zip("rkvx", (r, k, v, x))}
    o_ref, s_ref = wkv6_oracle(host["r"], host["k"], host["v"], host["x"], np.ascontiguousarray(u[heads].cpu().numpy()), None)
    bar = TOL_BF16 + (BF16_OUT_ROUNDING if out_dtype == torch.bfloat16 else 0.0)
    assert max_norm_err(out[:, first:, heads].float().cpu().numpy(), o_ref[:, lead:]) <= bar
    assert max_norm_err(s_out[:, heads].cpu().numpy(), s_ref) <= TOL_BF16
    assert bool(torch.isfinite(out[:, :first:997].float()).all())
    del r, k, v, x, out
    torch.cuda.empty_cache()
