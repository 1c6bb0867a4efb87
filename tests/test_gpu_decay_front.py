"""GPU parity of the operators in front of the decay path (Finch-C2 Time Mixing: lerp, lora, ddlerp,
d_t = lora_omega(ddlerp_d(x_t, x_{t-1}))): wkv6_decay_lora_input_bf16 against the fp64 oracle on the
same seeded inputs, and chained into the fused prefill against the chained oracles.

Tolerance: y = tanh(.) has magnitude below 1, so the stated 2e-3 (max |gpu - oracle| / max |oracle|) is
close to an absolute bound; gated on the fp32 output; the bf16 output must be the fp32 output
rounded once."""
import numpy as np
import pytest
import torch

import paper_2407_12077_amd as wkv
from oracle import decay_logits_numpy, decay_lora_input_numpy, finch_c2_oracle
from paper_2407_12077_amd.workloads import (CONFIGS, make_decay_front_inputs, make_inputs, make_uprime, round_to_bf16,
                                            scaled)

import front_shapes
from gpu_util import BF16_OUT_ROUNDING, TOL_BF16, error_report, fmt_report, max_norm_err, to_dev

pytestmark = pytest.mark.gpu


def run_front(fi, out_dtype=torch.float32, with_prev=True):
    B, T, D = fi["x"].shape
    x = to_dev(fi["x"], torch.bfloat16)
    xp = to_dev(fi["x_prev"], torch.bfloat16) if with_prev else None
    mu, lam = to_dev(fi["mu_x"], torch.float32), to_dev(fi["lam_d"], torch.float32)
    # the library takes the factors with the contraction index contiguous: A_d and A_omega column by column,
    # B_d column by column
    a_d = to_dev(np.ascontiguousarray(fi["A_d"].T), torch.bfloat16)
    b_d = to_dev(np.ascontiguousarray(fi["B_d"].T), torch.bfloat16)
    a_w = to_dev(np.ascontiguousarray(fi["A_omega"].T), torch.bfloat16)
    y = torch.full((B, T, 64), float("nan"), dtype=out_dtype, device="cuda")
    code = wkv.WKV6_DTYPE_F32 if out_dtype == torch.float32 else wkv.WKV6_DTYPE_BF16
    wkv.wkv6_decay_lora_input_bf16(B, T, D, 32, 64, x, xp, mu, lam, a_d, b_d, a_w, y, code)
    torch.cuda.synchronize()
    return y


def oracle_front(fi, with_prev=True):
    return decay_lora_input_numpy(fi["x"], fi["x_prev"] if with_prev else None, fi["mu_x"], fi["lam_d"], fi["A_d"],
                                  fi["B_d"], fi["A_omega"])


@pytest.mark.parametrize("B,T,H", [(1, 1, 2), (1, 63, 2), (2, 64, 2), (3, 65, 4), (2, 200, 12), (5, 37, 32), (1, 1000, 16)])
@pytest.mark.parametrize("with_prev", [True, False])
def test_matches_oracle(gpu_device, B, T, H, with_prev):
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=900 + T)
    ref = oracle_front(fi, with_prev)
    y32 = run_front(fi, torch.float32, with_prev).cpu().numpy()
    err = max_norm_err(y32, ref)
    print(f"decay front B={B} T={T} D={H * 64} prev={with_prev}: err={err:.3e} (|y|max {np.abs(ref).max():.3f})", flush=True)
    assert err <= TOL_BF16
    y16 = run_front(fi, torch.bfloat16, with_prev).float().cpu().numpy()
    assert np.array_equal(y16, round_to_bf16(y32))


# tiles of 16, 32 and 64 rows over whole and parts of sequences, one block of channels a wave or fewer (two with 10 and 12 heads), a last tile of one row
@pytest.mark.parametrize("B,T,H", [(17, 1, 6), (9, 2, 10), (33, 15, 2), (33, 16, 4), (31, 17, 12), (1, 33, 2), (131, 33, 4), (127, 65, 4), (2, 4097, 4)])
@pytest.mark.parametrize("with_prev", [True, False])
def test_rows_of_a_tile_and_their_predecessors(gpu_device, B, T, H, with_prev):
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=500 + B)
    y32 = run_front(fi, torch.float32, with_prev).cpu().numpy()
    assert max_norm_err(y32, oracle_front(fi, with_prev)) <= TOL_BF16
    assert np.array_equal(run_front(fi, torch.bfloat16, with_prev).float().cpu().numpy(), round_to_bf16(y32))


def test_special_weights(gpu_device):
    """B_d = 0 and lambda_d = 1: z is the previous token, so y_t = tanh(x_{t-1} A_omega); lambda_d = 0: y_t =
    tanh(x_t A_omega), whatever mu_x and A_d are."""
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=2, T=70, H=4), seed=77)
    fi["B_d"] = np.zeros_like(fi["B_d"])
    x = fi["x"].astype(np.float64)
    for lam, src in ((1.0, np.concatenate([fi["x_prev"][:, None].astype(np.float64), x[:, :-1]], axis=1)), (0.0, x)):
        fi["lam_d"] = np.full_like(fi["lam_d"], lam)
        want = np.tanh(src @ fi["A_omega"].astype(np.float64))
        got = run_front(fi).cpu().numpy()
        assert max_norm_err(got, want) <= 1e-3
        assert max_norm_err(got, oracle_front(fi)) <= 1e-3


def test_validation(gpu_device):
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=1, T=8, H=2), seed=3)
    t = lambda a, dt=torch.bfloat16: to_dev(a, dt)
    x, mu, lam = t(fi["x"]), t(fi["mu_x"], torch.float32), t(fi["lam_d"], torch.float32)
    a_d, b_d, a_w = t(fi["A_d"].T.copy()), t(fi["B_d"].T.copy()), t(fi["A_omega"].T.copy())
    y = torch.zeros((1, 8, 64), dtype=torch.bfloat16, device="cuda")
    ok = (x, None, mu, lam, a_d, b_d, a_w, y, wkv.WKV6_DTYPE_BF16)
    wkv.wkv6_decay_lora_input_bf16(1, 8, 128, 32, 64, *ok)
    wkv.wkv6_decay_lora_input_bf16(0, 8, 128, 32, 64, None, None, None, None, None, None, None, None, 0)
    for args, status in [((1, 8, 128, 16, 64) + ok, 3), ((1, 8, 128, 32, 32) + ok, 3), ((1, 8, 100, 32, 64) + ok, 3),
                         ((1, -1, 128, 32, 64) + ok, 2), ((1, 8, 128, 32, 64, None) + ok[1:], 1),
                         ((1, 8, 128, 32, 64) + ok[:8] + (9,), 3)]:
        with pytest.raises(wkv.Wkv6Error) as e:
            wkv.wkv6_decay_lora_input_bf16(*args)
        assert e.value.status == status


@pytest.mark.parametrize("B,T,H", [(2, 333, 4), (1, 1500, 8)])
def test_chained_into_the_fused_prefill(gpu_device, B, T, H):
    """From the layer input to the output of the time mix with nothing of the decay path in HBM but y:
    wkv6_decay_lora_input_bf16 -> wkv6_finch_c2_prefill_lora_bf16, against decay_lora_input_numpy ->
    decay_logits_numpy -> finch_c2_oracle.  The GPU chain rounds y to bf16 between the two calls (it is
    the interface tensor); the oracle chain is given that same rounding so that the comparison
    isolates the kernels (the logits are then exact functions of the same y on both sides)."""
    cfg = scaled(CONFIGS[2], B=B, T=T, H=H)
    N, D = 64, H * 64
    fi = make_decay_front_inputs(cfg, seed=41)
    inp = make_inputs(cfg, seed=42)
    up = make_uprime(cfg, seed=42)
    rng = np.random.default_rng(43)
    lam_w = rng.uniform(-5.5, 0.5, D).astype(np.float32)
    b_w = round_to_bf16((rng.standard_normal((64, D)) * 0.2).astype(np.float32))
    # GPU chain
    y_gpu = run_front(fi, torch.bfloat16)
    r, k, v, upd = (to_dev(a, torch.bfloat16) for a in (inp["r"], inp["k"], inp["v"], up))
    out = torch.full((B, T, H, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    s_out = torch.full((B, H, N, N), float("nan"), dtype=torch.float32, device="cuda")
    wkv.wkv6_finch_c2_prefill_lora_bf16(B, T, H, N, 64, r, k, v, y_gpu, to_dev(lam_w, torch.float32),
                                        to_dev(b_w, torch.bfloat16), upd, None, out, None, s_out)
    torch.cuda.synchronize()
    # oracle chain
    y_ref = oracle_front(fi)
    assert max_norm_err(y_gpu.float().cpu().numpy(), y_ref) <= TOL_BF16 + BF16_OUT_ROUNDING
    d = decay_logits_numpy(round_to_bf16(y_ref.astype(np.float32)), lam_w, b_w, H, N)
    o_ref, s_ref = finch_c2_oracle(inp["r"], inp["k"], inp["v"], d.astype(np.float32), up, None)
    # the GPU's y may differ from the oracle's by one bf16 step in a few entries, which moves a logit by
    # up to 2^-9 * |B_omega| and a decay by a comparable relative amount: allow twice the usual bar
    rep_o = error_report(out.float().cpu().numpy(), o_ref, "out")
    rep_s = error_report(s_out.cpu().numpy(), s_ref, "state")
    print(f"chain B={B} T={T} H={H}: out {fmt_report(rep_o)} | state {fmt_report(rep_s)}", flush=True)
    assert rep_o["global"] <= 2 * TOL_BF16 + BF16_OUT_ROUNDING and rep_s["global"] <= 2 * TOL_BF16


def test_full_size_every_token(gpu_device):
    """Config 2's tokens at full width: every token against the oracle."""
    cfg = CONFIGS[2]
    fi = make_decay_front_inputs(cfg)
    print("decay front config 2: oracle on every token ...", flush=True)
    ref = oracle_front(fi)
    y32 = run_front(fi, torch.float32).cpu().numpy()
    rows = np.abs(y32 - ref).max(axis=2)
    print(f"decay front config 2: global={max_norm_err(y32, ref):.3e} worst token={rows.max():.3e} "
          f"rel_l2={np.linalg.norm(y32 - ref) / np.linalg.norm(ref):.3e}", flush=True)
    assert max_norm_err(y32, ref) <= TOL_BF16
    y16 = run_front(fi, torch.bfloat16).float().cpu().numpy()
    assert np.array_equal(y16, round_to_bf16(y32))


def test_input_beyond_four_gib(gpu_device):
    """x of 4.83 GB (one sequence of 1 179 648 tokens of width 2048, drawn on the device from a seed): byte
    offsets into x pass 2^32.  Windows of tokens at the start, in the middle and at the end are compared with
    the oracle, each window's predecessor row given to the oracle as its x_prev."""
    B, T, D = 1, 9216 * 128, 2048
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=1, T=4, H=D // 64), seed=4321)      # weights and vectors
    gen = torch.Generator(device="cuda").manual_seed(98)
    x = torch.empty((B, T, D), dtype=torch.bfloat16, device="cuda")
    for t0 in range(0, T, 65536):
        x[:, t0:t0 + 65536] = torch.randn((B, 65536, D), generator=gen, device="cuda").to(torch.bfloat16)
    assert x.numel() * 2 > (1 << 32)
    xp = to_dev(fi["x_prev"], torch.bfloat16)
    mu, lam = to_dev(fi["mu_x"], torch.float32), to_dev(fi["lam_d"], torch.float32)
    a_d = to_dev(np.ascontiguousarray(fi["A_d"].T), torch.bfloat16)
    b_d = to_dev(np.ascontiguousarray(fi["B_d"].T), torch.bfloat16)
    a_w = to_dev(np.ascontiguousarray(fi["A_omega"].T), torch.bfloat16)
    y = torch.full((B, T, 64), float("nan"), dtype=torch.float32, device="cuda")
    wkv.wkv6_decay_lora_input_bf16(B, T, D, 32, 64, x, xp, mu, lam, a_d, b_d, a_w, y, wkv.WKV6_DTYPE_F32)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(y).all())
    for t0 in (0, (T // 2 // 128) * 128 + 100, T - 200):
        rows = x[:, t0:t0 + 200].float().cpu().numpy()
        prev = fi["x_prev"] if t0 == 0 else x[:, t0 - 1].float().cpu().numpy()
        ref = decay_lora_input_numpy(rows, prev, fi["mu_x"], fi["lam_d"], fi["A_d"], fi["B_d"], fi["A_omega"])
        err = max_norm_err(y[:, t0:t0 + 200].cpu().numpy(), ref)
        print(f"tokens {t0}..{t0 + 199}: err={err:.3e}", flush=True)
        assert err <= TOL_BF16
    del x, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("B,T,H", [(24, 1, 32), (17, 1, 2), (40, 2, 6), (9, 15, 4), (9, 16, 12), (9, 17, 2), (130, 31, 2),
                                   (131, 33, 2), (4, 1100, 2), (70, 60, 2), (256, 32, 2), (2, 4097, 2), (3, 5461, 2), (128, 127, 2),
                                   (1, 16385, 2)])
def test_split_contraction_tiles(gpu_device, B, T, H):
    """Every tile of the wave-split form (16, 32 and 64 rows) and the change to the 128-token form, with sequence starts at
    every place of a tile (T below, at and above the tile's rows), ragged last tiles, widths that leave waves without a
    block, and both kinds of first token.  The bar is the one of the 128-token form: fp16 operands, 2e-3 of the
    largest |y|."""
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=1300 + T)
    for with_prev in (True, False):
        y32 = run_front(fi, torch.float32, with_prev).cpu().numpy()
        assert max_norm_err(y32, oracle_front(fi, with_prev)) <= TOL_BF16
        y16 = run_front(fi, torch.bfloat16, with_prev).float().cpu().numpy()
        assert np.array_equal(y16, round_to_bf16(y32))


@pytest.mark.parametrize("B,T,H", [(17, 1, 4), (300, 1, 2), (600, 3, 2), (9, 17, 4), (130, 31, 4), (131, 33, 4), (4, 1100, 4), (70, 60, 4),
                                   (256, 32, 4), (2, 4097, 4), (3, 5461, 4), (128, 127, 4), (1, 16385, 4)])
def test_split_contraction_tiles_at_the_widths_that_take_them(gpu_device, B, T, H):
    """The same places of a tile as above at D = 256, where 16-, 32- and 64-row tiles are taken (at D = 128
    tiles of 128 tokens are the faster ones where 64 rows would fit).  Bar and rounding as above."""
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=1700 + T)
    for with_prev in (True, False):
        y32 = run_front(fi, torch.float32, with_prev).cpu().numpy()
        assert max_norm_err(y32, oracle_front(fi, with_prev)) <= TOL_BF16
        y16 = run_front(fi, torch.bfloat16, with_prev).float().cpu().numpy()
        assert np.array_equal(y16, round_to_bf16(y32))


# the outputs of a tile over four, two and one workgroups: both sides of each line, ragged last tiles, sequences that start in a tile
@pytest.mark.parametrize("B,T,H", [(1, 1024, 4), (1023, 1, 4), (1, 1025, 4), (205, 5, 4), (4, 512, 4), (2041, 1, 4), (1, 2049, 4)])
def test_outputs_of_a_tile_over_several_workgroups(gpu_device, B, T, H):
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=70 + B + T)
    y32 = run_front(fi, torch.float32).cpu().numpy()
    assert max_norm_err(y32, oracle_front(fi)) <= TOL_BF16
    assert np.array_equal(run_front(fi, torch.bfloat16).float().cpu().numpy(), round_to_bf16(y32))


@pytest.mark.parametrize("B,T,H", [s for shapes in front_shapes.SEVERAL_BLOCKS.values() for s in shapes] + front_shapes.WHOLE)
def test_several_blocks_a_wave(gpu_device, B, T, H):
    """Each tile with two to eight blocks of channels a wave, sequences that start in a tile, ragged last tiles, with and without carried rows; and
    tiles of 128 tokens with short sequences."""
    fi = make_decay_front_inputs(scaled(CONFIGS[2], B=B, T=T, H=H), seed=2100 + B + T)
    for with_prev in (True, False):
        y32 = run_front(fi, torch.float32, with_prev).cpu().numpy()
        assert max_norm_err(y32, oracle_front(fi, with_prev)) <= TOL_BF16
        y16 = run_front(fi, torch.bfloat16, with_prev).float().cpu().numpy()
        assert np.array_equal(y16, round_to_bf16(y32))
