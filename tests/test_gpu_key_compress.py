"""GPU parity of the key-compression entry point against the fp64 oracle (Method section, GOLD
Key Compression: c_t = x_t W^KD).  bf16 products are exact in fp32 and the accumulation is fp32,
so the fp32 output is held to 1e-5 (max-normalised) and the bf16 output must be the fp32 output
rounded once."""
import numpy as np
import pytest
import torch

import paper_2407_12077_amd as wkv
from oracle import key_compress_oracle
from paper_2407_12077_amd.workloads import make_key_compress_inputs, round_to_bf16

from gpu_util import max_norm_err, to_dev

pytestmark = pytest.mark.gpu


def run(x, w, out_dtype):
    M, D = x.shape
    xd, wd = to_dev(x, torch.bfloat16), to_dev(w, torch.bfloat16)
    c = torch.full((M, D // 16), float("nan"), dtype=out_dtype, device="cuda")
    code = wkv.WKV6_DTYPE_F32 if out_dtype == torch.float32 else wkv.WKV6_DTYPE_BF16
    wkv.wkv6_key_compress_bf16(M, D, xd, wd, c, code)
    torch.cuda.synchronize()
    return c.float().cpu().numpy()


@pytest.mark.parametrize("M,D", [(1, 2048), (127, 2048), (128, 2048), (129, 2048), (1000, 2048), (300, 4096), (200, 256),
                                 (333, 768), (500, 1024), (130, 2304), (1100, 4096)])
def test_matches_oracle(gpu_device, M, D):
    x, w = make_key_compress_inputs(M, D, seed=500 + M)
    ref = key_compress_oracle(x, w)
    c32 = run(x, w, torch.float32)
    assert max_norm_err(c32, ref) <= 1e-5
    c16 = run(x, w, torch.bfloat16)
    assert np.array_equal(c16, round_to_bf16(c32))


# tiles of 64 and 128 tokens with all waves alike: a last tile of one row, the fewest steps, column tiles of 16, 48 and 64 columns, a
# third column tile of 16; smaller tiles, the contraction over the waves: waves without a block, a last block of one row, 16 of 64 columns
@pytest.mark.parametrize("M,D", [(6849, 2048), (16384, 2048), (16385, 2048), (8200, 256), (16321, 256), (9000, 768), (30000, 768), (12000, 1024), (5400, 4352), (17, 2048), (2100, 2048), (4097, 2048), (3001, 768), (8191, 256), (1500, 2304)])
def test_tiles_that_fill_the_chip_at_most_once(gpu_device, M, D):
    x, w = make_key_compress_inputs(M, D, seed=900 + M)
    ref = key_compress_oracle(x, w)
    c32 = run(x, w, torch.float32)
    assert max_norm_err(c32, ref) <= 1e-5
    assert np.array_equal(run(x, w, torch.bfloat16), round_to_bf16(c32))


def test_selector_matrix_copies_channels(gpu_device):
    """W with one 1 per column: every output is one bf16 input copied exactly."""
    M, D = 200, 2048
    x, _ = make_key_compress_inputs(M, D, seed=77)
    pick = np.random.default_rng(78).integers(0, D, D // 16)
    w = np.zeros((D, D // 16), np.float32)
    w[pick, np.arange(D // 16)] = 1.0
    assert np.array_equal(run(x, w, torch.bfloat16), x[:, pick])


def test_empty_and_validation(gpu_device):
    z = torch.zeros((4, 2048), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((2048, 128), dtype=torch.bfloat16, device="cuda")
    c = torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda")
    wkv.wkv6_key_compress_bf16(0, 2048, None, None, None, wkv.WKV6_DTYPE_BF16)
    for args, status in [((4, 1000, z, w, c, 0), 3), ((4, 2048, z, w, c, 9), 3), ((4, 2048, None, w, c, 0), 1),
                         ((-1, 2048, z, w, c, 0), 2)]:
        with pytest.raises(wkv.Wkv6Error) as e:
            wkv.wkv6_key_compress_bf16(*args)
        assert e.value.status == status


@pytest.mark.parametrize("M,D", [(32768, 2048), (65536, 4096)])
def test_full_size_every_row(gpu_device, M, D):
    """The benchmark's sizes (the tokens of config 2 at D = 2048 and of config 5 at D = 4096):
    every row against the oracle."""
    x, w = make_key_compress_inputs(M, D)
    print(f"key compression M={M} D={D}: oracle on every row ...", flush=True)
    ref = key_compress_oracle(x, w)
    c32 = run(x, w, torch.float32)
    err = max_norm_err(c32, ref)
    rows = np.abs(c32 - ref).max(axis=1) / np.abs(ref).max(axis=1)
    print(f"key compression M={M} D={D}: global={err:.3e} worst row={rows.max():.3e} "
          f"rel_l2={np.linalg.norm(c32 - ref) / np.linalg.norm(ref):.3e}", flush=True)
    assert err <= 1e-5 and rows.max() <= 1e-5
    c16 = run(x, w, torch.bfloat16)
    assert np.array_equal(c16, round_to_bf16(c32))


def test_input_beyond_four_gib(gpu_device):
    """x of 4.83 GB (1 179 648 tokens of width 2048, drawn on the device from a seed): byte offsets into x
    pass 2^32.  The first, a middle and the last row tile are compared with the oracle."""
    M, D = 9216 * 128, 2048
    _, w = make_key_compress_inputs(16, D, seed=77)
    gen = torch.Generator(device="cuda").manual_seed(99)
    x = torch.empty((M, D), dtype=torch.bfloat16, device="cuda")
    for m0 in range(0, M, 65536):
        x[m0:m0 + 65536] = torch.randn((65536, D), generator=gen, device="cuda").to(torch.bfloat16)
    assert x.numel() * 2 > (1 << 32)
    wd = to_dev(w, torch.bfloat16)
    c = torch.full((M, D // 16), float("nan"), dtype=torch.float32, device="cuda")
    wkv.wkv6_key_compress_bf16(M, D, x, wd, c, wkv.WKV6_DTYPE_F32)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(c).all())
    for m0 in (0, (M // 2 // 128) * 128 + 64, M - 128):
        ref = key_compress_oracle(x[m0:m0 + 128].float().cpu().numpy(), w)
        err = max_norm_err(c[m0:m0 + 128].cpu().numpy(), ref)
        print(f"rows {m0}..{m0 + 127}: err={err:.3e}", flush=True)
        assert err <= 1e-5
    del x, c
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M,D", [(1, 256), (15, 256), (17, 768), (16, 4096), (512, 2048), (513, 2048), (1023, 2048), (1024, 2048),
                                 (1025, 2048), (2048, 2048), (2049, 2048), (4096, 2048), (4097, 2048), (2047, 768),
                                 (4095, 768), (8191, 768), (8193, 768), (8193, 2048), (4096, 4096), (4097, 4096), (40, 8192), (6816, 2048), (6817, 2048), (5440, 2304)])
def test_every_tile_of_the_split_contraction(gpu_device, M, D):
    """Both sides of every change of tile (256 workgroups of 16 x 16, 16 x 32, 16 x 64 and 32 x 64, five thirds of
    that at D = 2048 and twice that above), ragged token and column tails and one to sixteen of a workgroup's waves with work.  fp32 sums of bf16 products
    that are exact in fp32: 1e-5 of the largest value, as for the large tiles; a bf16 result is the fp32 result
    rounded once."""
    x, w = make_key_compress_inputs(M, D, seed=900 + M)
    c32 = run(x, w, torch.float32)
    assert max_norm_err(c32, key_compress_oracle(x, w)) <= 1e-5
    assert np.array_equal(run(x, w, torch.bfloat16), round_to_bf16(c32))


@pytest.mark.parametrize("M,D", [(8193, 4096), (16384, 4096), (16385, 4096), (8192, 2048), (32768, 1024), (32769, 1024), (5000, 8192), (8321, 4352)])
def test_large_tiles_around_one_per_compute_unit(gpu_device, M, D):
    """Both sides of the changes between tiles of 64 and of 128 tokens with all waves alike (at most 256 of them) and the tiles with loader
    waves, with a ragged last row tile and a partial last column tile."""
    x, w = make_key_compress_inputs(M, D, seed=77 + M)
    c32 = run(x, w, torch.float32)
    assert max_norm_err(c32, key_compress_oracle(x, w)) <= 1e-5
    assert np.array_equal(run(x, w, torch.bfloat16), round_to_bf16(c32))
