"""What the entry points launch, checked without a GPU (tests/launch_util.py): the dynamic-LDS limits are raised by an entry
point's first call whatever its size, since a later call may be captured, and each rule that chooses between kernels is
pinned on both sides of its line."""
import pytest

import front_shapes
import launch_util as lu
from split_shapes import SPLIT, WHOLE


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return lu.build_fake(tmp_path_factory.mktemp("fake_hip"))


SIZES = [(1, 1, 32), (3, 6, 4), (2, 7, 4), (1, 2000, 4), (300, 40, 4), (2, 33, 260)]      # (B, T, H): every kernel behind an entry


@pytest.mark.parametrize("make", [
    lambda B, T, H: lu.time_mix("wkv6_append_bf16", B, T, H),
    lambda B, T, H: lu.time_mix("wkv6_finch_c2_append_bf16", B, T, H),
    lambda B, T, H: lu.time_mix("wkv6_prefill_bf16", B, T, H),
    lambda B, T, H: lu.time_mix("wkv6_finch_c2_prefill_bf16_f32out", B, T, H),
    lambda B, T, H: lu.fused_c2(B, T, H),
    lambda B, T, H: lu.fused_c2(B, T, H, moments=False),
    lambda B, T, H: lu.fused_finch(B, T, H),
], ids=["append", "c2_append", "prefill", "c2_prefill_f32out", "fused_c2_moments", "fused_c2", "fused_finch"])
def test_first_call_raises_every_limit_of_its_entry(fake, make):
    for first in SIZES:
        per_call = lu.events(fake, [make(*first)] + [make(*s) for s in SIZES])
        limit = {e.kernel: e.bytes for e in per_call[0] if e.kind == "attribute"}
        for size, ev in zip(SIZES, per_call[1:]):
            assert not [e for e in ev if e.kind == "attribute"], (first, size)
            for e in ev:
                assert e.bytes <= max(65536, limit.get(e.kernel, 0)), (first, size, e.kernel)


@pytest.mark.parametrize("B,H,c2,longest", [(1, 4, True, 2), (8, 32, True, 2), (8, 32, False, 2), (9, 32, True, 3), (16, 32, False, 3),
                                            (17, 32, True, 4), (32, 32, True, 4), (33, 32, True, 2), (256, 32, True, 2), (17, 32, False, 4),
                                            (33, 32, False, 4), (256, 32, False, 4)])
def test_fused_decay_calls_are_token_by_token_up_to_two_to_four_tokens(fake, B, H, c2, longest):
    """By the number of units; 6 tokens of 32 units take twice as long token by token."""
    make = (lambda T: lu.fused_c2(B, T, H)) if c2 else (lambda T: lu.fused_finch(B, T, H))
    for T, kernels in zip(range(1, 9), lu.launched(fake, [make(T) for T in range(1, 9)])):
        assert kernels == ["recurrent_kernel" if T <= longest else "one_chunk_kernel"], T


@pytest.mark.parametrize("B,T,H,few", [(1, 1, 1, True), (24, 1, 32, True), (136, 15, 32, True), (137, 15, 32, False), (3, 16, 12, False),
                                       (256, 8, 12, True), (257, 8, 12, False), (4096, 2, 32, True), (4096, 3, 32, False), (4096, 2, 31, False),
                                       (65535, 1, 2, True), (65535, 2, 2, False), (4096, 8, 256, True), (4096, 9, 256, False), (1024, 4, 64, True), (1024, 5, 64, False),
                                       (1024, 8, 128, True), (1024, 9, 128, False)])
def test_fold_by_wave_per_token_only_for_few_tokens_or_many_heads(fake, B, T, H, few):
    """65 535 sequences of 15 tokens and 2 heads took nine times as long with a wave per token."""
    call = ("wkv6_layernorm_finalize", [B, T, H, 64, lu.at(0), 1e-5, lu.at(1), None])
    assert lu.launched(fake, [call])[0] == ["layernorm_finalize_few_kernel" if few else "layernorm_finalize_kernel"]


@pytest.mark.parametrize("tokens,H,through", [(1, 32, True), (8 * 2048, 32, True), (17 * 1024, 32, True), (17 * 1024 + 1, 32, False), (10 * 2048, 32, False),
                                              (8 * 1024, 64, True), (9 * 1024, 64, False), (24, 12, False), (1365, 12, False), (1366, 12, True), (24576, 12, True),
                                              (24577, 12, False), (1023, 16, False), (1024, 16, True), (16384, 16, True), (18433, 16, False)])
@pytest.mark.parametrize("f32", [False, True])
def test_normalised_rows_written_through_only_while_that_is_faster(fake, tokens, H, through, f32):
    """24 tokens of 12 heads written through took 4.3 us against 3.9."""
    call = ("wkv6_layernorm_apply_bf16", [1, tokens, H, 64, lu.at(0), lu.at(1), lu.at(2), lu.at(3), lu.at(4), int(f32), None])
    [run] = [e for e in lu.events(fake, [call])[0] if e.kind == "launch"]
    name = "layernorm_apply_strip_kernel" if H % 32 == 0 else "layernorm_apply_kernel"
    assert run.kernel.startswith("%s<%s, %d>(" % (name, str(f32).lower(), 16 if through and not f32 else 2)), run.kernel


@pytest.mark.parametrize("B,T,D,kernel", [
    (1, 1, 128, "split_kernel<1, 12,"), (24, 1, 128, "split_kernel<1, 12,"), (300, 1, 128, "split_kernel<1, 12,"), (16, 1024, 128, "decay_input_kernel<"),
    (33, 1024, 128, "decay_input_kernel<"), (1000, 20, 128, "split_kernel<1, 12,"), (1000, 40, 256, "split_kernel<2, 8,"), (33, 1024, 256, "decay_input_kernel<"),
    (24, 1, 256, "split_kernel<1, 12,"), (300, 129, 256, "split_kernel<4, 8,"), (33, 1024, 768, "decay_input_kernel<"), (16, 1024, 768, "split_kernel<4, 8,"),
    (24, 1, 2048, "split_kernel<1, 12,"), (8, 1000, 2048, "split_kernel<2, 8,"), (16, 1024, 2048, "split_kernel<4, 8,"), (24, 1000, 2048, "decay_input_kernel<"),
    (33, 1024, 2048, "split_kernel<4, 8,"), (33, 1024, 4096, "split_kernel<4, 8,"), (32, 1024, 2048, "decay_input_kernel<"),
    (130, 31, 256, "split_kernel<1, 12,"), (131, 33, 256, "split_kernel<2, 8,"), (256, 32, 256, "split_kernel<2, 8,"), (2, 4097, 256, "split_kernel<4, 8,"),
    (3, 5461, 256, "split_kernel<4, 8,"), (1, 16385, 256, "decay_input_kernel<"), (600, 3, 128, "split_kernel<1, 12,"), (1000, 40, 2048, "split_kernel<2, 8,"),
    (4, 1000, 128, "split_kernel<1, 12,"), (2, 2100, 128, "split_kernel<2, 8,"), (8, 1000, 128, "split_kernel<2, 8,"), (500, 50, 128, "decay_input_kernel<"),
    (500, 50, 768, "split_kernel<2, 8,"), (33, 1024, 1024, "split_kernel<4, 8,"), (5, 4000, 1024, "decay_input_kernel<")])
def test_decay_front_tiles_by_width(fake, B, T, D, kernel):
    """What a round of each tile takes depends on the width: at D = 128, 33 x 1024 tokens in 64-row tiles take 18 us against 14, and one token
    in a tile of 128 tokens 6.5 against 3.9."""
    call = ("wkv6_decay_lora_input_bf16", [B, T, D, 32, 64] + [lu.at(i) for i in range(8)] + [0, None])
    [ev] = lu.events(fake, [call])
    [launch] = [e for e in ev if e.kind == "launch"]
    assert kernel in launch.kernel, launch.kernel


@pytest.mark.parametrize("f32", [False, True])
def test_decay_front_shapes_of_the_gpu_tests(fake, f32):
    wanted = [(s, k % str(f32).lower()) for k, shapes in front_shapes.SEVERAL_BLOCKS.items() for s in shapes]
    wanted += [(s, "decay_input_kernel<%s>" % str(f32).lower()) for s in front_shapes.WHOLE]
    calls = [("wkv6_decay_lora_input_bf16", [B, T, 64 * H, 32, 64] + [lu.at(i) for i in range(8)] + [int(f32), None]) for (B, T, H), _ in wanted]
    for (shape, kernel), ev in zip(wanted, lu.events(fake, calls)):
        assert [e.kernel for e in ev if e.kind == "launch"] == [kernel], shape


@pytest.mark.parametrize("B,T,D,groups", [(1, 1, 2048, 4), (24, 1, 2048, 4), (1, 1024, 2048, 4), (1025, 1, 2048, 2), (4, 512, 768, 2), (1, 2049, 2048, 1), (4, 1024, 2048, 1)])
def test_decay_front_outputs_of_a_tile_over_workgroups(fake, B, T, D, groups):
    call = ("wkv6_decay_lora_input_bf16", [B, T, D, 32, 64] + [lu.at(i) for i in range(8)] + [0, None])
    [launch] = [e for e in lu.events(fake, [call])[0] if e.kind == "launch"]
    assert launch.kernel == "decay_input_split_kernel<1, 12, false, %d>" % groups
    assert launch.grid[0] == (B * T + 15) // 16 * groups


# shapes of tests/test_gpu_own_split.py beside those of the list
ALSO_SPLIT = [(1, 1100, 4), (2, 1531, 12), (2, 1201, 6), (1, 1000, 4), (1, 1300, 8)]


@pytest.mark.parametrize("make", [lambda B, T, H: lu.time_mix("wkv6_prefill_bf16", B, T, H), lambda B, T, H: lu.time_mix("wkv6_finch_c2_append_bf16", B, T, H),
                                  lambda B, T, H: lu.fused_c2(B, T, H), lambda B, T, H: lu.fused_finch(B, T, H)],
                         ids=["prefill", "c2_append", "fused_c2", "fused_finch"])
def test_own_split_where_it_is_said_to_be(fake, make):
    """Three segments of 384 tokens (85 units of 1100) took 7 % longer than the whole walk."""
    shapes = list(SPLIT) + ALSO_SPLIT + WHOLE
    for (B, T, H), ev in zip(shapes, lu.events(fake, [make(*s) for s in shapes])):
        run = [e for e in ev if e.kind == "launch"]
        if (B, T, H) in WHOLE:
            assert [e.base for e in run] == ["chunked_kernel"], (B, T, H)
            continue
        assert [e.base for e in run] == ["segment_state_kernel", "segment_fold_kernel", "chunked_kernel"], (B, T, H)
        if (B, T, H) in SPLIT:
            segs = SPLIT[B, T, H][0]
            assert [e.grid[0] for e in run] == [B * (segs - 1) * H, 4 * B * H, B * segs * H], (B, T, H)


@pytest.mark.parametrize("units,T,columns", [(32, 16, 2), (33, 17, 4), (128, 17, 4), (129, 16, 8), (129, 17, 0), (256, 18, 0), (256, 20, 0),
                                             (256, 21, 8), (256, 1000, 8), (257, 16, 0)])
@pytest.mark.parametrize("entry,bf16", [("wkv6_prefill_f32", False), ("wkv6_prefill_bf16_recurrent", True)])
def test_columns_of_few_units_over_workgroups(fake, entry, bf16, units, T, columns):
    """From 129 units on, 17 to 20 tokens are faster or level by the four-wave form (0: 256 units x 17 tokens 9.0 against 9.4 us)."""
    [ev] = lu.events(fake, [lu.time_mix(entry, 1, T, units)])
    if not bf16 and (units, T) == (256, 1000):                # fp32 tensors: only short sequences token by token
        assert [e.kernel for e in ev if e.kind == "launch"] == ["chunked_f32_kernel<4, 4>"]
        return
    ev = [e for e in ev if e.kind == "launch"]
    want = "recurrent_columns_kernel<%d, %s>" % (columns, str(bf16).lower()) if columns else "recurrent_wide_kernel<%s, false>" % str(bf16).lower()
    assert [e.kernel for e in ev] == [want]


@pytest.mark.parametrize("B,H", [(1, 1), (8, 32), (9, 32), (256, 32)])
@pytest.mark.parametrize("make,shortest", [
    (lambda B, T, H: lu.time_mix("wkv6_append_bf16", B, T, H), 7), (lambda B, T, H: lu.time_mix("wkv6_finch_c2_append_bf16", B, T, H), 7),
    (lambda B, T, H: lu.time_mix("wkv6_prefill_bf16", B, T, H), 1), (lambda B, T, H: lu.time_mix("wkv6_finch_c2_prefill_bf16_f32out", B, T, H), 1),
    (lambda B, T, H: lu.fused_c2(B, T, H), 5), (lambda B, T, H: lu.fused_finch(B, T, H), 5)],
    ids=["append", "c2_append", "prefill", "c2_prefill_f32out", "fused_c2", "fused_finch"])
def test_sequences_of_one_chunk_take_four_waves_a_unit(fake, make, shortest, B, H):
    for T, ev in zip((shortest, 32, 33), lu.events(fake, [make(B, T, H) for T in (shortest, 32, 33)])):
        [run] = [e for e in ev if e.kind == "launch"]
        assert (run.base, run.block, run.bytes <= 40 * 1024) == (("one_chunk_kernel", 256, True) if T <= 32 else ("chunked_kernel", 1024, False))
        assert T > 32 or run.grid[0] == B * H


@pytest.mark.parametrize("make,lengths", [
    (lambda B, T, H: lu.time_mix("wkv6_prefill_bf16", B, T, H, False), (1, 32)), (lambda B, T, H: lu.time_mix("wkv6_prefill_bf16_f32out", B, T, H, False), (1, 32)),
    (lambda B, T, H: lu.time_mix("wkv6_finch_c2_append_bf16", B, T, H, False), (7, 32)), (lambda B, T, H: lu.fused_c2(B, T, H), (5, 32)),
    (lambda B, T, H: lu.fused_finch(B, T, H), (5, 32))], ids=["prefill", "f32out", "c2_append", "fused_c2", "fused_finch"])
@pytest.mark.parametrize("B,H", [(524287, 32), (524288, 32), (65537, 256), (174763, 96)])
def test_one_chunk_of_more_units_than_a_grid_takes(fake, make, lengths, B, H):
    """A launch holds fewer than 2^32 work items: from 2^24 units on, the several units of a workgroup of the kernel for longer sequences."""
    for T, ev in zip(lengths, lu.events(fake, [make(B, T, H) for T in lengths])):
        [run] = [e for e in ev if e.kind == "launch"]
        assert run.grid[0] * run.block < 2 ** 32 and run.base == ("one_chunk_kernel" if B * H < 2 ** 24 else "chunked_kernel"), T


@pytest.mark.parametrize("entry,B,T,H,multi,traffic", [
    ("wkv6_prefill_bf16", 8, 33, 32, False, 0), ("wkv6_prefill_bf16", 8, 520, 32, False, 0), ("wkv6_prefill_bf16", 8, 530, 32, False, 1),
    ("wkv6_prefill_bf16", 8, 8000, 32, False, 1), ("wkv6_prefill_bf16", 16, 230, 32, True, 0), ("wkv6_prefill_bf16", 16, 240, 32, True, 1),
    ("wkv6_prefill_bf16", 64, 760, 32, True, 1), ("wkv6_prefill_bf16", 64, 790, 32, True, 2), ("wkv6_prefill_bf16_f32out", 16, 110, 32, True, 0),
    ("wkv6_prefill_bf16_f32out", 64, 620, 32, True, 1), ("wkv6_prefill_bf16_f32out", 64, 660, 32, True, 2),
    ("wkv6_finch_c2_prefill_bf16", 16, 190, 32, True, 0), ("wkv6_finch_c2_prefill_bf16", 256, 512, 32, True, 2), ("wkv6_finch_c2_prefill_bf16", 1, 4096, 32, False, 1)])
def test_cache_policies_by_the_bytes_of_a_call(fake, entry, B, T, H, multi, traffic):
    """0: less than 90 MiB of rows and states; 2: several units a workgroup and more than a GiB."""
    run = [e for e in lu.events(fake, [lu.time_mix(entry, B, T, H)])[0] if e.kind == "launch"][-1]
    assert run.base == "chunked_kernel" and run.kernel.endswith("%s, (Traffic)%d>" % (str(multi).lower(), traffic)), run.kernel


@pytest.mark.parametrize("B,T,multi,traffic", [(8, 340, False, 0), (8, 390, False, 1), (16, 150, True, 0), (16, 170, True, 1), (256, 512, True, 1)])
def test_cache_policies_of_a_call_inside_a_layer(fake, B, T, multi, traffic):
    run = [e for e in lu.events(fake, [lu.fused_c2(B, T, 32)])[0] if e.kind == "launch"][-1]
    assert run.kernel.endswith("%s, (Traffic)%d>" % (str(multi).lower(), traffic)), run.kernel


@pytest.mark.parametrize("units,shortest,column_blocks", [(1, 97, 1), (24, 97, 1), (25, 33, 1), (64, 33, 1), (65, 33, 2), (96, 33, 2), (97, 24, 2), (128, 24, 2),
                                                          (129, 24, 4), (256, 24, 4), (257, 48, 4), (512, 48, 4)])
def test_fp32_sequences_in_chunks_from_where_that_is_faster(fake, units, shortest, column_blocks):
    calls = [lu.time_mix("wkv6_prefill_f32", 1, T, units) for T in (shortest - 1, shortest, 201)]
    below, *above = [[e for e in ev if e.kind == "launch"] for ev in lu.events(fake, calls)]
    assert "recurrent" in below[0].kernel
    for launch in above:
        assert [e.kernel for e in launch] == ["chunked_f32_kernel<%d, 4>" % column_blocks]
        assert launch[0].grid[0] == (units + 7) // 8 * 8 * (4 // column_blocks)


@pytest.mark.parametrize("units,chunked", [(512, (48, 56, 57, 64, 65, 79, 80)), (513, (57, 64, 80, 200)), (768, (57, 64, 80)), (769, (48, 56, 57, 64, 65, 79, 80)),
                                           (1024, (48, 56, 57, 64, 65, 79, 80)), (1025, (57, 64, 80)), (2048, (57, 64, 80)), (4096, (57, 64, 80, 81))])
def test_fp32_of_many_units_in_chunks_only_where_that_is_faster(fake, units, chunked):
    """4096 units of 48 tokens took 159 us against 143 token by token, 2048 of 65 tokens 106 against 99."""
    lengths = [47, 48, 56, 57, 64, 65, 79, 80, 81, 200]
    for T, ev in zip(lengths, lu.events(fake, [lu.time_mix("wkv6_prefill_f32", 1, T, units) for T in lengths])):
        [run] = [e for e in ev if e.kind == "launch"]
        assert (run.base == "chunked_f32_kernel") == (T in chunked or T > 80), T


@pytest.mark.parametrize("units,chunked", [(2 ** 23 - 8, True), (2 ** 23 - 7, False), (2 ** 23, False), (2 ** 24 - 1, False)])
def test_fp32_of_more_units_than_a_grid_takes(fake, units, chunked):
    """The token-by-token form has half as many threads a unit."""
    [run] = [e for e in lu.events(fake, [lu.time_mix("wkv6_prefill_f32", units, 100, 1)])[0] if e.kind == "launch"]
    assert run.base == ("chunked_f32_kernel" if chunked else "recurrent_wide_kernel")


@pytest.mark.parametrize("compute_units,units,column_blocks", [(256, 64, 1), (256, 65, 2), (256, 129, 4), (128, 32, 1), (128, 33, 2), (128, 64, 2), (128, 65, 4), (304, 76, 1), (304, 152, 2)])
def test_fp32_column_groups_while_they_fit_the_chip(fake, compute_units, units, column_blocks):
    [run] = [e for e in lu.events(fake, [lu.time_mix("wkv6_prefill_f32", 1, 150, units)], compute_units)[0] if e.kind == "launch"]
    assert run.kernel == "chunked_f32_kernel<%d, 4>" % column_blocks


@pytest.mark.parametrize("units,shortest", [(1, 202), (32, 264), (64, 328), (65, None), (256, None)])
def test_fp32_scores_in_a_kernel_of_their_own(fake, units, shortest):
    """A wave a chunk; the second kernel's grid as without them."""
    lengths = [(shortest or 400) - 1, shortest or 400, 5000]
    for T, ev in zip(lengths, lu.events(fake, [lu.time_mix("wkv6_prefill_f32", 1, T, units) for T in lengths])):
        launch = [e for e in ev if e.kind == "launch"]
        if shortest and T >= shortest:
            assert [e.kernel for e in launch] == ["chunked_f32_scores_kernel", "chunked_f32_scored_kernel<1, 4>"]
            assert launch[0].grid[0] * 4 - units * ((T + 15) // 16) in range(4)
            assert launch[1].grid[0] == (units + 7) // 8 * 8 * 4
        else:
            assert [e.base for e in launch] == ["chunked_f32_kernel"]


@pytest.mark.parametrize("first", [(1, 1, 4), (2, 20, 16), (4, 100, 4), (40, 100, 4), (3, 100, 32), (300, 100, 4), (4, 300, 4)])
def test_first_fp32_call_raises_every_limit(fake, first):
    sizes = [(4, 100, 4), (40, 100, 4), (3, 100, 32), (300, 100, 4), (4, 300, 4)]
    per_call = lu.events(fake, [lu.time_mix("wkv6_prefill_f32", *first)] + [lu.time_mix("wkv6_prefill_f32", *s) for s in sizes])
    limit = {e.kernel: e.bytes for e in per_call[0] if e.kind == "attribute"}
    for ev in per_call[1:]:
        assert {e.kind for e in ev} == {"launch"} and ev[-1].bytes <= limit[ev[-1].kernel]


@pytest.mark.parametrize("M,D,kernel", [
    (16, 2048, "few_kernel<1, 1,"), (4096, 2048, "few_kernel<2, 4,"), (4097, 2048, "few_kernel<2, 4,"), (6816, 2048, "few_kernel<2, 4,"), (6817, 2048, "key_compress_kernel<128, 2,"),
    (8192, 2048, "key_compress_kernel<128, 2,"), (4096, 1792, "few_kernel<2, 4,"), (4097, 1792, "key_compress_kernel<128, 2,"), (5440, 2304, "few_kernel<2, 4,"), (5461, 2304, "key_compress_kernel<128, 2,"),
    (4096, 4096, "few_kernel<2, 4,"), (4097, 4096, "key_compress_kernel<128, 2,"), (16384, 4096, "key_compress_kernel<128, 2,"), (16385, 4096, "key_compress_kernel<256, 4,"), (32769, 2048, "key_compress_kernel<128, 4,")])
def test_key_compression_tiles(fake, M, D, kernel):
    """From D = 2048 on the small tiles, whose sums in sixteen parts are the closest to 64 bits, go on beyond one round: up to five thirds of
    it at D = 2048, to two above."""
    call = ("wkv6_key_compress_bf16", [M, D, lu.at(0), lu.at(1), lu.at(2), 0, None])
    [launch] = [e for e in lu.events(fake, [call])[0] if e.kind == "launch"]
    assert kernel in launch.kernel, launch.kernel


@pytest.mark.parametrize("make,T,four", [
    (lambda T, units: lu.decode("wkv6_decode_bf16", units, 1), 1, [(1024, True), (1025, False), (2559, False), (2560, True), (2 ** 24, False)]),
    (lambda T, units: lu.decode("wkv6_finch_c2_decode_bf16", units, 1), 1, [(1024, True), (1025, False), (2559, False), (2560, True)]),
    (lambda T, units: lu.time_mix("wkv6_append_bf16", units, T, 1), 1, [(1024, True), (1025, False), (2559, False), (2560, True)]),
    (lambda T, units: lu.time_mix("wkv6_append_bf16", units, T, 1), 6, [(1536, True), (1537, False), (2560, False), (8192, False)]),
    (lambda T, units: lu.time_mix("wkv6_finch_c2_append_bf16", units, T, 1), 2, [(1536, True), (1537, False), (2560, False)]),
    (lambda T, units: lu.time_mix("wkv6_prefill_f32", units, T, 1), 15, [(1536, True), (1537, False), (2560, False)]),
    (lambda T, units: lu.fused_c2(units, T, 1), 1, [(2048, True), (2049, False)]), (lambda T, units: lu.fused_c2(units, T, 1), 2, [(2048, True), (2049, False)]),
    (lambda T, units: lu.fused_finch(units, T, 1), 1, [(1024, True), (1025, False), (2048, False)]),
    (lambda T, units: lu.fused_finch(units, T, 1), 2, [(1280, True), (1281, False), (2048, False)]),
    (lambda T, units: lu.fused_finch(units, T, 1), 4, [(1280, True), (1281, False), (2048, False)])],
    ids=["decode", "c2_decode", "append_1", "append_6", "c2_append_2", "f32_15", "fused_c2_1", "fused_c2_2", "fused_finch_1", "fused_finch_2", "fused_finch_4"])
def test_four_waves_a_unit_only_where_that_is_faster(fake, make, T, four):
    """Finch with fused logits, 2048 units of one token: four waves 13.2 us against 10.4."""
    for (units, want), ev in zip(four, lu.events(fake, [make(T, units) for units, _ in four])):
        [run] = [e for e in ev if e.kind == "launch"]
        assert run.base == "recurrent_kernel" and run.grid[0] == units
        assert (run.block, run.kernel.endswith(", 4>")) == ((256, True) if want else (64, False)), units


@pytest.mark.parametrize("heads,kept", [(1, 1), (4, 1), (5, 4), (16, 4), (17, 8), (32, 8), (33, 12), (48, 12), (49, 16), (64, 16), (65, 24), (96, 24), (97, 32),
                                        (128, 32), (129, 40), (160, 40), (161, 48), (192, 48), (193, 64), (256, 64), (257, 64), (1000, 64)])
def test_fold_keeps_the_heads_of_a_wave_and_few_more(fake, heads, kept):
    """8 x 2048 tokens of 32 heads took 2.5 us with sixteen places against 2.2 with eight."""
    call = ("wkv6_layernorm_finalize", [2, 300, heads, 64, lu.at(0), 1e-5, lu.at(1), None])
    [run] = [e for e in lu.events(fake, [call])[0] if e.kind == "launch"]
    assert run.kernel == "layernorm_finalize_kernel<%d, %s>" % (kept, str(heads > 256).lower()) and (heads > 256 or 4 * kept >= heads)
