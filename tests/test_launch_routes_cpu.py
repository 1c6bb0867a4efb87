"""What the entry points launch, checked without a GPU (tests/launch_util.py): the dynamic-LDS limits are raised by an entry
point's first call whatever its size, since a later call may be captured, and each rule that chooses between kernels is
pinned on both sides of its line."""
import pytest

import launch_util as lu


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
