"""The binding refuses what ctypes refuses: strides and sizes in elements or bytes are whole numbers."""
import pytest

import paper_2407_12077_amd as wkv


class Address:                     # a tensor as far as the binding looks
    def data_ptr(self):
        return 0x1000


A = Address()


@pytest.mark.parametrize("entry", ["wkv6_prefill_bf16_strided", "wkv6_finch_c2_prefill_bf16_strided"])
def test_a_fractional_stride_is_refused(entry):
    with pytest.raises(TypeError):
        getattr(wkv, entry)(0, 8, 2, 64, A, A, A, A, A, None, A, A, 1024.5, 0, stream=0)
    getattr(wkv, entry)(0, 8, 2, 64, A, A, A, A, A, None, A, A, 1024, 0, stream=0)       # no sequence: nothing to launch


@pytest.mark.parametrize("entry", ["wkv6_prefill_bf16_split", "wkv6_finch_c2_prefill_bf16_split"])
def test_a_fractional_workspace_size_is_refused(entry):
    with pytest.raises(TypeError):
        getattr(wkv, entry)(0, 8, 2, 64, A, A, A, A, A, None, A, A, 0, 1, A, 4096.5, stream=0)
    getattr(wkv, entry)(0, 8, 2, 64, A, A, A, A, A, None, A, A, 0, 1, A, 4096, stream=0)
