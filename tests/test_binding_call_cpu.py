"""CPU tests of the binding's native calls: conversions, refusals and statuses are those of the C types they stand for.
Nothing is enqueued: every accepted call has nothing to do (no batch) or is refused by the library's own checks."""
import ctypes
import inspect

import pytest

import paper_2407_12077_amd as wkv
from paper_2407_12077_amd import binding

CALLS = [n for n in binding.EXPORTS
         if n not in ("wkv6_split_workspace_bytes", "wkv6_split_segments", "wkv6_arena_layout", "wkv6_status_string", "wkv6_version")]


class Buffer:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


class Whole:
    def __index__(self):
        return 0


def decode(B=0, H=2, N=64, ptr=None, stream=0):
    binding.wkv6_decode_bf16(B, H, N, ptr, ptr, ptr, ptr, ptr, ptr, ptr, stream=stream)


@pytest.mark.parametrize("name", CALLS)
def test_every_call_takes_the_header_s_arguments(name):
    """One argument a C parameter, in that order: the library answers, with a status for null addresses."""
    fn = getattr(binding, name)
    params = list(inspect.signature(fn).parameters)
    assert len(params) == len(getattr(binding.load(), name).argtypes) and params[-1] == "stream"
    whole = {"B", "T", "H", "N", "R", "R_d", "D", "M", "out_dtype", "segments", "batch_stride", "workspace_bytes"}
    args = {p: (64 if p in ("N", "D") else 1) if p in whole else 1e-5 if p == "eps" else None for p in params[:-1]}
    with pytest.raises(wkv.Wkv6Error):
        fn(**args, stream=0)
    with pytest.raises(TypeError):
        getattr(binding._bound(), name)(*args.values())            # no stream
    for p in whole & set(params):
        with pytest.raises((TypeError, wkv.Wkv6Error) if p in ("out_dtype", "segments") else TypeError) as e:
            fn(**{**args, p: 1.5}, stream=0)
        if p not in ("out_dtype", "segments"):
            assert isinstance(e.value, ctypes.ArgumentError)


def test_conversions():
    decode(B=Whole(), ptr=Buffer(4096))
    decode(B=1 << 32, ptr=Buffer(4096))                            # cut to the C type, as ctypes does
    with pytest.raises(wkv.Wkv6Error, match="NULL"):
        decode(ptr=Buffer(Whole()))
    decode(ptr=Buffer(4096), stream=Whole())
    with pytest.raises(AttributeError):
        decode(ptr=4096)
    with pytest.raises(TypeError):
        decode(ptr=Buffer("4096"))
    with pytest.raises(TypeError):
        decode(ptr=Buffer(4096), stream=[])
    with pytest.raises(TypeError):
        binding.wkv6_layernorm_finalize(1, 1, 1, 64, None, "1e-5", None, stream=0)


def test_failure_of_a_callback_is_passed_on():
    class Gone:
        def data_ptr(self):
            raise ValueError("gone")

    with pytest.raises(ValueError, match="gone"):
        decode(ptr=Gone())


def test_stream_sources():
    """None asks for the current stream: of the device that is current at the call, each time."""
    call, asked = binding._bound(), []

    def fail():
        raise LookupError("no device")

    try:
        call.stream_source(lambda device: asked.append(device) or 0, lambda: 3)
        decode(ptr=Buffer(4096), stream=None)
        decode(ptr=Buffer(4096), stream=None)
        assert asked == [3, 3]
        call.stream_source(lambda device: 0, fail)
        with pytest.raises(LookupError):
            decode(ptr=Buffer(4096), stream=None)
    finally:
        call.stream_source(None, None)
