"""Which kernels a sequence of calls launches, without a GPU: a child process loads a stand-in for the HIP runtime
(tests/launch_log/fake_hip.cpp) in front of the library and makes the calls with addresses that nothing reads."""
import json
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, json, sys
sys.path.insert(0, sys.argv[1])
fake = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
fake.launch_log.restype = ctypes.c_char_p
from paper_2407_12077_amd import binding
lib, res = binding.load(), []
for name, args in json.load(sys.stdin):
    fake.launch_log_clear()
    status = getattr(lib, name)(*args)
    res.append([status, fake.launch_log().decode()])
print(json.dumps(res))
"""


def build_fake(folder):
    so = os.path.join(str(folder), "libfake_hip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC",
                           os.path.join(ROOT, "tests", "launch_log", "fake_hip.cpp"), "-o", so])
    return so


class Event:
    def __init__(self, line):
        kind, gx, gy, bx, size, name = line.split("\t")
        self.kind, self.grid, self.block, self.bytes = kind, (int(gx), int(gy)), int(bx), int(size)
        name = re.sub(r"\(anonymous namespace\)::|wkv6::|^void ", "", name)
        self.kernel = name[:name.rindex("(")]                    # template arguments included
        self.base = self.kernel.split("<")[0]


def events(fake, calls, compute_units=256):
    """calls: [(entry, [arguments])]; per call the events in order.  All calls in one fresh process."""
    out = subprocess.run([sys.executable, "-c", CHILD, ROOT, fake], input=json.dumps(calls), capture_output=True, text=True,
                         env={**os.environ, "FAKE_HIP_COMPUTE_UNITS": str(compute_units)})
    assert out.returncode == 0, out.stderr
    res = []
    for (name, args), (status, text) in zip(calls, json.loads(out.stdout)):
        assert status == 0, (name, args, status)
        res.append([Event(line) for line in text.splitlines()])
    return res


# addresses: aligned, far apart, never read
def at(i, shift=0):
    return (0x10 + i) * 0x1000000000 + shift


def time_mix(entry, B, T, H, state=True):
    """Arguments of a prefill or append entry with the plain argument list."""
    return (entry, [B, T, H, 64, at(0), at(1), at(2), at(3), at(4), at(5) if state else None, at(6), at(7), None])


def decode(entry, B, H):
    return (entry, [B, H, 64, at(0), at(1), at(2), at(3), at(4), at(5), at(6), None])


def fused_c2(B, T, H, moments=True):
    return ("wkv6_finch_c2_prefill_lora_bf16", [B, T, H, 64, 64, at(0), at(1), at(2), at(3), at(4), at(8), at(9), at(5), at(6),
                                                at(10) if moments else None, at(7), None])


def fused_finch(B, T, H):
    return ("wkv6_prefill_lora_bf16", [B, T, H, 64, 64, at(0), at(1), at(2), at(3), at(4), at(8), at(9), at(5), at(6), at(7), None])


def launched(fake, calls):
    """Per call the names of the kernels that it launches, without template arguments."""
    return [[e.base for e in ev if e.kind == "launch"] for ev in events(fake, calls)]
