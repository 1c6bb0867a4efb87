"""Build ``libwkv6.so`` (HIP kernels + C ABI) for gfx950, in-tree, with hipcc, and the binding's extension with g++."""
import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libwkv6.so")
SOURCES = ["wkv6_api.hip", "wkv6_recurrent.hip", "wkv6_chunked.hip", "wkv6_chunked_f32.hip", "wkv6_segments.hip", "wkv6_short.hip",
           "key_compress.hip", "layernorm_finalize.hip", "decay_input.hip"]
CALL = os.path.join(PKG, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))      # plain host code: no HIP in it
# packed-fp32 VALU forms are switched off on purpose for the whole library
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]
# Per-source additions.  The chunked kernel's waves are latency bound (four per SIMD, long dependent
# chains): the compiler's maximum-ILP scheduling strategy measured 1 % faster on every configuration;
# the loader/worker kernels lose with it (the decay front 20 %), so it stays with this one source.
SOURCE_FLAGS = {"wkv6_chunked.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]}


def build(verbose=False, extra=()):
    """Compile every source to an object of its own (in parallel), then link the shared library, then the binding's
    extension; always recompiles."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    jobs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *SOURCE_FLAGS.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        jobs.append((cmd, obj, subprocess.Popen(cmd)))
    failed = [(cmd, proc.returncode) for cmd, _, proc in jobs if proc.wait() != 0]      # (every compiler has ended)
    if failed:
        raise subprocess.CalledProcessError(failed[0][1], failed[0][0])
    link = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *(obj for _, obj, _ in jobs)]
    if verbose:
        print(" ".join(link))
    subprocess.check_call(link)
    build_call(verbose)
    return LIB


def build_call(verbose=False):
    """The binding's extension.  It comes last: callers of the C ABI need neither g++ nor Python's headers, and have the library
    whether or not this succeeds."""
    call = ["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_path("include"),
            "-I", os.path.join(os.path.dirname(PKG), "include"), os.path.join(CSRC, "binding_call.cpp"), "-o", CALL]
    if verbose:
        print(" ".join(call))
    subprocess.check_call(call)


def ensure_built():
    """For the harness entry points (tests, smoke, bench): compile only what is not there.
    The binding itself never builds and never falls back: it raises when the library is missing."""
    if not os.path.exists(LIB):
        build()
    elif not os.path.exists(CALL):
        build_call()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
