"""Builds in-tree: librdkv.so (HIP kernels + C ABI) for gfx950 with hipcc, and _rdkv_call.so (the decode loop's calls from
Python) with the host compiler."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librdkv.so")
CALL = os.path.join(HERE, "_rdkv_call.so")
# The decode kernels are a walk over tiers, words and pieces whose conditions are the same for all lanes: numbers of a chunk, the
# grid's index, the wavefront's number.  By default the compiler's structurizer turns regions of such branches into flags and flow
# blocks too (per word of a channel-wise row three instructions, a wait, two jumps, and 20 registers in all).  The first option
# lets it leave a region as it is whose branches its uniformity analysis has proved uniform -- an analysis that takes a value it
# cannot prove for divergent --, the second takes back the exception for regions around a divergent one: a region with a single
# branch that lanes may take differently, at any depth, is structurized as ever.  (The outputs are the same bit for bit without the
# options.  One 64K sequence channel-wise 13.8 -> 12.1 us, 16 with one scale per channel 74.9 -> 68.6, 16 ragged ones token-wise
# 42.8 -> 41.6, 8 layers of 16K tokens 76.4 -> 75.0, launches bound by HBM 0 to 0.5 %.  The search and the packing gain nothing, the
# weights spill.)
UNIFORM = ["-mllvm", "-structurizecfg-skip-uniform-regions", "-mllvm", "-structurizecfg-relaxed-uniform-regions=false"]
# The scheduler counts live registers by the target's own trackers (only an estimate of pressure: which instruction order it
# prefers): the second weights pass, which has all 256, no longer keeps eight values in memory across its loop, for 32 instead of
# 11 scalars in lanes of a vector register (8 heads x 128K keys 79.2 -> 77.4 us, 128 heads x 20K keys 199 -> 188).  The other files'
# kernels come out the same.
EXACT_PRESSURE = ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"]
# (source, object, extra flags); the mixed-mode decode kernels are compiled once per head-set count and row length
# class so that their many instantiations build in parallel; the slowest objects come first
SOURCES = [
    ("decode_mixed_kernels.hip", "decode_mixed_hs2_long1.o", ["-DRDKV_MIXED_HS=2", "-DRDKV_MIXED_LONG=1"] + UNIFORM),
    ("decode_mixed_kernels.hip", "decode_mixed_hs2_long0.o", ["-DRDKV_MIXED_HS=2", "-DRDKV_MIXED_LONG=0"] + UNIFORM),
    ("decode_mixed_kernels.hip", "decode_mixed_hs1_long1.o", ["-DRDKV_MIXED_HS=1", "-DRDKV_MIXED_LONG=1"] + UNIFORM),
    ("decode_mixed_kernels.hip", "decode_mixed_hs1_long0.o", ["-DRDKV_MIXED_HS=1", "-DRDKV_MIXED_LONG=0"] + UNIFORM),
    ("decode_mfma_kernels.hip", "decode_mfma_kernels.o", UNIFORM),
    ("rdkv_api.hip", "rdkv_api.o", []),
    ("decode_rows_mfma.hip", "decode_rows_mfma.o", []),
    ("decode_kernels.hip", "decode_kernels.o", []),
    ("copy_kernels.hip", "copy_kernels.o", []),
    ("pack_kernels.hip", "pack_kernels.o", []),
    ("allocate_kernels.hip", "allocate_kernels.o", []),
    # (its copies into LDS set m0, a reserved register, and say so)
    ("weights_kernels.hip", "weights_kernels.o", ["-Wno-inline-asm"] + EXACT_PRESSURE),
    ("calib_kernels.hip", "calib_kernels.o", []),
]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the quantizer must be reproducible bit for bit: no implicit fused multiply-add
    "-ffp-contract=off",
    # MFMA results stay in ordinary vector registers (no copies through the accumulation registers)
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # the leading kernel arguments arrive in registers with the wavefront (no load before the first address is known)
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def call_command():
    """The host compiler's line for _rdkv_call.so: against the installed PyTorch's headers, without a HIP header."""
    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", "-I" + os.path.join(ROOT, "include")] +
            ["-isystem" + p for p in include_paths() + [sysconfig.get_paths()["include"]]] +
            [os.path.join(CSRC, "rdkv_call.cpp"), "-o", CALL, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10"])


def build(verbose=True, jobs=8):
    objs, procs = [], []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    cmd = call_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs.append(("rdkv_call.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, obj_name, extra in SOURCES:
        obj = os.path.join(HERE, "_build", obj_name)
        objs.append(obj)
        cmd = ["hipcc", "-c", os.path.join(CSRC, src), "-o", obj] + FLAGS + extra
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((obj_name, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = ["hipcc", "-shared", "-o", LIB] + objs + ["--offload-arch=gfx950"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def _drain(procs):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if out:
            print(out, flush=True)
        if p.returncode != 0:
            raise RuntimeError(f"the compiler failed on {src}")


if __name__ == "__main__":
    build()
    print("built", LIB)
