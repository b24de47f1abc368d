"""Build liblotts.so (HIP kernels + C ABI) for gfx950 with hipcc, and the extension _calls (the binding's host side) with g++, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "liblotts.so")
LIB_NO_POLLS = os.path.join(_HERE, "liblotts_no_polls.so")
LIB_FLAT = os.path.join(_HERE, "liblotts_flat.so")
CALIB = os.path.join(_HERE, "calib_copy")
PROBE = os.path.join(_HERE, "libread_probe.so")
CALLS = os.path.join(_HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["verify_attention.hip", "spec_accept.hip", "spec_accept_logits.hip", "majority_vote.hip",
           "confidence_vote.hip", "skinny_gemm.hip", "kv_append.hip", "kernel_timer.hip", "greedy_search.cpp"]


FLAGS = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build(verbose: bool = False) -> str:
    """Cross-compiles on a machine without a GPU too.  Packed-fp32 code generation is switched
    off for all device code."""
    lib = FLAGS + ["-fPIC", "-shared", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    sources = [os.path.join(CSRC, s) for s in SOURCES]
    import torch   # its version, its headers and its C++ ABI; no GPU is looked for
    torch_dir = os.path.dirname(torch.__file__)
    jobs = [
        lib + sources + ["-o", LIB],
        # the same library without patience, for the tests: whatever waits for another workgroup gives up at once
        lib + ["-DLOTTS_WAIT_POLLS=0"] + sources + ["-o", LIB_NO_POLLS],
        # and with attention's flat plan for calls of any length, for the tests
        lib + ["-DLOTTS_FLAT_STEPS=0"] + sources + ["-o", LIB_FLAT],
        # the counter-calibration copy program (profiling aid, not part of the library)
        FLAGS + [os.path.join(CSRC, "calib_copy.hip"), "-o", CALIB],
        # the read-only streaming probe bench.py puts next to the attention kernel (measurement aid, its own library)
        FLAGS + ["-fPIC", "-shared", os.path.join(CSRC, "read_probe.hip"), "-o", PROBE],
        # the Python extension that makes the shortest calls (host code only; torch is loaded before it)
        ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(),
         '-DLOTTS_TORCH="%s"' % torch.__version__, "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(torch_dir, "include"),
         "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "calls.cpp"), "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python",
         "-ltorch_cpu", "-lc10", "-o", CALLS],
    ]
    running = [subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for cmd in jobs]
    outputs = ["\n".join(l for l in p.communicate()[0].splitlines() if "not a recognized feature" not in l) for p in running]
    for p, out in zip(running, outputs):
        if p.returncode != 0:
            raise RuntimeError("%s failed:\n%s" % (p.args[0], out))
    if verbose and outputs[0].strip():
        print(outputs[0])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
