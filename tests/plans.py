"""The library's launch plans, from its own sources compiled for the host (plans_main.cpp)."""
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _program(flags=()):
    src, where = os.path.join(ROOT, "tests", "plans_main.cpp"), tempfile.mkdtemp(prefix="plans")
    out = [os.path.join(where, n) for n in ("plans.o", "runtime.o", "plans")]
    for cmd in (["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-w", "-I" + os.path.join(ROOT, "include"),
                 "-I" + os.path.join(ROOT, "paper_2505_19634_amd", "csrc"), *flags, "-x", "hip", "-c", src, "-o", out[0]],
                ["g++", "-DPLANS_RUNTIME", "-c", src, "-o", out[1]],
                ["g++", "-no-pie", out[0], out[1], "-Wl,--unresolved-symbols=ignore-all", "-o", out[2]]):
        subprocess.run(cmd, check=True, capture_output=True, text=True)
    return out[2]


def ask(lines, flags=()):
    """One dict per line, numbers where they are numbers."""
    res = subprocess.run([_program(flags)], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True)
    plans = []
    for line in res.stdout.splitlines():
        w = line.split()
        plans.append({n: int(v) if v.lstrip("-").isdigit() else v for n, v in zip(w[::2], w[1::2])})
    assert len(plans) == len(lines)
    return plans
