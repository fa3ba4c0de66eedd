"""Build libef.so (HIP kernels + C ABI) and libef_bench.so (the bandwidth probes bench.py runs
beside it) for gfx950 with hipcc, and the Python binding's native calls (ef_binding.cpp) with the C++ compiler, in-tree."""
import hashlib
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libef.so")
BENCH_LIB = os.path.join(HERE, "libef_bench.so")
BINDING = os.path.join(HERE, "_ef_binding.so")
# library -> (source, everything it is built from)
TARGETS = {
    LIB: (os.path.join(CSRC, "ef_api.hip"),
          [os.path.join(CSRC, h) for h in ("ef_device.h", "ef_tile.h", "ef_worker.h", "ef_server.h", "ef_finish.h", "ef_end.h",
                                           "ef_quality.h", "ef_small.h", "ef_layout.h")] +
          [os.path.join(ROOT, "include", h) for h in ("ef.h", "ef_debug.h")]),
    BENCH_LIB: (os.path.join(CSRC, "ef_bench.hip"),
                [os.path.join(CSRC, h) for h in ("ef_tile.h", "ef_layout.h", "ef_probe.h")] +
                [os.path.join(ROOT, "include", h) for h in ("ef.h", "ef_bench.h")]),
    BINDING: (os.path.join(CSRC, "ef_binding.cpp"), [os.path.join(ROOT, "include", "ef.h")]),
}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: Algorithm 4's fp32 operations round one by one (no FMA), so
#   sign bits are reproducible against a plain CPU evaluation.
# correctly rounded divide: the server's division by M is an IEEE division.
# packed-fp32 ops are switched off for the device pass.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
]


def binding_built_for():
    """What the binding has compiled in and its loader compares: the torch whose tensors it takes, and its sources (their
    contents: a copied tree's times say nothing)."""
    import torch
    digest = hashlib.sha256()
    src, deps = TARGETS[BINDING]
    for name in [src] + deps:
        with open(name, "rb") as f:
            digest.update(f.read())
    return "torch %s, sources %s" % (torch.__version__, digest.hexdigest()[:16])


def binding_command():
    """The binding sees tensors, so it is built against the torch that is installed; it has no device code."""
    import torch
    at = torch.__path__[0]
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DEF_BUILT_FOR="%s"' % binding_built_for(), "-I", os.path.join(ROOT, "include"),
             "-isystem", os.path.join(rocm, "include"), "-isystem", os.path.join(at, "include"),
             "-isystem", os.path.join(at, "include", "torch", "csrc", "api", "include"),
             "-isystem", sysconfig.get_paths()["include"]],
            ["-L", os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"])


def stale(lib=LIB):
    if not os.path.exists(lib):
        return True
    src, deps = TARGETS[lib]
    t = os.path.getmtime(lib)
    return any(os.path.exists(f) and os.path.getmtime(f) > t for f in [src] + deps)


def build(force=True, verbose=False, lib=None):
    """Compile the libraries (one of them if `lib` is given); with force=False only those whose
    sources are newer than the built file."""
    for target in ([lib] if lib else list(TARGETS)):
        if not force and not stale(target):
            continue
        tmp = target + ".tmp%d" % os.getpid()
        if target == BINDING:
            first, last = binding_command()
            cmd = first + ["-o", tmp, TARGETS[target][0]] + last
        else:
            cmd = [HIPCC] + FLAGS + ["-o", tmp, TARGETS[target][0]]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        os.replace(tmp, target)
    return LIB


if __name__ == "__main__":
    build(force=True, verbose=True)
    print("built", LIB, BENCH_LIB)
    sys.exit(0)
