"""Build libhistfit.so in-tree with hipcc for gfx950, and the binding's native
marshalling module _fastcall.so (host code against torch's headers).

Every translation unit under csrc/ is compiled in parallel to an object in
_build/, then linked into paper_2203_06139_amd/libhistfit.so.  Always
recompiles when called (the build check must exercise the compiler).
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhistfit.so")
BINDING = os.path.join(HERE, "_fastcall.so")
ARCH = os.environ.get("HF_OFFLOAD_ARCH", "gfx950")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
COMMON = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # no packed-FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument",
]


def _sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


# Kernels with more literals than scalar registers.  The compiler hoists what
# does not fit into vector registers before the outermost loop and holds or
# spills it there; materialised where it is used, the average over explicit
# edges takes 154 registers instead of 180 (4e6 bins 43.8 -> 38.9 us) and a
# fit of three Gaussians spills 15 instead of 98 (512 fits 297 -> 288 us).  The
# fits of one Gaussian have no spills and lose 3% (74.4 -> 76.7 us); the plain
# starts, with two exponentials in several loops, take 76 registers instead of
# 128 and two spilled (4096 of 64..512 bins 89 -> 71 us, 1e7 bins 24.3 -> 26.0
# ms).  The other kernels neither gain nor lose.
NO_HOIST = ("fit_ng2", "fit_ng3", "fit_ng4", "nll1d_avg_", "mlp.hip")


def _compile(src: str, build_dir: str = BUILD, extra=()) -> str:
    obj = os.path.join(build_dir, os.path.basename(src) + ".o")
    cmd = [HIPCC, *COMMON, *extra, "-c", src, "-o", obj]
    if os.path.basename(src).startswith(NO_HOIST):
        cmd[1:1] = ["-mllvm", "-disable-machine-licm"]
    if src.endswith(".cpp"):
        cmd[1:1] = ["-x", "hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s%s" % (src, r.stdout, r.stderr))
    noisy = [ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if noisy:
        sys.stderr.write("\n".join(noisy) + "\n")
    return obj


def build(jobs: int | None = None, out: str = LIB, build_dir: str = BUILD, extra=()) -> str:
    """Compile and link; `extra` hipcc flags (e.g. -DHF_CHUNK=16) and `out`
    allow building variants of the library side by side."""
    os.makedirs(build_dir, exist_ok=True)
    srcs = _sources()
    jobs = jobs or min(len(srcs), max(1, min(16, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, build_dir, extra), srcs))
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s%s" % (r.stdout, r.stderr))
    os.replace(tmp, out)
    if out == LIB:
        build_binding()
    return out


def build_binding(out: str = BINDING) -> str:
    import sysconfig

    from torch.utils import cpp_extension
    tmp = out + ".tmp%d" % os.getpid()
    libs = cpp_extension.library_paths(device_type="cuda")
    cmd = [HIPCC, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           *("-isystem" + d for d in cpp_extension.include_paths(device_type="cuda")),
           "-I" + sysconfig.get_path("include"), os.path.join(HERE, "binding", "fastcall.cpp"),
           "-o", tmp, *("-L" + d for d in libs), *("-Wl,-rpath," + d for d in libs),
           "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building %s failed:\n%s%s" % (out, r.stdout, r.stderr))
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build())
