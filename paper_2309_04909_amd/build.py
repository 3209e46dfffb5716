"""Build libbicop.so (the C ABI of include/bicop.h) for gfx950 with hipcc, and
the Python binding's native argument marshalling (_fastcall.so) with g++.

Every .hip file under csrc/ is compiled to an object in _build/ (in parallel),
then the objects are linked into paper_2309_04909_amd/libbicop.so.  The
packed-fp32 target feature is switched off for all device code.

    python -m paper_2309_04909_amd.build [-j N] [--asm]
"""

import argparse
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbicop.so")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc")
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # let '#pragma unroll' fully unroll the 33-slot loops of l_x = 32 (else
    # the slot arrays are indexed dynamically, through scratch)
    "-mllvm", "-pragma-unroll-threshold=200000",
]


FASTCALL = os.path.join(HERE, "_fastcall.so")


def build_fastcall(out: str = FASTCALL) -> str:
    """Compile csrc/fastcall.cpp, the binding's native argument marshalling (host code against torch's headers)."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    tmp = out + ".tmp"
    rc, log = _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    f"-I{root}/include", f"-I{root}/include/torch/csrc/api/include", "-I/opt/rocm/include",
                    f"-I{sysconfig.get_paths()['include']}", os.path.join(CSRC, "fastcall.cpp"), "-o", tmp,
                    f"-L{root}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", f"-Wl,-rpath,{root}/lib"])
    if rc != 0:
        raise RuntimeError("the _fastcall module failed to build:\n" + log)
    os.replace(tmp, out)
    return out


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature; that warning is harmless
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip())
    return r.returncode, out


def build(jobs: int | None = None, verbose: bool = False, asm: bool = False, extra_flags=(), out: str = LIB,
          build_dir: str = BUILD) -> str:
    """Compile every HIP source and link libbicop.so (or `out`).  Returns the library path."""
    os.makedirs(build_dir, exist_ok=True)
    # the replicated-sharing and record instantiations compile longest: first
    srcs = sorted(sources(), key=lambda s: not os.path.basename(s).startswith(("k_rss", "k_pre")))
    jobs = jobs or min(len(srcs), max(1, min(16, os.cpu_count() or 4)))

    def compile_one(src):
        obj = os.path.join(build_dir, os.path.basename(src).replace(".hip", ".o"))
        rc, log = _run([HIPCC, *FLAGS, *extra_flags, "-c", src, "-o", obj])
        if rc == 0 and asm:
            s = os.path.join(build_dir, os.path.basename(src).replace(".hip", ".s"))
            _run([HIPCC, *FLAGS, *extra_flags, "--cuda-device-only", "-S", src, "-o", s])
        return src, obj, rc, log

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(compile_one, srcs))
    errors = [(s, o) for s, _, rc, o in results if rc != 0]
    for s, _, rc, log in results:
        if log and (verbose or rc != 0):
            print(f"--- {os.path.basename(s)}\n{log}", file=sys.stderr)
    if errors:
        raise RuntimeError("hipcc failed for: " + ", ".join(os.path.basename(s) for s, _ in errors))
    tmp = out + ".tmp"
    rc, log = _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *[o for _, o, _, _ in results]])
    if rc != 0:
        raise RuntimeError("link failed:\n" + log)
    os.replace(tmp, out)
    if out == LIB:
        build_fastcall()
    return out


def clean():
    shutil.rmtree(BUILD, ignore_errors=True)
    for path in (LIB, FASTCALL):
        if os.path.exists(path):
            os.remove(path)


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("-j", type=int, default=None)
    ap.add_argument("-v", action="store_true")
    ap.add_argument("--asm", action="store_true", help="also write device assembly next to the objects")
    a = ap.parse_args()
    print(build(a.j, a.v, a.asm))
