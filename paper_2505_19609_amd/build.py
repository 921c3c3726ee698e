"""Build libskrull_attn.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from importlib.util import find_spec

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libskrull_attn.so")
AUTOGRAD = os.path.join(HERE, "_autograd.so")
SOURCES = ["api.hip", "plan.hip", "fwd.hip", "bwd.hip", "probe.hip", "dacp.cpp", "gds.cpp"]
# packed fp32 VALU ops are switched off for all device code
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
         "-I" + CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-inline-asm"]
# further compiler flags for experiments (space separated), e.g. SKRULL_EXTRA_FLAGS="-mllvm -align-loops=64"
FLAGS += os.environ.get("SKRULL_EXTRA_FLAGS", "").split()


def _compile(src: str) -> str:
    """Compile one source.  The compiler's per-kernel resource remarks are
    parsed and the build fails if any kernel uses scratch memory: register
    spills cost bandwidth in the hot loops, and a partially spilled MFMA
    operand tuple has been seen to be reloaded incompletely by this compiler
    (wrong results), so spilling kernels are not allowed in the library."""
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
    r = subprocess.run(["hipcc", *FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(CSRC, src), "-o", obj], stderr=subprocess.PIPE, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    name, report = None, []
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name:
            report.append((name, int(m.group(1))))
            if int(m.group(1)) != 0:
                raise RuntimeError(f"{src}: kernel {name} spills {m.group(1)} bytes/lane to scratch")
    if not os.environ.get("SKRULL_QUIET"):
        for line in r.stderr.splitlines():
            if "error" in line or ("warning" in line and "packed-fp32" not in line):
                print(line)
    return obj


def _torch_dir():
    """Where torch is installed, or None where it, or the compiler for its interface, is not: the library needs neither."""
    spec = find_spec("torch")
    return os.path.dirname(spec.origin) if spec and shutil.which("g++") else None


def _compile_autograd(torch_dir: str) -> str:
    """Compile the native side of autograd.py against torch's C++ interface (host code only)."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    obj = os.path.join(CSRC, "autograd.o")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(torch_dir, "include"),
                    "-I" + os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
                    "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(rocm, "include"),
                    "-c", os.path.join(CSRC, "autograd.cpp"), "-o", obj], check=True)
    return obj


def _link_autograd(torch_dir: str, obj: str) -> None:
    libs = os.path.join(torch_dir, "lib")
    subprocess.run(["g++", "-shared", "-fPIC", "-o", AUTOGRAD, obj, "-L" + libs, "-ltorch_python", "-ltorch", "-ltorch_cpu",
                    "-lc10", "-lc10_hip", "-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"], check=True)


def build_library(jobs: int = 4) -> str:
    """Compile every HIP source and link the shared library, and the extension module beside it where that can be built; returns the library's path."""
    torch_dir = _torch_dir()
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        autograd = ex.submit(_compile_autograd, torch_dir) if torch_dir else None
        objs = list(ex.map(_compile, SOURCES))
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
        if autograd:
            _link_autograd(torch_dir, autograd.result())
    return LIB


if __name__ == "__main__":
    print(build_library())
