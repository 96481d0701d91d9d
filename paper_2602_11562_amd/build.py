"""Build liblaser.so (HIP kernels + C ABI) for gfx950 with hipcc and laser_fast.so (the binding's native part) with g++, in-tree.

    python -m paper_2602_11562_amd.build

Cross-compiles without a GPU. The shared library is written next to this file so it
travels with the source tree; nothing is installed.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblaser.so")
FAST = os.path.join(HERE, "laser_fast.so")
OBJDIR = os.path.join(HERE, "_build")

SOURCES = ["laser_api.hip", "sta_generic.hip", "sta_f32.hip", "sta_mfma.hip", "sta_ring.hip", "sta_stream.hip", "sta_few.hip", "gsta_generic.hip",
           "gsta_tiled.hip", "gsta_one.hip", "gsta_project.hip", "fused_forward.hip", "multires.hip", "segment_ffn.hip", "ffn_gsta.hip", "project.hip", "sta_backward.hip", "sta_backward_mfma.hip", "gsta_backward.hip", "gsta_backward_tile.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _compile(src: str, extra=()) -> str:
    obj = os.path.join(OBJDIR, ("tuning_" if extra else "") + src.replace(".hip", ".o"))
    cmd = [_hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(jobs: int = 6, tuning: bool = False, out: str = LIB) -> str:
    """Compile every HIP source and link liblaser.so, and the binding's native part beside it. Always rebuilds. `tuning` builds the variant whose launch
    shapes can be overridden through environment variables (parameter sweeps only; never the shipped library)."""
    os.makedirs(OBJDIR, exist_ok=True)
    extra = ("-DLASER_TUNING",) if tuning else ()
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda src: _compile(src, extra), SOURCES))
    tmp = out + ".tmp"
    r = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, out)
    if out == LIB:
        build_fast_binding_or_do_without()
    return out


def build_fast_binding_or_do_without() -> None:
    """The binding's native part needs g++ and torch's headers. Without them the binding marshals every call in Python, and one built
    earlier, for a library that is gone, must not stay."""
    try:
        build_fast_binding()
    except (ImportError, OSError, RuntimeError) as e:
        if os.path.exists(FAST):
            os.remove(FAST)
        warnings.warn(f"laser_fast.so was not built, laser_forward is marshalled in Python: {e}")


def build_fast_binding(out: str = FAST) -> str:
    """Compile the binding's native part (csrc/binding_fast.cpp) against the headers of the installed torch."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths

    from .binding import torch_stamp
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = out + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DLASER_TORCH_STAMP="{torch_stamp()}"',
           *["-I" + d for d in include_paths()], "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "binding_fast.cpp"),
           "-L" + lib, "-lc10", "-ltorch_cpu", "-ltorch_python", "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on binding_fast.cpp:\n" + r.stderr[-4000:])
    os.replace(tmp, out)
    return out


def build_host_check(out: str) -> str:
    """Build tests/abi_host_check.cpp into an executable whose host code of laser_api.hip (argument validation,
    kernel selection, size arithmetic) is instrumented with AddressSanitizer and UndefinedBehaviorSanitizer; the
    kernel launchers are the objects of the last build_library() (device code is never sanitized, and nothing
    here reaches a launch). No GPU needed to build or run it."""
    os.makedirs(OBJDIR, exist_ok=True)
    objs = [os.path.join(OBJDIR, src.replace(".hip", ".o")) for src in SOURCES if src != "laser_api.hip"]
    if not all(os.path.exists(o) for o in objs):
        build_library()
    san = ["-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=undefined"]
    api_obj = os.path.join(OBJDIR, "san_laser_api.o")
    arch_host = [x for f in san for x in ("-Xarch_host", f)]
    steps = [
        [_hipcc(), *[f for f in HIPCC_FLAGS if f != "-O3"], "-O1", "-g", *arch_host, "-c",
         os.path.join(CSRC, "laser_api.hip"), "-o", api_obj],
        ["/opt/rocm/lib/llvm/bin/clang++", "-O1", "-g", *san, "-I" + os.path.join(ROOT, "include"), "-c",
         os.path.join(ROOT, "tests", "abi_host_check.cpp"), "-o", os.path.join(OBJDIR, "abi_host_check.o")],
        [_hipcc(), "--offload-arch=gfx950", "-fno-gpu-sanitize", *san, os.path.join(OBJDIR, "abi_host_check.o"),
         api_obj, *objs, "-o", out],
    ]
    for cmd in steps:
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("host check build failed:\n" + " ".join(cmd) + "\n" + r.stderr[-4000:])
    return out


def build_launch_recorder(out: str) -> str:
    """Build a library of the same entry points whose launches are recorded instead of made (tests/launch_recorder.cpp): the
    host halves of the sources, with the overrides of a tuning build. No GPU needed to build or use it."""
    os.makedirs(OBJDIR, exist_ok=True)
    no_kernels = os.path.join(OBJDIR, "no_kernels.bin")      # what stands in the place of the device code
    with open(no_kernels, "wb") as f:
        f.write(b"none")
    flags = [f for f in HIPCC_FLAGS if not f.startswith("--offload-arch")] + [
        "-O1", "-DLASER_TUNING", "-Xclang", "-fcuda-include-gpubinary", "-Xclang", no_kernels]

    def compile_one(src: str) -> str:
        obj = os.path.join(OBJDIR, "launches_" + os.path.basename(src).rsplit(".", 1)[0] + ".o")
        cmd = [_hipcc(), "-x", "hip", "--offload-host-only", *flags, "-c", src, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"host half of {src}:\n" + r.stderr[-4000:])
        return obj

    srcs = [os.path.join(CSRC, s) for s in SOURCES] + [os.path.join(ROOT, "tests", "launch_recorder.cpp")]
    with ThreadPoolExecutor(max_workers=6) as ex:
        objs = list(ex.map(compile_one, srcs))
    # (bound to its own functions, whatever runtime the process has loaded)
    r = subprocess.run(["/opt/rocm/lib/llvm/bin/clang++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", out, *objs, "-ldl"],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("launch recorder link failed:\n" + r.stderr[-4000:])
    return out


if __name__ == "__main__":
    if len(sys.argv) > 2 and sys.argv[1] == "--tuning":      # python -m paper_2602_11562_amd.build --tuning OUT.so
        print(build_library(tuning=True, out=os.path.abspath(sys.argv[2])))
    else:
        print(build_library())
