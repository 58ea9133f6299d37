"""Ahead-of-time build of the C-ABI library (libcvx.so) for gfx950 with hipcc.

    python -m paper_1910_00078_amd.build

hipcc cross-compiles without a GPU.  Objects and the shared library are written next to this file
(csrc/_obj/*.o, libcvx.so); they are git-ignored but travel with the source tree.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_obj")
LIB = os.path.join(HERE, "libcvx.so")
TORCH_LIB = os.path.join(HERE, "_cvx_torch" + sysconfig.get_config_var("EXT_SUFFIX"))      # for this interpreter alone
SOURCES = ["cvx_api.cpp", "kernels_direct.hip", "kernels_igemm.hip", "kernels_stem.hip", "kernels_pointwise.hip",
           "kernels_tiled_f32.hip", "kernels_split_f32.hip", "kernels_grouped.hip"]
# Sources whose kernels are dealt over further objects (the same file with -DCVX_PART=1..n), so that a build uses the
# machine's cores: one kernel of the implicit-GEMM family takes the compiler about ten seconds.
PARTS = {"kernels_igemm.hip": 12}
HEADERS = ["cvx_internal.h", "cvx_device.h", os.path.join("..", "..", "include", "cvx.h")]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
    "-mllvm", "-amdgpu-mfma-vgpr-form",   # MFMA accumulators stay in VGPRs: no AGPR<->VGPR copies around the k-loop
    "-Wno-unused-command-line-argument",
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _extra_headers():
    return [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".h", ".inc"))]


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = False, verbose: bool = False, defines=(), lib_path: str = LIB, obj_dir: str = OBJ) -> str:
    """Compile csrc/ into the shared library.  `defines` adds -D flags (developer builds, written to
    another lib_path / obj_dir so the product library is untouched)."""
    return _build(force, verbose, list(defines), lib_path, obj_dir)


def _build(force, verbose, defines, LIB, OBJ) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()
    hdrs = _extra_headers() + [os.path.join(CSRC, HEADERS[2])]
    jobs = []
    objs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        for part in range(PARTS.get(src, 0), -1, -1):
            o = os.path.join(OBJ, os.path.splitext(src)[0] + (".%d.o" % part if part else ".o"))
            objs.append(o)
            if force or _stale(o, [s] + hdrs):
                jobs.append([hipcc, "-x", "hip", "-c", s, "-o", o] + FLAGS + ["-D" + d for d in defines]
                            + (["-DCVX_PART=%d" % part] if part else []))

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("build failed: %s\n%s" % (" ".join(cmd), r.stdout))
        if verbose and r.stdout.strip():
            print(r.stdout)

    if jobs:
        with ThreadPoolExecutor(max_workers=min(len(jobs), 8)) as ex:
            list(ex.map(run, jobs))
    if jobs or force or _stale(LIB, objs):
        tmp = LIB + ".tmp%d" % os.getpid()
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        os.replace(tmp, LIB)
    if not defines and LIB == globals()["LIB"]:
        _build_torch(force, run, hdrs)
    return LIB


def _torch_prerequisites():
    """What the native one-call function is compiled with -- torch, the C++ compiler -- or what of it is missing, as text."""
    cxx = os.environ.get("CXX", "g++")
    try:
        import torch
    except ImportError:
        return "torch"
    for header in (os.path.join(os.path.dirname(torch.__file__), "include", "ATen", "core", "Tensor.h"),
                   os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        if not os.path.exists(header):
            return header
    return (torch, cxx) if shutil.which(cxx) else cxx


def _build_torch(force, run, hdrs, obj=OBJ):
    """The native one-call function on torch tensors (host code, compiled against the installed torch, whose version it carries).  The C ABI
    library does not need it, and conv_fwd_fused goes through that alone where it is missing."""
    found = _torch_prerequisites()
    if isinstance(found, str):
        print("no native conv_fwd_fused: %s is missing" % found, file=sys.stderr)
        return
    torch, cxx = found
    src, t, stamp = os.path.join(CSRC, "cvx_torch.cpp"), os.path.dirname(torch.__file__), os.path.join(obj, "_cvx_torch.version")
    version = str(torch.__version__)
    built_for = open(stamp).read() if os.path.exists(stamp) else ""
    if not (force or built_for != version or _stale(TORCH_LIB, [src] + hdrs)):
        return
    tmp = TORCH_LIB + ".tmp%d" % os.getpid()
    run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", '-DCVX_TORCH_VERSION="%s"' % version,
         "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(), "-I" + os.path.join(t, "include"),
         "-I" + os.path.join(t, "include", "torch", "csrc", "api", "include"), "-I/opt/rocm/include",
         "-I" + sysconfig.get_paths()["include"], src, "-o", tmp, "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu",
         "-lc10", "-lc10_hip", "-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, TORCH_LIB)
    with open(stamp, "w") as f:
        f.write(version)


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
