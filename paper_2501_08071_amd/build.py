"""Compile the HIP sources into the in-tree C-ABI shared library (gfx950 only)."""
from __future__ import annotations

import hashlib
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libattn_gfx950.so")
SOURCES = ["attn_fwd_gfx950.hip", "attn_fwd_stream_gfx950.hip", "attn_fwd_rows64_gfx950.hip", "attn_api.cpp", "rowops_gfx950.hip", "rowops_api.cpp",
           "gemm_gfx950.hip", "gemm_api.cpp", "probe_gfx950.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# packed-fp32 VALU forms are switched off for all device code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument", "-Wno-inline-asm"]
# Per source.  The kernel whose wavefronts own the whole register file (one per SIMD) asks the compiler to keep matrix
# results where vector instructions can read them (the scores are consumed by the vector pipe); left to its own
# heuristic it puts every matrix result of such a kernel into accumulation registers and copies the scores out
# element by element.
SOURCE_FLAGS = {"attn_fwd_rows64_gfx950.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}
NOISE = "is not a recognized feature for this target"


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if NOISE not in l)
    if res.returncode != 0:
        raise RuntimeError(f"the compiler failed:\n{' '.join(cmd)}\n{err}")
    return err


def _whole(out: str, make):
    """make(path) writes a file; it takes the name `out` only when it is complete, so that another process never loads half of one."""
    part = f"{out[:-3]}.{os.getpid()}.part.so"
    try:
        res = make(part)
        os.replace(part, out)
        return res
    finally:
        if os.path.exists(part):
            os.remove(part)


def build_lib(extra_flags=(), out: str = LIB, verbose: bool = False, jobs: int = 4) -> str:
    """Every source to an object of its own (with its own flags), then one link."""
    tmp = tempfile.mkdtemp(prefix="attn_build_")
    try:
        def compile_one(src):
            obj = os.path.join(tmp, src + ".o")
            cmd = [HIPCC, *FLAGS, *SOURCE_FLAGS.get(src, ()), *extra_flags, "-c", "-x", "hip", os.path.join(CSRC, src), "-o", obj]
            return obj, _run(cmd)

        with ThreadPoolExecutor(max_workers=jobs) as ex:
            done = list(ex.map(compile_one, SOURCES))
        err = "".join(e for _, e in done)
        err += _whole(out, lambda part: _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *[o for o, _ in done], "-o", part]))
        if verbose and err.strip():
            print(err)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return out


BINDING_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]


def binding_path() -> str:
    """The module behind the Python entry points: torch tensors to the C ABI of LIB.  It is compiled against the insides of torch and
    Python and calls LIB by address, so its name carries all it was made from: one left from another torch, another Python or other
    sources has another name and is not loaded."""
    import sysconfig

    import torch
    h = hashlib.sha256(repr((torch.__version__, torch.version.git_version, sysconfig.get_config_var("EXT_SUFFIX"), BINDING_FLAGS)).encode())
    for f in (os.path.join(CSRC, "binding_fast.cpp"), *(os.path.join(HERE, "..", "include", x) for x in ("attn.h", "gemm.h", "rowops.h"))):
        with open(f, "rb") as fh:
            h.update(hashlib.sha256(fh.read()).digest())
    return os.path.join(HERE, f"_binding_fast_{h.hexdigest()[:16]}.so")


def build_binding(out: str | None = None, verbose: bool = False) -> str:
    """That module (host code only, against torch's headers)."""
    import sysconfig

    import torch
    out = out or binding_path()
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include",
           sysconfig.get_paths()["include"]]
    # (no path to torch's libraries is recorded: the process that imports the module has loaded them)
    err = _whole(out, lambda part: _run([os.environ.get("CXX", "g++"), *BINDING_FLAGS, *[a for d in inc for a in ("-isystem", d)],
                                         os.path.join(CSRC, "binding_fast.cpp"), "-L" + os.path.join(t, "lib"), "-ltorch_python",
                                         "-ltorch_cpu", "-lc10", "-lc10_hip", "-o", part]))
    if verbose and err.strip():
        print(err)
    return out


if __name__ == "__main__":
    print(build_lib(verbose=True), build_binding(verbose=True))
