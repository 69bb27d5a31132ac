"""Build libmsda.so (the HIP kernels and the C ABI) in-tree with hipcc for gfx950,
and _msda_torch.so (the PyTorch side of the single call) with g++.

    python -m paper_2601_10819_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libmsda.so")
SOURCES = [os.path.join(CSRC, f) for f in
           ("msda_fwd.hip", "msda_bwd.hip", "msda_tiles.hip", "msda_sort.hip", "msda_batch.hip",
            "msda_util.hip", "msda_vis.hip", "msda_softmax.hip", "msda_noalloc.hip",
            "msda_api.cpp")]
HEADERS = [os.path.join(CSRC, "msda_internal.h"), os.path.join(CSRC, "msda_common.h"),
           os.path.join(CSRC, "msda_rows.h"), os.path.join(CSRC, "msda_grads.h"),
           os.path.join(ROOT, "include", "msda.h")]

TORCH_SOURCE = os.path.join(CSRC, "msda_torch.cpp")
TORCH_LIB = os.path.join(PKG, "_msda_torch.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    f"--offload-arch={ARCH}",
    # hardware float atomics (no compare-and-swap loops) for the grad_feat scatter
    "-munsafe-fp-atomics",
    # no packed-FP32 instructions: write plain scalar float code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"),
]


def torch_command(out: str):
    """The g++ line of _msda_torch.so (host code only)."""
    import sysconfig
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", os.path.join(ROOT, "include"), "-isystem", inc,
            "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
            "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
            TORCH_SOURCE, "-o", out, "-L", lib, "-lc10", "-lc10_hip", "-ltorch_cpu",
            "-ltorch_python", f"-Wl,-rpath,{lib}"]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l and l.strip())
    return res.returncode, out


def _replace(built: str, target: str):
    """target replaced by the built file at once (also across file systems);
    a copy that fails leaves nothing beside it."""
    import shutil
    tmp = target + ".tmp%d" % os.getpid()
    try:
        shutil.copyfile(built, tmp)
        shutil.copymode(built, tmp)
        os.replace(tmp, target)
    finally:
        if os.path.exists(tmp):
            os.unlink(tmp)


def build(verbose: bool = False) -> str:
    """Compile every HIP source into libmsda.so (always recompiles): one
    object per source, compiled in parallel, then one link; and
    _msda_torch.so beside it."""
    import shutil
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    tmpdir = tempfile.mkdtemp(prefix="msda_build_")
    try:
        objs = [os.path.join(tmpdir, os.path.basename(src) + ".o") for src in SOURCES]
        cflags = [f for f in FLAGS if f != "-shared"]
        cmds = [[HIPCC] + cflags + ["-c", src, "-o", obj] for src, obj in zip(SOURCES, objs)]
        torch_obj = os.path.join(tmpdir, os.path.basename(TORCH_LIB))
        cmds.append(torch_command(torch_obj))
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        jobs = max(1, min(len(cmds), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4))))
        with ThreadPoolExecutor(jobs) as pool:
            results = list(pool.map(_run, cmds))
        for (rc, out), src in zip(results, SOURCES + [TORCH_SOURCE]):
            if rc != 0:
                raise RuntimeError(f"the compiler failed on {os.path.basename(src)} ({rc}):\n{out}")
            if verbose and out:
                print(out)
        lib_obj = os.path.join(tmpdir, os.path.basename(LIB))
        link = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}"] + objs + ["-o", lib_obj]
        if verbose:
            print(" ".join(link), flush=True)
        rc, out = _run(link)
        if rc != 0:
            raise RuntimeError(f"link failed ({rc}):\n{out}")
        for obj, target in ((lib_obj, LIB), (torch_obj, TORCH_LIB)):
            _replace(obj, target)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


def is_stale() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(TORCH_LIB)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(TORCH_LIB))
    return any(os.path.getmtime(s) > t for s in SOURCES + HEADERS + [TORCH_SOURCE])


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
