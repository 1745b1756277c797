"""Build libspecfp8.so (HIP for gfx950) and its torch binding in-tree.

    python -m paper_2606_18502_amd.build [-v]

(`python paper_2606_18502_amd/build.py` where torch is not installed: the
library is a plain C ABI and is built without it.)

Every HIP source is compiled with hipcc for gfx950 only, without packed-fp32
instructions (-packed-fp32-ops) and without floating-point contraction
(-ffp-contract=off keeps the documented rounding of every scale, exp and
epilogue step); the host-only validation unit is plain C++.  The objects are
linked into paper_2606_18502_amd/libspecfp8.so, next to this file, and the
torch-facing argument marshalling (torch_bind.cpp, against the installed torch)
into _torch_bind.so beside it.
"""

from __future__ import annotations

import argparse
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libspecfp8.so")
ARCH = "gfx950"

# longest compiles first: they run in parallel
HIP_SOURCES = ["gemm_k0_1.hip", "gemm_k2_3.hip", "gemm_k4_6.hip", "gemm_k7_12.hip", "accept.hip", "quantize.hip",
               "gemm.hip", "kvcache.hip", "tree_mask.hip", "api.cpp", "plan.cpp"]
HOST_SOURCES = ["validate.cpp"]
BIND_SOURCE = "torch_bind.cpp"
BIND = os.path.join(HERE, "_torch_bind.so")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def _hip_flags():
    return [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", f"-I{os.path.join(ROOT, 'include')}"]


def _torch():
    """The installed torch, or None: only the binding needs it."""
    try:
        import torch
    except ImportError:
        return None
    return torch


def _bind_compile(obj: str, torch):
    torch_dir = os.path.dirname(torch.__file__)
    inc = [os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}"]
            + [x for d in inc for x in ("-isystem", d)] + ["-c", os.path.join(CSRC, BIND_SOURCE), "-o", obj])


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("build step failed:\n" + " ".join(cmd) + "\n" + res.stdout + res.stderr)
    return res


def build(verbose: bool = False) -> str:
    """Compile every source and link libspecfp8.so, then the torch binding where
    torch is installed; returns the library path."""
    os.makedirs(BUILD, exist_ok=True)
    cc = hipcc()
    jobs = []
    objs = []
    for src in HIP_SOURCES:
        obj = os.path.join(BUILD, src.replace(".", "_") + ".o")
        lang = ["-x", "hip"] if src.endswith(".cpp") else []
        jobs.append([cc] + lang + _hip_flags() + ["-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    for src in HOST_SOURCES:
        obj = os.path.join(BUILD, src.replace(".", "_") + ".o")
        jobs.append(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", f"-I{os.path.join(ROOT, 'include')}",
                     "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    torch = _torch()
    bind_obj = os.path.join(BUILD, BIND_SOURCE.replace(".", "_") + ".o")
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        bind = ex.submit(_run, _bind_compile(bind_obj, torch)) if torch else None
        for res in ex.map(_run, jobs):
            if verbose and (res.stdout or res.stderr):
                print(res.stdout + res.stderr)
    tmp = LIB + ".tmp"
    _run([cc, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-Wl,-soname,libspecfp8.so", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    if bind is None:
        print("torch is not installed: the torch binding is not built", file=sys.stderr)
        return LIB
    res = bind.result()
    if verbose and (res.stdout or res.stderr):
        print(res.stdout + res.stderr)
    # torch's own libraries are loaded by `import torch` before the binding is
    tmp = BIND + ".tmp"
    _run(["g++", "-shared", "-o", tmp, bind_obj, f"-L{HERE}", "-lspecfp8", "-Wl,-rpath,$ORIGIN",
          f"-L{os.path.join(os.path.dirname(torch.__file__), 'lib')}", "-lc10", "-lc10_hip", "-ltorch_cpu",
          "-ltorch_python"])
    os.replace(tmp, BIND)
    return LIB


def main(argv=None) -> int:
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("-v", "--verbose", action="store_true")
    args = ap.parse_args(argv)
    print(build(verbose=args.verbose))
    return 0


if __name__ == "__main__":
    sys.exit(main())
