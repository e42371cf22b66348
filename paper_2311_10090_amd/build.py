"""Build libmpe.so (HIP, gfx950) and the binding's native host path _mpe_call.so in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmpe.so")
CALL = os.path.join(HERE, "_mpe_call.so")
SOURCES = ["mpe_api.hip", "mpe_env_kernels.hip", "mpe_env_agents.hip", "mpe_policy_wide.hip", "mpe_policy_f32.hip", "mpe_policy_dispatch.hip", "mpe_tag.hip", "mpe_policy_gru.hip", "mpe_gru_waves.hip",
           "mpe_small_spread.hip", "mpe_small_spread_ac.hip", "mpe_small_tag.hip", "mpe_small_tag_ac.hip", "mpe_waves_spread.hip",
           "mpe_waves_tag.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def compile_call(hipcc: str, obj: str) -> str:
    """The Python extension of the binding's hot calls: host code only, against torch's headers."""
    from torch.utils.cpp_extension import include_paths
    import torch
    inc = [a for d in (*include_paths(), sysconfig.get_paths()["include"]) for a in ("-I", d)]
    cmd = [hipcc, "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-w", *inc, "-I", "/opt/rocm/include",
           "-c", os.path.join(CSRC, "mpe_call.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compilation of mpe_call.cpp failed:\n" + r.stderr)
    return obj


def link_call(hipcc: str, obj: str) -> None:
    """Link it against the libmpe.so beside it (found through $ORIGIN) and the libraries that torch has loaded."""
    import torch
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = CALL + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc, "-shared", "-fPIC", "-o", tmp, obj, "-L", HERE, "-l:libmpe.so", "-Wl,-rpath,$ORIGIN", "-L", torch_lib,
                        "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of _mpe_call.so failed:\n" + r.stderr)
    os.replace(tmp, CALL)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source and link libmpe.so.  force=False skips when up to date."""
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "mpe.h")]
    if not force and all(os.path.exists(f) and os.path.getmtime(f) >= os.path.getmtime(d) for f in (LIB, CALL) for d in deps):
        return LIB
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        call_obj = ex.submit(compile_call, hipcc, os.path.join(objdir, "mpe_call.o"))
        objs = list(ex.map(compile_one, SOURCES))
        call_obj = call_obj.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    link_call(hipcc, call_obj)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
