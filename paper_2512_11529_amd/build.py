"""Builds libgr.so (the C-ABI HIP library) for gfx950 with hipcc and gr_bind.so (argument marshalling of the Python binding) with g++,
in-tree."""
import os
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libgr.so")
BIND_PATH = os.path.join(PKG_DIR, "gr_bind.so")
SOURCES = ["gr_api.hip", "gr_mask.hip", "gr_select.hip", "gr_attn.hip", "gr_reorder.hip", "gr_diag.hip"]
# packed-fp32 VALU forms are disabled on purpose (hipcc would otherwise form them from scalar code)
COMMON = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Wno-inline-asm", "-Xclang", "-target-feature", "-Xclang",
          "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
PER_FILE = {"gr_select.hip": ["-ffp-contract=off"]}


def _bind_command():
    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    dirs = [*include_paths(), sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *[a for d in dirs for a in ("-isystem", d)], os.path.join(CSRC, "gr_bind.cpp"), "-o", BIND_PATH, "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_lib(verbose: bool = False) -> str:
    """Compile every HIP source and link libgr.so, and compile gr_bind.so.  Always recompiles."""
    objs = []
    bind = _bind_command()
    procs = [("gr_bind.cpp", subprocess.Popen(bind, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))]
    if verbose:
        print(" ".join(bind), flush=True)
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc", *COMMON, *PER_FILE.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
        if pr.returncode != 0:
            failed = True
            print(f"--- {src} failed\n" + "\n".join(lines), file=sys.stderr)
        elif verbose and lines:
            print("\n".join(lines))
    if failed:
        raise RuntimeError("compilation failed")
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL if not verbose else None, stderr=subprocess.STDOUT if not verbose else None)
    return LIB_PATH


if __name__ == "__main__":
    print(build_lib(verbose=True))
