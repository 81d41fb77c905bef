"""Build liblonggen_attn.so from csrc/*.hip with hipcc for gfx950 (cross-compiles without a GPU) and the extension
module _lg_bind, the tensor side of the binding, from csrc/lg_bind.cpp with the C++ compiler that hipcc drives (it needs
the headers of Python and torch; without the module the binding goes through ctypes).

    python -m paper_2410_01485_amd.build
"""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblonggen_attn.so")
# (the interpreter's tag in the name: another one's build is not found instead of being loaded)
BIND_NAME = "_lg_bind" + sysconfig.get_config_var("EXT_SUFFIX")
BIND_SRC = os.path.join(CSRC, "lg_bind.cpp")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.path.join(os.path.dirname(HIPCC), "..", "lib", "llvm", "bin", "clang++")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed-fp32 instructions are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]

# flags of one file: the forward's tile loop runs up to 5 % slower where its code happens to start off a 64-byte boundary
# (the backward kernels' unrolled steps do not: within 0.3 %)
FILE_FLAGS = {"lg_fwd_bf16.hip": ["-falign-loops=64"], "lg_fwd_list_bf16.hip": ["-falign-loops=64"]}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


# host code (argument checks, host build of the tile scheduler, launch set-up) under AddressSanitizer and
# UndefinedBehaviorSanitizer; the device code is built as usual
SAN_COMPILE = ["-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
               "-Xarch_host", "-fno-sanitize-recover=undefined"]
SAN_LINK = ["-fno-gpu-sanitize", "-fsanitize=address", "-fsanitize=undefined", "-shared-libsan"]
# (no check of dynamic types: it would need the type information of torch's own libraries)
SAN_BIND = ["-O1", "-g", "-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize=vptr",
            "-fno-sanitize-recover=undefined", "-shared-libsan"]


def start_bind(out, sanitize=False):
    """Start compiling the extension module (host code only; torch's C++ headers, no library of ours linked)."""
    import torch
    from torch.utils import cpp_extension
    cmd = [CXX if os.path.exists(CXX) else "g++"] + (SAN_BIND if sanitize else ["-O2"])
    cmd += ["-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            BIND_SRC, "-o", out, "-I", sysconfig.get_paths()["include"]]
    for d in cpp_extension.include_paths():
        cmd += ["-isystem", d]
    for d in cpp_extension.library_paths():
        cmd += ["-L", d]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)


def build(verbose=True, jobs=8, sanitize_host=False, out=None):
    """Compile every translation unit (in parallel) and link the shared library; the extension module next to it.

    sanitize_host: build a second library (path `out`) whose HOST code, and the module's, runs under ASan + UBSan; a
    process that loads it must have the clang ASan runtime preloaded (tests/test_sanitized_host.py does that).
    If only the module fails, the library is in place before this raises."""
    lib = out or LIB
    objdir = os.path.join(HERE, "_build_san" if sanitize_host else "_build")
    os.makedirs(objdir, exist_ok=True)
    flags = FLAGS + (SAN_COMPILE if sanitize_host else [])
    bind = os.path.join(os.path.dirname(os.path.abspath(lib)), BIND_NAME)
    bind_tmp = bind + ".tmp%d" % os.getpid()
    try:
        bind_proc, bind_out = start_bind(bind_tmp, sanitize_host), ""
    except (ImportError, OSError) as e:  # no torch, no compiler
        bind_proc, bind_out = None, str(e)
    procs = []
    objs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        cmd = [HIPCC] + flags + FILE_FLAGS.get(os.path.basename(src), []) + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            procs[0][1].wait()
    failed = False
    for src, p in procs:
        out = p.communicate()[0].decode()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            print("FAILED: %s\n%s" % (src, out), file=sys.stderr)
        elif verbose and out.strip():
            print(out)
    if bind_proc is not None:
        bind_out = bind_proc.communicate()[0].decode()
    if failed:
        raise RuntimeError("compilation failed")
    tmp = lib + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + (SAN_LINK if sanitize_host else []) + ["-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, lib)
    if bind_proc is None or bind_proc.returncode != 0:
        raise RuntimeError("%s is built, the extension module is not (calls go through ctypes):\n%s" % (lib, bind_out))
    os.replace(bind_tmp, bind)
    untagged = os.path.join(os.path.dirname(bind), "_lg_bind.so")  # of an earlier build
    if os.path.exists(untagged):
        os.remove(untagged)
    return lib


if __name__ == "__main__":
    print(build())
