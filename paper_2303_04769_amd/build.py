"""Builds libsmall_hip.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
import os
import subprocess
import sysconfig
import threading

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsmall_hip.so")
# The single-layer calls from Python, in front of the ctypes binding. It reads torch's tensors through its C++ headers: the name says
# for which Python and which torch it was built, so that no other one loads it.
FASTCALL = os.path.join(HERE, f"_fastcall.{sysconfig.get_config_var('SOABI')}.torch-{torch.__version__}.so")
PROBE_LIB = os.path.join(HERE, "libsmall_probe.so")       # the benchmark's matrix-rate probe, a library of its own
SOURCES = ["elementwise.hip", "window.hip", "window_rows.hip", "window_dpp.hip", "window_dpp_u8.hip", "pool_dpp_u8.hip", "quant_ends.hip", "pool_dpp.hip", "conv.hip", "conv_same.hip", "conv_pw.hip", "conv_split.hip", "conv_split3.hip", "conv_split3_wide.hip", "dwpw.hip", "dwpw_run.hip", "dwpw_team.hip", "chain.hip", "resident.hip", "quant.hip", "conv_u8_tile.hip", "conv_u8_pw.hip", "layout_u8.hip", "resident_u8.hip", "table2.hip", "small_api.hip"]
# packed fp32 VALU ops are switched off for every device translation unit
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc", "-Wall", "-Wno-unused-function", "-Wno-pass-failed",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# SMALL_RES_TIMING=1 in the environment builds the image-resident run with cycle stamps per layer and wave (read back by
# `bench.py --resident-timing`); the stamps cost a few store instructions per layer, so the default build has none.
if os.environ.get("SMALL_RES_TIMING"):
    FLAGS = FLAGS + ["-DSMALL_RES_TIMING"]


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def build_fastcall(force=False):
    """Host code only, against torch's headers (its libraries are loaded before it)."""
    src = os.path.join(CSRC, "fastcall.cpp")
    if not (force or _stale(FASTCALL, [src, os.path.join(HERE, "..", "include", "small.h")])):
        return
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    # (written beside its place and moved there whole: another process may load it, or build it too, at the same time)
    part = f"{FASTCALL[:-3]}.{os.getpid()}-{threading.get_ident()}.part.so"
    cmd += [a for d in include for a in ("-isystem", d)] + [src, "-o", part, "-L" + os.path.join(root, "lib")]
    try:
        out = subprocess.run(cmd + ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], stdout=subprocess.PIPE,
                             stderr=subprocess.STDOUT, text=True)
        if out.returncode:
            raise RuntimeError("g++ failed\nfastcall.cpp:\n" + out.stdout)
        os.replace(part, FASTCALL)
    finally:
        if os.path.exists(part):
            os.remove(part)


def build_lib(force=False, verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    # objects built with other flags (the timing build) are never mixed with this build's
    stamp = os.path.join(OBJ, "flags.txt")
    flags = " ".join(FLAGS)
    if not os.path.exists(stamp) or open(stamp).read() != flags:
        force = True
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    headers = [os.path.join(CSRC, "small_internal.h"), os.path.join(HERE, "..", "include", "small.h")]
    objs, procs = [], []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, src.replace(".hip", ".o"))
        objs.append(o)
        if force or _stale(o, [s] + headers):
            cmd = [hipcc] + FLAGS + ["-c", s, "-o", o]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode:
            failed.append(f"{src}:\n{out}")
        elif verbose and out:
            print(out)
    if failed:
        raise RuntimeError("hipcc failed\n" + "\n".join(failed))
    with open(stamp, "w") as f:
        f.write(flags)
    if force or procs or _stale(LIB, objs):
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    probe_src = os.path.join(CSRC, "probe.hip")
    if force or _stale(PROBE_LIB, [probe_src, os.path.join(HERE, "..", "include", "small_probe.h")]):
        out = subprocess.run([hipcc] + FLAGS + ["-shared", probe_src, "-o", PROBE_LIB], stdout=subprocess.PIPE,
                             stderr=subprocess.STDOUT, text=True)
        if out.returncode:
            raise RuntimeError("hipcc failed\nprobe.hip:\n" + out.stdout)
    return LIB


def build_all(force=False, verbose=False):
    """The libraries, and the extension, which the binding can do without."""
    lib = build_lib(force, verbose)
    build_fastcall(force)
    return lib


if __name__ == "__main__":
    print(build_all(force=True, verbose=True))
