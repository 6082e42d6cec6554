"""Builds libtw.so (HIP, gfx950 only) with hipcc and the Python module over it with g++, both in-tree."""
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtw.so")
PYMODULE = os.path.join(HERE, "_twpy" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["tw_host.hip", "tw_fused.hip", "tw_unfused.hip", "tw_gemm.hip", "tw_gemm_tile.hip", "tw_probe.hip"]

# Packed fp32 VALU instructions are switched off for every kernel (the compiler
# would otherwise form them from plain float code). Kernel arguments that stand ahead of the
# first struct arrive in scalar registers with the wave, as many as fit (14), instead of being
# fetched from memory by its first instructions.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-mllvm", "-amdgpu-kernarg-preload-count=14",
               "-Wall", "-Wno-unused-command-line-argument"]


def hipcc_path():
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: libtw can only be built with the ROCm toolchain")


def build_libtw(verbose=False):
    """Compile every kernel source for gfx950 and link libtw.so next to this file."""
    hipcc = hipcc_path()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + HIPCC_FLAGS + inc + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        # the host pass does not know the device-only feature flag; that warning is noise
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s" % r.stdout)
    os.replace(tmp, LIB)
    return LIB


def start_pymodule():
    """Starts compiling tw_python.cpp; finish_pymodule() links it against libtw.so."""
    import torch
    base = os.path.join(os.path.dirname(torch.__file__), "include")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    obj = os.path.join(objdir, "tw_python.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I", os.path.join(ROOT, "include"), "-isystem", base,
           "-isystem", os.path.join(base, "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
           "-c", os.path.join(CSRC, "tw_python.cpp"), "-o", obj]
    return obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def finish_pymodule(started):
    import torch
    obj, proc = started
    out, _ = proc.communicate()
    if proc.returncode != 0:
        raise RuntimeError("g++ failed on tw_python.cpp:\n%s" % out)
    tmp = PYMODULE + ".tmp.%d" % os.getpid()
    # libtw.so is found next to the module; torch's libraries are in the process already
    cmd = ["g++", "-shared", "-o", tmp, obj, "-L", HERE, "-ltw", "-L", os.path.join(os.path.dirname(torch.__file__), "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,--disable-new-dtags,-rpath,$ORIGIN",
           "-Wl,--allow-shlib-undefined"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of the Python module failed:\n%s" % r.stdout)
    os.replace(tmp, PYMODULE)
    return PYMODULE


def build_all(verbose=False):
    """libtw.so and the Python module. Returns libtw.so's path."""
    started = start_pymodule()
    path = build_libtw(verbose)
    finish_pymodule(started)
    return path


if __name__ == "__main__":
    print(build_all(verbose=True))
