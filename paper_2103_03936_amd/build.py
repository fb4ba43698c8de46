"""Compile the HIP sources under csrc/ for gfx950 into libpufferfish.so and the Python binding (in-tree)."""
import glob
import os
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpufferfish.so")
BINDING = os.path.join(HERE, "_binding.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed-FP32 instruction selection is switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose=False, jobs=8):
    """Compile every csrc/*.hip to an object (in parallel) and link libpufferfish.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs, objs = [], []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [hipcc] + [f for f in FLAGS if f != "-shared"] + ["-c", src, "-o", obj]
        log = tempfile.TemporaryFile("w+")  # (a pipe that nobody reads yet stops a compiler that says much)
        procs.append((log, subprocess.Popen(cmd, stdout=log, stderr=subprocess.STDOUT)))
        while len([p for _, p in procs if p.poll() is None]) >= jobs:
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    failed = False
    for log, p in procs:
        p.wait()
        with log:
            log.seek(0)
            lines = [l for l in log.read().splitlines() if "packed-fp32-ops" not in l]
        if p.returncode != 0 or verbose:
            sys.stderr.write("\n".join(lines) + "\n")
        failed |= p.returncode != 0
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    build_binding()
    return LIB


def build_binding():
    """csrc/pf_binding.cpp (host code only) -> _binding.so, linked against torch and libpufferfish.so."""
    import torch
    tdir = os.path.dirname(torch.__file__)
    subprocess.check_call(
        ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
         "-I" + os.path.join(tdir, "include"), "-I" + os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
         "-I/opt/rocm/include", "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "pf_binding.cpp"), "-o", BINDING,
         "-L" + os.path.join(tdir, "lib"), "-L" + HERE, "-lpufferfish", "-ltorch_python", "-ltorch_cpu", "-ltorch_hip",
         "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"])
    return BINDING


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
