"""Build libpex.so (HIP, gfx950) in-tree with hipcc, and the binding's native calls with g++.  Run as ``python -m paper_2510_00236_amd.build``."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libpex.so")
_OBJ = os.path.join(_HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra", "-Wno-inline-asm",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(_ROOT, "include"), "-I", CSRC]


HOST_SOURCE = os.path.join(_HERE, "host", "pex_host.cpp")
HOST_MODULE = os.path.join(_HERE, "_pex_host.so")


def host_command():
    """Compiles the binding's native calls against the headers of the installed torch and links them to libpex.so beside them.  As torch itself
    without assertions: those of its headers bring a thread-local counter, and with glibc before 2.39 a library with thread-local storage that
    nobody touches puts every look-up of torch's own on the slow path (an allocation 1.11 -> 1.36 us, a random fill 4.4 -> 5.5)."""
    import importlib.util
    spec = importlib.util.find_spec("torch")
    if spec is None:
        raise ImportError("no torch to compile the native calls against")
    torch_dir = spec.submodule_search_locations[0]
    include = [os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"],
               os.path.join(_ROOT, "include"), "/opt/rocm/include"]
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-w", "-DNDEBUG", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", *["-I" + d for d in include],
            HOST_SOURCE, "-o", HOST_MODULE, "-L" + os.path.join(torch_dir, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python", "-L" + _HERE, "-l:libpex.so",
            "-Wl,-rpath,$ORIGIN", "-Wl,--allow-shlib-undefined"]


def build_host() -> bool:
    """Compile the native calls.  The binding works without them, at 1 to 3 us more a call: where they cannot be built that is said, and none of
    an earlier build stays beside the new library."""
    if os.path.exists(HOST_MODULE):
        os.remove(HOST_MODULE)
    try:
        subprocess.run(host_command(), check=True)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        print(f"warning: the binding's native calls are not built ({e}); every call goes through the Python checks", file=sys.stderr)
        return False
    return True


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every translation unit, link libpex.so and, where it can be built, the module beside it.  Always recompiles."""
    os.makedirs(_OBJ, exist_ok=True)
    objs = []
    procs = []
    for src in sources():
        obj = os.path.join(_OBJ, os.path.basename(src)[:-4] + ".o")
        cmd = [HIPCC, *FLAGS, *extra_flags, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    # what the four-wave, Gram and fp32 kernels assume about their own machine code, checked while the objects compile
    from . import isa_check
    isa_error = None
    try:
        at = lambda name: os.path.join(CSRC, name)
        isa_check.check_all(HIPCC, [*FLAGS, *extra_flags], at("pex_stat_bf16.hip"), (at("pex_gram.hip"), at("pex_gram_wide.hip")), (at("pex_stat_f32.hip"), at("pex_stat_f32_split.hip"), at("pex_stat_small.hip")))
    except (isa_check.IsaCheckError, subprocess.CalledProcessError) as e:
        isa_error = e
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        # hipcc's host pass does not know the packed-fp32 target feature and says so; that is harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if out.strip() and (verbose or p.returncode != 0):
            print(out, flush=True)
        if p.returncode != 0:
            print(f"hipcc failed on {src}", file=sys.stderr)
            failed = True
    if failed:
        raise RuntimeError("libpex build failed")
    if isa_error is not None:
        raise RuntimeError(f"libpex build failed: {isa_error}")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    build_host()
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
