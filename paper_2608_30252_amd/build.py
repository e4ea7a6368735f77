"""Build libmad.so (HIP, gfx950) and the Python binding's _fastcall.so in-tree.

    python -m paper_2608_30252_amd.build            # the library
    python -m paper_2608_30252_amd.build --trace    # + libmad_trace.so, the diagnostic phase-trace build

Every translation unit in csrc/ is compiled by hipcc for gfx950 only and
linked into paper_2608_30252_amd/libmad.so.  Packed-fp32 instructions are
disabled for the device code (the compiler still emits ordinary fp32 math).
"""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmad.so")
FASTCALL = os.path.join(HERE, "_fastcall.so")
BUILD_DIR = os.path.join(HERE, "_build")
# the same sources with the kernels' phase marks compiled in (MAD_PHASE_TRACE):
# read by paper_2608_30252_amd/phase_trace.py, never by the product path
TRACE_LIB = os.path.join(HERE, "libmad_trace.so")
TRACE_BUILD_DIR = os.path.join(HERE, "_build", "trace")

ARCH = "gfx950"
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def build(verbose: bool = False, out: str = LIB, build_dir: str = BUILD_DIR, defines=()) -> str:
    os.makedirs(build_dir, exist_ok=True)
    cc = hipcc()
    common = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
              "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")] + DEVICE_FLAGS + \
             [f"-D{d}" for d in defines]

    def compile_one(src):
        obj = os.path.join(build_dir, os.path.basename(src) + ".o")
        cmd = [cc] + common + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if err.strip() and verbose:
            print(err, flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, sources()))
    tmp = out + ".tmp"
    cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


def build_fastcall(verbose: bool = False) -> str:
    """csrc/fastcall.cpp against the installed torch's headers and libraries (the ones its import loads).

    NDEBUG leaves out a thread-local debugging counter of pybind11's headers.  It was the module's only thread-local
    variable, and glibc up to 2.38 sends every access to the thread-local variables of the libraries loaded before
    (torch's) through its slow path for good once a library with one is loaded behind them: a call through ctypes
    took 15.0 us of host time without the module and 17.1 with it loaded."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    tmp = FASTCALL + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-DNDEBUG",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(HERE, "..", "include"), "-I", sysconfig.get_paths()["include"]]
    for p in include_paths():
        cmd += ["-isystem", p]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd += [os.path.join(CSRC, "fastcall.cpp"), "-o", tmp, "-L", libs, f"-Wl,-rpath,{libs}", "-ltorch_python",
            "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on fastcall.cpp:\n{r.stderr}")
    if r.stderr.strip() and verbose:
        print(r.stderr, flush=True)
    os.replace(tmp, FASTCALL)
    return FASTCALL


def build_trace(verbose: bool = False) -> str:
    return build(verbose, out=TRACE_LIB, build_dir=TRACE_BUILD_DIR, defines=("MAD_PHASE_TRACE",))


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
    print(build_fastcall(verbose="-v" in sys.argv))
    if "--trace" in sys.argv:
        build_trace(verbose="-v" in sys.argv)
        print(TRACE_LIB)
