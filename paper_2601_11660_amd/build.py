"""Builds the HIP library in-tree, paper_2601_11660_amd/libmbu_hip.so (gfx950 only), and the module of the
binding's calls, paper_2601_11660_amd/_native.so (host code)."""
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmbu_hip.so")
NATIVE = os.path.join(HERE, "_native.so")
OBJ_DIR = os.path.join(ROOT, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 instruction forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off",
    # the first kernel arguments arrive in scalar registers with the wave instead of behind a load: part of
    # the latency chain of the small layers (64x96 network, 20 launches: 85.3 -> 83.1 us)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
]

# per-source additions
EXTRA_FLAGS = {
    # the first layer reads its few accumulators straight back with vector instructions:
    # keep them in ordinary vector registers instead of accumulation registers
    "stem_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_native(verbose: bool = False) -> str:
    """Compile csrc/native_calls.cpp against the installed torch (always recompiles)."""
    import torch
    t = os.path.dirname(torch.__file__)
    # NDEBUG: without it pybind11's reference counter gives the module a thread-local segment that nothing
    # touches, and glibc's accesses to the thread-local state of older libraries (torch's dispatch keys, read
    # several times by every operator) then take the slow path: 160 torch calls 661 -> 720 us
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"],
           "-isystem", os.path.join(t, "include"),
           "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           os.path.join(CSRC, "native_calls.cpp"), "-o", NATIVE,
           "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return NATIVE


def build_native_or_none(verbose: bool = False) -> bool:
    """build_native() where a host compiler and the headers of Python and torch are at hand.  Elsewhere no module is
    left behind, an older one included: the binding does without."""
    try:
        build_native(verbose)
        return True
    except (OSError, subprocess.CalledProcessError) as e:
        print(f"no module of the binding's calls: {e}", file=sys.stderr, flush=True)
        if os.path.exists(NATIVE):
            os.remove(NATIVE)
        return False


def build(verbose: bool = False) -> str:
    """Compile every HIP source, link the shared library, and build the module of the binding's calls
    where that is possible (always recompiles)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def compile_one(src):
        obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
        cmd = [hipcc] + HIPCC_FLAGS + EXTRA_FLAGS.get(os.path.basename(src), []) + inc + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    workers = min(8, len(os.sched_getaffinity(0)))
    with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as pool:
        native = pool.submit(build_native_or_none, verbose)
        objs = list(pool.map(compile_one, sources()))
        native.result()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
