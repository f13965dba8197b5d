"""Build libchsim.so (the HIP library behind include/chsim.h) for gfx950.

Every .hip source under csrc/ is compiled with hipcc into _build/ and linked
into paper_1808_00128_amd/libchsim.so, in-tree.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build", "chsim")
LIB = os.path.join(PKG, "libchsim.so")

ARCH = os.environ.get("CHSIM_OFFLOAD_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
    # Packed FP32 arithmetic stays off in every device code object.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


# The evolution kernels pick a tableau row by a chain of scalar branches with a
# compile-time register index in each case; sinking the identical cases into
# one block would turn that back into a dynamic index into stack memory.
EXTRA_FLAGS = {
    name: ["-mllvm", "-simplifycfg-sink-common=false"]
    for name in ("evolve_l4.hip", "evolve_l8.hip", "evolve_wide.hip")
}
# The column kernels branch on the gate alone (uniform over the wave).  Making
# that control flow structured, as divergent branches need, would keep two copies
# of the columns alive (454 spilled registers instead of none at n = 50).
EXTRA_FLAGS.update({
    name: ["-mllvm", "-structurizecfg-skip-uniform-regions=true"]
    for name in ("evolve_c4a.hip", "evolve_c4b.hip", "evolve_c8.hip", "evolve_c16.hip", "quad_pairs.hip")
})


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


# Host code with AddressSanitizer and UndefinedBehaviorSanitizer (the device
# code objects unsanitized and at -O1): the same sources, for checking the
# library's host paths (argument validation, decompositions, planning) on a
# machine without a GPU.  Load it with the clang ASan runtime preloaded.
SAN_BUILD = os.path.join(ROOT, "_build", "chsim_san")
SAN_LIB = os.path.join(SAN_BUILD, "libchsim_san.so")
SAN_FLAGS = [
    f"--offload-arch={ARCH}", "-O1", "-g", "-std=c++17", "-fPIC", "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
    "-Xarch_host", "-fno-sanitize-recover=all", "-Xarch_host", "-fno-omit-frame-pointer",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def build_host_sanitized(verbose: bool = False) -> str:
    os.makedirs(SAN_BUILD, exist_ok=True)

    def one(src):
        obj = os.path.join(SAN_BUILD, os.path.basename(src) + ".o")
        cmd = [HIPCC, *SAN_FLAGS, *EXTRA_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        return obj

    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(one, srcs))
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", SAN_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return SAN_LIB


def asan_runtime() -> str:
    """The clang ASan runtime that matches hipcc's host compiler."""
    out = subprocess.run([HIPCC, "--print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True,
                         text=True).stdout.strip()
    if out and os.path.isabs(out) and os.path.exists(out):
        return out
    import glob

    hits = sorted(glob.glob("/opt/rocm/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so"))
    if not hits:
        raise RuntimeError("clang ASan runtime not found")
    return hits[-1]


if __name__ == "__main__":
    if "--sanitize-host" in sys.argv:
        print(build_host_sanitized(verbose="-v" in sys.argv))
    else:
        build(verbose="-v" in sys.argv)
        print(LIB)
