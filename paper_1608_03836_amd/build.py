"""Build the HIP library ``libwadg.so`` in-tree for gfx950.

Usage: ``python paper_1608_03836_amd/build.py`` (or ``__graft_entry__.build()``); run as a
script, since importing the package loads the library this builds.
"""

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libwadg.so")
DEMO = os.path.join(PKG, "abi_demo")

SOURCES = ["reference.cpp", "stage_kernel.hip", "resident_kernel.hip", "split_kernel.hip",
           "quarter_kernel.hip", "pipe_kernel.hip",
           "adjoint_kernel.hip",
           "norms_kernel.hip", "l2_kernel.hip", "convert_kernel.hip", "parareal_kernel.hip", "launch.hip",
           "api.hip", "api_adjoint.hip", "api_batch.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Per-source flags.  The pipelined kernel loops over work items, and the
# one-launch sweep over stages, with every operator entry a compile-time
# constant; machine-level loop-invariant code motion would keep all of them
# in scalar registers across the loop and spill most, so it is switched off
# for those files (the constants are then rebuilt where they are used, as in
# the kernels without a loop).
SOURCE_FLAGS = {f: ["-mllvm", "-disable-machine-licm"]
                for f in ("pipe_kernel.hip", "quarter_kernel.hip")}

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed FP32 instructions are kept out of every code object
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


# Host-sanitizer build (CPU tests only): host code under AddressSanitizer
# and UndefinedBehaviorSanitizer, device code unsanitized.
SAN_DIR = os.path.join(PKG, "_build_san")
SAN_LIB = os.path.join(SAN_DIR, "libwadg.so")
SAN_FLAGS = "-Xarch_host -fsanitize=address -Xarch_host -fsanitize=undefined".split() + [
    "-Xarch_host", "-fno-omit-frame-pointer", "-Xarch_host", "-fno-sanitize-recover=all"]


def sanitizer_runtime():
    """Path of the compiler's AddressSanitizer runtime (preloaded into the
    Python process that loads the sanitized library)."""
    out = subprocess.run([os.path.join(os.path.dirname(os.path.realpath(HIPCC)), "..", "llvm",
                                       "bin", "clang"), "-print-file-name=libclang_rt.asan-x86_64.so"],
                         check=True, capture_output=True, text=True).stdout.strip()
    if not os.path.isabs(out) or not os.path.exists(out):
        raise RuntimeError("AddressSanitizer runtime not found")
    return out


def _source_stamp(flags):
    import hashlib
    h = hashlib.sha256(" ".join(flags).encode())
    for d, names in ((CSRC, sorted(os.listdir(CSRC))), (INCLUDE, sorted(os.listdir(INCLUDE)))):
        for n in names:
            with open(os.path.join(d, n), "rb") as f:
                h.update(n.encode() + f.read())
    return h.hexdigest()


def build_host_sanitized(verbose=False, jobs=None):
    """Build ``_build_san/libwadg.so``: every source with the host pass under
    ASan + UBSan (-O1, frame pointers kept).  Skips the build when the
    sources, headers and flags are unchanged since the last one.  Returns the
    library path."""
    from concurrent.futures import ThreadPoolExecutor
    flags = ["--offload-arch=gfx950", "-O1", "-g1", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"] + SAN_FLAGS
    stamp = _source_stamp(flags)
    stamp_file = os.path.join(SAN_DIR, "stamp")
    if os.path.exists(SAN_LIB) and os.path.exists(stamp_file) and open(stamp_file).read() == stamp:
        return SAN_LIB
    os.makedirs(SAN_DIR, exist_ok=True)
    common = flags + ["-I", INCLUDE, "-I", CSRC]

    def compile_one(src):
        obj = os.path.join(SAN_DIR, os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"] if src.endswith(".cpp") else []
        cmd = [HIPCC] + common + SOURCE_FLAGS.get(src, []) + ["-c"] + lang + \
            [os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, capture_output=not verbose)
        return obj

    n = jobs or min(len(SOURCES), max(1, os.cpu_count() or 1))
    with ThreadPoolExecutor(max_workers=n) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-shared-libsan"] + SAN_FLAGS + \
        objs + ["-o", SAN_LIB]
    subprocess.run(cmd, check=True, capture_output=not verbose)
    with open(stamp_file, "w") as f:
        f.write(stamp)
    return SAN_LIB


def build(verbose=False, extra_flags=(), jobs=None):
    """Compile every source into ``libwadg.so`` next to this file: one
    relocatable device-and-host object per source, compiled in parallel, then
    one link.  Always recompiles; raises CalledProcessError on failure."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    common = [f for f in FLAGS if f != "-shared"] + list(extra_flags) + ["-I", INCLUDE, "-I", CSRC]

    def compile_one(src):
        path = os.path.join(CSRC, src)
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"] if src.endswith(".cpp") else []
        cmd = [HIPCC] + common + SOURCE_FLAGS.get(src, []) + ["-c"] + lang + [path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    n = jobs or min(len(SOURCES), max(1, os.cpu_count() or 1))
    with ThreadPoolExecutor(max_workers=n) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    # the plain-C consumer of the library (csrc/abi_demo.c), linked against
    # it with the library's directory as run path
    cmd = ["gcc", "-std=c99", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", INCLUDE,
           "-I", "/opt/rocm/include", os.path.join(CSRC, "abi_demo.c"), "-o", DEMO,
           "-L", PKG, "-lwadg", "-L", "/opt/rocm/lib", "-lamdhip64",
           "-Wl,-rpath,$ORIGIN", "-Wl,-rpath,/opt/rocm/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])
