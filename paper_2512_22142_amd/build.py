"""Builds libcleave.so (HIP kernels + C ABI, hipcc for gfx950) and _native.so (the
binding's argument checks) in-tree."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcleave.so")
NATIVE = os.path.join(HERE, "_native.so")

SOURCES = ["plan.cpp", "scheduler.cpp", "api.cpp", "execute.hip", "execute_direct.hip", "reduce.hip", "verify.hip", "subset.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # the host-side planners compare doubles the oracle must reproduce: no fused multiply-adds
    "-Xarch_host", "-ffp-contract=off",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
    # no packed-fp32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _compile(src):
    obj = os.path.join(OBJ_DIR, src + ".o")
    cmd = [HIPCC] + COMMON + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    return src, obj, res


def native_tag():
    """What _native.so is tied to: it is compiled against torch's C++ classes and CPython's."""
    import torch
    return "cleave checks for torch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])


def native_fits(path=NATIVE):
    """Whether the built file is there and was made for this torch and this Python."""
    if not os.path.exists(path):
        return False
    with open(path, "rb") as f:
        return native_tag().encode() + b"\0" in f.read()


def _compile_native():
    """The binding's argument checks (host code against torch's headers), linked
    to the library beside it; the HIP runtime is the one torch has loaded."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    inc = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__",
           "-DUSE_ROCM", '-DCLEAVE_NATIVE_TAG="%s"' % native_tag(), "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           os.path.join(CSRC, "native.cpp"), "-o", NATIVE]
    for d in inc + [os.path.join(rocm, "include")]:
        cmd += ["-isystem", d]
    for d in cpp_extension.library_paths():
        cmd += ["-L" + d]
    cmd += ["-L" + HERE, "-l:libcleave.so", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed on native.cpp:\n%s" % (res.stdout + res.stderr))


def build(verbose=True, extra=None):
    """Compiles every source (always; the call is the build check) and links."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    if extra:
        COMMON.extend(extra)
    with ThreadPoolExecutor(max_workers=4) as pool:
        results = list(pool.map(_compile, SOURCES))
    objs = []
    for src, obj, res in results:
        text = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                         if "packed-fp32-ops" not in l and l.strip())
        if res.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, text))
        if verbose and text:
            print(text, file=sys.stderr)
        objs.append(obj)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    _compile_native()
    return LIB


def ensure_built(verbose=False):
    """Builds the library only if none is there that fits this torch and Python
    (tests, the smoke check and the benchmark use what is built; after a change
    to a source, build again)."""
    if not (os.path.exists(LIB) and native_fits()):
        build(verbose=verbose)
    return LIB


if __name__ == "__main__":
    print(build(extra=sys.argv[1:]))
