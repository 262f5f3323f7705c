"""Build the HIP library (csrc/*.hip -> libla_hip.so, in-tree) for gfx950 with hipcc, and the extension
module that marshals its Python calls (csrc/la_binding.cpp -> _la_native.so) with the host compiler."""
import glob
import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libla_hip.so")
NATIVE = os.path.join(_HERE, "_la_native.so")
NATIVE_SOURCE = os.path.join(CSRC, "la_binding.cpp")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 arithmetic is kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep MFMA accumulators in ordinary vector registers: the softmax arithmetic reads and
    # rescales them, and copies to and from the accumulation registers dominated the inner loop
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def is_stale():
    if not os.path.exists(LIB) or not os.path.exists(NATIVE):
        return True
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(d) > os.path.getmtime(LIB) for d in sources() + headers) or \
        any(os.path.getmtime(d) > os.path.getmtime(NATIVE) for d in [NATIVE_SOURCE] + headers)


def build_native(verbose=False):
    """The extension module: host code over torch's C++ tensors, linked to the library beside it."""
    import torch
    from torch.utils import cpp_extension
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I", os.path.join(ROOT, "include")]
    for path in cpp_extension.include_paths() + [os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    cmd += [NATIVE_SOURCE, "-o", tmp, "-L" + _HERE, "-l:libla_hip.so", "-Wl,-rpath,$ORIGIN", "-L" + lib_dir,
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    _run(cmd, tmp, verbose)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose=False, extra_flags=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + \
        ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", tmp] + sources()
    _run(cmd, tmp, verbose)
    os.replace(tmp, LIB)
    build_native(verbose)
    return LIB


def _run(cmd, tmp, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only target feature; that warning is harmless
    noise = ("packed-fp32-ops", "is not a recognized feature")
    log = "\n".join(l for l in res.stdout.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("%s failed:\n" % cmd[0] + log)
    if verbose and log.strip():
        print(log)


if __name__ == "__main__":
    print(build(verbose=True))
