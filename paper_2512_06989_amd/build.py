"""Compile the HIP sources under csrc/ into paper_2512_06989_amd/libmhffn.so
for gfx950 with hipcc (cross-compiles without a GPU).

    python -m paper_2512_06989_amd.build        # rebuild everything
"""
import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmhffn.so")
HOST_LIB = os.path.join(HERE, "_host.so")             # argument marshalling (csrc/binding.cpp)
CALIB_LIB = os.path.join(HERE, "libmhffn_calib.so")   # calibration kernels of the bench
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["api.cpp", "module.cpp", "fwd_bf16.hip", "fwd_f32.hip", "bwd.hip", "bwd_f32.hip",
           "bwd_finish.hip", "unfused.hip", "gemm_bf16.hip"]
# Packed-fp32 VALU forms are switched off for all device code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


def _deps_mtime():
    m = 0.0
    for root in (CSRC, os.path.join(os.path.dirname(HERE), "include")):
        for f in os.listdir(root):
            m = max(m, os.path.getmtime(os.path.join(root, f)))
    return m


def _compile(src):
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    return obj, err


def _rocm_include():
    """The headers beside the compiler; HIPCC may be a name on PATH or a link to it."""
    hipcc = os.path.realpath(shutil.which(HIPCC) or HIPCC)
    return os.path.join(os.path.dirname(os.path.dirname(hipcc)), "include")


def _compile_binding():
    """csrc/binding.cpp with the host compiler, against the headers of the installed torch."""
    import sysconfig
    from torch.utils import cpp_extension
    obj = os.path.join(OBJDIR, "binding.o")
    inc = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], _rocm_include()]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           *["-I" + d for d in inc], "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on binding.cpp:\n%s" % r.stderr)
    return obj


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and all(os.path.exists(f) and os.path.getmtime(f) >= _deps_mtime() for f in (LIB, HOST_LIB)):
        return LIB
    os.makedirs(OBJDIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        binding = ex.submit(_compile_binding)
        results = list(ex.map(_compile, SOURCES))
        binding_obj = binding.result()
    if verbose:
        for _, err in results:
            if err.strip():
                print(err, file=sys.stderr)
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp,
                           *[o for o, _ in results]])
    os.replace(tmp, LIB)
    # (torch's own libraries are in the process before this one is imported: no path to them)
    from torch.utils import cpp_extension
    tmp = HOST_LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call(["g++", "-shared", "-fPIC", "-o", tmp, binding_obj, "-L" + HERE, "-l:libmhffn.so",
                           "-Wl,-rpath,$ORIGIN", *["-L" + d for d in cpp_extension.library_paths()],
                           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])
    os.replace(tmp, HOST_LIB)
    # the bench's calibration kernels: a library of their own, never loaded by the binding
    obj, _ = _compile("calib.hip")
    tmp = CALIB_LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, obj])
    os.replace(tmp, CALIB_LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
