"""Build the C-ABI library (hand-written HIP for gfx950) into paper_2605_29639_amd/libkvq.so.

`python -m paper_2605_29639_amd.build` or `build()`.  hipcc cross-compiles without a GPU.
"""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libkvq.so")
OBJ_PROF = os.path.join(HERE, "_build", "prof")
LIB_PROF = os.path.join(HERE, "libkvq_prof.so")
LIB_FAST = os.path.join(HERE, "_kvq_fast.so")
SOURCES = ["kvq_api.hip", "kvq_write.hip", "kvq_attn.hip", "kvq_prefill.hip", "kvq_repack.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # Matrix-instruction results stay in ordinary vector registers.  With the 512-register
         # budget of a one-wavefront-per-SIMD kernel the compiler otherwise puts them into
         # accumulation registers, which no vector instruction can address, and copies every
         # logit and (on each rescale) every output accumulator out and back in.
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-Wno-unused-command-line-argument"]


def _compile(job):
    src, objdir, defines = job
    obj = os.path.join(objdir, src.replace(".hip", ".o"))
    subprocess.check_call(["hipcc", *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", obj])
    return obj


def _link(objs, lib):
    tmp = lib + ".tmp%d" % os.getpid()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, lib)


def _fast():
    """The native half of the Python binding, on torch's headers and libraries (without them there is none,
    and kvq.py does without)."""
    if os.path.exists(LIB_FAST):
        os.remove(LIB_FAST)   # (one of another torch would be worse than none)
    try:
        import torch
        from torch.utils import cpp_extension
        paths = cpp_extension.include_paths()
    except ImportError:
        paths = []
    if not any(os.path.exists(os.path.join(p, "torch", "csrc", "autograd", "python_variable.h")) for p in paths):
        print("no torch headers: %s is not built" % os.path.basename(LIB_FAST))
        return
    tmp = LIB_FAST + ".tmp%d" % os.getpid()
    include = [x for p in paths for x in ("-isystem", p)]
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                           "-I", sysconfig.get_paths()["include"], *include, os.path.join(CSRC, "kvq_fast.cpp"),
                           "-o", tmp, "-L", os.path.join(os.path.dirname(torch.__file__), "lib"),
                           "-ltorch_python", "-ltorch_cpu", "-lc10"])
    os.replace(tmp, LIB_FAST)


def build(verbose: bool = False) -> str:
    """libkvq.so (the library), libkvq_prof.so (the same sources with -DKVQ_PROFILE: the
    measurement switches of include/kvq_prof.h on top) and _kvq_fast.so (the native half of the
    Python binding)."""
    jobs = []
    for objdir, defines in ((OBJ, []), (OBJ_PROF, ["-DKVQ_PROFILE"])):
        os.makedirs(objdir, exist_ok=True)
        jobs += [(src, objdir, defines) for src in SOURCES]
    with ThreadPoolExecutor(max_workers=8) as ex:
        fast = ex.submit(_fast)
        objs = list(ex.map(_compile, jobs))
        fast.result()
    _link(objs[:len(SOURCES)], LIB)
    _link(objs[len(SOURCES):], LIB_PROF)
    if verbose:
        print("built", LIB, "and", LIB_PROF)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
