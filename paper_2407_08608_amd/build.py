"""Build libfa_mi355.so in-tree with hipcc for gfx950 (cross-compiles without a GPU), and the native part of binding.py."""
import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libfa_mi355.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # hipcc -O3 otherwise emits packed-fp32 VALU ops for plain float code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# "#pragma unroll" silently leaves a loop rolled when its unrolled size passes a threshold; the
# backward kernels index register arrays by the loop variable and must be unrolled whatever their size.
EXTRA_FLAGS = {"fa_bwd.hip": ["-mllvm", "-pragma-unroll-threshold=1000000"]}


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    extra = EXTRA_FLAGS.get(os.path.basename(src), [])
    subprocess.run([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], check=True)
    return obj


# Sources with MFMAs or loads written as inline assembly: their device assembly is generated once more as text and checked
# for instructions that touch an MFMA result, or write what such an instruction reads, too close to it (mfma_hazard_check.py).
HAZARD_CHECKED = ["fa_bwd.hip", "fa_fwd.hip", "fa_fwd_fp8.hip"]


def _check_hazards(name):
    from . import mfma_hazard_check
    src, listing = os.path.join(CSRC, name), os.path.join(OBJ, name + ".s")
    subprocess.run([HIPCC, *FLAGS, *EXTRA_FLAGS.get(name, []), "-S", "--cuda-device-only", src, "-o", listing],
                   check=True, stderr=subprocess.DEVNULL)
    text = open(listing).read()
    problems = mfma_hazard_check.check(text) + mfma_hazard_check.check_loads(text)
    if problems:
        lines = "\n".join(f"  {f} +{ln}: {text} ({waited} wait states)" for f, ln, text, waited in problems[:20])
        raise RuntimeError(f"{name}: {len(problems)} instructions come too close to an inline-assembly MFMA or load:\n{lines}")
    return name


# The native part of binding.py: host code against torch's C++ interface, which stays out of the library.  Object layouts
# of this Python and this torch go into it: the name keeps other Pythons from finding it, the module refuses another torch.
BINDING = os.path.join(HERE, "_fa_binding" + sysconfig.get_config_var("EXT_SUFFIX"))


def _build_binding():
    import torch
    for old in glob.glob(os.path.join(HERE, "_fa_binding*.so")):
        os.unlink(old)
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"]]
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
                    f'-DFA_TORCH_VERSION="{torch.__version__}"',
                    *(f for d in include for f in ("-isystem", d)), os.path.join(CSRC, "fa_binding.cpp"), "-o", BINDING,
                    "-L" + os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"], check=True)


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + len(HAZARD_CHECKED) + 1)) as ex:
        binding = ex.submit(_build_binding)
        checks = [ex.submit(_check_hazards, n) for n in HAZARD_CHECKED]
        objs = list(ex.map(_compile, srcs))
        for c in checks:
            c.result()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    # binding.py does without its native part, so a missing compiler, torch or header costs that part only
    if binding.exception() is not None:
        print(f"not built: {BINDING} ({binding.exception()}); calls will take the Python way, about 3 us more each", file=sys.stderr)
    if verbose:
        print("built", LIB, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build()
