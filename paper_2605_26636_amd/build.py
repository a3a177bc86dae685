"""Compile the HIP sources under csrc/ into paper_2605_26636_amd/libjetvit.so for gfx950, and the
argument marshalling of the Python binding (csrc/jv_native.cpp) into paper_2605_26636_amd/_native.so."""
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libjetvit.so")
NATIVE = os.path.join(HERE, "_native.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
    "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(what, cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that is harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{what} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False) -> str:
    import torch
    from torch.utils import cpp_extension
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run("hipcc", [hipcc] + FLAGS + sources() + ["-o", OUT], verbose)
    includes = cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    libs = cpp_extension.library_paths("cuda")
    _run("g++", ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                 f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}"]
         + [f for i in includes for f in ("-isystem", i)] + [os.path.join(CSRC, "jv_native.cpp"), "-o", NATIVE]
         + ["-L" + d for d in libs] + ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip",
                                       "-L" + HERE, "-l:libjetvit.so", "-Wl,-rpath,$ORIGIN"], verbose)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
