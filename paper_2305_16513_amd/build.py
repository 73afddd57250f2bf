"""Builds libsws.so (HIP, gfx950) in-tree with hipcc.  Run: python -m paper_2305_16513_amd.build"""
import concurrent.futures
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsws.so")
CALLS = os.path.join(HERE, "_calls.so")

# Packed fp32 VALU instructions are switched off for every device object.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra", "-Wno-unused-parameter",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# The sliding-sum and pooling kernels: C's fmax / fmin must ignore a signalling NaN where the hardware's max / min
# (IEEE mode) would return it quieted, so the compiler quiets every element it has loaded first, one more vector
# instruction per element (70 of 915 in the scan kernel's max instance).  The library leaves NaN propagation through
# max / min unspecified (inputs are finite), so these files are compiled without NaN guarantees; + is unaffected.
NO_NAN_SRCS = {"slide1d.hip", "slide_reg.hip", "slide_long.hip", "slide_rows.hip", "slide16.hip", "pool2d.hip",
               "pool2d_padded.hip", "pool2d_small.hip", "pool_grad_large.hip"}


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    extra = ["-fno-honor-nans"] if os.path.basename(src) in NO_NAN_SRCS else []
    cmd = ["hipcc", *HIPCC_FLAGS, *extra, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    return obj, err


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        results = list(ex.map(_compile, srcs))
    if verbose:
        for _, err in results:
            if err.strip():
                print(err, file=sys.stderr)
    objs = [o for o, _ in results]
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if os.path.exists(CALLS):                         # (linked to the library that is about to be replaced)
        os.remove(CALLS)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    try:
        _build_calls()
    except (ImportError, OSError, RuntimeError) as e:
        print("without native calls (the binding's Python code serves them all): %s" % e, file=sys.stderr)
    return LIB


def _build_calls():
    """The binding's small calls in native code: host code against torch's headers, beside the library and linked to it.  The library needs none of these."""
    import sysconfig
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DSWS_TORCH_VERSION="%s"' % torch.__version__, "-I", os.path.join(ROOT, "include"),
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "calls.cpp"), "-o", CALLS,
           "-L", HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN", "-L", lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        if os.path.exists(CALLS):
            os.remove(CALLS)
        raise RuntimeError("g++ failed for calls.cpp:\n" + r.stderr)
    if r.stderr.strip():
        print(r.stderr, file=sys.stderr)


if __name__ == "__main__":
    print(build(verbose=True))
