"""Compiles named device functions of the kernels' own source for the host, so that a test can
call them without a GPU.  The hardware reciprocal, reciprocal square root and square root (within
1 ulp) become IEEE operations times `scale` (set_scale)."""
import ctypes
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2207_08207_amd", "csrc")
PRELUDE = """
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstring>
#include <algorithm>
#define __forceinline__ inline
#include "lst_select.hpp"
#include "lst_ws.hpp"
using std::min;
using std::max;
static float host_scale = 1.0f;
extern "C" void set_scale(float s) { host_scale = s; }
namespace lst {
inline float frcp(float x) { return (1.0f / x) * host_scale; }
inline float frsq(float x) { return (1.0f / sqrtf(x)) * host_scale; }
#define __builtin_amdgcn_sqrtf(x) (sqrtf(x) * host_scale)
template <class T> inline const T *gp(const T *p) { return p; }
template <class T> inline T *gp(T *p) { return p; }
template <class T> inline T gload(const T *p, long i) { return p[i]; }
inline int uload(const int *p) { return *p; }
"""


def _definition(src, name):
    """The text of function or struct `name`, from its start of line to its closing brace."""
    m = re.search(rf"^(struct {name} \{{|[^\n;/]*\b{name}\([^;{{]*\{{)", src, re.M)
    assert m, name
    depth, i = 0, src.index("{", m.start())
    for k in range(i, len(src)):
        depth += (src[k] == "{") - (src[k] == "}")
        if depth == 0:
            return src[m.start():k + 1] + (";" if m.group(0).startswith("struct") else "")
    raise AssertionError(name)


def build(tmp_path, names, code):
    """`names` of lst_kernels.hip, then `code` (extern "C" functions that call them), as a ctypes library."""
    with open(os.path.join(CSRC, "lst_kernels.hip")) as f:
        src = f.read()
    text = PRELUDE + "\n".join(_definition(src, n) for n in names) + "\n}  // namespace lst\nusing namespace lst;\n" + code
    cpp, so = os.path.join(tmp_path, "k.cpp"), os.path.join(tmp_path, "k.so")
    with open(cpp, "w") as f:
        f.write(text)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    f"-I{rocm}/include", f"-I{CSRC}", cpp, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.set_scale.argtypes = [ctypes.c_float]
    return lib
