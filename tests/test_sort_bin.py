"""The sort cell of a coordinate is worked out by the key, the scatter and the
search kernel each, which must agree to the last bit: the function rounds after
every operation, whatever the compiler would contract around it.  It is taken
from the kernels' source and built for the host with the FP32 unit's own
contraction mode and FMA instructions, out of line so that nothing is shared."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.join(os.path.dirname(__file__), "..", "paper_1210_8084_amd")
CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("amdclang++"), shutil.which("clang++"))
              if c and os.path.exists(c)), None)

SHELL = """
#include <algorithm>
#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ __attribute__((noinline))
using std::fmin; using std::min;
template <typename real> struct Inst { int nl[3], kl[3]; real lo[3], inv_wl[3]; };
%s
extern "C" void bins(int n, const float* x, float lo, float inv_w, int nl, int kl, int* out) {
    Inst<float> I{{nl, nl, nl}, {kl, kl, kl}, {lo, lo, lo}, {inv_w, inv_w, inv_w}};
    for (int i = 0; i < n; ++i) out[i] = sort_bin(I, 0, x[i]);
}
"""


def function(text, name):
    i = text.rindex("template <typename real>", 0, text.index(" " + name + "("))
    return text[i:text.index("\n}\n", i) + 3]


@pytest.mark.skipif(CLANG is None, reason="no clang to build the function with")
@pytest.mark.parametrize("nl,kl", [(1000, 3), (37, 2), (1, 5), (9000, 1), (100, 0)])
def test_sort_bin_rounds_every_operation(tmp_path, nl, kl):
    text = open(os.path.join(ROOT, "csrc", "tpkmc_kernels.h")).read()
    mode = re.search(r'"tpkmc_f32.hip": \["(-ffp-contract=[\w-]+)"\]', open(os.path.join(ROOT, "build.py")).read()).group(1)
    src = tmp_path / "bins.cpp"
    src.write_text(SHELL % (function(text, "axis_bin") + function(text, "sort_bin")))
    lib = tmp_path / "bins.so"
    subprocess.run([CLANG, "-O3", "-std=c++17", "-mfma", mode, "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    n = 1_000_000
    x = np.random.default_rng(nl).uniform(-0.01, 1.31, n).astype(np.float32)
    lo, inv_w = np.float32(0.1), np.float32(nl / 1.2)
    got = np.empty(n, dtype=np.int32)
    fn = ctypes.CDLL(str(lib)).bins
    fn.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_float, ctypes.c_float, ctypes.c_int, ctypes.c_int,
                   ctypes.c_void_p]
    fn(n, x.ctypes.data, lo, inv_w, nl, kl, got.ctypes.data)
    t = (x - lo) * inv_w
    c = np.clip(np.floor(np.maximum(t, 0)), 0, nl - 1).astype(np.int32)
    k = 1 << kl
    f = (t - c.astype(np.float32)) * np.float32(k)
    want = c * k + np.clip(np.trunc(np.clip(f, 0, k)), 0, k - 1).astype(np.int32)
    assert np.array_equal(got, want), f"{(got != want).sum()} of {n} differ"
