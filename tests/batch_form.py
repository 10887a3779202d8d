"""The batched step's kernel and placement rules (plain C++ of the library), compiled for the tests."""
import ctypes as C
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2004_03972_amd", "csrc")
FORMS = {"f32": 0, "bf16": 1, "fp8": 2, "bit": 3}
SHIM = """
#include "batch_plan.h"
using namespace hqa;
static std::vector<BatchShape> shapes(int n, const int *N, const int *form) {
    std::vector<BatchShape> v;
    for (int k = 0; k < n; k++) v.push_back({k, N[k], (N[k] + 127) / 128 * 128, form[k]});
    std::stable_sort(v.begin(), v.end(), [](const BatchShape &a, const BatchShape &b) { return a.Np > b.Np; });
    return v;
}
extern "C" void form(int n, const int *N, const int *f, int R, int *out) {
    const std::vector<BatchShape> v = shapes(n, N, f);
    const BatchForm b = batch_form_for(v, R, batch_bytes(v, R));
    out[0] = b.rt; out[1] = b.wide; out[2] = b.stream;
}
extern "C" int place(int n, const int *N, const int *f, int R, int reps, int f32, int cap, int *out) {
    const std::vector<BatchTile> t = batch_place(shapes(n, N, f), R, reps, f32);
    for (size_t k = 0; k < t.size() && (int)k < cap; k++) {
        out[3 * k] = t[k].inst; out[3 * k + 1] = t[k].i0; out[3 * k + 2] = t[k].r0;
    }
    return (int)t.size();
}
"""
_lib = None


def lib():
    global _lib
    if _lib is None:
        d = tempfile.mkdtemp(prefix="batch_form_")
        src, so = os.path.join(d, "shim.cc"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                        "-o", so, src], check=True)
        _lib = C.CDLL(so)
    return _lib


def _args(sizes, kinds):
    n = len(sizes)
    return n, (C.c_int * n)(*sizes), (C.c_int * n)(*[FORMS[k] for k in kinds])


def form(sizes, kinds, R):
    """"narrow 1", "narrow 2", "narrow 4", "cached" or "streamed": the kernel of these BF16, FP8 and
    one-bit instances (one handle)."""
    out = (C.c_int * 3)()
    lib().form(*_args(sizes, kinds), R, out)
    rt, wide, stream = out
    assert wide <= (rt == 4) and stream <= wide
    return "streamed" if stream else "cached" if wide else f"narrow {rt}"


def place(sizes, kinds, R, reps, f32=False):
    """Launch order: (instance, first row, first replica), instance -1 for a placeholder."""
    cap = 16 + 64 * sum((-(-N // 128)) * (-(-R // reps)) for N in sizes)
    out = (C.c_int * (3 * cap))()
    n = lib().place(*_args(sizes, kinds), R, reps, int(f32), cap, out)
    assert n <= cap
    return [tuple(out[3 * k:3 * k + 3]) for k in range(n)]
