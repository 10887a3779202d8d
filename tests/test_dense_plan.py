"""Block shape of the dense per-step kernel by size (host code, compiled here): it divides every
padded state, and takes the larger blocks where their rounds over the chip cost least."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2004_03972_amd", "csrc")
SHIM = """
#include "dense_plan.h"
extern "C" int64_t plan(int Np, int Rp, int f32, int *out) {
    const hqa::StepBlock b = hqa::step_block(Np, Rp, f32 != 0);
    out[0] = b.tm; out[1] = b.tn; out[2] = b.cb;
    return hqa::step_blocks(Np, Rp, b.tm, b.tn);
}
extern "C" int tiles(int Np, int64_t steps) { return hqa::step_reads_tiles(Np, steps); }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("dense_plan")
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                    "-o", str(d / "shim.so"), str(d / "shim.cc")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.plan.restype = C.c_int64

    def f(N, R, f32):
        out = (C.c_int * 3)()
        n = lib.plan(-(-N // 128) * 128, -(-R // 16) * 16, int(f32), out)
        return n, tuple(out)
    f.tiles = lambda Np, steps: bool(lib.tiles(Np, C.c_int64(steps)))
    return f


def test_every_size(plan):
    for N in (1, 128, 129, 509, 1000, 2048, 5445, 10000, 46341, 100000):
        for R in (1, 16, 17, 32, 33, 48, 64, 100, 128, 640, 1500, 65536):
            for f32 in (False, True):
                n, (tm, tn, cb) = plan(N, R, f32)
                Np, Rp = -(-N // 128) * 128, -(-R // 16) * 16
                assert (tm, tn) in ((1, 1), (2, 1), (2, 2), (2, 4)) and cb in (4, 8)
                assert Rp % (16 * tn) == 0 and n * tm * tn * 256 == Np * Rp, (N, R)
                assert (cb == 8) == (f32 and Np >= 1024 and tm == 2 and n >= 512), (N, R)


@pytest.mark.parametrize("N,R,shape", [
    (387, 7, (1, 1)), (4096, 16, (1, 1)), (4097, 16, (2, 1)),       # one round of small blocks, then none
    (5445, 13, (2, 1)), (10000, 16, (2, 1)), (4469, 19, (2, 2)),
    (2513, 32, (2, 1)), (5035, 60, (2, 4)), (2048, 64, (2, 1)), (2049, 64, (2, 2)),
    (4096, 64, (2, 2)), (4097, 64, (2, 4)),
    (1105, 128, (2, 2)), (1000, 112, (2, 1)), (8756, 384, (2, 4)),
])
def test_line_between_shapes(plan, N, R, shape):
    for f32 in (False, True):
        assert plan(N, R, f32)[1][:2] == shape, plan(N, R, f32)


def test_short_runs_of_small_problems_set_up_no_copies(plan):
    for Np, line in ((128, 20), (512, 5), (640, 4), (1024, 3), (1280, 2), (2432, 2), (2560, 1), (10112, 1)):
        assert [plan.tiles(Np, s) for s in (line - 1, line, 2 ** 62)] == [False, True, True], Np
