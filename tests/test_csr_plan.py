"""The form of the sparse per-step kernel over all sizes (host code, compiled here): every launch
stays within 2^32 threads, covers every row and replica, and slices only whole chunks of replicas
over the XCDs of a large graph; the turned copies of a state likewise."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2004_03972_amd", "csrc")
SHIM = """
#include "csr_plan.h"
extern "C" uint64_t plan(int N, int64_t nnz, int max_deg, uint32_t Rp, int *out) {
    const hqa::CsrPlan p = hqa::csr_plan(N, nnz, max_deg, Rp);
    out[0] = p.rows; out[1] = p.vec; out[2] = (int)p.chunks; out[3] = p.sliced;
    return p.rows ? ((uint64_t)N * (Rp / 4) + 255) / 256 : hqa::csr_wave_blocks(N, p);
}
extern "C" int export_turn(int N) { return hqa::export_turn_fits(N); }
extern "C" int features_turn(int N, int R) { return hqa::features_turn_fits(N, R); }
"""


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("csr_plan")
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                    "-o", str(d / "shim.so"), str(d / "shim.cc")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.plan.restype = C.c_uint64
    lib.plan.argtypes = [C.c_int, C.c_int64, C.c_int, C.c_uint32, C.c_void_p]
    return lib


def test_every_size(L):
    out = (C.c_int * 4)()
    for N in (1, 3, 64, 511, 4096, 10000, 100003, 1 << 20, (1 << 26) - 1, 1 << 26, 1 << 28, 2 ** 31 - 1):
        for d in (0, 1, 6, 9.9, 10, 12, 20, 30, 700):
            nnz = min(int(N * d), 2 ** 31 - 2)
            for Rp in (4, 8, 16, 32, 36, 48, 64, 68, 96, 124, 128, 132, 192, 196, 256, 260, 320, 512, 516,
                       1024, 2048, 65536):
                if N * (Rp // 4) >= 2 ** 32 - 256:        # beyond what the state's set-up launches
                    continue
                for max_deg in (6, 100):
                    blocks = L.plan(N, nnz, max_deg, Rp, out)
                    rows, vec, chunks, sliced = out
                    where = (N, nnz, max_deg, Rp, rows, vec, chunks, sliced)
                    assert blocks * 256 < 2 ** 32, where
                    if rows:
                        assert rows in (2, 6), where
                        continue
                    assert vec in (1, 2, 4), where
                    assert 64 * vec * chunks >= Rp > 64 * vec * (chunks - 1), where
                    assert not sliced or (vec == 1 and (chunks in (2, 4) or chunks % 8 == 0)
                                          and Rp >= 57.6 * chunks), where
                    if N >= 6500 and N * N >= (600 if Rp > 4 else 900) * nnz:   # many: no half-empty chunks
                        assert Rp <= 64 or Rp >= 57.6 * vec * chunks, where
                        assert Rp > 32 or nnz >= 20 * N or Rp % 256 == 0, where


@pytest.mark.parametrize("N,d,Rp,form", [
    (1000000, 6, 4, "rows"), (1000000, 6, 64, "rows"), (100000, 30, 16, "rows"), (100000, 30, 68, "rows"),
    (1 << 26, 0, 4, "rows"), (10000, 30, 128, "wave"), (100000, 30, 256, "wave"), (4096, 6, 1024, "wave"),
    (2000, 12, 64, "wave"), (3388, 5, 8, "wave"), (6499, 5, 8, "wave"), (6500, 5, 8, "rows"),
    (4096, 5, 100, "rows"), (13186, 12, 1000, "wave"), (13186, 12, 900, "rows"), (7329, 30, 768, "rows"),
    (7278, 30, 100, "wave")])
def test_named_sizes(L, N, d, Rp, form):
    out = (C.c_int * 4)()
    L.plan(N, N * d, 3 * d + 7, Rp, out)
    assert (out[0] > 0) == (form == "rows")


def test_short_rows_of_a_lattice(L):
    out = (C.c_int * 4)()
    for N, deg, rows in ((4096, 6, True), (4096, 7, False), (3375, 6, False), (6859, 7, True)):
        L.plan(N, 6 * N, deg, 8, out)
        assert (out[0] > 0) == rows, (N, deg)


def test_turned_copies_stay_within_a_launch(L):
    for N in (1, 31, 32, 4096, (1 << 27) - 16, (1 << 27) - 15, 1 << 27, (1 << 29) - 32, (1 << 29) - 31,
              1 << 29, 2 ** 31 - 1):
        assert bool(L.export_turn(N)) == (-(-N // 32) * 256 < 2 ** 32), N
        for R in (1, 33, 32 * 65535, 32 * 65535 + 1, 2 ** 31 - 1):
            assert bool(L.features_turn(N, R)) == (-(-N // 16) * 512 < 2 ** 32 and -(-R // 32) <= 65535), (N, R)
