"""The launch shape of the exact energies over all sizes (host code, compiled here): every dense
instance has a plan whose partial sums fit the scratch, and the scratch is what it always was."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2004_03972_amd", "csrc")
SHIM = """
#include "energy_plan.h"
extern "C" void plan(int N, int V, int D, int *out) {
    const hqa::EnergyPlan p = hqa::energy_plan(N, V, D);
    out[0] = p.vec; out[1] = p.P; out[2] = p.piece;
}
extern "C" size_t part_bytes(int N, int V) { return hqa::energy_part_bytes(N, V); }
extern "C" int digits(int k) { return k < hqa::MV_NDIGITS ? hqa::MV_DIGITS[k] : 0; }
"""


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("energy_plan")
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                    "-o", str(d / "shim.so"), str(d / "shim.cc")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.part_bytes.restype = C.c_size_t
    return lib


SIZES = [1, 2, 15, 16, 17, 63, 64, 65, 100, 300, 767, 768, 1000, 5000, 20000, 1 << 20]
VECTORS = [1, 2, 3, 4, 16, 17, 64, 65, 255, 1024, 8191, 8192, 8193, 16368, 16369, 16400, 20000,
           100000, 1 << 20, 5000000]


def test_every_size_has_a_plan(L):
    out = (C.c_int * 3)()
    for N in SIZES:
        for V in VECTORS:
            if N * V > 1 << 36:
                continue
            words = L.part_bytes(N, V) // 8
            for k in range(9):
                D = L.digits(k)
                L.plan(N, V, D, out)
                vec, P, piece = out
                where = (N, V, D, vec, P, piece)
                assert 1 <= piece <= V and vec in (16, 32, 64), where
                assert 1 <= P <= max(1, (N + 15) // 16), where
                assert P * D * (piece + 1) <= words, where
                assert -(-piece // vec) <= 65535, where
                # few launches, and none cut short where the sums fit
                assert -(-V // piece) <= 4 or V * 16 > 65535 * vec or V <= 3, where
                if D * (V + 1) <= words and V <= 65535 * vec:
                    assert piece == V, where


@pytest.mark.parametrize("N,V,nbytes", [
    (1, 1, 392), (64, 1, 1280), (200, 7, 8512), (800, 64, 214656), (5000, 256, 1212928),
    (100, 8192, 1151360), (64, 16369, 2095232), (1000, 20000, 3784320), (300, 100000, 12800000),
    (20000, 3, 422400)])
def test_scratch_is_unchanged(L, N, V, nbytes):
    """It counts towards the limit of the read-out without allocation: what that accepts and
    refuses stays."""
    assert L.part_bytes(N, V) == nbytes
