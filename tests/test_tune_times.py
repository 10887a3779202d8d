"""The tuner's measure of a candidate (host code, compiled here): a run that something else held up
does not change it, and only a candidate that would be chosen is measured twice."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2004_03972_amd", "csrc")
SHIM = """
#include "tune_times.h"
// the times of up to TUNE_PASSES runs; how many were made, and the measure
extern "C" int measure(const float *t, float best, float *slope) {
    hqa::TuneTimes m;
    int pass = 0;
    for (; pass < hqa::TUNE_PASSES && !hqa::tune_done(pass, m, best); pass++)
        if (pass > 0) m.add(hqa::tune_pass_twice(pass), t[pass]);
    *slope = m.slope();
    return pass;
}
"""


@pytest.fixture(scope="module")
def measure(tmp_path_factory):
    d = tmp_path_factory.mktemp("tune_times")
    (d / "shim.cc").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC,
                    "-o", str(d / "shim.so"), str(d / "shim.cc")], check=True)
    lib = C.CDLL(str(d / "shim.so"))
    lib.measure.argtypes = [C.c_void_p, C.c_float, C.c_void_p]

    def f(times, best):
        s = C.c_float()
        return lib.measure((C.c_float * 5)(*times), best, C.byref(s)), s.value
    return f


@pytest.mark.parametrize("held", range(5))
def test_one_run_held_up(measure, held):
    t = [9.0, 3.0, 5.0, 3.0, 5.0]                       # a fixed cost of 1 and 2 a run of `steps`
    t[held] += 4.0
    runs, slope = measure(t, 6.5)
    assert (runs, slope) == (5, 2.0)


def test_measured_twice_only_if_chosen(measure):
    assert measure([9.0, 3.0, 5.0, 0.0, 0.0], 2.0) == (3, 2.0)
    assert measure([9.0, 3.0, 5.0, 3.0, 5.0], 2.1) == (5, 2.0)
    assert measure([9.0, 5.0, 4.0, 5.0, 4.0], 1.0) == (5, 0.0)
