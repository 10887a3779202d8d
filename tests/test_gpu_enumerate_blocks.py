"""Exact enumeration of real couplings at every number of low bits walked in blocks of 16 codes
(none to twelve), with and without near-ties, against the oracle's exact brute force."""
import numpy as np
import pytest

import oracle as orc
from paper_2004_03972_amd import instances as inst
from test_gpu_enumerate import _solve_real

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa
    hqa.lib()
    return hqa


@pytest.mark.parametrize("n", [1, 2, 8, 12, 13, 14, 15, 17, 18, 19, 21])
@pytest.mark.parametrize("kind", ["glass", "ties"])
def test_low_bits(H, n, kind):
    J, h = inst.uniform_glass(40, n)
    if kind == "ties":                                   # quarters, one coupling off by 2^-45
        J, h = np.rint(2 * J) * 0.25, np.rint(h) * 0.5
        J[3, 4] = J[4, 3] = J[3, 4] + 2.0 ** -45
    _solve_real(H, J, n, 2, seed=n, h=h)


@pytest.mark.parametrize("n", [3, 14, 18])
@pytest.mark.parametrize("e", [-900, -500, 90])
def test_scales(H, n, e):
    """Couplings near the smallest and the largest exponents that the exact sums take."""
    J, h = inst.uniform_glass(30, n)
    if e > 0:                                            # a fraction keeps the instance real
        J, h = np.rint(J * 2.0 ** 20) * 2.0 ** (e - 20), np.rint(h * 2.0 ** 20) * 2.0 ** (e - 20)
        h[0] += 0.5 if abs(h[0]) < 2.0 ** 50 else 0.0
        J[1, 2] = J[2, 1] = 0.5
    else:
        J, h = J * 2.0 ** e, h * 2.0 ** e
    _solve_real(H, J, n, 2, seed=n, h=h)


@pytest.mark.parametrize("n", [8, 13, 16])
def test_many_candidates(H, n):
    """Couplings so small that nearly every code is within the rescoring bound of the others:
    more candidates than a workgroup rescores together."""
    J = np.zeros((30, 30))
    h = np.zeros(30)
    h[0] = 0.5                                           # a fraction keeps the instance real
    J[0, 1] = J[1, 0] = 2.0 ** -60
    J[2, 3] = J[3, 2] = -(2.0 ** -61)
    _solve_real(H, J, n, 3, seed=n, h=h)
