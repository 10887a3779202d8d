"""Checks of dense couplings by 64 x 64 tiles and their mirrors."""
import numpy as np
import pytest

from paper_2004_03972_amd import instances as inst

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa
    hqa.lib()
    return hqa


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 128, 129, 200])
def test_dense_checks_by_tiles(H, N):
    """One wrong entry anywhere is found: at the corners of a tile, in the last rows, in either
    triangle; and the exponents come from the whole matrix."""
    s = np.ones((1, N), np.int8)
    J = inst.small_int(N, 2)
    H.ising_energy(H.Problem(J), s)
    spots = {(i, j) for i in (0, 63, 64, N // 2, N - 1) for j in (0, 1, 62, 64, N - 1) if max(i, j) < N}
    for i, j in sorted(spots):
        for v in (0.5, np.nan, np.inf):
            B = J.copy()
            B[i, j] = v
            with pytest.raises(H.HQAError) as e:
                H.ising_energy(H.Problem(B), s)
            assert ("diagonal" if i == j and v == 0.5 else
                    "symmetric" if v == 0.5 else "non-finite") in str(e.value), (i, j, v)
        if i != j:                                       # a far exponent: the exact sums refuse it
            B = J.copy()
            B[i, j] = B[j, i] = 2.0 ** -200
            B[0, 1] = B[1, 0] = 1.0 if {i, j} != {0, 1} else B[0, 1]
            if np.any(np.abs(B) >= 1):
                with pytest.raises(H.HQAError):
                    H.ising_energy(H.Problem(B), s)
