"""Exact energies and cuts of dense instances at the edges of the many-vector kernel: its
16-row, 16- and 64-column blocks, its 16, 32 and 64 vectors a wavefront, each digit count and
each storage copy; bit for bit with the oracle, which accumulates exactly and rounds once."""
import numpy as np
import pytest

import oracle as orc
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


def couplings(N, bits, seed):
    """Symmetric integers of up to `bits` bits times 2^-40, some small so that spans fill."""
    rng = np.random.default_rng(seed)
    m = rng.integers(-(1 << bits) + 1, 1 << bits, size=(N, N)).astype(np.float64)
    if bits > 52:                                        # spans beyond one binary64 significand
        m = rng.normal(size=(N, N)) * 2.0 ** rng.integers(0, bits - 52, size=(N, N))
        m = np.rint(m * 2.0 ** 20)
    U = np.triu(m, 1)
    return (U + U.T) * 2.0 ** -40


def check(H, J, h, V, seed):
    N = J.shape[0]
    s = np.where(np.random.default_rng(seed).random((V, N)) < 0.5, -1, 1).astype(np.int8)
    E, C = H.ising_energy(H.Problem(J, h=h), s)
    Eo, Co = orc.energy(orc.Problem(N, J=J, h=h), s)
    assert np.array_equal(E, Eo)
    assert np.array_equal(C, Co)


@pytest.mark.parametrize("N", [1, 2, 15, 16, 17, 63, 64, 65, 79, 81, 130, 257])
@pytest.mark.parametrize("bits", [1, 50])
def test_sizes(H, N, bits):
    J = couplings(N, bits, N)
    h = np.random.default_rng(N).normal(size=N)
    for V in (1, 16, 17):
        check(H, J, h if bits > 1 else None, V, V)


@pytest.mark.parametrize("bits", [1, 5, 6, 13, 14, 29, 30, 45, 52])
@pytest.mark.parametrize("V", [3, 33, 64, 65, 130])
def test_digit_counts(H, bits, V):
    check(H, couplings(100, bits, bits), None, V, bits)


@pytest.mark.parametrize("spread", [0, 6, 20, 40, 70, 100, 140])
@pytest.mark.parametrize("V", [5, 40, 70])
def test_wide_spans(H, spread, V):
    """Couplings of very different exponents: 8 to 20 digits; more than 150 binades between the
    lowest and the highest set bit are refused."""
    rng = np.random.default_rng(spread)
    N = 70
    U = np.triu(rng.normal(size=(N, N)) * 2.0 ** rng.integers(-spread, 1, size=(N, N)), 1)
    h = rng.normal(size=N)
    x = np.concatenate([U[U != 0], h])
    low = min(-(float(t).as_integer_ratio()[1].bit_length() - 1) for t in x)
    if np.frexp(np.abs(x))[1].max() - 1 - low > 150:
        with pytest.raises(H.HQAError):
            H.ising_energy(H.Problem(U + U.T, h=h), np.ones((V, N), np.int8))
        return
    check(H, U + U.T, h, V, spread)


@pytest.mark.parametrize("prec,scale", [("fp8", 1.0), ("bf16", 1.0), ("f32", 1.0), ("f32", 2.0 ** -30)])
@pytest.mark.parametrize("N,R", [(33, 5), (130, 70)])
def test_storage_copies(H, prec, scale, N, R):
    """Read-outs take the couplings from the anneal's storage copy when it is exact."""
    J = inst.small_int(N, N, -3, 3) * scale
    md = H.MD(H.Problem(J), H.make_schedule(10, 5), R, prec, seed=3)
    md.run()
    g = md.classify(4)
    E, C = orc.energy(orc.Problem(N, J=J), g["spins"])
    assert np.array_equal(g["energy"], E) and np.array_equal(g["cut"], C)
    md.close()
