"""Sort and reduction of the read-out at their edges: keys kept in LDS or read again (8192 spins,
4096 in binary64), replicas of a line dealt over the XCDs, many equal keys; row sums in one, two
and three words and in the accumulator.  Equal to the oracle, h_eff bit for bit."""
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


def readout(H, prob, N, R, prec, S, ns, pb=None):
    md = H.MD(prob, H.make_schedule(10, 5), R, prec, seed=1)
    md.set_state(H.HQA_STATE_WSUM, S)
    H.hqa_md_set_step(md.h, 10)
    bar = md.state(H.HQA_STATE_PHIBAR)
    for n in ns:
        g = md.classify(n, solve=0 < n <= 24)
        A, s = orc.classify(bar, n)
        assert np.array_equal(g["amb_idx"], A), n
        if pb is not None and 0 < n <= 24:
            he, _ = orc.reduce(pb, A, s)
            assert np.array_equal(g["h_eff"], he), n
    md.close()


@pytest.mark.parametrize("N,R,prec", [(1, 3, "f32"), (255, 300, "f32"), (257, 515, "f32"),
                                      (4096, 260, "f32"), (8192, 5, "f32"), (8193, 5, "f32"),
                                      (4096, 3, "f64"), (4097, 3, "f64")])
def test_sort(H, N, R, prec):
    """A ring (CSR: the binary32 state is replica-minor); window sums of few distinct sizes."""
    i = np.arange(N)
    rp = np.arange(N + 1, dtype=np.int32) * (2 if N > 2 else 0)
    col = np.sort(np.stack([(i - 1) % N, (i + 1) % N], 1), 1).ravel() if N > 2 else np.zeros(0)
    prob = H.Problem(row_ptr=rp, col=col, val=np.ones(col.size))
    rng = np.random.default_rng(N)
    S = rng.integers(-40, 41, (R, N)) * np.where(rng.random((R, N)) < 0.3, 1.0, 1e-3)
    readout(H, prob, N, R, prec, S, sorted({0, 1, min(N, 5), min(N, 70), N // 2, N}))


@pytest.mark.parametrize("bits", [3, 40, 52, 70, 95, 110, 130])
@pytest.mark.parametrize("N", [21, 64, 333])
def test_row_sums(H, bits, N):
    """Couplings of up to `bits` bits between the lowest and the highest: 1, 2 and 3 words, and
    beyond them the accumulator."""
    rng = np.random.default_rng(bits + N)
    m = rng.integers(-(1 << min(bits, 52)) + 1, 1 << min(bits, 52), (N, N)).astype(np.float64)
    if bits > 52:
        m = m * 2.0 ** rng.integers(0, bits - 52, (N, N))
    U = np.triu(m, 1) * 2.0 ** -60
    J, h = U + U.T, rng.integers(-3, 4, N).astype(np.float64)
    S = rng.normal(size=(4, N))
    readout(H, H.Problem(J, h=h), N, 4, "f32", S, [1, 5, 14], orc.Problem(N, J=J, h=h))
