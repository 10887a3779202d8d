"""Tabu read-out at the edges of its launch shapes (one spin a thread up to 512, two, four;
one to sixteen wavefronts) and in each form of the couplings, bit for bit with the oracle.

Window means are imported, so no anneal is needed; small integer and quarter-integer
couplings make ties between gains common.
"""
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


def _check(H, J, h, prec, R, ns, iters):
    N = J.shape[0]
    md = H.MD(H.Problem(J, h=h), H.make_schedule(10, 5), R, prec)
    S = np.random.default_rng(N).normal(size=(R, N)).astype(np.float32).astype(np.float64)
    md.set_state(H.HQA_STATE_WSUM, S)
    H.hqa_md_set_step(md.h, 10)
    bar = md.state(H.HQA_STATE_PHIBAR)
    pb = orc.Problem(N, J=J, h=h)
    for n in ns:
        tenure = max(1, n // 10)
        g = md.classify_tabu(n, iters, tenure)
        A, s = orc.classify(bar, n)
        he, Je = orc.reduce(pb, A, s)
        x0 = np.stack([s[r, A[r]] for r in range(R)])
        xb, db = orc.tabu(Je, he, x0, iters, tenure)
        assert np.array_equal(g["h_eff"], he), n
        assert np.array_equal(g["e_reduced"], db), n
        assert np.array_equal(g["spins"], orc.merge_x(s, A, xb)), n


WIDTHS = [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049]


@pytest.mark.parametrize("kind", ["int", "quarter"])
def test_every_width(H, kind):
    N = 2060
    J = inst.small_int(N, 3, -2, 2, density=0.2)
    if kind == "quarter":
        J = J * 0.25
    _check(H, J, None, "fp8", 2, WIDTHS, 80)


@pytest.mark.parametrize("prec,hi", [("fp8", 4), ("bf16", 100), ("f32", 100), ("fp8", 100),
                                     ("f32", 3000)])
def test_coupling_forms(H, prec, hi):
    """Exact in FP8, in BF16, in binary32; integers FP8 does not hold (the binary64 couplings);
    sums beyond the integer kernel's range (the binary64 search).  With integer fields."""
    N = 90
    J = inst.small_int(N, 5 + hi, -hi, hi, density=0.5)
    h = np.random.default_rng(hi).integers(-hi, hi + 1, N).astype(float)
    _check(H, J, h, prec, 3, [5, 64, 70, 90], 300)
