"""MD Hamiltonian of dense instances (binary64 matrix product) at the edges of its tiles.

The reference is the oracle's H_MD on the exported state.  Both sides add the same
binary64 terms in different orders, so each sum of m terms may differ by m eps times the
sum of the terms' magnitudes, and the force enters the momentum once per spin.
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


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("N,R", [(1, 1), (2, 17), (15, 16), (16, 33), (17, 3), (63, 64), (65, 65),
                                 (80, 32), (131, 130)])
def test_dense_hamiltonian_tile_edges(H, N, R, prec):
    J, h = inst.uniform_glass(N, 500 + N)
    T = 40
    md = H.MD(H.Problem(J, h=h), H.make_schedule(T, 5), R, prec, seed=N + R)
    pb, mp = orc.Problem(N, J=J, h=h), orc.MDParams(T=T, W=5)
    for q in (0, 23):
        md.run(q)
        phi, p = md.state(H.HQA_STATE_PHI), md.state(H.HQA_STATE_P)
        pi = orc.integer_p(pb, mp, q, phi, p)
        ref = orc.hmd(pb, mp, q, phi, pi)
        mag = 0.04 * (0.5 * pi * pi + np.abs(phi) ** 6).sum(1) + 0.12 * (
            np.abs(phi) * (np.abs(phi) @ np.abs(J)) + np.abs(h) * phi * phi).sum(1)
        # the momentum term's own share: alpha |p| times the force's rounding
        mag += (0.04 * np.abs(pi) * 0.12 * (np.abs(phi) @ np.abs(J) + 2 * np.abs(h * phi))).sum(1)
        got = md.hamiltonian()
        assert np.all(np.abs(got - ref) <= 4.0 * (N + 16) * np.finfo(float).eps * (mag + 1e-300))
