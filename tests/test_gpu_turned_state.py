"""Features and exports of a replica-minor (CSR) state at the edges of their tiles: 16 and 32 spins,
32 replicas, four replicas a workgroup of the sums."""
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


def run(H, prob, N, R, p0):
    md = H.MD(prob, H.make_schedule(60, 20), R, "f32", p0=p0)
    md.stats_window(10, 30, 2)
    md.run(30)
    out = [md.features()] + [md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P,
                                                   H.HQA_STATE_STATMEAN)]
    md.run()
    out.append(md.state(H.HQA_STATE_PHIBAR))
    md.close()
    return out


@pytest.mark.parametrize("N", [5, 15, 16, 17, 31, 33, 257, 600])
def test_replicas_do_not_depend_on_their_number(H, N):
    """Replica r has the same features and states whatever R is, bit for bit; and the features'
    scales follow from the exported fluxes: a binary32 sum of N squares in 256 chains and a tree
    is within (N / 256 + 9) 2^-24, a root and two quotients add less than 4 2^-24."""
    rp, ci, v = inst.dense_to_csr(inst.small_int(N, N, -2, 2, density=min(1.0, 8 / N)))
    prob = H.Problem(row_ptr=rp, col=ci, val=v)
    p0 = inst.random_pm1((70, N), 3)
    full = run(H, prob, N, 70, p0)
    for R in (1, 3, 4, 5, 31, 32, 33, 64):
        for x, y in zip(run(H, prob, N, R, p0[:R].copy()), full):
            assert np.array_equal(x, y[:R]), R
    f, phi, _, mean, _ = full
    sig = np.sqrt(np.mean(phi ** 2, axis=1, keepdims=True))
    tol = (N / 256 + 16) * 2.0 ** -24
    assert np.allclose(f[..., 3], phi / sig, rtol=tol, atol=0)
    assert np.allclose(f[..., 0], mean / sig, rtol=tol + 2.0 ** -22, atol=0)


@pytest.mark.parametrize("R", [1, 31, 33, 64])
def test_random_start(H, R):
    """The seeded momenta: those of the dense (replica-major) state."""
    N = 70
    J = inst.small_int(N, 1, density=0.2)
    rp, ci, v = inst.dense_to_csr(J)
    out = []
    for prob in (H.Problem(row_ptr=rp, col=ci, val=v), H.Problem(J)):
        md = H.MD(prob, H.make_schedule(60, 20), R, "f32", seed=9)
        out.append([md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P)])
        md.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)
