"""Exact energies of more vectors than the partial sums of one launch hold, with couplings of 10 to
20 digits: bit for bit with the oracle, which accumulates exactly and rounds once."""
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


def glass(N, spread, seed):
    """Symmetric normal couplings over `spread` binades (0: 10 digits, 80: 20), fields."""
    rng = np.random.default_rng(seed)
    U = np.triu(rng.normal(size=(N, N)) * 2.0 ** rng.integers(-spread, 1, size=(N, N)), 1)
    return U + U.T, rng.normal(size=N)


@pytest.mark.parametrize("N,spread,V", [(21, 0, 16400), (130, 0, 16400), (21, 80, 8193),
                                        (100, 80, 8192), (7, 80, 40)])
def test_vectors(H, N, spread, V):
    J, h = glass(N, spread, N)
    s = np.where(np.random.default_rng(V).random((V, N)) < 0.5, -1, 1).astype(np.int8)
    E, C = H.ising_energy(H.Problem(J, h=h), s)
    Eo, Co = orc.energy(orc.Problem(N, J=J, h=h), s)
    assert np.array_equal(E, Eo)
    assert np.array_equal(C, Co)


@pytest.mark.parametrize("spread,R", [(0, 16400), (80, 8193)])
def test_readouts(H, spread, R):
    """The same counts as replicas: one instance's read-out, several instances', and the pass."""
    import torch
    probs, orcs = [], []
    for k, N in enumerate((17, 24)):
        J, h = glass(N, spread, k)
        probs.append(H.Problem(J, h=h))
        orcs.append(orc.Problem(N, J=J, h=h))
    md = H.MD(probs, H.make_schedule(6, 3), R, "f32", seed=3)
    md.run()
    for k in range(2):
        g = md.classify(3, solve=True, k=k)
        Eo, Co = orc.energy(orcs[k], g["spins"])
        assert np.array_equal(g["energy"], Eo) and np.array_equal(g["cut"], Co)
        Em, Cm = md.classify_many(3, solve=True, instances=[k, 1 - k])
        assert np.array_equal(Em[0], Eo) and np.array_equal(Cm[0], Co)
        Ep, Cp = md.run_pass(3, 3, solve=True, graph=False)
        md.sync()
        torch.cuda.synchronize()
        assert np.array_equal(Ep[k].cpu().numpy(), Eo) and np.array_equal(Cp[k].cpu().numpy(), Co)
    md.close()


@pytest.mark.parametrize("N", [1, 2, 15, 16, 17])
@pytest.mark.parametrize("spread", [None, 0, 80])
def test_few_spins(H, N, spread):
    """The vector counts on both sides of the line between a workgroup a vector and the products."""
    J, h = glass(N, spread or 0, N)
    if spread is None:
        J, h = np.sign(J), None
    for V in (1, 17, 2048, 2049):
        s = np.where(np.random.default_rng(V).random((V, N)) < 0.5, -1, 1).astype(np.int8)
        E, C = H.ising_energy(H.Problem(J, h=h), s)
        Eo, Co = orc.energy(orc.Problem(N, J=J, h=h), s)
        assert np.array_equal(E, Eo) and np.array_equal(C, Co), V
