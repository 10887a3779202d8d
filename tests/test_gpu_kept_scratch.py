"""Scratch kept with a handle, and couplings read where they lie: calls of changing sizes on one
handle give what a fresh handle gives, and closing it returns the memory."""
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


KEYS = ("spins", "amb_idx", "energy", "cut")


def test_changing_sizes(H):
    prob, sched = H.Problem(inst.sk(300, 1)), H.make_schedule(20, 5)
    md = H.MD(prob, sched, 96, "f32", seed=3)
    md.run()
    for n in (1, 14, 6, 0, 18, 3, 14):
        g = md.classify(n, solve=n > 0)
        fresh = H.MD(prob, sched, 96, "f32", seed=3)
        fresh.run()
        want = fresh.classify(n, solve=n > 0)
        assert np.array_equal(md.state(H.HQA_STATE_PHIBAR), fresh.state(H.HQA_STATE_PHIBAR))
        assert np.array_equal(md.hamiltonian(), fresh.hamiltonian())
        fresh.close()
        for k in KEYS:
            assert np.array_equal(g[k], want[k]), (n, k)
    md.close()


def test_large_scratch_is_given_back(H):
    """A read-out whose scratch is beyond what a handle keeps (R n^2 couplings of 8 bytes)
    leaves at most 64 MiB with it, and the handle's end leaves nothing."""
    import torch
    md = H.MD(H.Problem(inst.sk(64, 1)), H.make_schedule(10, 5), 40000, "f32", seed=3)
    md.run()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    md.classify(18, solve=True)                          # 104 MB of reduced couplings
    assert free0 - torch.cuda.mem_get_info()[0] <= (64 << 20)
    md.close()


@pytest.mark.parametrize("N", [5, 64, 201])
@pytest.mark.parametrize("offset", [0, 1])
def test_couplings_in_place(H, N, offset):
    """Dense device couplings from any 8-byte boundary; the caller's array is only read."""
    import torch
    J = inst.sk(N, 7)
    buf = torch.zeros(N * N + 1, dtype=torch.float64, device="cuda")
    buf[offset:offset + N * N] = torch.from_numpy(J.ravel())
    s = inst.random_pm1((40, N), 3).astype(np.int8)
    sd = torch.from_numpy(s).cuda()
    E = torch.zeros(40, dtype=torch.float64, device="cuda")
    C = torch.zeros_like(E)
    torch.cuda.synchronize()
    prob = H.hqa_problem(n=N, layout=H.HQA_DENSE, mem=H.HQA_DEVICE)
    prob.j = buf.data_ptr() + 8 * offset
    for _ in range(2):
        H.hqa_ising_energy(prob, sd, 40, E, C, H.HQA_DEVICE)
        Eo, Co = orc.energy(orc.Problem(N, J=J), s)
        assert np.array_equal(E.cpu().numpy(), Eo) and np.array_equal(C.cpu().numpy(), Co)
    assert np.array_equal(buf[offset:offset + N * N].cpu().numpy(), J.ravel())
