"""hqa_ising_energy on device couplings: the whole N x N array has to lie in its allocation."""
import ctypes as C

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


@pytest.mark.parametrize("N,spare", [(33, 0), (33, 3), (100, 0)])
def test_couplings_end_with_their_allocation(H, N, spare):
    """Couplings that end at the allocation's last byte are read; an array that is one value too
    short is refused (8 bytes, within the memory page, so that no access leaves mapped memory)."""
    import torch
    L = H.lib()
    J = inst.sk(N, 7)
    s = inst.random_pm1((5, N), 3).astype(np.int8)
    sd = torch.from_numpy(s).cuda()
    E = torch.zeros(5, dtype=torch.float64, device="cuda")
    cut = torch.zeros_like(E)
    p = C.c_void_p()
    n = N * N + spare
    assert L.hipMalloc(C.byref(p), C.c_size_t(8 * n)) == 0
    try:
        host = np.zeros(n)
        host[spare:] = J.ravel()
        assert L.hipMemcpy(p, C.c_void_p(host.ctypes.data), C.c_size_t(8 * n), 1) == 0
        torch.cuda.synchronize()
        prob = H.hqa_problem(n=N, layout=H.HQA_DENSE, mem=H.HQA_DEVICE)
        prob.j = p.value + 8 * spare
        H.hqa_ising_energy(prob, sd, 5, E, cut, H.HQA_DEVICE)
        Eo, Co = orc.energy(orc.Problem(N, J=J), s)
        assert np.array_equal(E.cpu().numpy(), Eo) and np.array_equal(cut.cpu().numpy(), Co)
        assert (8 * n) % 4096 != 0
        prob.j = p.value + 8 * (spare + 1)
        with pytest.raises(H.HQAError):
            H.hqa_ising_energy(prob, sd, 5, E, cut, H.HQA_DEVICE)
        # the refusal leaves nothing behind for the next call
        prob.j = p.value + 8 * spare
        H.hqa_ising_energy(prob, sd, 5, E, cut, H.HQA_DEVICE)
        assert np.array_equal(E.cpu().numpy(), Eo)
    finally:
        assert L.hipFree(p) == 0
