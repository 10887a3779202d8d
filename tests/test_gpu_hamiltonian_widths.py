"""MD Hamiltonian of dense instances over the replica blocks it takes by size: blocks of 32 and 64
replicas where they give 256 workgroups, of 16 otherwise; the same bits for the same replica."""
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


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("N,R,width", [(131, 1101, 32), (131, 1923, 64), (33, 64 * 86 - 5, 64)])
def test_widths_agree(H, N, R, width, prec):
    tiles = -(-N // 16)
    assert -(-R // width) * tiles >= 256 and (width == 64 or -(-R // 64) * tiles < 256)
    J, h = inst.uniform_glass(N, 7)
    prob, sched = H.Problem(J, h=h), H.make_schedule(20, 5)
    p0 = inst.random_pm1((R, N), 3)

    def run(p):
        md = H.MD(prob, sched, p.shape[0], prec, p0=p)
        md.run(9)
        out = md.hamiltonian()
        md.close()
        return out
    whole = run(p0)
    for r in (0, 32, R - 16):                            # 16 replicas: one narrow block
        assert np.array_equal(whole[r:r + 16], run(np.ascontiguousarray(p0[r:r + 16])))
