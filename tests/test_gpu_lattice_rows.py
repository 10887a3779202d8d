"""Replica-resident anneal of graphs whose rows all have four or six couplings, or not: equal to
the streamed sparse kernel bit for bit, whatever the parity and the start of the steps."""
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


def circulant(N, hops, cut):
    """Every spin coupled to those 1 .. hops away on a ring; `cut` takes one bond out."""
    rng = np.random.default_rng(N)
    J = np.zeros((N, N))
    for k in range(1, hops + 1):
        i = np.arange(N)
        w = rng.normal(size=N)
        J[i, (i + k) % N] = w
        J[(i + k) % N, i] = w
    if cut:
        J[0, 1] = J[1, 0] = 0.0
    return J


@pytest.mark.parametrize("N", [9, 1000, 1024, 1025, 2049, 4096])
@pytest.mark.parametrize("hops,cut", [(2, False), (3, False), (3, True), (4, False)])
def test_rows(H, N, hops, cut):
    rp, ci, v = inst.dense_to_csr(circulant(N, hops, cut))
    prob = H.Problem(row_ptr=rp, col=ci, val=v, h=np.random.default_rng(1).normal(size=N))
    R, sched = 6, H.make_schedule(9, 4)
    out = []
    for plan, stops in (("step", [9]), ("resident", [9]), ("resident", [1, 2, 5, 8, 9]),
                        ("resident", [2, 3, 9])):
        md = H.MD(prob, sched, R, "f32", seed=2, plan=plan)
        for q in stops:
            md.run(q)
        assert md.last_plan == plan
        out.append([md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM)])
        md.close()
    for o in out[1:]:
        for x, y in zip(out[0], o):
            assert np.array_equal(x, y)
