"""Batches above and below the last-level cache's size, whose state passes it by or stays in it:
each streamed form equals the same instance run alone, one launch per step, bit for bit."""
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


@pytest.mark.parametrize("kind", ["bf16", "fp8", "bit"])
@pytest.mark.parametrize("N,R", [(129, 64 * 110 + 3), (260, 64 * 900 + 37)])
def test_state_size(H, kind, N, R):
    """20 N R bytes of state: 18 MB and 300 MB, with ragged rows and replicas."""
    J, h = inst.uniform_glass(N, 1)
    if kind == "fp8":
        J = inst.small_int(N, 2, -2, 2, density=0.4)
    elif kind == "bit":
        J = inst.er_maxcut(N, 0.2, 3)
    p = H.Problem(J, h=h, storage="bf16" if kind == "bf16" else "fp8")
    out = []
    for plan in ("batch", "step"):
        md = H.MD(p, H.make_schedule(4, 3), R, "bf16", seed=6, plan=plan)
        md.run(2)
        md.run()
        assert md.last_plan == plan
        out.append([md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM)])
        md.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)
