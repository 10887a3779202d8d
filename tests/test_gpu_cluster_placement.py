"""The cluster plan runs whichever XCD the device deals a launch's first workgroup to: after
other launches of 1 .. 9 workgroups, and back to back, it gives the per-step plan's states."""
import numpy as np
import pytest

from paper_2004_03972_amd import instances as inst

pytestmark = pytest.mark.gpu


def test_cluster_after_uneven_launches():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa as H
    T, R = 20, 40
    prob = H.Problem(inst.er_maxcut(400, 0.05, 9))
    want = H.MD(prob, H.make_schedule(T, 5), R, "fp8", seed=4, plan="step")
    want.run()
    want = want.state(H.HQA_STATE_WSUM)
    md = H.MD(prob, H.make_schedule(T, 5), R, "fp8", seed=4, plan="cluster")
    for k in range(1, 10):
        torch.ones(1024 * k, device="cuda").add_(1.0)
        other = H.MD(H.Problem(inst.sk(16 * k, k)), H.make_schedule(4, 2), 16, "f32", seed=k)
        other.run()
        other.sync()
        md.reset(4)
        md.run()
        md.sync()                                    # no placement error
        assert md.last_plan == "cluster"
        assert np.array_equal(md.state(H.HQA_STATE_WSUM), want)
        other.close()
