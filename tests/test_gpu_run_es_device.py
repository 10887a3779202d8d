"""The checkpointed run's probabilities on the device: complete when the call returns, whatever the
handles' streams, and unharmed by the calls that follow at once on the same handle."""
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


@pytest.mark.parametrize("N,R", [(37, 5), (2000, 500)])
@pytest.mark.parametrize("own_es_stream", [False, True])
def test_device_prob_on_nonblocking_streams(H, N, R, own_es_stream):
    """12 R N bytes of probabilities (12 MB in the larger case, kept with the handle beside the
    features) go to a device tensor; host probabilities of an equal run are the reference."""
    import torch
    rp, ci, v = inst.er_sparse(N, 6.0, 3)
    prob, sched = H.Problem(row_ptr=rp, col=ci, val=v), H.make_schedule(60, 20)
    sm, se = torch.cuda.Stream(), torch.cuda.Stream()     # non-blocking
    es = H.ES(seed=4, stream=(se if own_es_stream else sm).cuda_stream)
    host = np.empty((R, N, 3), dtype=np.float32)
    md = H.MD(prob, sched, R, "f32", seed=2, stream=sm.cuda_stream)
    want_stop = md.run_es(es, 30, 10, 2, 2.0, prob=host)
    want = md.classify(0, prob=host)
    other = np.ascontiguousarray(host[::-1])
    for _ in range(3):
        md.reset(2)
        dev = torch.zeros((R * N, 3), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        assert md.run_es(es, 30, 10, 2, 2.0, prob=dev) == want_stop
        got = md.classify(0, prob=dev)
        md.classify(0, prob=other)                        # its scratch is the run's
        assert np.array_equal(dev.cpu().numpy().reshape(R, N, 3), host)
        for k in ("spins", "energy", "cut"):
            assert np.array_equal(got[k], want[k]), k
    md.close()
    es.close()
