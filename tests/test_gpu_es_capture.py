"""A training step on device data without a loss is stream work alone: it may be captured as a
classifier's first call, and later calls on larger batches leave the captured step intact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa
    hqa.lib()
    return hqa


@pytest.mark.parametrize("n", [1, 65, 5000])
def test_first_step_captured(H, n):
    """The captured step holds Adam's step 1; parameters set anew make every replay that step,
    with eager work on 40,000 samples (512 partial sums instead of a few) in between."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    big = 40000
    x = torch.randn((big, 12), generator=g, device="cuda")
    y = torch.randint(0, 3, (big,), generator=g, device="cuda", dtype=torch.int32)
    cw = torch.tensor([0.8, 0.9, 1.4], device="cuda")
    xb, yb = x.cpu().numpy(), y.cpu().numpy()
    torch.cuda.synchronize()
    ref = H.ES(seed=5)
    P0 = ref.params
    H.hqa_es_train_step(ref.h, x, y, n, cw, 3e-3, None, H.HQA_DEVICE)
    want = ref.params
    assert not np.array_equal(want, P0)
    s = torch.cuda.Stream()
    es = H.ES(seed=5, stream=s.cuda_stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s, capture_error_mode="thread_local"):
        H.hqa_es_train_step(es.h, x, y, n, cw, 3e-3, None, H.HQA_DEVICE)
    for k in range(3):
        es.params = P0
        with torch.cuda.stream(s):
            graph.replay()
        assert np.array_equal(es.params, want), k
        assert es.grad(xb, yb, cw.cpu().numpy())[0] > 0.0      # eager, the largest batch
        torch.cuda.synchronize()
    es.close()
    ref.close()
