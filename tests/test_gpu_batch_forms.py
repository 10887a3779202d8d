"""Each kernel of the batched step, on sizes that the dispatch gives to it: ragged rows and replicas,
one instance and several, each streamed form; bit for bit with one launch per step and instance."""
import numpy as np
import pytest

from batch_form import form
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


def _problem(H, N, kind, seed):
    if kind == "bf16":
        J, h = inst.uniform_glass(N, seed)
    else:
        J = inst.small_int(N, seed, -2, 2, density=0.4) if kind == "fp8" else inst.er_maxcut(N, 0.2, seed)
        h = np.random.default_rng(seed).uniform(-1, 1, N)
    return H.Problem(J, h=h, storage="bf16" if kind == "bf16" else "fp8")


@pytest.mark.parametrize("sizes,kinds,R,want", [
    ([260], ["fp8"], 64 * 200 + 37, "cached"),
    ([260], ["bit"], 64 * 220 + 1, "cached"),
    ([2500], ["bf16"], 64 * 26 + 5, "cached"),
    ([2437, 2500, 2561], ["fp8", "bf16", "bit"], 64 * 9 - 7, "cached"),
    ([129], ["bf16"], 64 * 300 + 3, "narrow 4"),
    ([385, 129, 300, 256], ["bf16", "fp8", "bit", "bf16"], 64 * 45 + 1, "narrow 4"),
    ([200, 333, 520], ["bf16", "bit", "fp8"], 64 * 18 + 9, "narrow 2"),
    ([70, 200, 333], ["bit", "fp8", "bf16"], 100, "narrow 1"),
    ([2437, 2500, 2561], ["bf16", "fp8", "bit"], 64 * 28 - 3, "streamed")])
def test_forms(H, sizes, kinds, R, want):
    assert form(sizes, kinds, R) == want
    probs = [_problem(H, N, k, 3 + x) for x, (N, k) in enumerate(zip(sizes, kinds))]
    md = H.MD(probs, H.make_schedule(4, 3), R, "bf16", seed=6, plan="batch" if len(sizes) == 1 else "auto")
    md.run(1)
    md.run()
    assert md.last_plan == "batch"
    assert [md.batch_form(k) for k in range(len(sizes))] == kinds
    ref = H.MD(probs, H.make_schedule(4, 3), R, "bf16", seed=6, plan="step")
    ref.run()
    assert ref.last_plan == "step"
    for k in range(len(sizes)):
        for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM):
            assert np.array_equal(md.state(w, k), ref.state(w, k)), (k, w)
    md.close()
    ref.close()
