"""Batch plan in each replica width of its tiles (64, 32 and 16): instances of every
streamed form equal the same instances run alone, one launch per step, bit for bit."""
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


def _check(H, sizes, R, T):
    probs = []
    for k, N in enumerate(sizes):
        J, h = [(inst.sk(N, k), None), (inst.er_maxcut(N, 0.1, k), None),
                (inst.small_int(N, k, -2, 2, density=0.3), None), inst.uniform_glass(N, k)][k % 4]
        probs.append(H.Problem(J, h=h, storage="fp8" if k % 4 in (1, 2) else "bf16"))
    md = H.MD(probs, H.make_schedule(T, 3), R, "bf16", seed=6)
    md.run(T // 2)
    md.run()
    assert md.last_plan == "batch"
    for k, p in enumerate(probs):
        one = H.MD(p, H.make_schedule(T, 3), R, "bf16", seed=6, plan="step")
        one.run()
        for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM):
            assert np.array_equal(md.state(w, k), one.state(w)), (k, w)
        one.close()


@pytest.mark.parametrize("R", [1, 16, 17, 32, 33, 64, 65, 100])
def test_small_batches(H, R):
    """Up to 96 tiles: 16 replicas a tile, ragged in rows and replicas."""
    _check(H, [1, 127, 200, 385], R, 6)


@pytest.mark.parametrize("R", [20, 64, 96])
def test_medium_batches(H, R):
    """97 .. 320 tiles of 64: 32 replicas a tile."""
    _check(H, [2600, 2500, 2450, 2400, 2300, 900], R, 4)


def test_large_batches(H):
    """Above 320 tiles: 64 replicas a tile, the last one ragged."""
    _check(H, [600, 500, 450, 300], 64 * 21 + 5, 4)
