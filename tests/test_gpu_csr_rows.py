"""Sparse per-step kernel over its replica chunks: row degrees around the batches of 8 and
16 couplings, replica counts around the lanes and chunks of every dispatch.

Replicas are independent and every chunk runs the same operations, so a run of R replicas
must equal, bit for bit, runs of its replicas 64 at a time (one chunk, one replica a lane);
those are checked against the oracle within the derived binary32 error bound.
"""
import numpy as np
import pytest

import oracle as orc
from f32_bound import f32_bound
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


def _graph(kind):
    """Symmetric couplings whose rows have 0 .. 35 entries ("few": below 10 on average)."""
    rng = np.random.default_rng(77 if kind == "few" else 78)
    N = 61 if kind == "few" else 83
    J = np.zeros((N, N))
    for i in range(N - 1):
        want = [0, 1, 7, 8, 9][i % 5] if kind == "few" else [0, 15, 16, 17, 24, 31, 33][i % 7]
        for j in rng.permutation(np.arange(i + 1, N))[:want // 2 + want % 2]:
            J[i, j] = J[j, i] = rng.uniform(-0.5, 0.5)
    return J, rng.uniform(-1, 1, N)


@pytest.mark.parametrize("kind", ["few", "many"])
@pytest.mark.parametrize("R", [1, 63, 64, 65, 128, 129, 191, 256, 260, 511, 1024])
def test_replica_chunks_agree(H, kind, R):
    J, h = _graph(kind)
    N, T = J.shape[0], 14
    assert (np.count_nonzero(J) < 10 * N) == (kind == "few")
    rp, ci, v = inst.dense_to_csr(J)
    prob = H.Problem(row_ptr=rp, col=ci, val=v, h=h)
    p0 = inst.random_pm1((R, N), 5)

    def run(p):
        md = H.MD(prob, H.make_schedule(T, 6), p.shape[0], "f32", p0=p, plan="step")
        md.run()
        return [md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM)] + [md.field()]
    whole = run(p0)
    for r in range(0, R, 64):
        for x, y in zip(whole, run(p0[r:r + 64])):
            assert np.array_equal(x[r:r + 64], y)
    if R <= 64:
        e, phis = f32_bound(orc, orc.Problem(N, row_ptr=rp, col=ci, val=v, h=h),
                            orc.MDParams(T=T, W=6), np.zeros((R, N)), p0, T)
        assert np.max(np.abs(whole[0] - phis[T])) <= e[T]
