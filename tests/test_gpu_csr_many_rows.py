"""Sparse per-step kernel on many rows (rows side by side in a wavefront): a graph made of copies of
a small one, whose own run takes a wavefront a row, must give the small run in every copy, bit for
bit; and a state of 2^26 rows, more than a wavefront a row can launch."""
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


def _graph(kind):
    """Rows of 0 .. 13 ("few"), 0 .. 33 ("some") and 5 .. 60 couplings ("many")."""
    rng = np.random.default_rng(len(kind))
    N = {"few": 61, "some": 83, "many": 89}[kind]
    want = {"few": [0, 1, 2, 5, 6, 7], "some": [0, 15, 6, 17, 24, 5, 33], "many": [5, 60, 23, 44, 37]}[kind]
    J = np.zeros((N, N))
    for i in range(N - 1):
        w = want[i % len(want)]
        for j in rng.permutation(np.arange(i + 1, N))[:w // 2 + w % 2]:
            J[i, j] = J[j, i] = rng.uniform(-0.5, 0.5)
    return J, rng.uniform(-1, 1, N)


@pytest.mark.parametrize("kind,R", [(k, R) for k in ("few", "some", "many")
                                    for R in (1, 4, 5, 31, 32, 33, 63, 64, 65, 68, 96, 128, 129, 192, 257)])
def test_copies(H, kind, R):
    J, h = _graph(kind)
    N0, T = J.shape[0], 14
    rp, ci, v = inst.dense_to_csr(J)
    d = len(ci) / N0
    lo, hi = {"few": (0, 10), "some": (10, 20), "many": (20, 60)}[kind]
    assert lo <= d < hi
    K = max(int(600 * d / N0), 6500 // N0) + 2           # copies: at least 600 d rows, and 6500
    ci_k = (ci[None, :] + N0 * np.arange(K)[:, None]).astype(np.int32).ravel()
    rp_k = np.concatenate([[0], (rp[None, 1:] + len(ci) * np.arange(K)[:, None]).ravel()]).astype(np.int32)
    p0 = inst.random_pm1((R, N0), 5)

    def run(prob, p):
        md = H.MD(prob, H.make_schedule(T, 6), R, "f32", p0=p, plan="step")
        md.run(4)
        md.stats_window(4, 9)
        md.run()
        assert md.last_plan == "step"
        out = [md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM, H.HQA_STATE_STATMEAN)]
        out.append(md.field())
        md.close()
        return out
    small = run(H.Problem(row_ptr=rp, col=ci, val=v, h=h), p0)
    large = run(H.Problem(row_ptr=rp_k, col=ci_k, val=np.tile(v, K), h=np.tile(h, K)), np.tile(p0, (1, K)))
    for s, x in zip(small, large):
        assert np.array_equal(x.reshape(R, K, N0), np.broadcast_to(s[:, None, :], (R, K, N0)))


def test_rows_beyond_a_wavefront_each(H):
    """2^26 rows of one replica: one thread each, where a wavefront each is 2^32 threads, which a
    launch cannot have.  The first 400 rows are a ring; the start's signs depend on the seed and the
    row alone, so a ring of 400 rows with 600 rows beside it must run the same."""
    import torch
    ring = 400
    i = np.arange(ring)
    ci = np.sort(np.stack([(i - 1) % ring, (i + 1) % ring], 1), 1).astype(np.int32).ravel()
    v = np.where((ci.reshape(ring, 2) + i[:, None]) % 3 == 0, 1.0, -1.0).ravel()
    out = []
    for N in (1000, 1 << 26):
        rp = np.minimum(2 * np.arange(N + 1, dtype=np.int64), 2 * ring).astype(np.int32)
        md = H.MD(H.Problem(row_ptr=rp, col=ci, val=v), H.make_schedule(6, 3), 1, "f32", seed=9, plan="step")
        md.run()
        phi = torch.empty((1, N), dtype=torch.float64, device="cuda")
        H.hqa_md_state(md.h, 0, H.HQA_STATE_PHI, phi, H.HQA_DEVICE)
        out.append(phi)
        md.close()
    assert torch.equal(out[0][0], out[1][0, :1000])
    alone = out[0][0, ring:].abs()
    assert torch.equal(alone, alone[:1].expand_as(alone))
    tail = out[1][0, ring:].abs()
    assert bool((tail == alone[0]).all())
