"""Per-step plan: the default block shape and the tiled form with its operand-order fluxes
give the states of a pinned untiled 1 x 1 block, bit for bit."""
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


def _run(H, prob, T, R, prec, tiles, cuts):
    md = H.MD(prob, H.make_schedule(T, 4), R, prec, seed=3)
    if tiles:
        md.set_step_tiles(*tiles[:3], tiled=tiles[3])
    out = []
    for q in cuts:
        md.run(q)
        out += [md.state(w) for w in (H.HQA_STATE_PHI, H.HQA_STATE_P, H.HQA_STATE_WSUM)]
        out.append(md.field())
    assert md.last_plan == "step"
    md.close()
    return out


# sizes whose default shapes are 1x1, 1x1, 2x1, 2x2 and 2x4
@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("N,R", [(1, 1), (130, 33), (1500, 64), (1500, 128), (1500, 256)])
def test_default_block_equals_pinned(H, N, R, prec):
    prob = H.Problem(inst.sk(N, N) if N > 1 else np.zeros((1, 1)))
    a = _run(H, prob, 9, R, prec, None, (4, 9))
    b = _run(H, prob, 9, R, prec, (1, 1, 4, False), (4, 9))
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


# 4608 rows and more: the update's state is requested with the last batch
@pytest.mark.parametrize("N,R", [(300, 5), (4500, 3), (4600, 17), (4737, 16)])
def test_tiled_runs_in_pieces(H, N, R):
    prob = H.Problem(inst.sk(N, 7))
    want = _run(H, prob, 10, R, "bf16", (1, 1, 4, False), (1, 4, 10))
    for cb in (4, 8):
        got = _run(H, prob, 10, R, "bf16", (1, 1, cb, True), (1, 4, 10))
        assert all(np.array_equal(x, y) for x, y in zip(got, want))


# the smallest sizes of a larger block, and of binary32's deeper one (2x1, 2x2 and 2x4)
@pytest.mark.parametrize("prec", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("N,R", [(4097, 16), (2049, 64), (4097, 64), (1100, 240), (1409, 1248), (3970, 256)])
def test_default_block_at_the_lines(H, N, R, prec):
    J = np.sign(inst.sk(N, 3)) if prec == "fp8" else inst.sk(N, 3)
    prob = H.Problem(J)
    a = _run(H, prob, 5, R, prec, None, (5,))
    b = _run(H, prob, 5, R, prec, (1, 1, 4, False), (5,))
    assert all(np.array_equal(x, y) for x, y in zip(a, b))


# short runs, which read the row-major state, between long ones, which read the copies
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("N,R", [(300, 5), (1300, 33), (2432, 17), (2433, 3)])
def test_tiled_short_and_long_runs(H, N, R, prec):
    J = np.sign(inst.sk(N, 2)) if prec == "fp8" else inst.sk(N, 2)
    prob = H.Problem(J)
    cuts = (1, 8, 9, 10, 32, 34, 35)
    want = _run(H, prob, 35, R, prec, (1, 1, 4, False), cuts)
    got = _run(H, prob, 35, R, prec, (1, 1, 8, True), cuts)
    assert all(np.array_equal(x, y) for x, y in zip(got, want))
