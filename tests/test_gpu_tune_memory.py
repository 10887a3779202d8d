"""Tuning keeps the operand-order copies of the state only where its choice reads them."""
import numpy as np
import pytest

from paper_2004_03972_amd import instances as inst

pytestmark = pytest.mark.gpu


# a size whose state is large beside its couplings (one-launch plans win), and one that streams them
@pytest.mark.parametrize("N,R,prec", [(100, 131072, "bf16"), (60, 262144, "fp8"), (3000, 4096, "bf16")])
def test_copies_kept_by_choice(N, R, prec, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa as H
    monkeypatch.delenv("HQA_TUNE_CACHE", raising=False)
    J = np.sign(inst.sk(N, 1)) if prec == "fp8" else inst.sk(N, 1)
    md = H.MD(H.Problem(J), H.make_schedule(40, 5), R, prec, seed=1)
    md.run(2)
    copies = 2 * 2 * R * (-(-N // 128) * 128)               # two of BF16
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    md.tune(3)
    plan, *_, tiled = md.tuned_plan()
    torch.cuda.synchronize()
    kept = free - torch.cuda.mem_get_info()[0]
    print(N, R, prec, plan, tiled, kept / copies, flush=True)
    assert kept < copies / 2 or tiled
    md.run(9)                                                # the choice runs on, and a pinned tiled form after it
    md.set_step_tiles(1, 1, 8, tiled=True)
    md.run(40)
    x = md.state(H.HQA_STATE_PHI)
    md.close()
    md = H.MD(H.Problem(J), H.make_schedule(40, 5), R, prec, seed=1)
    md.run(40)
    assert np.array_equal(x, md.state(H.HQA_STATE_PHI))
    md.close()
