"""Head-only update of a fragment-packed bf16 head at the edges of its
matrix-core step: a few buffered positions, one more than a 16-position
contraction step, and the full 64; a drafter vocabulary whose row blocks do
not fill the last workgroup.  Against the oracle's step with the bounds of
test_gpu_adapt."""
import pytest
import torch

import synth
import test_gpu_adapt as base

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

SHAPE = synth.ModelShape(1, 512, 8, 2, 128, 1536, 8192)
W = synth.Workload("adapt-edge", "bf16", SHAPE, 1, K=4, M=2, B_max=4,
                   budget=16, n_seqs=1, prompt_len=(16, 16))


@pytest.mark.parametrize("n", [4, 17, 64])
def test_head_update_edges(monkeypatch, n):
    monkeypatch.setitem(synth.WORKLOADS, W.name, W)
    monkeypatch.setitem(base.CASES, "edge", (W.name, 8128, 64, n, 0.05))
    c = base._setup("edge")
    loss = torch.zeros(1, dtype=torch.float32, device=c["rt"].dev)
    torch.cuda.synchronize()
    c["rt"].head_update(c["buf"], c["lm0"], c["train"], c["lr"], c["kl"], loss)
    torch.cuda.synchronize()
    assert int(c["buf"]["count"][0]) == 0
    base._check_against_oracle(c, c["train"], loss)
