"""Next-block starts of a block of more than 64 nodes, some of them with a
cumulative log-probability that is not a number: those are never picked, and
hide no other candidate (a lane of the selection holds nodes 64 apart).  Eight
starts get ten nodes each and no chain end; one start's own cumulative
log-probability is NaN, so that its nodes' are; the picks must be the rank >= 2
nodes by cumulative log-probability, ties to the lower id, of the others."""
import numpy as np
import pytest
import torch

import synth
from gpu_harness import host, models, runtime

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]


@pytest.mark.parametrize("nan_start", [0, 3, 7])
def test_nan_candidates_hide_no_other(nan_start):
    w = synth.Workload("starts-nan", "f32", synth.TINY, 1, K=2, M=2, B_max=8,
                       budget=128, n_seqs=1, prompt_len=(12, 12),
                       branch_map=(0, 10, 10, 0))
    weights, _, _ = models(w)
    rt = runtime(w, weights, max_pages=4)
    buckets = np.zeros((1, rt.row_cap), np.int32)
    buckets[0, :2] = 1                       # block 1: ten nodes per row
    buckets[0, 2::2] = 1                     # block 2: ten at k = 1, none at 2
    rt.set_buckets(torch.as_tensor(buckets).to(rt.dev))
    rt.prefill(synth.prompts(w))
    rt.expand(1)
    torch.cuda.synchronize()
    assert int(rt.tree["n_nodes"][0]) == 21
    assert int(rt.tree["n_starts"][0]) == 8
    starts = host(rt.tree["starts"])[0]
    for b, n in enumerate(starts):           # the last starts' nodes are best
        rt.tree["cum_logp"][0, int(n)] = \
            float("nan") if b == nan_start else -100.0 + 10.0 * b
    print("[starts-nan]", nan_start, flush=True)
    rt.expand(2)
    torch.cuda.synchronize()
    t = {f: host(rt.tree[f])[0] for f in ("parent", "rank", "cum_logp")}
    assert int(rt.tree["n_nodes"][0]) == 101
    mine = [n for n in range(21, 101) if t["parent"][n] == starts[nan_start]]
    assert len(mine) == 10 and np.isnan(t["cum_logp"][mine]).all()
    cand = [n for n in range(21, 101)
            if t["rank"][n] >= 2 and not np.isnan(t["cum_logp"][n])]
    cand.sort(key=lambda n: (-t["cum_logp"][n], n))
    assert int(rt.tree["n_starts"][0]) == 8
    assert list(host(rt.tree["starts"])[0]) == cand[:8]
    rt.set_buckets(None)
