"""The commit's catch-up forward under a tight length bound: a catch-up row at
position T + a + 1 attends to every committed drafter entry, the a accepted
ones of this iteration among them, also when the bound is the one that a
prefill leaves (T + 1) or the least that the caller may set (T).  A two-layer
drafter, whose second layer's committed K/V depends on the first layer's
attention; paths that end at a node with no continuing row.  One iteration
against the oracle with the suite's fp32 tolerance, every drafter layer's
entries among the outputs."""
import pytest
import torch

import synth
from gpu_harness import inject, models, runtime
from parity_checks import Tally, oracle_iteration, run_and_compare
from test_gpu_configs import synthetic_state

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]
TOL = 1e-4


@pytest.mark.parametrize("lens,slack", [((7,), 0), ((7,), 1), ((3, 40), 1)])
def test_catch_up_sees_the_accepted_entries(lens, slack):
    w = synth.Workload("bound-fp32", "f32", synth.TINY, 2, K=3, M=2, B_max=4,
                       budget=40, n_seqs=len(lens),
                       prompt_len=(min(lens), max(lens)))
    w = synth.uniform_tree(w, 3)
    weights, tgt, dr = models(w)
    states = [synthetic_state(w, tgt, dr, s, n, 17) for s, n in enumerate(lens)]
    rt = runtime(w, weights, max_pages=(max(lens) + w.M * w.K + 16) // 16 + 1)
    forced = synth.uniform_buckets(w.n_seqs, rt.row_cap)
    rt.set_buckets(torch.as_tensor(forced).to(rt.dev))
    seqs = {}
    for s, st in enumerate(states):
        inject(rt, s, st)
        seqs[s] = (st,) + oracle_iteration(tgt, dr, st, w, w.M * w.K,
                                           forced[s])
        rec = seqs[s][2]
        assert rec["fallback"] and len(rec["path"]) == w.M * w.K, s
    rt.set_length_bound(max(lens) + slack)
    print("[bound]", lens, slack, flush=True)
    run_and_compare(rt, seqs, w, tgt, dr, TOL, Tally(), forced=forced)
    rt.set_buckets(None)
