"""Stochastic acceptance of many rows, where the statistics of leaves are
taken only for the nodes that the walks end at (96 MiB of logits and more):
same results as the small-call path on the same trees, logits and uniforms,
for trees of one node (the walk ends at a leaf at once), chains and bushy
ones, and against the oracle's walk."""
import numpy as np
import pytest
import torch

import synth
from oracle.sampling import accept_sample

from gpu_harness import host, runtime
from parity_checks import inject_tree
from test_gpu_sampling import MARGIN, random_tree, synthetic_logits

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]


def test_inner_nodes_first_matches_one_pass():
    w = synth.with_layers(synth.WORKLOADS["llama3-8b-k4"], 1)
    V, budget, cap = w.target.vocab, w.budget, w.M * w.K
    S = 4                                   # 4 x 60 x 128256 x 4 B: 123 MB
    rt = runtime(w, None, n_seqs=S)
    rt.vout["logits"] = torch.zeros(S * budget, V, dtype=torch.float32,
                                    device=rt.dev)
    one = runtime(w, None, n_seqs=1)        # 31 MB: the one-pass path
    one.vout["logits"] = torch.zeros(budget, V, dtype=torch.float32,
                                     device=one.dev)
    for trial in range(4):
        rng = np.random.default_rng([29, trial])
        sizes = [budget, 1, 2, int(rng.integers(3, budget))]
        trees, zs = [], []
        for s in range(S):
            t = random_tree(rng, sizes[s], cap, V)
            trees.append(t)
            zs.append(synthetic_logits(rng, t, V))
            inject_tree(rt, s, t, len(t))
        rows = np.concatenate(zs)
        rt.vout["logits"][:len(rows)] = torch.as_tensor(rows)
        ua = rng.random((S, budget)).astype(np.float32)
        ub = rng.random((S, budget)).astype(np.float32)
        print("[inner] trial", trial, [len(t) for t in trees], flush=True)
        rt.accept_sample(1.0, torch.as_tensor(ua).to(rt.dev),
                         torch.as_tensor(ub).to(rt.dev))
        torch.cuda.synchronize()
        for s, t in enumerate(trees):
            a = int(rt.aout["n_accepted"][s])
            path = list(host(rt.aout["path"][s, :a]))
            bonus = int(rt.aout["bonus"][s])
            inject_tree(one, 0, t, len(t))
            one.vout["logits"][:len(t)] = torch.as_tensor(zs[s])
            one.accept_sample(1.0, torch.as_tensor(ua[s:s + 1]).to(rt.dev),
                              torch.as_tensor(ub[s:s + 1]).to(rt.dev))
            torch.cuda.synchronize()
            assert a == int(one.aout["n_accepted"][0]), (trial, s)
            assert path == list(host(one.aout["path"][0, :a])), (trial, s)
            assert bonus == int(one.aout["bonus"][0]), (trial, s)
            ref = accept_sample(t, zs[s].astype(np.float64), 1.0,
                                ua[s].astype(np.float64),
                                ub[s].astype(np.float64))
            if ref["test_margin"] > MARGIN:
                assert path == ref["path"], (trial, s)
