"""Stochastic acceptance over rows with special values.  A row that holds a NaN
or +inf has no distribution: nothing is accepted and the bonus is token 0, also
where only one 1024-token block of the row holds it.  A row of the type's
lowest value throughout is uniform (temperature above 1, so that it does not
overflow).  Masks of -inf and of the lowest value leave the tokens mass 0, in
single tokens and in whole blocks: the walk and the draw are the oracle's.  Both
entry points, with few rows and with the many that take the inner nodes'
statistics first."""
import numpy as np
import pytest
import torch

import synth
from oracle.sampling import accept_sample
from oracle.tree import DraftTree

from gpu_harness import host, runtime
from parity_checks import inject_tree

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]
LOWEST = np.finfo(np.float32).min


@pytest.fixture(scope="module", params=[1, 4], ids=["one-pass", "inner-first"])
def rt(request):
    w = synth.with_layers(synth.WORKLOADS["llama3-8b-k4"], 1)
    r = runtime(w, None, n_seqs=request.param)     # 4 x 60 rows: 123 MB
    r.vout["logits"] = torch.zeros(r.S * w.budget, w.target.vocab,
                                   dtype=torch.float32, device=r.dev)
    return r


def walk(rt, tree, z, ua, ub, temperature, noalloc):
    """The same tree and logits in every sequence; the last one's result."""
    n = len(tree)
    for s in range(rt.S):
        inject_tree(rt, s, tree, n)
        rt.vout["logits"][s * n:(s + 1) * n] = torch.as_tensor(z)
    u = [torch.as_tensor(np.tile(x, (rt.S, 1)).astype(np.float32)).to(rt.dev)
         for x in (ua, ub)]
    rt.accept_sample(temperature, *u, noalloc=noalloc)
    torch.cuda.synchronize()
    s = rt.S - 1
    a = int(rt.aout["n_accepted"][s])
    return list(host(rt.aout["path"][s, :a])), int(rt.aout["bonus"][s])


def two_children(V, tokens):
    t = DraftTree(5, 60)
    for x in tokens:
        t.add(x, 0, 0, 1, 0.0)
    return t


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("at", [0, 5000, 128255])
def test_row_without_a_distribution(rt, value, at, noalloc):
    V = rt.V
    t = two_children(V, [7000, 90000])
    z = np.random.default_rng(3).standard_normal((3, V)).astype(np.float32)
    z[0, [7000, 90000]] = 14.0
    z[0, at] = value
    print("[values]", value, at, noalloc, flush=True)
    u = np.full(60, 0.3)
    assert walk(rt, t, z, u, u, 1.0, noalloc) == ([], 0)


def test_row_of_the_lowest_value_is_uniform(rt):
    V = rt.V
    t = two_children(V, [])
    z = np.full((1, V), LOWEST, np.float32)
    for u in (0.0, 0.25, 0.7):
        path, bonus = walk(rt, t, z, np.zeros(60), np.full(60, u), 2.0, False)
        assert path == [] and abs(bonus - np.float32(u) * V) <= 1, (u, bonus)


@pytest.mark.parametrize("mask", [-np.inf, LOWEST])
@pytest.mark.parametrize("temperature", [0.7, 1.0, 1.6])
def test_masked_tokens_have_no_mass(rt, mask, temperature):
    V = rt.V
    rng = np.random.default_rng(4)
    t = two_children(V, [2048, 7000, 90000])
    z = rng.standard_normal((4, V)).astype(np.float32)
    z[0, 2048:2048 + 3 * 1024] = mask          # whole blocks, a child's token
    z[0, rng.choice(V, 5000, replace=False)] = mask
    z[0, 7000], z[0, 90000] = 9.0, 10.0
    exact = 0
    for trial in range(6):
        ua, ub = rng.random((2, 60)).astype(np.float32)
        with np.errstate(over="ignore"):
            ref = accept_sample(t, z.astype(np.float64), temperature, ua, ub)
        path, bonus = walk(rt, t, z, ua, ub, temperature, False)
        if ref["test_margin"] > 1e-4:
            assert path == ref["path"], trial
            end = path[-1] if path else 0
            assert z[end, bonus] > LOWEST, trial
            if ref["cdf_margin"] > 2e-6:
                assert bonus == ref["bonus"], trial
            exact += 1
    assert exact >= 4
