"""Prefill passes where they can go wrong, against the oracle's prefill: a
prompt of more rows than one pass takes (2048), prompts that begin, end and
continue inside a pass, lengths on and beside the 64-row pieces that the
attention works on, and a last piece of one row.  fp32 (16-row attention) and
bf16 with grouped queries (32x32 attention); caches of both models, roots and
condition taps."""
import numpy as np
import pytest
import torch

import synth
from oracle import specdec
from oracle.model import rmsnorm

from gpu_harness import host, models, rel_err, runtime

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

BF16 = synth.ModelShape(2, 512, 8, 2, 128, 1536, 4032)


def _workload(dtype, n):
    return synth.Workload("passes-" + dtype, dtype,
                          synth.TINY if dtype == "f32" else BF16, 1, K=4, M=2,
                          B_max=4, budget=16, n_seqs=n, prompt_len=(1, 2200))


@pytest.mark.parametrize("dtype,lens", [
    ("f32", [63, 64, 65, 1, 129, 1790, 40]),
    ("f32", [2113]),
    ("bf16", [65, 1, 64, 63, 1900, 128, 17]),
    ("bf16", [2049]),
])
def test_prefill_passes(dtype, lens):
    w = _workload(dtype, len(lens))
    tol = 1e-4 if dtype == "f32" else 2e-2     # the suite's bounds
    weights, tgt, dr = models(w)
    prompts = synth.prompts(w, lengths=lens)
    rt = runtime(w, weights, max_pages=(max(lens) + 16) // 16)
    print("[passes]", dtype, lens, flush=True)
    rt.prefill(prompts)
    torch.cuda.synchronize()
    for s, pr in enumerate(prompts):
        st = specdec.prefill(tgt, dr, pr)
        assert int(rt.T[s]) == st.T
        if dtype == "f32":
            assert int(rt.root[s]) == st.root
        else:
            # a near-tie may fall either way, another row's or another
            # prompt's root may not: the oracle's logits of the last position
            # (the last tap layer is the last layer) may each be off by tol
            h = tgt.num.act(rmsnorm(st.cond_taps[2], tgt.final_norm,
                                    tgt.shape.norm_eps))
            z = h @ tgt.lm_head.T
            assert z.argmax() == st.root
            assert z[int(rt.root[s])] >= z.max() - 2 * tol * np.abs(z).max(), s
        assert rel_err(host(rt.cond_taps[s]), st.cond_taps).max() < tol
        for which, kv in (("target", st.tkv), ("drafter", st.dkv)):
            got = rt.read_cache(which, s, st.T)
            for layer in range(len(kv.k)):
                for x, ref in ((got[0], kv.k), (got[1], kv.v)):
                    e = rel_err(x[layer].reshape(st.T, -1),
                                np.asarray(ref[layer]).reshape(st.T, -1))
                    assert e.max() < tol, (which, s, layer, e.argmax())


@pytest.mark.parametrize("dtype,chunk,lens", [
    ("f32", 16, [63, 1, 40]),
    ("f32", 48, [97, 17]),
    ("bf16", 16, [33, 65, 1]),
    ("bf16", 96, [200, 31]),
    ("bf16", 512, [513]),
])
def test_prefill_passes_in_the_least_workspace(dtype, chunk, lens):
    """Passes of prefill_chunk rows: pieces of fewer rows than 64, passes that
    end inside a prompt and that one piece fills."""
    w = _workload(dtype, len(lens))
    tol = 1e-4 if dtype == "f32" else 2e-2
    weights, tgt, dr = models(w)
    prompts = synth.prompts(w, lengths=lens)
    rt = runtime(w, weights, max_pages=(max(lens) + 16) // 16,
                 prefill_chunk=chunk, prefill_rows=0)
    print("[passes] least workspace", dtype, chunk, lens, flush=True)
    rt.prefill(prompts)
    torch.cuda.synchronize()
    for s, pr in enumerate(prompts):
        st = specdec.prefill(tgt, dr, pr)
        assert int(rt.T[s]) == st.T
        assert rel_err(host(rt.cond_taps[s]), st.cond_taps).max() < tol
        for which, kv in (("target", st.tkv), ("drafter", st.dkv)):
            got = rt.read_cache(which, s, st.T)
            for layer in range(len(kv.k)):
                for x, ref in ((got[0], kv.k), (got[1], kv.v)):
                    e = rel_err(x[layer].reshape(st.T, -1),
                                np.asarray(ref[layer]).reshape(st.T, -1))
                    assert e.max() < tol, (which, s, layer, e.argmax())
