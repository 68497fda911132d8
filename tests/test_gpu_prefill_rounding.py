"""Rounding of the attention probabilities in a long prefill piece (32x32
kernel, bf16): P is rounded to bf16 relative to each tile of 64 keys' own
largest score, whose probability is then exact, and not relative to one
reference for a whole split.  Both are emulated in the oracle (everything else
in float64, rounded where the device rounds); the device's distance from the
unrounded oracle has to be on the tile side of the two, by more than halfway on
a log scale.  Scores are spread (queries and keys of layer 0 scaled by 4, exact
in bf16), so that few keys carry a row and the two differ by far more than the
last-bit flips that another summation order gives."""
import numpy as np
import pytest
import torch

import oracle.model
import synth
from gpu_harness import runtime
from oracle import specdec
from oracle.model import Drafter, Target
from oracle.numerics import round_bf16

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

SHAPE = synth.ModelShape(2, 512, 8, 2, 128, 1536, 4032)
W = synth.Workload("rounding", "bf16", SHAPE, 1, K=4, M=2, B_max=4, budget=16,
                   n_seqs=1, prompt_len=(1024, 1024))
TILE = 64


def rounded_attend(per_tile):
    def attend(q, keys, vals):
        n, H = len(keys), q.shape[0]
        kh = np.arange(H) // (H // keys.shape[1])
        s = np.einsum("hd,nhd->hn", q, keys[:, kh]) / np.sqrt(q.shape[1])
        s *= np.log2(np.e)
        ref = np.full(H, -1e30)
        o, l = np.zeros_like(q), np.zeros(H)
        for a in range(0, n, TILE):
            t = s[:, a:a + TILE]
            mx = t.max(1)
            new = mx if per_tile else np.where(mx > ref + 8, mx, ref)
            scale = np.exp2(np.maximum(ref - new, -1e4))
            p = np.exp2(t - new[:, None])
            l = l * scale + p.sum(1)
            o = o * scale[:, None] + np.einsum(
                "hn,nhd->hd", round_bf16(p), vals[a:a + TILE][:, kh])
            ref = new
        return (o / l[:, None]).reshape(-1)
    return attend


def emulated(prompt, weights, dw, attend=None):
    """Layer-1 K and V of the oracle's prefill, with `attend` in its place."""
    tgt = Target(weights, W.target, W.dtype, W.tap_layers)
    dr = Drafter(dw, W.target, W.dtype, W.drafter_layers, tgt.embed)
    plain = oracle.model.attend
    oracle.model.attend = attend or plain
    try:
        kv = specdec.prefill(tgt, dr, prompt).tkv
    finally:
        oracle.model.attend = plain
    return np.stack([kv.k[1], kv.v[1]])


def setup():
    tw = synth.make_weights(synth.target_specs(SHAPE), 0, W.dtype, jitter=0.1)
    dw = synth.drafter_weights(W, 0, jitter=0.1)
    for n in ("layers.0.wq", "layers.0.wk"):
        tw[n] = tw[n] * 4
    return tw, dw, synth.prompts(W)


def test_prefill_rounds_relative_to_each_tile():
    tw, dw, prompts = setup()
    ref = emulated(prompts[0], tw, dw)
    rel = lambda x: np.linalg.norm(x - ref) / np.linalg.norm(ref)  # noqa: E731
    tile = rel(emulated(prompts[0], tw, dw, rounded_attend(True)))
    split = rel(emulated(prompts[0], tw, dw, rounded_attend(False)))
    rt = runtime(W, {**tw, **dw}, max_pages=65)
    print("[rounding] prefill", flush=True)
    rt.prefill(prompts)
    torch.cuda.synchronize()
    k, v = rt.read_cache("target", 0, 1024)
    got = rel(np.stack([k[1], v[1]]).reshape(ref.shape))
    print(f"[rounding] device {got:.3e}, emulated per tile {tile:.3e}, per "
          f"split {split:.3e}", flush=True)
    assert tile < split
    assert got < np.sqrt(tile * split), (got, tile, split)
