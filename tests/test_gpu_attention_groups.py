"""Tree attention with key groups (launches of few workgroups: the tiles of a
split are dealt to four, or two, groups of waves and combined in LDS), one
iteration against the oracle: prefixes of fewer tiles than groups, whole and
ragged numbers of 32-key tiles, trees of one to four q-tiles per KV head, with
head widths 64 and 128 and both element types.  Tolerances are the suite's:
1e-4 relative in fp32, 2e-2 in bf16."""
import pytest

import synth
from gpu_harness import inject, models, runtime
from parity_checks import Tally, oracle_iteration, run_and_compare
from test_gpu_configs import synthetic_state

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

WIDE = synth.ModelShape(2, 256, 2, 2, 128, 512, 1024)
GROUPED = synth.ModelShape(2, 512, 8, 2, 128, 1536, 4096)


@pytest.mark.parametrize("dtype,shape,budget,length", [
    ("f32", synth.TINY, 12, 1), ("f32", synth.TINY, 16, 31),
    ("f32", synth.TINY, 32, 97), ("f32", synth.TINY, 40, 128),
    ("f32", synth.TINY, 60, 129),
    ("f32", WIDE, 16, 33), ("f32", WIDE, 32, 127),
    ("bf16", GROUPED, 4, 32), ("bf16", GROUPED, 8, 95),
    ("bf16", GROUPED, 16, 64), ("bf16", GROUPED, 24, 200),
])
def test_key_groups(dtype, shape, budget, length):
    w = synth.Workload("groups", dtype, shape, 1, K=3, M=2, B_max=4,
                       budget=budget, n_seqs=1, prompt_len=(length, length))
    print("[groups]", dtype, shape.head_dim, budget, length, flush=True)
    weights, tgt, dr = models(w)
    st = synthetic_state(w, tgt, dr, 0, length, 300 + length)
    rt = runtime(w, weights, max_pages=(length + w.M * w.K + 16) // 16 + 1)
    inject(rt, 0, st)
    tol = 1e-4 if dtype == "f32" else 2e-2
    seqs = {0: (st,) + oracle_iteration(tgt, dr, st, w, 2)}
    run_and_compare(rt, seqs, w, tgt, dr, tol, Tally())
