"""The caller bounds the workspace: the least one holds prefill passes of
prefill_chunk rows and is no larger than it was when a prefill ran in chunks
of that many rows (sizes recorded below; an embedder may have fixed its
workspace by them), a workspace of that size binds, and longer passes are the
caller's choice (sb_workspace_bytes_prefill).  No device is touched."""
import ctypes as C

import pytest

from paper_2605_07243_amd import binding as B
from test_abi import Fake, cfg, lib  # noqa: F401

LLAMA_8B = ((32, 4096, 32, 8, 128, 14336, 128256), (0, 16, 31))
LLAMA_70B = ((80, 8192, 64, 8, 128, 28672, 128256), (0, 40, 79))
BF16 = dict(dtype=B.SB_BF16, K=4, M=2, B_max=8, budget=60, max_pages=100)

CHUNKED = {
    # name: (model, configuration, bytes when prefill ran in chunks)
    "tiny": (None, dict(max_pages=20), 8768256),
    "8b": (LLAMA_8B, BF16, 198842624),
    "8b-small": (LLAMA_8B, {**BF16, "B_max": 2, "budget": 16,
                            "prefill_chunk": 16}, 25080320),
    "8b-16-sequences": (LLAMA_8B, {**BF16, "budget": 64, "max_seqs": 16,
                                   "max_pages": 200}, 1683372032),
    "8b-long": (LLAMA_8B, {**BF16, "K": 8, "B_max": 16, "budget": 128,
                           "max_pages": 300, "prefill_chunk": 512}, 794692096),
    "8b-adapting": (LLAMA_8B, {**BF16, "drafter_layers": 2,
                               "draft_vocab": 32000, "adapt_cap": 64},
                    216387840),
    "70b": (LLAMA_70B, {**BF16, "K": 6, "budget": 96, "max_seqs": 4,
                        "max_pages": 200, "prefill_chunk": 96}, 942242560),
}


@pytest.mark.parametrize("name", list(CHUNKED))
def test_workspace_is_bounded_by_the_caller(lib, name):  # noqa: F811
    model, kw, chunked = CHUNKED[name]
    c = cfg(**kw)
    if model is not None:
        c.target = B.ModelDims(*model[0], 500000.0, 1e-5)
        c.tap_layers[:] = model[1]
    least = lib.sb_workspace_bytes(C.byref(c))
    assert 0 < least <= chunked
    size = [lib.sb_workspace_bytes_prefill(C.byref(c), r)
            for r in (0, c.prefill_chunk, 1024, 2048, 4096)]
    assert least == size[0] == size[1] <= size[2] <= size[3] == size[4]
    if c.draft_vocab:      # binding reads d2t through the device's runtime
        return
    f = Fake()
    tl = (B.LayerWeights * c.target.n_layers)(
        *[B.LayerWeights(*[f.at()] * 6, None)] * c.target.n_layers)
    dl = (B.LayerWeights * c.drafter_layers)(
        *[B.LayerWeights(*[f.at()] * 7)] * c.drafter_layers)
    tw = B.TargetWeights(f.at(), tl, f.at(), f.at())
    dw = B.DrafterWeights(*([f.at()] * 6), dl, *([f.at()] * 4), None)
    ctx = C.c_void_p()
    assert lib.sb_create(C.byref(c), C.byref(ctx)) == B.SB_OK
    for n, code in ((least - 1, B.SB_EBUDGET), (least, B.SB_OK),
                    (chunked, B.SB_OK), (size[3], B.SB_OK)):
        assert lib.sb_bind(ctx, C.byref(tw), C.byref(dw), f.at(), n) == code, n
    lib.sb_destroy(ctx)


def test_invalid_configuration_has_no_size(lib):  # noqa: F811
    c = cfg(prefill_chunk=100)
    assert lib.sb_workspace_bytes_prefill(C.byref(c), 2048) == 0
