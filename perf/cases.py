"""The work that a program gives this library, as cases that can be timed and compared.

A serving loop calls, per verifier iteration, M block expansions, one tree
verification, the acceptance walk and the commit; a prefill when a prompt
arrives; and now and then a head-only update of the drafter.  Each case is
one of these calls (acceptance and commit together) at the layer shapes and
tree sizes of the repository's workloads, with a target of a few layers.

``prepare`` builds what the program holds before the call: random weights
N(0, 0.02), page tables in random order, a prefix of random K/V, trees whose
shape depends on the case alone (so that every seed does the same work) and
whose tokens come from the seed.  Trees are grown as the library grows them,
with the rank-head buckets drawn from a fixed mix instead of from logits, so
that a near-tie of two logits cannot change which rows a later call has.  For
the same reason token ids that an argmax or a top-10 picks (the verify argmax,
the prefill's root, the drafter's top-10 ids, buckets, new tree nodes) are not
among the outputs; the logits, the sorted top-10 values, psi, hidden states
and K/V they are taken from are.
"""
from __future__ import annotations

import math
import random
import types
import zlib

import numpy as np
import torch

from paper_2605_07243_amd.runtime import Runtime

# layer shapes: d, query heads, KV heads, head dim, MLP width, vocabulary
SHAPES = {"8b": (4096, 32, 8, 128, 14336, 128256),
          "70b": (8192, 64, 8, 128, 28672, 128256),
          "tiny": (256, 4, 4, 64, 1024, 1024)}
BRANCH = (2, 4, 6, 4)        # bucket -> tokens attached
# rank-head buckets of the trees: the class frequencies of a trained rank
# head (three rows in four attach two tokens: narrow trees that stay below
# the budget), or every row in b1 (wide trees that fill it)
MIXES = {"trained": (0.752, 0.902, 0.943), "wide": None}
BASE = dict(model="8b", dtype="bf16", layers=4, drafter_layers=1,
            draft_vocab=0, K=4, M=2, B_max=8, budget=60, seqs=1, lo=1024,
            hi=1024, mix="wide", chunk=128)


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one tree of a toy model in fp32, where launches
        # and host time count
        _case(name="verify-tiny-fp32", kind="verify", model="tiny",
              dtype="f32", layers=2, M=3, B_max=4, budget=32, lo=128, hi=128),
        # block 1 of a single conversation: K rows, a stream of all drafter
        # weights and of a full-vocabulary LM head
        _case(name="first-block-8b", kind="first"),
        # a later block of the two-layer drafter with the reduced vocabulary
        _case(name="next-block-8b-2layer", kind="next", drafter_layers=2,
              draft_vocab=32000),
        # a later block of a batch of 16 conversations of mixed lengths
        _case(name="next-block-8b-batch16", kind="next", budget=64, seqs=16,
              lo=512, hi=2048),
        # verification of one conversation's tree, the call that an iteration
        # spends most of its time in
        _case(name="verify-8b", kind="verify", layers=8),
        # a deep tree over a long prefix
        _case(name="verify-8b-long", kind="verify", K=8, B_max=16, budget=128,
              lo=4096, hi=4096),
        # trees of 16 conversations of mixed lengths
        _case(name="verify-8b-batch16", kind="verify", budget=64, seqs=16,
              lo=512, hi=2048),
        # four trees through the wider model's layers
        _case(name="verify-70b-batch4", kind="verify", model="70b", layers=2,
              K=6, budget=96, seqs=4, lo=2048, hi=2048),
        # one prompt arriving
        _case(name="prefill-8b-1024", kind="prefill"),
        # a batch of prompts of mixed lengths arriving
        _case(name="prefill-8b-batch16", kind="prefill", budget=64, seqs=16,
              lo=512, hi=2048),
        # sampled acceptance (temperature 1) and the commit of 16 trees
        _case(name="accept-commit-8b-batch16", kind="commit", budget=64,
              seqs=16, lo=512, hi=2048, mix="trained"),
        # a full buffer of rejected positions stepping the drafter's heads
        _case(name="head-update-8b", kind="update", positions=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["first", "next", "verify", "verify", "prefill",
                       "prefill", "commit", "update"])
    if kind == "update":
        return _case(kind=kind, positions=_log(rng, 1, 64),
                     draft_vocab=rng.choice([0, 64 * _log(rng, 125, 1000)]))
    model = rng.choice(["8b", "8b", "8b", "tiny", "70b"])
    seqs = _log(rng, 1, 4 if model == "70b" else 16)
    K = rng.randint(2, 8)
    M = rng.randint(2, 3)
    B_max = min(_log(rng, 2, 16), (512 - K) // ((M - 1) * K))
    lo = _log(rng, 5, 1400)
    hi = min(2048 if seqs > 1 else 4096, lo + rng.choice([0, _log(rng, 8, 1500)]))
    if seqs == 1 and rng.random() < 0.3:
        lo = hi = _log(rng, 1500, 4096)
    chunk = rng.choice([64, 128, 128, 256])
    if kind == "prefill":                    # no dearer than the listed ones
        most = (4096 if model == "70b" else 16384) // seqs
        lo, hi = min(lo, most), min(hi, most)
        chunk = 128 if seqs * hi > 4096 else chunk
    budget = min(_log(rng, 16, 160), 1024 // seqs)
    if kind in ("next", "commit"):
        budget = max(budget, 4 * K + 8)      # room after the first block
    return _case(kind=kind, model=model,
                 dtype="f32" if model == "tiny" else "bf16",
                 layers=rng.randint(1, 3 if model == "70b" else 4),
                 drafter_layers=rng.choice([1, 1, 2]),
                 draft_vocab=0 if model == "tiny" else
                 rng.choice([0, 0, 32 * _log(rng, 250, 1500)]),
                 K=K, M=M, B_max=B_max,
                 budget=budget, seqs=seqs,
                 lo=lo, hi=hi, mix=rng.choice(["wide", "trained"]),
                 chunk=chunk)


# ---------------------------------------------------------------------------
# what a case stands for, from the case alone

def _workload(c):
    """The workload description the runtime takes."""
    d, H, Hkv, hd, F, V = SHAPES[c["model"]]
    L = c["layers"]
    t = types.SimpleNamespace(n_layers=L, d_model=d, n_heads=H,
                              n_kv_heads=Hkv, head_dim=hd, d_ff=F, vocab=V,
                              rope_theta=500000.0, norm_eps=1e-5,
                              q_dim=H * hd, kv_dim=Hkv * hd)
    return types.SimpleNamespace(
        name="case", dtype=c["dtype"], target=t,
        drafter_layers=c["drafter_layers"], K=c["K"], M=c["M"],
        B_max=c["B_max"], budget=c["budget"], n_seqs=c["seqs"],
        prompt_len=(c["lo"], c["hi"]), branch_map=BRANCH,
        draft_vocab=c["draft_vocab"], tap_layers=(0, L // 2, L - 1))


def _lengths(c):
    """Prefix (or prompt) lengths of the sequences."""
    r = random.Random("%d %d %d" % (c["lo"], c["hi"], c["seqs"]))
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["seqs"])]


def _max_pages(c):
    return (c["hi"] + 64 * (c["M"] * c["K"] + 1) + 15) // 16


def _grow(c, s, blocks):
    """Nodes, drafter rows and next starts of sequence s after `blocks`
    expansions: siblings attached in (k, start, rank) order within the
    budget, then chain ends and the likeliest b1/b2 siblings as starts."""
    K, budget = c["K"], c["budget"]
    r = random.Random("%d %d %d %d %s %d" % (K, c["M"], c["B_max"], budget,
                                             c["mix"], s))
    edges = MIXES[c["mix"]]
    nodes = [dict(parent=-1, depth=0, row=-1, rank=0, logp=0.0, cum=0.0)]
    rows, starts = [], [0]
    for m in range(1, blocks + 1):
        base, first_new = len(rows), len(nodes)
        buckets = []
        for b, sn in enumerate(starts):
            old = rows[nodes[sn]["row"]]["vis"] if m > 1 else []
            for k in range(1, K + 1):
                own = [base + b * K + q for q in range(k)]
                rows.append(dict(block=m, start=sn, k=k,
                                 depth=nodes[sn]["depth"] + k, vis=old + own))
                u = r.random()
                buckets.append(1 if edges is None
                               else sum(u >= e for e in edges))
        alive, chain = [True] * len(starts), list(starts)
        for k in range(1, K + 1):
            for b in range(len(starts)):
                if not alive[b]:
                    continue
                i = b * K + k - 1
                first, p = len(nodes), nodes[chain[b]]
                for rank in range(1, BRANCH[buckets[i]] + 1):
                    if len(nodes) >= budget:
                        break
                    lp = -0.5 * rank - r.random()
                    nodes.append(dict(parent=chain[b], depth=p["depth"] + 1,
                                      row=base + i, rank=rank, logp=lp,
                                      cum=p["cum"] + lp))
                alive[b] = first < budget
                if alive[b]:
                    chain[b] = first
        starts = []
        if len(nodes) < budget:
            starts = [chain[b] for b in range(len(chain)) if alive[b]]
            sib = [n for n in range(first_new, len(nodes))
                   if nodes[n]["rank"] >= 2
                   and buckets[nodes[n]["row"] - base] in (1, 2)]
            sib.sort(key=lambda n: (-nodes[n]["cum"], n))
            starts = (starts + sib)[:c["B_max"]]
    return nodes, rows, starts


def _rows(c):
    """Live rows of the call the case makes."""
    if c["kind"] == "first":
        return c["seqs"] * c["K"]
    if c["kind"] == "next":
        return sum(len(_grow(c, s, 1)[2]) * c["K"] for s in range(c["seqs"]))
    return sum(len(_grow(c, s, c["M"])[0]) for s in range(c["seqs"]))


def work(c):
    """What the call cannot do without: weights, prefix K/V and inputs read
    once, outputs written once."""
    d, H, Hkv, hd, F, V = SHAPES[c["model"]]
    es = 2 if c["dtype"] == "bf16" else 4
    layer = d * (H + 2 * Hkv) * hd + d * H * hd + 3 * d * F
    Vd = c["draft_vocab"] or V
    if c["kind"] == "update":
        n = c["positions"]
        return {"bytes": 3 * Vd * d * es + n * d * 4, "flops": 6 * n * Vd * d}
    L, LD, S = c["layers"], c["drafter_layers"], c["seqs"]
    T = _lengths(c)
    kv = 2 * Hkv * hd * es
    if c["kind"] == "prefill":
        n = sum(T)
        par = L * layer + 5 * d * d + LD * (layer + 2 * d * d)
        return {"bytes": es * (par + V * d + n * d) + n * kv * (L + LD)
                + S * 3 * d * 4,
                "flops": 2 * n * par + 2 * S * V * d
                + 2 * sum(t * t for t in T) * H * hd * (L + LD)}
    if c["kind"] == "commit":
        a = 3 * S                      # accepted tokens, about
        return {"bytes": (a + S) * V * 4 + 2 * (a + S) * kv * (L + LD)
                + S * 3 * d * 8, "flops": 4 * (a + S) * V}
    R = _rows(c)
    per = R / S
    if c["kind"] == "verify":
        return {"bytes": es * (L * layer + V * d + R * d) + L * sum(T) * kv
                + R * (V + 3 * d) * 4,
                "flops": 2 * R * (L * layer + V * d)
                + sum(4 * per * (t + per / 4) * H * hd * L for t in T)}
    par = 2 * d * d + LD * (layer + 2 * d * d) + Vd * d
    cond = 3 * d * d if c["kind"] == "first" else 0
    return {"bytes": es * (par + cond + R * d) + LD * sum(T) * kv
            + R * (Vd + d) * 4,
            "flops": 2 * R * par + 2 * S * cond
            + sum(4 * per * (t + per / 4) * H * hd * LD for t in T)}


def tolerance(c):
    """About four times the distance from `exact` that was measured: fp32
    5e-7; bf16 drafter calls 5e-3, target and prefill 1e-2 to 1.5e-2 over 1 to
    8 layers (a changed summation order moves values across rounding
    boundaries, and those differences travel through the layers that follow),
    head updates 7e-5 (a step far below the spacing of most bf16 weights)."""
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 4e-4}
    if c["kind"] == "update":
        return {"rel": 3e-4, "max": 0.05}
    if c["kind"] in ("first", "next"):
        return {"rel": 2e-2, "max": 0.3}
    return {"rel": 3e-2, "max": 0.4}


# ---------------------------------------------------------------------------
# inputs

def _gen(seed, name, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed((seed * 1000003 + zlib.crc32(name.encode())) % (2 ** 63))
    return g


def _normal(seed, name, shape, dtype, std):
    t = torch.randn(shape, generator=_gen(seed, name), device="cuda",
                    dtype=torch.float32)
    return t.mul_(std).to(dtype)


class _Weights(dict):
    """Weights by the runtime's names, made when asked for."""

    def __init__(self, c, seed):
        super().__init__()
        d, H, Hkv, hd, F, V = SHAPES[c["model"]]
        self.c, self.seed, self.V = c, seed, V
        self.Vd = c["draft_vocab"] or V
        self.shapes = {"wq": (H * hd, d), "wk": (Hkv * hd, d),
                       "wv": (Hkv * hd, d), "wo": (d, H * hd), "wg": (F, d),
                       "wu": (F, d), "wd": (d, F), "w_shift": (d, 2 * d),
                       "embed": (V, d), "lm_head": (V, d),
                       "d.lm_head": (self.Vd, d), "d.w_cond": (d, 3 * d),
                       "d.w_fuse": (d, 3 * d), "d.pos_query": (c["K"], d),
                       "d.rank_w": (4, d + 15), "d.rank_b": (4,)}
        self.d = d

    def __missing__(self, name):
        if name == "d.d2t":
            if self.Vd == self.V:
                raise KeyError(name)
            r = np.random.default_rng([self.seed, 7])
            return np.sort(r.choice(self.V, self.Vd, replace=False)).astype(
                np.int32)
        key = name if name in self.shapes else name.split(".")[-1]
        if "norm" in key:
            return 1 + _normal(self.seed, name, (self.d,), torch.float32, 0.1)
        dt = (torch.float32 if name.startswith("d.rank")
              or self.c["dtype"] == "f32" else torch.bfloat16)
        return _normal(self.seed, name, self.shapes[key], dt, 0.02)


def _tables(c, seed):
    n = c["seqs"] * _max_pages(c)
    r = np.random.default_rng([seed, 3])
    return [r.permutation(n).astype(np.int32).reshape(c["seqs"], -1)
            for _ in range(2)]


def _pools(c, seed):
    """Contents of the target's and drafter's K and V pools."""
    _, _, Hkv, hd, _, _ = SHAPES[c["model"]]
    n = c["seqs"] * _max_pages(c)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    out = []
    for name, L in (("t", c["layers"]), ("d", c["drafter_layers"])):
        for x, shape in (("k", (16, hd)), ("v", (hd, 16))):
            t = torch.empty((L, n, Hkv) + shape, dtype=dt, device="cuda")
            out.append(t.normal_(generator=_gen(seed, name + x)))
    return out


def _words(bits, n_words):
    w = np.zeros(n_words, np.uint32)
    for b in bits:
        w[b >> 5] |= np.uint32(1 << (b & 31))
    return w.view(np.int32)


def _tokens(c, seed):
    r = np.random.default_rng([seed, 5])
    V = SHAPES[c["model"]][5]
    return np.stack([r.choice(V, c["budget"], replace=False)
                     for _ in range(c["seqs"])]).astype(np.int32)


def _tree(c, seed, blocks, row_cap):
    """The runtime's tree fields (all but h_last) after `blocks` expansions."""
    S, bud = c["seqs"], c["budget"]
    tok, T = _tokens(c, seed), _lengths(c)
    i32 = lambda *s: np.zeros(s, np.int32)  # noqa: E731
    rw = (row_cap + 31) // 32
    t = dict(n_nodes=i32(S), token=tok, parent=i32(S, bud), depth=i32(S, bud),
             row=i32(S, bud), rank=i32(S, bud),
             logp=np.zeros((S, bud), np.float32),
             cum_logp=np.zeros((S, bud), np.float32),
             anc=i32(S, bud, (bud + 31) // 32), n_rows=i32(S),
             row_block=i32(S, row_cap), row_start=i32(S, row_cap),
             row_k=i32(S, row_cap), row_pos=i32(S, row_cap),
             row_vis=i32(S, row_cap, rw), n_starts=i32(S),
             starts=i32(S, c["B_max"]))
    for s in range(S):
        nodes, rows, starts = _grow(c, s, blocks)
        for i, n in enumerate(nodes):
            for f, g in (("parent", "parent"), ("depth", "depth"),
                         ("row", "row"), ("rank", "rank"), ("logp", "logp"),
                         ("cum_logp", "cum")):
                t[f][s, i] = n[g]
            t["anc"][s, i] = _words(_anc(nodes, i), t["anc"].shape[2])
        for i, r in enumerate(rows):
            t["row_block"][s, i], t["row_start"][s, i] = r["block"], r["start"]
            t["row_k"][s, i], t["row_pos"][s, i] = r["k"], T[s] + r["depth"]
            t["row_vis"][s, i] = _words(r["vis"], rw)
        t["n_nodes"][s], t["n_rows"][s] = len(nodes), len(rows)
        t["n_starts"][s] = len(starts)
        t["starts"][s, :len(starts)] = starts
    return t


def _anc(nodes, i):
    out = []
    while i >= 0:
        out.append(i)
        i = nodes[i]["parent"]
    return out[::-1]


def _put(rt, t):
    for f, a in t.items():
        rt.tree[f].copy_(torch.from_numpy(a))


def _taps_in(c, seed):
    return _normal(seed, "cond_taps", (c["seqs"], 3, SHAPES[c["model"]][0]),
                   torch.float32, 1.0)


def _accept_inputs(c, seed):
    """Target logits of every node (children's tokens likely, as a drafter
    that is right three times in four has them) and the uniforms."""
    S, bud, V = c["seqs"], c["budget"], SHAPES[c["model"]][5]
    z = torch.randn((S * bud, V), generator=_gen(seed, "z"), device="cuda")
    tok = _tokens(c, seed)
    rest = math.log(V) + 0.5
    idx, val, base = [], [], 0
    for s in range(S):
        nodes = _grow(c, s, c["M"])[0]
        for i, n in enumerate(nodes):
            if n["parent"] >= 0:
                idx.append((base + n["parent"], int(tok[s, i])))
                val.append(rest + (1.5 if n["rank"] == 1 else -1.0))
        base += len(nodes)
    if idx:
        ij = torch.tensor(idx, device="cuda")
        z[ij[:, 0], ij[:, 1]] = torch.tensor(val, device="cuda")
    u = torch.rand((2, S, bud), generator=_gen(seed, "u"), device="cuda")
    return z, u[0].contiguous(), u[1].contiguous()


def _prompts(c, seed):
    r = np.random.default_rng([seed, 11])
    return [r.integers(0, SHAPES[c["model"]][5], n) for n in _lengths(c)]


def prepare(c, seed):
    rt = Runtime(_workload(c), _Weights(c, seed), max_pages=_max_pages(c),
                 prefill_chunk=c["chunk"],
                 adapt_cap=64 if c["kind"] == "update" else 0)
    st = dict(kind=c["kind"], rt=rt)
    if c["kind"] == "update":
        buf = rt.adapt_buffer()
        n = c["positions"]
        buf["h"][:n] = _normal(seed, "h", (n, rt.w.target.d_model),
                               torch.float32, 1.0)
        buf["target"][:n] = torch.from_numpy(_targets(c, seed)).to("cuda")
        train = rt.head_copy()
        train["lm_head"].add_(_normal(seed, "step", train["lm_head"].shape,
                                      torch.bfloat16, 0.002))
        st.update(buf=buf, n=n, train=train, lm0=rt._keep[4]["lm_head"],
                  loss=torch.zeros(1, dtype=torch.float32, device="cuda"))
        return st
    tables = _tables(c, seed)
    rt.tpt.copy_(torch.from_numpy(tables[0]))
    rt.dpt.copy_(torch.from_numpy(tables[1]))
    if c["kind"] == "prefill":
        st["prompts"] = _prompts(c, seed)
        return st
    for dst, src in zip((rt.tk, rt.tv, rt.dk, rt.dv), _pools(c, seed)):
        dst.copy_(src)
    T = _lengths(c)
    rt.T.copy_(torch.tensor(T, dtype=torch.int32))
    rt.root.copy_(torch.from_numpy(_tokens(c, seed)[:, 0].copy()))
    rt.cond_taps.copy_(_taps_in(c, seed))
    rt.set_length_bound(max(T) + 1)
    if c["kind"] == "verify":
        _put(rt, _tree(c, seed, c["M"], rt.row_cap))
    if c["kind"] == "next":
        rt.expand(1)
        _put(rt, _tree(c, seed, 1, rt.row_cap))
        fields = [rt.tree[f] for f in ("n_nodes", "n_rows", "n_starts",
                                       "starts")]
        st.update(fields=fields, saved=[f.clone() for f in fields])
    if c["kind"] == "commit":
        for m in range(1, c["M"] + 1):
            rt.expand(m)
            _put(rt, _tree(c, seed, m, rt.row_cap))
        rt.verify(want_logits=True)
        z, st["u_accept"], st["u_bonus"] = _accept_inputs(c, seed)
        rt.vout["logits"].copy_(z)
        st.update(T=rt.T.clone(), bound=max(T) + 1)
    return st


def run(st):
    rt = st["rt"]
    if st["kind"] == "prefill":
        rt.prefill(st["prompts"])
        return dict(tk=rt.tk, tv=rt.tv, dk=rt.dk, dv=rt.dv, T=rt.T,
                    cond_taps=rt.cond_taps)
    if st["kind"] == "verify":
        rt.verify(want_logits=True)
        return dict(logits=rt.vout["logits"], taps=rt.vout["taps"])
    if st["kind"] == "commit":
        # the same iteration each time: T back to where it was
        rt.T.copy_(st["T"])
        rt.set_length_bound(st["bound"])
        rt.accept_sample(1.0, st["u_accept"], st["u_bonus"])
        rt.commit()
        return dict(n_accepted=rt.aout["n_accepted"], path=rt.aout["path"],
                    bonus=rt.aout["bonus"], r_reject=rt.aout["r_reject"],
                    T=rt.T, root=rt.root, cond_taps=rt.cond_taps,
                    tk=rt.tk, tv=rt.tv, dk=rt.dk, dv=rt.dv)
    if st["kind"] == "update":
        st["buf"]["count"].fill_(st["n"])
        rt.head_update(st["buf"], st["lm0"], st["train"], 0.1, 0.1,
                       st["loss"])
        return dict(st["train"], loss=st["loss"])
    if st["kind"] == "next":
        # the same block each time: the tree back to where block 1 left it
        torch._foreach_copy_(st["fields"], st["saved"])
        rt.expand(2, want_logits=True)
    else:
        rt.expand(1, want_logits=True)
    o = rt.dout
    return dict(logits=o["logits"], topk_logit=o["topk_logit"], lse=o["lse"],
                psi=o["psi"], h_last=rt.tree["h_last"])


# ---------------------------------------------------------------------------
# the same in float64

def _targets(c, seed):
    r = np.random.default_rng([seed, 13])
    return r.integers(0, SHAPES[c["model"]][5], c["positions"]).astype(np.int32)


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5) * g


def _rope(x, pos):
    half = x.shape[-1] // 2
    j = torch.arange(half, dtype=torch.float64, device="cuda")
    ang = pos.double()[:, None] * 500000.0 ** (-2.0 * j / (2 * half))
    co, si = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * co - b * si, b * co + a * si], -1)


class _Ref:
    """Rows are grouped by sequence: `n[s]` rows of sequence s, each with a
    position, a segment slot and a mask over segment slots."""

    def __init__(self, c, seed, pools=None):
        self.c, self.w = c, _Weights(c, seed)
        self.d, self.H, self.Hkv, self.hd, _, _ = SHAPES[c["model"]]
        self.T = _lengths(c)
        self.tables = [torch.from_numpy(t).long().to("cuda")
                       for t in _tables(c, seed)]
        self.pools = pools
        cap = max(_row_cap(c), c["budget"])
        z = lambda L: [torch.zeros((L, c["seqs"], cap, self.Hkv, self.hd),  # noqa: E731
                                   dtype=torch.float64, device="cuda")
                       for _ in range(2)]
        self.seg = ([z(c["layers"]), z(c["drafter_layers"])]
                    if pools is not None else None)
        self.emb = self.w["embed"]

    def lin(self, x, name):
        return x @ self.w[name].double().t()

    def prefix(self, which, layer, s):
        k, v = self.pools[2 * which][layer], self.pools[2 * which + 1][layer]
        n = self.T[s]
        pg = self.tables[which][s, :(n + 15) // 16]
        K = k[pg].double().permute(0, 2, 1, 3).reshape(-1, self.Hkv, self.hd)
        V = v[pg].double().permute(0, 3, 1, 2).reshape(-1, self.Hkv, self.hd)
        return K[:n], V[:n]

    def layer(self, which, layer, x, n, pos, slots, masks, kv_out=None):
        p = ("d." if which else "") + "layers.%d." % layer
        H, Hkv, hd = self.H, self.Hkv, self.hd
        a = _rms(x, self.w[p + "attn_norm"].double())
        q = _rope(self.lin(a, p + "wq").view(-1, H, hd), pos)
        k = _rope(self.lin(a, p + "wk").view(-1, Hkv, hd), pos)
        v = self.lin(a, p + "wv").view(-1, Hkv, hd)
        del a
        o = torch.empty_like(q)
        at = 0
        for s, m in enumerate(n):
            r = slice(at, at + m)
            at += m
            if m == 0:
                continue
            if self.pools is None:           # causal, no prefix
                K, V, mask = k[r], v[r], masks
            else:
                sk, sv = self.seg[which][0][layer, s], self.seg[which][1][layer, s]
                sk[slots[s]], sv[slots[s]] = k[r], v[r]
                pk, pv = self.prefix(which, layer, s)
                m_ = masks[s].shape[1]
                K, V = torch.cat([pk, sk[:m_]]), torch.cat([pv, sv[:m_]])
                mask = torch.cat([torch.ones((m, len(pk)), dtype=torch.bool,
                                             device="cuda"), masks[s]], 1)
            G = H // Hkv
            for h in range(H):
                sc = q[r, h] @ K[:, h // G].t() / math.sqrt(hd)
                if isinstance(mask, str):      # "causal"
                    sc = sc.masked_fill(torch.ones_like(
                        sc, dtype=torch.bool).triu(1), -math.inf)
                else:
                    sc = sc.masked_fill(~mask, -math.inf)
                o[r, h] = torch.softmax(sc, -1) @ V[:, h // G]
        x = x + self.lin(o.reshape(-1, H * hd), p + "wo")
        del q, o
        if kv_out is not None:
            kv_out.append((k, v))
        b = _rms(x, self.w[p + "mlp_norm"].double())
        g = self.lin(b, p + "wg")
        g = g * torch.sigmoid(g)
        g *= self.lin(b, p + "wu")
        return x + self.lin(g, p + "wd")

    def target(self, tok, n, pos, slots, masks, kv_out=None):
        x = self.emb[tok].double()
        L = self.c["layers"]
        taps = []
        for i in range(L):
            x = self.layer(0, i, x, n, pos, slots, masks, kv_out)
            taps += [(j, x) for j, t in enumerate((0, L // 2, L - 1)) if t == i]
        return x, torch.stack([t for _, t in sorted(taps, key=lambda e: e[0])], 1)

    def cond(self, taps):
        return self.lin(taps.reshape(len(taps), -1), "d.w_cond")

    def drafter(self, cond, tok, k, pred, n, pos, slots, masks, kv_out=None):
        w = self.w
        x = torch.cat([_rms(cond, w["d.norm_c"].double()),
                       _rms(self.emb[tok].double(), w["d.norm_e"].double()),
                       _rms(w["d.pos_query"][k - 1].double(),
                            w["d.norm_q"].double())], 1)
        x = self.lin(x, "d.w_fuse")
        for i in range(self.c["drafter_layers"]):
            x = self.lin(torch.cat([x, x[pred]], 1), "d.layers.%d.w_shift" % i)
            x = self.layer(1, i, x, n, pos, slots, masks, kv_out)
        return x

    def head(self, x):
        return self.lin(_rms(x, self.w["d.final_norm"].double()), "d.lm_head")

    # drafter rows of block m of every sequence, in call order
    def block(self, m, tokens, h_last, taps):
        c, K = self.c, self.c["K"]
        tok, ks, pred, n, pos, slots, masks, cond, where = ([] for _ in range(9))
        c1 = self.cond(taps) if m == 1 else None
        at = 0
        for s in range(c["seqs"]):
            nodes, _, starts = _grow(c, s, m - 1)
            rows = _grow(c, s, m)[1] if starts else _grow(c, s, m - 1)[1]
            base = len(_grow(c, s, m - 1)[1])
            new = list(range(base, len(rows)))
            mask = torch.zeros((len(new), len(rows)), dtype=torch.bool)
            for i, r in enumerate(new):
                row = rows[r]
                sn = row["start"]
                tok.append(int(tokens[s, sn]))
                ks.append(row["k"])
                pred.append(at + i - (1 if row["k"] > 1 else 0))
                pos.append(self.T[s] + row["depth"])
                mask[i, row["vis"]] = True
                cond.append(c1[s] if m == 1 else h_last[s, nodes[sn]["row"]])
                where.append((s, r))
            at += len(new)
            n.append(len(new))
            slots.append(torch.tensor(new, dtype=torch.long, device="cuda"))
            masks.append(mask.to("cuda"))
        t = lambda a: torch.tensor(a, dtype=torch.long, device="cuda")  # noqa: E731
        if not where:
            return None, where
        x = self.drafter(torch.stack(cond), t(tok), t(ks), t(pred), n, t(pos),
                         slots, masks)
        for i, (s, r) in enumerate(where):
            h_last[s, r] = x[i]
        return x, where


def _row_cap(c):
    return c["K"] + (c["M"] - 1) * c["B_max"] * c["K"]


def _psi(z):
    lse = torch.logsumexp(z, -1, keepdim=True)
    top = z.topk(10, -1).values
    lp = top - lse
    ent = -(torch.exp(z - lse) * (z - lse)).sum(-1, keepdim=True)
    psi = torch.cat([lp, top[:, :1] - top[:, [1, 2, 4]], torch.exp(lp[:, :1]),
                     ent], 1)
    return top, lse[:, 0], psi


def _exact_update(c, seed):
    w = _Weights(c, seed)
    n, d = c["positions"], w.d
    Vd = w.Vd
    rb, kb = Vd // 32, d // 64
    pack = lambda t: t.view(rb, 32, kb, 2, 4, 8).permute(2, 0, 4, 3, 1, 5)  # noqa: E731
    w0 = w["d.lm_head"]
    packed = pack(w0).reshape(Vd, d)
    packed = packed.add(_normal(seed, "step", (Vd, d), torch.bfloat16, 0.002))
    w1 = packed.view(kb, rb, 4, 2, 32, 8).permute(1, 4, 0, 3, 2, 5)
    w1 = w1.reshape(Vd, d).double()
    h = _normal(seed, "h", (n, d), torch.float32, 1.0).double()
    a = _rms(h, w["d.final_norm"].double())
    z, z0 = a @ w1.t(), a @ w0.double().t()
    y = _targets(c, seed)
    if Vd != w.V:
        d2t = w["d.d2t"]
        i = np.minimum(np.searchsorted(d2t, y), Vd - 1)
        y = np.where(d2t[i] == y, i, -1)
    y = torch.from_numpy(y).long().to("cuda")
    has = y >= 0
    at = y.clamp(min=0)[:, None]
    lp, lp0 = torch.log_softmax(z, 1), torch.log_softmax(z0, 1)
    p = lp.exp()
    kl = (p * (lp - lp0)).sum(1, keepdim=True)
    g = p.clone()
    g.scatter_add_(1, at, -torch.ones_like(g[:, :1]))
    g = g * has[:, None] + 0.1 * p * (lp - lp0 - kl)
    rank = (z > z.gather(1, at)).sum(1) + 1
    b = torch.where(rank == 1, 0, torch.where(rank <= 4, 1,
                    torch.where(rank <= 10, 2, 3)))
    b = torch.where(has, b, torch.full_like(b, 3))
    x = torch.cat([h, _psi(z)[2]], 1)
    rw, rbias = w["d.rank_w"].double(), w["d.rank_b"].double()
    ls = torch.log_softmax(x @ rw.t() + rbias, 1)
    q = ls.exp()
    q.scatter_add_(1, b[:, None], -torch.ones_like(q[:, :1]))
    loss = (-(lp.gather(1, at)[:, 0] * has) + 0.1 * kl[:, 0]
            - ls.gather(1, b[:, None])[:, 0]).mean()
    w1 -= 0.1 / n * (g.t() @ a)
    return dict(lm_head=pack(w1).reshape(Vd, d), rank_w=rw - 0.1 / n * (q.t() @ x),
                rank_b=rbias - 0.1 / n * q.sum(0), loss=loss.reshape(1))


def _scatter(k, v, table, s, e, K, V):
    """K, V [L][n] of entries e of sequence s into the pools."""
    pg, sl = table[s][e // 16], e % 16
    for i in range(len(K)):
        k[i][pg, :, sl, :] = K[i].to(k.dtype)
        v[i][pg, :, :, sl] = V[i].to(v.dtype)


def _exact_prefill(c, seed):
    ref = _Ref(c, seed)
    prompts, n = _prompts(c, seed), ref.T
    tok = torch.from_numpy(np.concatenate(prompts)).long().to("cuda")
    pos = torch.cat([torch.arange(m, device="cuda") for m in n])
    tkv, dkv = [], []
    _, taps = ref.target(tok, n, pos, None, "causal", tkv)
    ends = np.cumsum(n)
    cond = torch.cat([torch.zeros((1, 3, ref.d), dtype=torch.float64,
                                  device="cuda"), taps[:-1]])
    first = torch.from_numpy(ends - np.array(n)).long().to("cuda")
    cond[first] = 0
    one = torch.ones_like(tok)
    ref.drafter(ref.cond(cond), tok, one, torch.arange(len(tok), device="cuda"),
                n, pos + 1, None, "causal", dkv)
    del cond
    out = [torch.zeros_like(p, dtype=torch.float64) for p in _pools(c, 0)]
    for which, kv in ((0, tkv), (1, dkv)):
        at = 0
        for s, m in enumerate(n):
            _scatter(out[2 * which], out[2 * which + 1], ref.tables[which], s,
                     torch.arange(m, device="cuda"),
                     [k[at:at + m] for k, _ in kv],
                     [v[at:at + m] for _, v in kv])
            at += m
    return dict(tk=out[0], tv=out[1], dk=out[2], dv=out[3], T=None,
                cond_taps=taps[torch.from_numpy(ends - 1).to("cuda")])


def _verify(ref, c, seed):
    tokens, n, tok, pos, slots, masks = _tokens(c, seed), [], [], [], [], []
    for s in range(c["seqs"]):
        nodes = _grow(c, s, c["M"])[0]
        m = torch.zeros((len(nodes), len(nodes)), dtype=torch.bool)
        for i, nd in enumerate(nodes):
            m[i, _anc(nodes, i)] = True
            pos.append(ref.T[s] + nd["depth"])
        n.append(len(nodes))
        tok += [int(t) for t in tokens[s, :len(nodes)]]
        slots.append(torch.arange(len(nodes), device="cuda"))
        masks.append(m.to("cuda"))
    t = lambda a: torch.tensor(a, dtype=torch.long, device="cuda")  # noqa: E731
    x, rows = ref.target(t(tok), n, t(pos), slots, masks)
    taps = torch.zeros((c["seqs"], c["budget"], 3, ref.d), dtype=torch.float64,
                       device="cuda")
    at = 0
    for s, m in enumerate(n):
        taps[s, :m] = rows[at:at + m]
        at += m
    return x, taps


def _exact_commit(c, seed, ref, h_last):
    S, K, bud = c["seqs"], c["K"], c["budget"]
    tokens = _tokens(c, seed)
    _, taps = _verify(ref, c, seed)
    z, ua, ub = _accept_inputs(c, seed)
    out = [p.double() for p in ref.pools]
    T = torch.zeros(S, dtype=torch.int32)
    r_rej = torch.zeros(S, dtype=torch.float64)
    na, bonus, path = T.clone(), T.clone(), torch.zeros((S, c["M"] * K), dtype=torch.int32)
    ctaps = torch.zeros((S, 3, ref.d), dtype=torch.float64, device="cuda")
    base, catch = 0, []
    for s in range(S):
        nodes, rows, _ = _grow(c, s, c["M"])
        cur, walk = 0, []
        while True:
            p = torch.softmax(z[base + cur].double(), 0)
            kids = [i for i, nd in enumerate(nodes) if nd["parent"] == cur]
            mass, seen, hit = 1.0, [], None
            for i in kids:
                x = int(tokens[s, i])
                px = float(p[x])
                if x in seen:
                    continue
                if float(ua[s, i]) < px / mass:
                    hit = i
                    break
                seen.append(x)
                mass -= px
            if hit is None:
                break
            walk.append(hit)
            cur = hit
        p[seen] = 0
        cdf = p.cumsum(0)
        b = int(torch.searchsorted(cdf, float(ub[s, cur]) * cdf[-1], right=True))
        base += len(nodes)
        cont = None
        nd = nodes[cur]
        if cur == 0:
            cont = 0
        elif nd["rank"] == 1 and rows[nd["row"]]["k"] < K:
            cont = nd["row"] + 1
        else:
            cont = next((j for j, r in enumerate(rows)
                         if r["start"] == cur and r["k"] == 1), None)
        na[s], bonus[s], T[s] = len(walk), b, ref.T[s] + len(walk) + 1
        path[s, :len(walk)] = torch.tensor(walk, dtype=torch.int32)
        ctaps[s] = taps[s, cur]
        ids = torch.tensor([0] + walk, device="cuda")
        e = ref.T[s] + torch.arange(len(walk) + 1, device="cuda")
        _scatter(out[0], out[1], ref.tables[0], s, e,
                 [k[s][ids] for k in ref.seg[0][0]],
                 [v[s][ids] for v in ref.seg[0][1]])
        dr = [nodes[i]["row"] for i in walk] + ([cont] if cont is not None else [])
        if dr:
            ids = torch.tensor(dr, device="cuda")
            _scatter(out[2], out[3], ref.tables[1], s, e[:len(dr)],
                     [k[s][ids] for k in ref.seg[1][0]],
                     [v[s][ids] for v in ref.seg[1][1]])
        if cont is None:
            r_rej[s] = -1
            catch.append((s, cur, max(nd["parent"], 0), len(walk)))
            continue
        if ref.w.Vd != ref.w.V:
            d2t = ref.w["d.d2t"]
            j = min(int(np.searchsorted(d2t, b)), ref.w.Vd - 1)
            if d2t[j] != b:
                continue
            b = j
        lz = ref.head(h_last[s, cont][None])[0]
        r_rej[s] = torch.exp(lz[b] - torch.logsumexp(lz, 0))
    # catch-up rows: committed entries first, then the row itself
    if catch:
        ref.pools = [out[0], out[1], out[2], out[3]]
        for s, cur, parent, a in catch:
            keep, ref.T = ref.T, list(ref.T)
            ref.T[s] += a
            n = [1 if q == s else 0 for q in range(S)]
            ones = torch.ones((1, 1), dtype=torch.bool, device="cuda")
            kv, t = [], lambda v: torch.tensor([v], device="cuda")  # noqa: E731
            ref.drafter(ref.cond(taps[s, parent][None]), t(int(tokens[s, cur])),
                        t(1), t(0), n, t(ref.T[s] + 1), [t(0)] * S, [ones] * S, kv)
            _scatter(out[2], out[3], ref.tables[1], s, t(ref.T[s]),
                     [k for k, _ in kv], [v for _, v in kv])
            ref.T = keep
    return dict(n_accepted=na, path=path, bonus=bonus, r_reject=r_rej, T=T,
                root=bonus, cond_taps=ctaps, tk=out[0], tv=out[1], dk=out[2],
                dv=out[3])


def exact(c, seed):
    if c["kind"] == "update":
        return _exact_update(c, seed)
    if c["kind"] == "prefill":
        return _exact_prefill(c, seed)
    ref = _Ref(c, seed, _pools(c, seed))
    S, cap = c["seqs"], _row_cap(c)
    if c["kind"] == "verify":
        x, taps = _verify(ref, c, seed)
        x = _rms(x, ref.w["final_norm"].double())
        logits = torch.zeros((S * c["budget"], ref.w.V), dtype=torch.float64,
                             device="cuda")
        logits[:len(x)] = ref.lin(x, "lm_head")
        return dict(logits=logits, taps=taps)
    tokens, taps = _tokens(c, seed), _taps_in(c, seed).double()
    z64 = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")  # noqa: E731
    h_last = z64(S, cap, ref.d)
    if c["kind"] == "commit":
        for m in range(1, c["M"] + 1):
            ref.block(m, tokens, h_last, taps)
        return _exact_commit(c, seed, ref, h_last)
    out = dict(logits=z64(S * c["B_max"] * c["K"], ref.w.Vd),
               topk_logit=z64(S, cap, 10), lse=z64(S, cap),
               psi=z64(S, cap, 15), h_last=h_last)
    for m in range(1, 2 if c["kind"] == "first" else 3):
        x, where = ref.block(m, tokens, h_last, taps)
        if x is None:
            break
        z = ref.head(x)
        top, lse, psi = _psi(z)
        for i, (s, r) in enumerate(where):
            out["topk_logit"][s, r], out["lse"][s, r] = top[i], lse[i]
            out["psi"][s, r] = psi[i]
    if c["kind"] == "first" or x is not None:
        out["logits"][:len(z)] = z
    return out
