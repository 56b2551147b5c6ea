"""What a user has this framework do, as cases that can be timed and compared.

Every case runs a decoder over sequences whose prefixes are cached already, through the public entry points of
`paper_2602_12957_amd`: `Engine.verify` / `commit` / `read_acceptance` (one verification round), `Engine.greedy_decode`
(token by token), `Engine.prefill` (prefixes) and `SpecDecoder.run` (rounds driven from draft sets to completion).

The model sizes are the two of the workload configurations.  The weights are random, with one thing added: the LM head
holds, for every token, a share of the embedding of a fixed predecessor, so that the decoder continues text with a margin
of several logits, as a trained document reader does.  A draft is that continuation with tokens replaced at a given rate,
and acceptance lengths follow from the seed.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2602_12957_amd.runtime import Engine, pack_prefix_tree
from paper_2602_12957_amd.specdecode import SpecDecoder

MODELS = {
    "M": dict(n_layers=24, d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, d_ffn=4096, vocab=32768, dtype="bf16"),
    "T": dict(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=1024, vocab=4096, dtype="fp32"),
}
PROMPT = 16          # prefix rows that are token ids (at most); the rest are rows of a vision encoder
SUCC_SHARE, EMBED_STD = 0.06, 0.5


def listed():
    return [
        # one user, no draft left: a single token per pass, the latency of the smallest call
        dict(name="step_1", kind="round", model="M", mode="region", n_seq=1, ctx=1055, k=0, tau=1.0),
        # plain decoding of the 16 regions of a page side by side, token after token
        dict(name="decode_16", kind="decode", model="M", n_seq=16, ctx=1055, steps=16),
        # plain decoding of 64 regions whose prefixes differ in length
        dict(name="decode_64", kind="decode", model="M", n_seq=64, ctx=512, ctx_hi=2048, steps=8),
        # a late round: few regions are left, each with a short odd rest of its draft
        dict(name="tail_7", kind="round", model="M", mode="region", n_seq=7, ctx=900, ctx_hi=1400, k=1, k_hi=47, tau=1.0),
        # eight packed prefix trees under the 128-row cap, relaxed acceptance at the usual threshold
        dict(name="tree_8", kind="tree", model="M", mode="region", n_seq=8, ctx=1055, depth=56, tau=0.75),
        # a whole document part driven from draft sets: matching, packing, rounds, commits
        dict(name="spec_8", kind="spec", model="M", mode="region", n_seq=8, ctx=1055, tokens=96, tau=0.75),
        # first round of a page's 16 regions (the headline workload)
        dict(name="region_16", kind="round", model="M", mode="region", n_seq=16, ctx=1055, k=16, k_hi=256, tau=1.0),
        # one long page draft over a long prefix, attention keys split
        dict(name="page_1", kind="round", model="M", mode="page", n_seq=1, ctx=4127, k=2048, tau=1.0, key_chunk=1024),
        # 64 ragged regions in one batch
        dict(name="ragged_64", kind="round", model="M", mode="region", n_seq=64, ctx=512, ctx_hi=2048, k=8, k_hi=1024, k_mu=4.5, tau=1.0),
        # four long pages, each with a draft as long as its prefix: the largest call
        dict(name="longdoc_4", kind="round", model="M", mode="page", n_seq=4, ctx=8192, k=8192, tau=1.0),
        # the prefixes of 16 regions, rows of the vision encoder on the device
        dict(name="prefill_16", kind="prefill", model="M", n_seq=16, ctx=1055),
        # the small fp32 model that is used to check a deployment
        dict(name="fp32_4", kind="round", model="T", mode="region", n_seq=4, ctx=271, k=32, tau=1.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["round", "round", "round", "page", "tree", "decode", "decode", "spec", "prefill", "fp32"])
    shape = rng.randrange(1 << 20)
    if kind == "round":
        n = _log(rng, 1, 64)
        lo, k = _log(rng, 64, 2048), _log(rng, 1, min(1024, 8192 // n)) - 1
        return dict(kind="round", model="M", mode="region", n_seq=n, ctx=lo, ctx_hi=rng.randint(lo, 2 * lo), k=k,
                    k_hi=rng.randint(k, 2 * k + 1), tau=rng.choice([1.0, 0.75]), shape=shape)
    if kind == "page":
        n = rng.randint(1, 4)
        return dict(kind="round", model="M", mode="page", n_seq=n, ctx=_log(rng, 1024, 8192), k=_log(rng, 256, 4096), tau=1.0,
                    key_chunk=1024 if n == 1 else 0, shape=shape)
    if kind == "tree":
        return dict(kind="tree", model="M", mode="region", n_seq=_log(rng, 1, 32), ctx=_log(rng, 64, 2048), depth=_log(rng, 4, 56),
                    tau=rng.choice([1.0, 0.75]), shape=shape)
    if kind == "decode":
        lo = _log(rng, 64, 4096)
        return dict(kind="decode", model="M", n_seq=_log(rng, 1, 64), ctx=lo, ctx_hi=rng.randint(lo, 2 * lo), steps=rng.randint(4, 12), shape=shape)
    if kind == "spec":
        return dict(kind="spec", model="M", mode="region", n_seq=_log(rng, 1, 16), ctx=_log(rng, 64, 2048), tokens=_log(rng, 32, 160),
                    tau=rng.choice([1.0, 0.75]), shape=shape)
    if kind == "prefill":
        lo = _log(rng, 64, 2048)
        return dict(kind="prefill", model="M", n_seq=_log(rng, 1, 16), ctx=lo, ctx_hi=rng.randint(lo, 2 * lo), shape=shape)
    return dict(kind="round", model="T", mode="region", n_seq=rng.randint(1, 16), ctx=_log(rng, 16, 1024), k=_log(rng, 1, 128), tau=1.0, shape=shape)


# ---------------------------------------------------------------------------------------------------- sizes
def _sizes(case):
    """(cached rows, draft rows) of every sequence; they follow from the case alone."""
    rng = random.Random(case.get("shape", 7))
    ctx = [rng.randint(case["ctx"], case.get("ctx_hi", case["ctx"])) for _ in range(case["n_seq"])]
    k_lo, k_hi = case.get("k", 0), case.get("k_hi", case.get("k", 0))
    if "k_mu" in case:
        k = [min(max(int(round(rng.lognormvariate(case["k_mu"], 0.8))), k_lo), k_hi) for _ in ctx]
    else:
        k = [rng.randint(k_lo, k_hi) for _ in ctx]
    if case["kind"] == "tree":
        k = [_tree_rows(case["depth"]) - 1 for _ in ctx]
    return ctx, k


def _tree_rows(depth):
    """Three candidates of `depth` tokens that part from the first after a quarter and after a half of it."""
    return 1 + depth + (depth - depth // 4) + (depth - depth // 2)


def work(case):
    m = SimpleNamespace(**MODELS[case["model"]])
    es = 2 if m.dtype == "bf16" else 4
    qd, kvd = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    layer = m.d_model * (qd + 2 * kvd) + qd * m.d_model + 3 * m.d_model * m.d_ffn
    ctx, k = _sizes(case)

    def one_pass(have, rows, head=True):
        """bytes and flops of a pass over `rows` new rows per sequence on top of `have` cached ones"""
        t = sum(rows)
        params = layer * m.n_layers + (m.d_model * m.vocab if head else 0)
        flops = 2.0 * params * t + m.n_layers * 4.0 * qd * sum(r * s + r * (r + 1) / 2 for s, r in zip(have, rows))
        kv = m.n_layers * 2 * kvd * es
        return params * es + kv * (sum(have) + t) + t * m.d_model * (es if head else 4), flops

    if case["kind"] == "prefill":
        b, f = one_pass([0] * len(ctx), ctx, head=False)
    elif case["kind"] == "decode":
        b = f = 0.0
        for i in range(case["steps"]):
            x, y = one_pass([c + i for c in ctx], [1] * len(ctx))
            b, f = b + x, f + y
    elif case["kind"] == "spec":     # every token scored once, no more rounds than the cap of a packed tree asks for
        b = f = 0.0
        left, at = case["tokens"], 0
        while left > 0:
            rows = min(left, 128)
            x, y = one_pass([c + at for c in ctx], [rows] * len(ctx))
            b, f, at, left = b + x, f + y, at + rows, left - rows
    else:
        b, f = one_pass(ctx, [1 + v for v in k])
    return {"bytes": b, "flops": f}


def tolerance(case):
    if MODELS[case["model"]]["dtype"] == "fp32":
        # against fp64 the logits are off by 2.8e-6 of their root mean square at most
        return {"rel": 1e-5, "max": 5e-5, "differ": 0.0}
    # the matrix-core path against the library's plain fp32-FMA kernels (other sums, other rounding of intermediates, the
    # same bf16 storage through 24 layers): logits rel 1.1e-2, largest difference 5.9e-2, no token differs
    return {"rel": 3e-2, "max": 0.25, "differ": 2e-3}


# ---------------------------------------------------------------------------------------------------- inputs
class _ResidentEngine(Engine):
    """An Engine whose weights are on the GPU already, as a program that has loaded a checkpoint there holds them."""

    def _up_mat(self, t):
        self._keep.append(t)
        return t.data_ptr()

    _up_f32 = _up_mat


def _weights(m, gen, succ):
    kind = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    dev = dict(device="cuda:0", generator=gen)

    def mat(rows, cols, std=0.02):
        return torch.empty((rows, cols), dtype=kind, device="cuda:0").normal_(0.0, std, generator=gen)

    def gain():
        return 1.0 + 0.1 * torch.randn(m.d_model, **dev)

    qd, kvd = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    embed, head = mat(m.vocab, m.d_model, EMBED_STD), mat(m.vocab, m.d_model)
    head[succ] += (SUCC_SHARE * embed.float()).to(kind)
    return {"tok_embed": embed, "lm_head": head, "final_norm": gain(),
            "layers": [dict(attn_norm=gain(), wqkv=mat(qd + 2 * kvd, m.d_model), wo=mat(m.d_model, qd), ffn_norm=gain(),
                            w_gate_up=mat(2 * m.d_ffn, m.d_model), w_down=mat(m.d_model, m.d_ffn)) for _ in range(m.n_layers)]}


def _chain(succ, pending, n):
    out, t = np.empty(n, np.int32), int(pending)
    for i in range(n):
        t = int(succ[t])
        out[i] = t
    return out


def _corrupt(rng, tokens, p, vocab):
    hit = rng.random(len(tokens)) < p
    return np.where(hit, rng.integers(0, vocab, len(tokens)), tokens).astype(np.int32)


def _tree(rng, chain, pending, vocab):
    """Three candidates that share a prefix, in an order that is drawn: the likely one and two that part from it."""
    n = len(chain)
    base = _corrupt(rng, chain, 0.02, vocab)
    cands = [base]
    for at in (n // 4, n // 2):
        other = base.copy()
        other[at:] = _corrupt(rng, chain[at:], 0.02, vocab)
        first = {int(c[at]) for c in cands}
        while int(other[at]) in first:
            other[at] = (other[at] + 1 + rng.integers(0, vocab - 1)) % vocab
        cands.append(other)
    order = rng.permutation(3)
    return pack_prefix_tree(pending, [cands[i] for i in order])


def prepare(case, seed):
    m = SimpleNamespace(**MODELS[case["model"]], rms_eps=1e-6, rope_theta=10000.0, kv_block_tokens=16)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    rng = np.random.default_rng(seed)
    succ = rng.permutation(m.vocab)
    ctx, k = _sizes(case)
    n = case["n_seq"]
    grow = {"decode": case.get("steps", 0) + 1, "spec": case.get("tokens", 0) + 2 * 129}.get(case["kind"], 0)
    need = [(c + v + 1 + grow + 15) // 16 + 1 for c, v in zip(ctx, k)]
    rows = max(sum(v + 1 for v in k), min(sum(ctx), 32768), 129 * n if case["kind"] == "spec" else 0, n)
    eng = _ResidentEngine(m, _weights(m, gen, torch.from_numpy(succ).cuda()), sum(need) + 8, n, max(need), rows, max_dump=n,
                          attn_key_chunk=case.get("key_chunk", 0))
    toks, embs, pend = [], [], []
    for c in ctx:
        t = np.full(c, -1, np.int32)
        p = min(PROMPT, c // 2)
        t[c - p:] = rng.integers(0, m.vocab, p)
        toks.append(t)
        embs.append(torch.randn((c, m.d_model), device="cuda:0", generator=gen))
        pend.append(int(rng.integers(0, m.vocab)))
    st = SimpleNamespace(eng=eng, case=case, slots=list(range(n)), toks=toks, embs=embs, pend=pend, n=n,
                         log_tau=0.0 if case.get("tau", 1.0) >= 1.0 else math.log(case["tau"]))
    if case["kind"] == "prefill":
        return st
    eng.prefill(st.slots, toks, embs)
    st.toks = st.embs = None
    eng.snapshot()
    st.trees = None
    if case["kind"] == "round":
        st.blocks = [np.concatenate([[p], _corrupt(rng, _chain(succ, p, v), 0.05, m.vocab)]).astype(np.int32) for p, v in zip(pend, k)]
    elif case["kind"] == "tree":
        packed = [_tree(rng, _chain(succ, p, case["depth"]), p, m.vocab) for p in pend]
        st.blocks, st.trees = [t[0] for t in packed], [(t[1], t[2]) for t in packed]
    elif case["kind"] == "spec":
        chains = [_chain(succ, p, case["tokens"] + 32) for p in pend]
        st.drafts = [[_corrupt(rng, c, 0.05, m.vocab).tolist() for _ in range(2)] for c in chains]
        st.driver = SpecDecoder(eng, n_window=3, max_packed=128, log_tau=st.log_tau, mode=case["mode"])
    if case["kind"] in ("round", "tree"):
        ends = np.cumsum([len(b) for b in st.blocks]) - 1
        st.dump = ends.astype(np.int32)         # the logits of every sequence's last row
    return st


# ---------------------------------------------------------------------------------------------------- one pass
def _state(eng):
    kind = torch.bfloat16 if eng.bf16 else torch.float32
    return {"k": eng.k_pool.view(kind), "v": eng.v_pool.view(kind), "len": eng.seq_len, "table": eng.block_table}


def run(st):
    eng, case = st.eng, st.case
    if case["kind"] == "prefill":
        eng.reset()
        eng.prefill(st.slots, st.toks, st.embs)
        return _state(eng)
    eng.restore()            # back to the cached prefixes (bookkeeping only), so that a pass can be repeated
    if case["kind"] == "decode":
        tokens = eng.greedy_decode(st.slots, st.pend, case["steps"])
        return {"tokens": tokens, "margin": eng.margin[:st.n], **_state(eng)}
    if case["kind"] == "spec":
        tokens, stats = st.driver.run(st.slots, st.pend, st.drafts, [case["tokens"]] * st.n)
        return {"tokens": tokens, "counts": [stats["rounds"], stats["rows"], stats["accepted"]], "len": eng.seq_len, "margin": eng.margin[:st.n]}
    out = eng.verify(st.slots, st.blocks, case["mode"], dump_rows=st.dump, log_tau=st.log_tau, trees=st.trees)
    eng.commit()
    alpha, bonus, status = eng.read_acceptance(st.n)     # the host needs them to slice the next round
    res = {"alpha": alpha, "bonus": bonus, "status": status, "argmax": out.argmax, "margin": out.margin, "logits": out.logits, **_state(eng)}
    if out.gap is not None:
        res["gap"] = out.gap
    return res
