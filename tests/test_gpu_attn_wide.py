"""k_attn_wide (passes of few query sets) against k_attn_mfma, bit for bit: the same blocks scored alone and in one
batch with a block so long that the pass takes the general kernel.  Both kernels run the same instructions on a row's
keys in the same order, so the tolerance is zero.  Block lengths around the set sizes (8, 16, 32 rows), cached lengths
around the 64-key groups, the 256-key steps and the 2048 and 4096 keys after which a wave fetches page ids again, chains and
packed trees, every grouping of query heads.  And batches whose tasks are dealt one group after the other."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from paper_2602_12957_amd.runtime import Engine

pytestmark = pytest.mark.gpu

BLOCKS = [(0, 1), (1, 8), (55, 9), (63, 1), (64, 16), (191, 65), (192, 17), (255, 1), (256, 7), (511, 33), (513, 2), (1300, 32),
          (2040, 20), (2049, 5), (4090, 7), (4097, 33), (8200, 9)]


def _tree(rng, rows):
    """(tokens, end, depth) of a random packed tree of `rows` nodes in pre-order."""
    depth = np.zeros(rows, np.int32)
    for i in range(1, rows):
        depth[i] = rng.integers(max(1, depth[i - 1] - 2), depth[i - 1] + 2)
    end = np.array([next((j for j in range(i + 1, rows) if depth[j] <= depth[i]), rows) for i in range(rows)], np.int32)
    return rng.integers(0, 256, size=rows).astype(np.int32), end, depth


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("n_q, n_kv", [(16, 4), (8, 1), (4, 2), (2, 2)])
def test_wide_attention_matches_the_general_kernel(n_q, n_kv, tree):
    desc = W.tiny_model(2, 128, n_q, n_kv, 64, 128, 256, "bf16")
    weights = W.make_weights(desc, 41)
    rng = np.random.default_rng(n_q + 100 * tree)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    long_rows = 32 * (3 * n_cu // n_q + 1)     # more than 2.25 query sets per compute unit on its own
    n = len(BLOCKS)
    blocks, trees = [], []
    for _, rows in BLOCKS + [(0, long_rows)]:
        if tree and rows < long_rows:
            tok, end, dep = _tree(rng, rows)
        else:
            tok = rng.integers(0, desc.vocab, size=rows).astype(np.int32)
            end, dep = np.full(rows, rows, np.int32), np.arange(rows, dtype=np.int32)
        blocks.append(tok)
        trees.append((end, dep))
    rows = sum(len(b) for b in blocks[:n])
    maxb = max(max((s + r) // 16 + 2 for s, r in BLOCKS), long_rows // 16 + 2)
    pool = sum((s + len(b)) // 16 + 2 for (s, _), b in zip(BLOCKS + [(0, 0)], blocks))
    eng = Engine(desc, weights, pool, n + 1, maxb, rows + long_rows, rows)
    cached = [i for i in range(n) if BLOCKS[i][0]]
    eng.prefill(cached, [rng.integers(0, desc.vocab, size=BLOCKS[i][0]).astype(np.int32) for i in cached])
    eng.snapshot()

    def score(members):
        eng.restore()
        out = eng.verify(members, [blocks[i] for i in members], "region", dump_rows=np.arange(rows), log_tau=-0.3,
                         trees=[trees[i] for i in members] if tree else None)
        return [x[:rows].cpu().numpy().copy() for x in (out.logits, out.argmax, out.margin, out.gap)]

    general = score(list(range(n + 1)))
    for a, b in zip(general, score(list(range(n)))):
        np.testing.assert_array_equal(a, b)
    at = 0
    for i in range(n):                          # each block alone as well: other set counts, other task tables
        eng.restore()
        out = eng.verify([i], [blocks[i]], "region", dump_rows=np.arange(len(blocks[i])), log_tau=-0.3, trees=[trees[i]] if tree else None)
        np.testing.assert_array_equal(general[0][at:at + len(blocks[i])], out.logits.cpu().numpy(), err_msg=str(BLOCKS[i]))
        at += len(blocks[i])
    assert int(eng.status.item()) == 0
    eng.close()


# Rows and cached keys of uneven batches in which a list of the task table comes near its length on 256 compute units, so that
# groups are dealt singly; in all but the first the list with the least work is full at least once.
UNEVEN = {
    "wide": (4, 4, "region", [220, 46, 32], [100, 0, 0]),
    "wide_full": (8, 2, "page", [263, 454, 133, 277, 451], [8000, 100, 100, 2000, 0]),
    "region_full": (16, 4, "region", [33, 185, 399, 539, 424, 471], [547, 2774, 695, 123, 433, 2182]),
    "page_full": (4, 1, "page", [216, 527, 110, 587, 385, 8, 585, 344, 399, 319, 22, 373, 3, 190, 411, 181],
                  [1210, 1688, 1395, 427, 207, 2158, 1351, 2924, 3266, 1668, 1459, 3651, 3967, 3781, 3820, 989]),
}


@pytest.mark.parametrize("name", UNEVEN)
def test_uneven_batches_match_their_members(name):
    """A task that is dealt twice or not at all, or past the end of its list, would leave rows unwritten."""
    n_q, n_kv, mode, rows, cached = UNEVEN[name]
    desc = W.tiny_model(2, 128, n_q, n_kv, 64, 128, 256, "bf16")
    rng = np.random.default_rng(len(rows))
    blocks = [rng.integers(0, desc.vocab, size=r).astype(np.int32) for r in rows]
    total, n = sum(rows), len(rows)
    eng = Engine(desc, W.make_weights(desc, 43), sum((r + c) // 16 + 2 for r, c in zip(rows, cached)), n,
                 max((r + c) // 16 + 2 for r, c in zip(rows, cached)), total, total)
    have = [i for i in range(n) if cached[i]]
    eng.prefill(have, [rng.integers(0, desc.vocab, size=cached[i]).astype(np.int32) for i in have])
    eng.snapshot()
    eng.ws.zero_()
    batch = eng.verify(list(range(n)), blocks, mode, dump_rows=np.arange(total)).logits.cpu().numpy().copy()
    at = 0
    for i in range(n):
        eng.restore()
        out = eng.verify([i], [blocks[i]], mode, dump_rows=np.arange(rows[i]))
        np.testing.assert_array_equal(batch[at:at + rows[i]], out.logits.cpu().numpy(), err_msg=str(i))
        at += rows[i]
    assert int(eng.status.item()) == 0
    eng.close()


# Scores far from 0: a reference point other than 0 is set at the first group (beyond +-64 binary orders of magnitude) and
# moves where a later score lies 96 above it.  Queries and keys are `factor` times the usual, so that the scores' standard
# deviation is 0.07 factor^2 binary orders.
@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("factor", [4, 8, 16])
def test_extreme_scores(factor, tree):
    """Both kernels alike bit for bit, and near the plain kernels, which take a running maximum.  One layer, so that the two paths
    store the same queries and keys but for roundings to bf16 that fall the other way: one in a term of a score moves it by
    2^-8 of the term, at the largest factor (terms of standard deviation 2.3, the largest of 64 about 8) by 0.03, a
    probability by 2 %, an attention output by less than 2 % of a value; the bar is the one of all shallow bf16 models, 2e-2 of
    a logit.  (A second layer's scores would carry the roundings of all its inputs: 2.1e-2 at factor 16.)"""
    desc = W.tiny_model(1, 128, 16, 4, 64, 128, 256, "bf16")
    weights = W.make_weights(desc, 47)
    qk = (desc.n_q_heads + desc.n_kv_heads) * 64
    for layer in weights["layers"]:
        layer["wqkv"] = np.concatenate([layer["wqkv"][:qk] * np.float32(factor), layer["wqkv"][qk:]]).astype(layer["wqkv"].dtype)
    rng = np.random.default_rng(factor)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = [(0, 1), (40, 3), (63, 70), (300, 1), (700, 33), (1300, 5), (0, 32 * (3 * n_cu // 16 + 1))]
    n, rows = len(shapes), sum(r for _, r in shapes[:-1])
    blocks, trees = [], []
    for i, (_, r) in enumerate(shapes):
        if tree and i < n - 1:
            tok, end, dep = _tree(rng, r)
        else:
            tok, end, dep = rng.integers(0, 256, size=r).astype(np.int32), np.full(r, r, np.int32), np.arange(r, dtype=np.int32)
        blocks.append(tok)
        trees.append((end, dep))
    prefix = {i: rng.integers(0, 256, size=s).astype(np.int32) for i, (s, _) in enumerate(shapes) if s}

    def score(members, debug=None):
        eng = Engine(desc, weights, sum((s + r) // 16 + 2 for s, r in shapes), n, max((s + r) // 16 + 2 for s, r in shapes),
                     sum(r for _, r in shapes), rows, debug=debug)
        eng.prefill(list(prefix), list(prefix.values()))
        out = eng.verify(members, [blocks[i] for i in members], "region", dump_rows=np.arange(rows),
                         trees=[trees[i] for i in members] if tree else None).logits.cpu().numpy().copy()
        assert int(eng.status.item()) == 0
        eng.close()
        return out

    general, wide, plain = score(range(n)), score(range(n - 1)), score(range(n - 1), {"force_simple": 1})
    np.testing.assert_array_equal(general, wide)
    assert np.abs(wide - plain).max() <= 2e-2


def _points(x):
    """Reference points [groups of 64 keys, queries] along a walk over the scores x [queries, keys], keys not seen -inf."""
    m, walk = np.full(len(x), -np.inf), []
    for at in range(0, x.shape[1], 64):
        mx = x[:, at:at + 64].max(axis=1)
        with np.errstate(invalid="ignore"):
            first = np.where(np.abs(np.ceil(mx)) <= 64, 0, np.ceil(mx))
            m = np.where(m == -np.inf, first, np.where(mx - m >= 96, np.ceil(mx), m))
        walk.append(m)
    return np.array(walk)


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("factor", [24, 32])
@pytest.mark.parametrize("n_q, n_kv", [(16, 4), (4, 2), (2, 2)])
def test_reference_points_in_every_form(n_q, n_kv, factor, tree):
    """The workgroups of eight query sets give the bits of k_attn_wide, and key splits, whose chunks set reference points of
    their own, come as near the plain kernels (see test_extreme_scores: at factor 32 a rounding that falls the other way, one in
    10^4, moves a probability by 8 % and with it one head's output; the bar stays).  The drawn scores ask for it: computed here
    from layer 0, points are set away from 0, move within a walk, differ between chunks of 256 keys, and some rows see no key of
    a chunk whose workgroup walks it."""
    desc = W.tiny_model(1, 128, n_q, n_kv, 64, 128, 256, "bf16")
    weights = W.make_weights(desc, 53)
    qk = (n_q + n_kv) * 64
    for layer in weights["layers"]:
        layer["wqkv"] = np.concatenate([layer["wqkv"][:qk] * np.float32(factor), layer["wqkv"][qk:]]).astype(layer["wqkv"].dtype)
    rng = np.random.default_rng(n_q + factor)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = [(0, 1), (40, 3), (63, 70), (120, 20), (300, 1), (700, 33), (1300, 5), (4300, 3), (0, 32 * (3 * n_cu // n_q + 1))]
    n, rows = len(shapes), sum(r for _, r in shapes[:-1])
    blocks, trees = [], []
    for i, (_, r) in enumerate(shapes):
        if tree and i < n - 1:
            tok, end, dep = _tree(rng, r)
        else:
            tok, end, dep = rng.integers(0, 256, size=r).astype(np.int32), np.full(r, r, np.int32), np.arange(r, dtype=np.int32)
        blocks.append(tok)
        trees.append((end, dep))
    prefix = {i: rng.integers(0, 256, size=s).astype(np.int32) for i, (s, _) in enumerate(shapes) if s}

    lay, away, moved, apart, blind = weights["layers"][0], 0, 0, 0, 0
    for i, (s, r) in list(enumerate(shapes))[1:-1]:
        x = weights["tok_embed"][np.concatenate([prefix[i], blocks[i]])].astype(np.float64)
        pos = np.concatenate([np.arange(s), s + trees[i][1]])
        y = O.rmsnorm(x, lay["attn_norm"], desc.rms_eps) @ lay["wqkv"][:qk].astype(np.float64).T
        y = O.rope_rotate_half(y.reshape(s + r, n_q + n_kv, 64), pos, desc.rope_theta)
        row, key = np.arange(r)[:, None], np.arange(s + r)[None] - s
        sees = (key <= row) & ((key < 0) | (np.concatenate([np.zeros(s, np.int32), trees[i][0]])[None] > row))
        for h in range(n_q):
            score = np.where(sees, y[s:, h] @ y[:, n_q + h * n_kv // n_q].T / 8 * np.log2(np.e), -np.inf)
            walk = _points(score)
            away += np.isfinite(walk).any() and (np.where(np.isfinite(walk), walk, 0) != 0).sum()
            moved += ((walk[1:] != walk[:-1]) & np.isfinite(walk[:-1])).sum()
            ends = np.array([_points(score[:, c:c + 256])[-1] for c in range(0, s + r, 256)])
            apart += (ends[1:] != ends[:-1]).sum()
        blind += (s + np.arange(r) < (s + r - 1) // 128 * 128).sum()
    assert min(away, moved, apart, blind) > 0, (away, moved, apart, blind)

    def score(members, mode="region", chunk=0, debug=None):
        eng = Engine(desc, weights, sum((s + r) // 16 + 2 for s, r in shapes), n, max((s + r) // 16 + 2 for s, r in shapes),
                     sum(r for _, r in shapes), rows, attn_key_chunk=chunk, debug=debug)
        eng.prefill(list(prefix), list(prefix.values()))
        out = eng.verify(members, [blocks[i] for i in members], mode, dump_rows=np.arange(rows),
                         trees=[trees[i] for i in members] if tree else None).logits.cpu().numpy().copy()
        assert int(eng.status.item()) == 0
        eng.close()
        return out

    wide, plain = score(range(n - 1)), score(range(n - 1), debug={"force_simple": 1})
    np.testing.assert_array_equal(score(range(n), "page"), wide)
    np.testing.assert_array_equal(score(range(n), "region"), wide)
    for chunk in (128, 256):
        region, page = score(range(n - 1), "region", chunk), score(range(n - 1), "page", chunk)
        np.testing.assert_array_equal(region, page)
        assert np.abs(region - plain).max() <= 2e-2
    assert np.abs(wide - plain).max() <= 2e-2


@pytest.mark.parametrize("n_q, n_kv", [(16, 4), (2, 2)])
@pytest.mark.parametrize("elements", [1, 2, 4])
def test_pools_need_no_more_than_their_elements_alignment(n_q, n_kv, elements):
    """K and V pools a few elements past a 16-byte boundary give the bits of aligned ones, with one block and with so many rows
    that aligned pools take the general kernel, from both entry points; a key split is without effect on them."""
    import paper_2602_12957_amd.binding as B
    from paper_2602_12957_amd.runtime import _ptr
    desc = W.tiny_model(2, 128, n_q, n_kv, 64, 128, 256, "bf16")
    weights = W.make_weights(desc, 59)
    rng = np.random.default_rng(elements)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    prefix = rng.integers(0, 256, size=300).astype(np.int32)
    blocks = [rng.integers(0, 256, size=r).astype(np.int32) for r in (7, 32 * (3 * n_cu // n_q + 1))]
    rows, n_dump = sum(len(b) for b in blocks), 200

    def score(shift, members, mode, chunk=0):
        eng = Engine(desc, weights, (rows + 300) // 16 + 4, 2, (rows + 300) // 16 + 4, rows, n_dump, attn_key_chunk=chunk)
        if shift:
            keep = [torch.zeros(p.numel() + shift, dtype=p.dtype, device=p.device) for p in (eng.k_pool, eng.v_pool)]
            eng.k_pool, eng.v_pool = keep[0][shift:], keep[1][shift:]
            assert eng.k_pool.data_ptr() % 16 == 2 * shift
            eng.cpool = B.hsd_kv_pool(_ptr(eng.k_pool), _ptr(eng.v_pool), eng.n_blocks, _ptr(eng.free_list), _ptr(eng.free_count))
        eng.reset()
        eng.prefill([0], [prefix])
        dump = np.arange(min(n_dump, sum(len(blocks[i]) for i in members)))
        out = eng.verify(members, [blocks[i] for i in members], mode, dump_rows=dump).logits.cpu().numpy().copy()
        assert int(eng.status.item()) == 0
        eng.close()
        return out

    for members, mode in (([0], "region"), ([0, 1], "region"), ([0, 1], "page")):
        aligned = score(0, members, mode)
        np.testing.assert_array_equal(aligned, score(elements, members, mode))
    np.testing.assert_array_equal(aligned, score(elements, members, mode, 128))


# A row that sees one key gets that key's value, to the last bit: the probability, whatever its rounding to bf16, cancels in the
# quotient.  mode, sequences, rows of a further sequence, key chunk: 16 and 32 columns of k_attn_wide, k_attn_mfma with 4 and 8
# query sets and with a key split.
ONE_KEY = {"wide_16": ("region", 8, 0, 0), "wide_32": ("region", 8, 9, 0), "general": ("region", 0, 0, 0), "general_page": ("page", 0, 0, 0),
           "split": ("page", 8, 9, 128)}


@pytest.mark.parametrize("name", ONE_KEY)
@pytest.mark.parametrize("n_q, n_kv", [(16, 4), (16, 8), (16, 16)])
def test_one_key_gives_its_value(n_q, n_kv, name):
    """One layer in which every number but the probability is exact.  Embeddings are +-V with V the largest mantissa (an error of
    2^-9 is a whole unit of it), so that norms make them +-1; the values are the embeddings again; the output projection takes the
    attention's output off the residual: what is left is 0, and so are the logits (one-hot rows of the LM head), in every
    column whose value came back whole.  The last head's columns stay, to keep the last norm finite.  Scores: q = a number per
    head, k = a random sum of signs, so that the probabilities' mantissas are spread."""
    mode, n, more, chunk = ONE_KEY[name]
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n == 0:
        n = 9 * n_cu // (4 * n_kv) + 1                  # more than 2.25 query sets per compute unit: the general kernel
    d, group, big = n_q * 64, n_q // n_kv, 255 / 128
    desc = W.ModelDesc(1, d, n_q, n_kv, 64, 128, 1024, "bf16")
    rng = np.random.default_rng(n_q + n_kv)
    sign = rng.choice([-1.0, 1.0], (desc.vocab, n_kv, 64)).astype(np.float32)
    wqkv = np.zeros(((n_q + 2 * n_kv) * 64, d), np.float32)
    at = lambda h, i: h * 64 + i
    for h in range(n_q):
        wqkv[at(h, 0), at(group * (h // group), 0)] = rng.uniform(2, 20)          # q . k = q_0 k_0
    for g in range(n_kv):
        wqkv[at(n_q + g, 0), [at(group * g, i) for i in range(64)]] = rng.normal(0, 0.25, 64)
        for i in range(64):
            wqkv[at(n_q + n_kv + g, i), at(group * g, i)] = big
    wo = -np.eye(d, dtype=np.float32)
    wo[d - 64:] = 0
    ones = np.ones(d, np.float32)
    weights = dict(tok_embed=big * np.repeat(sign, group, axis=1).reshape(desc.vocab, d), lm_head=np.eye(desc.vocab, d, dtype=np.float32),
                   final_norm=ones, layers=[dict(attn_norm=ones, wqkv=wqkv, wo=wo, ffn_norm=ones,
                                                 w_gate_up=np.zeros((256, d), np.float32), w_down=np.zeros((d, 128), np.float32))])
    blocks = [rng.integers(0, desc.vocab, 1).astype(np.int32) for _ in range(n)]
    if more:
        blocks.append(rng.integers(0, desc.vocab, more).astype(np.int32))
    first = np.cumsum([0] + [len(b) for b in blocks[:-1]]).astype(np.int32)
    eng = Engine(desc, weights, len(blocks) + 1, len(blocks), 1, n + more, len(blocks), attn_key_chunk=chunk)
    logits = eng.verify(list(range(len(blocks))), blocks, mode, dump_rows=first).logits.cpu().numpy().copy()
    assert int(eng.status.item()) == 0
    eng.close()
    assert np.isfinite(logits).all() and (np.abs(logits[:, d - 64:]) > 0.5).all()
    np.testing.assert_array_equal(logits[:, :d - 64], 0)


@pytest.mark.parametrize("value", [np.inf, 60.0])
@pytest.mark.parametrize("mode, rows, more, chunk", [("region", 4, 0, 0), ("region", 40, 0, 0), ("region", 40, 1, 0), ("page", 40, 1, 0), ("region", 40, 0, 128)])
def test_one_query_leaves_the_others_alone(mode, rows, more, chunk, value):
    """One token's queries are infinite, or so large that its reference points are far from 0 and move (keys and values as ever): the
    other rows of its block, which share its wave, give the bits they give beside an ordinary query.  16 and 32 columns of
    k_attn_wide, k_attn_mfma with 4 and 8 query sets and with a key split."""
    desc = W.tiny_model(1, 128, 16, 4, 64, 128, 256, "bf16")
    weights = W.make_weights(desc, 67)
    weights["tok_embed"][:, 5] = 0
    weights["tok_embed"][7, 5] = 0.02                 # token 7 alone has column 5, about 1 after the norm
    rng = np.random.default_rng(rows)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    prefix = rng.integers(8, 256, size=300).astype(np.int32)
    blocks = [rng.integers(8, 256, size=rows).astype(np.int32)] + [rng.integers(8, 256, size=32 * (3 * n_cu // 16 + 1)).astype(np.int32)] * more
    blocks[0][rows // 2] = 7

    def score(gain):
        wqkv = weights["layers"][0]["wqkv"].copy()
        wqkv[:16 * 64, 5] = 0 if gain == 0 else np.where(np.arange(16 * 64) % 2, 1, -1) * np.float32(3e38 if np.isinf(gain) else gain)
        wqkv[16 * 64:, 5] = 0
        total = sum(len(b) for b in blocks)
        eng = Engine(desc, {**weights, "layers": [{**weights["layers"][0], "wqkv": wqkv}]}, (total + 300) // 16 + 4, 2, (total + 300) // 16 + 4, total,
                     rows, attn_key_chunk=chunk)
        eng.prefill([0], [prefix])
        out = eng.verify(list(range(1 + more)), blocks, mode, dump_rows=np.arange(rows)).logits.cpu().numpy().copy()
        assert int(eng.status.item()) == 0
        eng.close()
        return out

    plain, odd = score(0), score(value)
    others = np.arange(rows) != rows // 2
    np.testing.assert_array_equal(odd[others], plain[others])
    assert not np.array_equal(odd[rows // 2], plain[rows // 2]) and np.isfinite(odd[rows // 2]).all() == np.isfinite(value)
