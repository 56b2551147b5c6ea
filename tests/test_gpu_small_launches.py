"""Kernels chosen for launches of few rows against the general ones, bit for bit: the 16-row kernel's tiles for the bf16
projections, and its weights read past the caches, against a tile set by hand; tiles dealt to the XCDs in bands; the smaller
tiles of the fp32 path against the 64-row ones that a block with enough rows takes at every projection.  Every output sums its products in one fixed
order in all of them, so the tolerance is zero.  The LM head's record where logits are not finite.  And the plain kernels
on a bf16 model against the oracle, with the bar of the bf16 parity tests."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from workloads.generators import SequenceSpec

from hsd_testlib import gated_compare_argmax, make_engine, prefix_rows

pytestmark = pytest.mark.gpu


def _round(desc, weights, seed, draft, debug=None):
    spec = SequenceSpec(0, 37, 3, len(draft), 0.0)
    n = len(draft) + 1
    eng = make_engine(desc, weights, [spec], max_total_q=max(n, 64), max_dump=n, debug=debug)
    _, _, tok, emb, pending = prefix_rows(desc, seed, spec)
    eng.prefill([0], [tok], [emb])
    out = eng.verify([0], [np.concatenate([[pending], draft]).astype(np.int32)], "region", dump_rows=np.arange(n))
    res = out.argmax.cpu().numpy().copy(), out.margin.cpu().numpy().copy(), out.logits.cpu().numpy().copy()
    eng.close()
    return res


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 65, 225])
def test_narrow_tiles_match_the_general_tile(rows):
    desc, seed = W.ModelDesc(3, 256, 8, 2, 64, 512, 1024, "bf16"), 17
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    chosen = _round(desc, weights, seed, draft)
    for cfg in (2, 12):
        for a, b in zip(chosen, _round(desc, weights, seed, draft, {"gemm_cfg": (cfg, cfg, cfg, cfg, 0)})):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("rows", [1, 33])
@pytest.mark.parametrize("d_model", [640, 768, 2048, 2176])
def test_row_sums_of_a_wide_model_with_one_head(rows, d_model):
    """One head of 64: the further planes of row sums (d_model / 64 floats a row each) lie in q and the attention output.  The
    three planes of 16-column tiles fit up to d_model 640, the one of 32-column tiles fills them exactly at 2048; at 768 and
    2176 the next wider tile has to be taken."""
    desc, seed = W.ModelDesc(2, d_model, 1, 1, 64, 128, 512, "bf16"), 23
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    for a, b in zip(_round(desc, weights, seed, draft), _round(desc, weights, seed, draft, {"gemm_cfg": (2, 2, 2, 2, 0)})):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("rows", [16, 17, 129, 257, 513, 700, 1025, 2049, 4097])
@pytest.mark.parametrize("d_model, d_ffn", [(256, 512), (384, 640)])
def test_16_row_tiles_match_the_general_tile(rows, d_model, d_ffn):
    """Row counts on both sides of the lines between the 16-row kernel's tiles from 16 x 16 to 128 x 64 for these widths,
    and contraction lengths that are whole stages of 512 or 256 (256, 512) or leave a partly filled one (384, 640)."""
    desc, seed = W.ModelDesc(2, d_model, 8, 2, 64, d_ffn, 512, "bf16"), 31
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    for a, b in zip(_round(desc, weights, seed, draft), _round(desc, weights, seed, draft, {"gemm_cfg": (2, 2, 2, 2, 0)})):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("heads, d_model, d_ffn, cols", [((8, 2), 256, 512, 768), ((8, 2), 384, 640, 384), ((9, 9), 384, 512, 384)])
@pytest.mark.parametrize("end", ["first", "last", "past"])
def test_144_row_tiles_match_the_general_tile(heads, d_model, d_ffn, cols, end):
    """The widest tile, 144 x 64, at the projection with `cols` outputs (QKV, or output and down): taken from the first row
    count at which 128 x 64 tiles outnumber the compute units to the last at which its own do not.  Nine heads: the output
    projection's contraction (576) leaves a stage of 128 half filled."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    first, last = n_cu // (cols // 64) * 128 + 1, n_cu // (cols // 64) * 144
    rows = {"first": first, "last": last, "past": last + 1}[end]
    assert -(-first // 128) * (cols // 64) > n_cu >= -(-last // 144) * (cols // 64) and -(-(last + 1) // 144) * (cols // 64) > n_cu
    assert last < 6144                       # from there on 256 x 256 tiles
    desc, seed = W.ModelDesc(1, d_model, *heads, 64, d_ffn, 512, "bf16"), 31
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    for a, b in zip(_round(desc, weights, seed, draft), _round(desc, weights, seed, draft, {"gemm_cfg": (2, 2, 2, 2, 0)})):
        np.testing.assert_array_equal(a, b)


# nine layers of 31 MB: more than the memory-side cache, so that passes of up to 128 rows read them past the caches.  On 256
# compute units every projection takes the 16-row kernel at the rows tested: gate/up 32 x 32, 32 x 64 and 64 x 64 tiles.
DEEP = W.ModelDesc(9, 1024, 16, 4, 64, 4096, 512, "bf16")


@pytest.fixture(scope="module")
def deep_engines():
    d = DEEP
    assert 2 * d.n_layers * d.d_model * ((d.n_q_heads + 2 * d.n_kv_heads + d.n_q_heads) * 64 + 3 * d.d_ffn) > 256 << 20
    weights, spec = W.make_weights(d, 37), SequenceSpec(0, 37, 3, 128, 0.0)
    _, _, tok, emb, pending = prefix_rows(d, 37, spec)
    engines = []
    for debug in (None, {"gemm_cfg": (2, 2, 2, 2, 0)}):
        engines.append(make_engine(d, weights, [spec], max_total_q=160, max_dump=160, debug=debug))
        engines[-1].prefill([0], [tok], [emb])
        engines[-1].snapshot()
    yield engines, pending
    for eng in engines:
        eng.close()


@pytest.mark.parametrize("rows", [1, 17, 33, 65, 128, 129])
def test_weights_read_past_the_caches(deep_engines, rows):
    engines, pending = deep_engines
    draft = np.random.default_rng(rows).integers(0, DEEP.vocab, size=rows - 1).astype(np.int32)
    res = []
    for eng in engines:
        eng.restore()
        out = eng.verify([0], [np.concatenate([[pending], draft]).astype(np.int32)], dump_rows=np.arange(rows))
        res.append([x.cpu().numpy().copy() for x in (out.argmax, out.margin, out.logits)])
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("rows", [1, 200])
def test_lm_head_record_without_finite_logits(rows):
    """The running top two of a lane whose logits are all -inf or NaN, and of one that meets some of them in any place.
    A column of the LM head that is -inf (and 0 elsewhere) makes a token's logit -inf or +inf by the sign of the row's
    operand there, a NaN makes it NaN.  The record: lowest id among the largest logits that are numbers, and its distance
    to the second largest; both tile sizes of the LM head."""
    desc, seed = W.ModelDesc(1, 128, 2, 1, 64, 128, 512, "bf16"), 47
    weights = W.make_weights(desc, seed)
    rng = np.random.default_rng(rows)
    draft = rng.integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    ids = np.arange(desc.vocab)
    none, half, every, thirds, scattered = ids < 0, ids < 256, ids >= 0, ids % 3, rng.integers(0, 3, size=desc.vocab)
    for nan, inf, column in ((half, none, 0), (ids != 300, none, 0), (none, half, 3), (none, half, 4), (none, every, 3),
                             (thirds == 1, thirds == 2, 3), (thirds == 0, none, 0), (scattered == 0, scattered == 1, 4)):
        head = weights["lm_head"].copy()
        head[inf] = 0.0
        head[inf, column] = -np.inf
        head[nan] = np.nan
        argmax, margin, logits = _round(desc, {**weights, "lm_head": head}, seed, draft)
        seen = np.where(np.isnan(logits), -np.inf, logits)
        top = seen.max(axis=1)
        np.testing.assert_array_equal(argmax, np.argmax((seen == top[:, None]) & ~np.isnan(logits), axis=1))
        second = np.sort(seen, axis=1)[:, -2]
        with np.errstate(invalid="ignore"):
            np.testing.assert_array_equal(margin, top - second)


LARGE_FP32 = W.ModelDesc(1, 1024, 16, 4, 64, 1024, 1024, "fp32")


@pytest.fixture(scope="module")
def large_block():
    """A block long enough that every projection of the fp32 model takes 64-row tiles (the last tile has 16 rows)."""
    desc, seed = LARGE_FP32, 19
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 64 * -(-n_cu // 16) + 16
    qkv = (desc.n_q_heads + 2 * desc.n_kv_heads) * desc.head_dim
    for cols in (qkv, desc.d_model, desc.d_ffn, desc.vocab):
        assert cols // 64 * -(-n // 32) > 2 * n_cu
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(3).integers(0, desc.vocab, size=n - 1).astype(np.int32)
    return weights, seed, draft, _round(desc, weights, seed, draft)


@pytest.mark.parametrize("first, rows", [(0, 1), (0, 15), (0, 64), (500, 17), (1008, 32)])
def test_fp32_small_tiles_match_the_large_block(large_block, first, rows):
    """Rows first .. first + rows - 1 of the large block, scored on top of the rows before them, which come in 64 at a
    time: 16-row tiles at every projection, in the K/V they leave as in the rows compared."""
    desc = LARGE_FP32
    weights, seed, draft, large = large_block
    spec = SequenceSpec(0, 37, 3, len(draft), 0.0)
    eng = make_engine(desc, weights, [spec], max_total_q=64, max_dump=64)
    _, _, tok, emb, pending = prefix_rows(desc, seed, spec)
    block = np.concatenate([[pending], draft]).astype(np.int32)
    eng.prefill([0], [tok], [emb])
    if first:
        eng.prefill([0], [block[:first]], chunk=64)
    out = eng.verify([0], [block[first:first + rows]], "region", dump_rows=np.arange(rows))
    for a, b in zip(large, (out.argmax, out.margin, out.logits)):
        np.testing.assert_array_equal(a[first:first + rows], b.cpu().numpy())
    eng.close()


def _bands(rows, cols, bp, bq, k, n_cu):
    """log2 of the activation bands that a launch of tiles of bp x bq over rows x cols is cut into on the XCDs, -1: none."""
    if bp < 128 and k < 2048:
        return -1
    act, wgt, best = -(-rows // bp), cols // bq, -1
    least = 8 * (act * bp + -(-wgt // 8) * bq) // 10
    for band in (1, 2):
        a, w = 1 << band, 8 >> band
        reads = -(-act // a) * bp + -(-wgt // w) * bq
        if act >= a and wgt >= w and 8 * -(-act // a) * -(-wgt // w) <= n_cu and reads < least:
            best, least = band, reads
    return best


@pytest.mark.parametrize("rows", [576, 577, 641, 897, 1025, 1281, 1300, 1856, 2049, 2304])
def test_banded_tile_order(rows):
    """Launches whose tiles are dealt to the XCDs in rectangles (2 bands of activation tiles by 4 of weight tiles, or 4 by 2; also
    where the tiles do not divide evenly, so that workgroups stay without one) against the generic kernel: a tile left out or
    taken twice would leave rows or columns of O, down (64x64, 128x64 and 144x64 tiles) or QKV wrong."""
    desc, seed = W.ModelDesc(1, 1024, 16, 4, 64, 2048, 512, "bf16"), 31
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if n_cu == 256:
        tile = 64 if rows <= 1024 else 128 if rows <= 2048 else 144
        assert _bands(rows, 1024, tile, 64, 2048, n_cu) == (-1 if rows <= 576 else 1 if rows <= 1280 else 2)     # down
        assert _bands(rows, 1024, tile, 64, 1024, n_cu) == (-1 if rows <= 1024 else 1 if rows <= 1280 else 2)    # O
        if 640 < rows <= 1440:
            assert _bands(rows, 1536, 128 if rows <= 1280 else 144, 64, 1024, n_cu) == (1 if rows > 896 else -1)
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    for a, b in zip(_round(desc, weights, seed, draft), _round(desc, weights, seed, draft, {"gemm_cfg": (2, 2, 2, 2, 0)})):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n_q, n_kv", [(16, 4), (3, 3), (1, 1)])
def test_fp32_tile_forms_agree(n_q, n_kv):
    """The forms of the fp32 GEMM -- half a column group or a whole one by 16 rows, 32 and 64 rows through LDS -- give a row the same
    bits at every projection: blocks of a length for each on the way through one that takes the last form everywhere.  K of
    the output projection is 64 n_q: 64 and 192 are no multiples of the longest chunk.  The first rows against the oracle."""
    desc, seed = W.ModelDesc(1, 1024, n_q, n_kv, 64, 1024, 1024, "fp32"), 23
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    groups = {"qkv": n_q + 2 * n_kv, "o": 16, "gate_up": 16, "lm_head": 16}
    least = min(groups.values())

    def form(g, rows, lm=False):                       # the launch's rule
        t16, t32 = g * -(-rows // 16), g * -(-rows // 32)
        return 0 if 2 * t16 <= n_cu and not lm else 1 if t16 <= n_cu else 2 if t32 <= 2 * n_cu else 3

    large = 32 * (2 * n_cu // least + 1)
    sizes = sorted({16 * max(1, n_cu // (4 * g)) for g in groups.values()} | {16 * (n_cu // g) for g in groups.values()}
                   | {32 * (2 * n_cu // g) - 5 for g in groups.values()})
    for name, g in groups.items():
        seen = {form(g, r, name == "lm_head") for r in sizes} | {form(g, large, name == "lm_head")}
        assert seen >= ({1, 2, 3} if name == "lm_head" else {0, 1, 2, 3}), (name, seen)
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(n_q).integers(0, desc.vocab, size=large - 1).astype(np.int32)
    want = _round(desc, weights, seed, draft)
    for rows in sizes:
        got = _round(desc, weights, seed, draft[:rows - 1])
        for a, b in zip(want, got):
            np.testing.assert_array_equal(a[:rows], b)
    vis, prompt = W.make_prefix(desc, seed, 0, 37, 3)
    cache, pending = O.prefill(desc, weights, vis, prompt)
    ref = O.verify_block(desc, weights, cache, pending, draft[:15])[3]
    assert np.abs(want[2][:16] - ref).max() <= 1e-4


@pytest.mark.parametrize("rows", [1, 33])
def test_plain_kernels_on_a_bf16_model(rows):
    desc, seed = W.ModelDesc(3, 256, 8, 2, 64, 512, 1024, "bf16"), 29
    weights = W.make_weights(desc, seed)
    vis, prompt = W.make_prefix(desc, seed, 0, 37, 3)
    draft = np.random.default_rng(rows).integers(0, desc.vocab, size=rows - 1).astype(np.int32)
    cache, pending = O.prefill(desc, weights, vis, prompt)
    _, _, u_hat, ref = O.verify_block(desc, weights, cache, pending, draft)
    argmax, _, logits = _round(desc, weights, seed, draft, {"force_simple": 1})
    assert np.abs(logits - ref).max() <= 2e-2
    assert len(gated_compare_argmax(argmax, u_hat, O.top2_margin(ref))[0]) == 0
