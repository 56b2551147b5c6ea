"""Kernels chosen for launches of few rows against the general ones, bit for bit: the narrow (32-column) tiles of the
bf16 projections against a tile set by hand, the 16-row tiles of the fp32 path against the 64-row ones that a block
with enough rows takes.  Every output sums its products in one fixed order in all of them, so the tolerance is zero."""
import numpy as np
import pytest

import workloads as W
from workloads.generators import SequenceSpec

from hsd_testlib import make_engine, prefix_rows

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


@pytest.mark.parametrize("rows", [1, 15, 17, 64])
def test_fp32_small_tiles_match_the_large_block(rows):
    """1040 rows x 1024 gate/up columns or vocabulary entries are 17 x 16 tiles of 64 rows, one per compute unit and more."""
    desc, seed = W.ModelDesc(2, 128, 4, 1, 64, 1024, 1024, "fp32"), 19
    weights = W.make_weights(desc, seed)
    draft = np.random.default_rng(3).integers(0, desc.vocab, size=1039).astype(np.int32)
    large, small = _round(desc, weights, seed, draft), _round(desc, weights, seed, draft[:rows - 1])
    for a, b in zip(large, small):
        np.testing.assert_array_equal(a[:rows], b)
