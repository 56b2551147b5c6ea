"""The library's native matching, cutting and packing (hsd_drafts_tree, hsd_tree_path) against the Python definitions it
stands for: match_candidates, cap_candidates and pack_prefix_tree, exactly."""
import ctypes as C

import numpy as np
import pytest

import paper_2602_12957_amd.binding as B
from paper_2602_12957_amd.runtime import pack_prefix_tree
from paper_2602_12957_amd.specdecode import DraftTrees, cap_candidates, match_candidates


@pytest.mark.parametrize("vocab", [1, 2, 3, 50])
def test_native_trees_equal_the_python_definitions(vocab):
    rng = np.random.default_rng(vocab)
    for _ in range(400):
        drafts = [rng.integers(0, vocab, size=int(rng.integers(0, 25))).tolist() for _ in range(int(rng.integers(0, 5)))]
        accepted = rng.integers(0, vocab, size=int(rng.integers(0, 9))).tolist()
        n, cap = int(rng.integers(0, 5)), int(rng.choice([1, 2, 3, 5, 8, 20, 128, 10 ** 6]))
        expect = pack_prefix_tree(7, cap_candidates(match_candidates(accepted, drafts, n), cap))
        got = DraftTrees(drafts).tree(accepted, n, 7, cap)
        for a, b in zip(expect, got):
            assert b.dtype == np.int32
            np.testing.assert_array_equal(a, b)
        tok, end, dep = got
        stop = int(rng.integers(0, len(tok)))
        path = np.empty(int(dep[stop]), np.int32)
        B.hsd_tree_path(tok, end, stop, len(path), path)
        s, back = stop, []
        while dep[s] > 0:                              # up from the stop node: the nearest earlier row one level higher
            back.append(int(tok[s]))
            s = max(r for r in range(s) if dep[r] == dep[s] - 1)
        assert path.tolist() == back[::-1]


def test_inputs_of_every_kind_and_long_drafts():
    long = list(range(5000))
    for drafts in ([long], [np.arange(5000)], [tuple(long)], [np.arange(5000, dtype=np.int16)], [[float(t) for t in long]]):
        tok, end, dep = DraftTrees(drafts).tree([], 3, 1, 10 ** 6)     # more rows than the first buffer holds
        assert tok[1:].tolist() == long and (end == 5001).all() and dep.tolist() == list(range(5001))
    with pytest.raises(OverflowError):
        DraftTrees([[2 ** 40]]).tree([], 1, 0, 8)
    assert DraftTrees([[2 ** 40, 5, 6]]).tree([5], 1, 0, 8)[0].tolist() == [0, 6]


@pytest.mark.parametrize("cap", [float("inf"), float("-inf"), float("nan"), 4.5, -1, 0, 2 ** 31, 2 ** 63, 2 ** 64 + 2, -2 ** 70])
def test_any_number_as_the_cap(cap):
    drafts = [[1, 2, 3], [1, 5, 6]]
    for a, b in zip(pack_prefix_tree(0, cap_candidates(match_candidates([], drafts, 3), cap)), DraftTrees(drafts).tree([], 3, 0, cap)):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("pending", [2 ** 31, -2 ** 31 - 1, 2 ** 63, 2 ** 64 + 5])
def test_a_pending_token_out_of_range_is_refused(pending):
    with pytest.raises(OverflowError):
        DraftTrees([[1, 2]]).tree([], 3, pending, 8)


def test_bad_arguments_are_refused():
    out, n = C.c_void_p(), C.c_int32()
    off = np.array([0, 2, 1], np.int64)
    tok = np.zeros(4, np.int64)
    assert B.lib.hsd_drafts_create(tok.ctypes.data, off.ctypes.data, 2, C.byref(out)) == B.HSD_EINVAL
    assert B.lib.hsd_drafts_create(None, np.array([0, 2], np.int64).ctypes.data, 1, C.byref(out)) == B.HSD_EINVAL
    assert B.lib.hsd_drafts_tree(None, None, 0, 0, 8, 0, None, None, None, C.byref(n)) == B.HSD_EINVAL
    t, e = np.array([1, 2, 3], np.int32), np.array([3, 2, 3], np.int32)
    path = np.zeros(3, np.int32)
    for args in ((3, 3, 1), (3, 0, 1), (3, 1, 2), (0, 0, 0)):
        assert B.lib.hsd_tree_path(t.ctypes.data, e.ctypes.data, *args, path.ctypes.data) == B.HSD_EINVAL
