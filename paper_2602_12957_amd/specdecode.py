"""Host orchestration of decoupled speculative verification on top of the HIP verification library
(paper Section 3.2; host logic only: everything numeric runs in the library's kernels).

Per round and sequence: match the reference window (the last n accepted tokens) against the fixed draft set
(Eq. 5-6), cap and pack the candidate continuations into one prefix tree, verify all sequences' trees in one
batched pass, commit, and continue from the bonus token.  A sequence without candidates takes a plain decoding
step in the same pass (its tree is the root alone).  Stage 1 / Stage 2 of the hierarchy (Eq. 2-4) are two calls
of the same driver: regions in one batch, then the page with the regions' outputs as its draft set.
"""
from __future__ import annotations

from typing import List, Optional, Sequence

import numpy as np

from . import binding as B
from .runtime import Engine


def match_candidates(accepted: Sequence[int], drafts: Sequence[Sequence[int]], n: int) -> List[List[int]]:
    """Suffixes that follow an occurrence of the window (last n accepted tokens) in any draft (Eq. 5-6); while fewer
    than n tokens are accepted the window is everything accepted so far, and with nothing accepted every draft is
    a candidate from its start.  Duplicates removed; order: by draft, then by position."""
    w = [int(t) for t in accepted[-n:]] if n > 0 and len(accepted) else []
    out, seen = [], set()
    for d in drafts:
        d = [int(t) for t in d]
        if not w:
            starts = [0]
        else:
            arr = np.asarray(d, dtype=np.int64)
            hit = np.ones(max(len(d) - len(w) + 1, 0), dtype=bool)
            for k, t in enumerate(w):
                hit &= arr[k:k + len(hit)] == t
            starts = np.nonzero(hit)[0].tolist()
        for j in starts:
            suf = tuple(d[j + len(w):])
            if suf and suf not in seen:
                seen.add(suf)
                out.append(list(suf))
    return out


def cap_candidates(candidates: Sequence[Sequence[int]], max_packed: int) -> List[List[int]]:
    """Cuts every candidate at one common depth, the largest whose packed tree (root included) has at most
    max_packed rows.  The tree has one row per distinct candidate prefix, so its size at cut depth L is
    1 + sum over depths k <= L of the number of distinct length-k prefixes: one pass over the depths."""
    cands = [tuple(int(t) for t in c) for c in candidates if len(c)]
    if not cands:
        return []
    rows, depth = 1, 0
    for k in range(1, max(len(c) for c in cands) + 1):
        level = len({c[:k] for c in cands if len(c) >= k})
        if rows + level > max_packed and k > 1:
            break
        rows, depth = rows + level, k
    out, seen = [], set()
    for c in cands:
        head = c[:depth]
        if head not in seen:
            seen.add(head)
            out.append(list(head))
    return out


class DraftTrees:
    """A sequence's draft set in the library: `tree` is match_candidates, cap_candidates and runtime.pack_prefix_tree in
    one native call."""

    def __init__(self, drafts: Sequence[Sequence[int]]):
        rows = [self._ints(d) for d in drafts]
        offsets = np.zeros(len(rows) + 1, dtype=np.int64)
        np.cumsum([len(r) for r in rows], out=offsets[1:])
        self._set = B.hsd_drafts_create(np.concatenate(rows) if rows else np.zeros(0, np.int64), offsets)

    @staticmethod
    def _ints(d):
        a = np.asarray(d)
        return np.ascontiguousarray(a, dtype=np.int64) if a.ndim == 1 and a.dtype.kind in "iu" and a.dtype != np.uint64 else \
            np.fromiter((int(t) for t in d), dtype=np.int64, count=len(d))

    def tree(self, accepted: Sequence[int], n: int, pending: int, max_packed: int):
        """(tokens, tree_end, tree_depth) of the capped, packed candidates that follow the last n accepted tokens.
        max_packed is any number, as cap_candidates takes it: infinity cuts nothing."""
        window = np.asarray(accepted[-n:] if n > 0 else [], dtype=np.int64)
        # ctypes hands the low 64 bits of an int to the library without a word: both numbers are brought into range here
        pending, most = int(pending), 2 ** 31 - 1
        if not -2 ** 63 <= pending < 2 ** 63:
            raise OverflowError("the pending token does not fit 32 bits")
        cap = int(max(max_packed, 0)) if max_packed < most else most
        out = np.empty((3, max(min(cap, 4096), 1)), dtype=np.int32)
        rc, rows = B.hsd_drafts_tree(self._set, window, pending, cap, out)
        if rc == B.HSD_ENOSPC and rows > out.shape[1]:
            out = np.empty((3, rows), dtype=np.int32)
            rc, rows = B.hsd_drafts_tree(self._set, window, pending, cap, out)
        if rc == B.HSD_ERANGE:
            raise OverflowError("a token of the packed tree does not fit 32 bits")
        B.check("hsd_drafts_tree", rc)
        return out[0, :rows], out[1, :rows], out[2, :rows]

    def close(self):
        if self._set is not None:
            B.hsd_drafts_destroy(self._set)
            self._set = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


class SpecDecoder:
    """SpecDecode(p_theta, z, Y~) (Eq. 1) for a batch of sequences whose prefixes are already in the engine's cache."""

    def __init__(self, engine: Engine, n_window: int = 3, max_packed: int = 128, log_tau: float = 0.0,
                 mode: str = "region"):
        self.eng, self.n_window, self.max_packed, self.log_tau, self.mode = engine, n_window, max_packed, log_tau, mode

    def run(self, slots: Sequence[int], pending: Sequence[int], draft_sets: Sequence[Sequence[Sequence[int]]],
            n_tokens: Sequence[int], eos: Optional[int] = None):
        """Generates n_tokens[i] tokens (or up to `eos`) for sequence slots[i] from its draft set.
        Returns (outputs: list of int arrays, stats: dict with rounds, verified rows, accepted tokens, plain steps)."""
        n = len(slots)
        out: List[List[int]] = [[] for _ in range(n)]
        pend = [int(p) for p in pending]
        done = [False] * n
        stats = dict(rounds=0, rows=0, accepted=0, plain_steps=0, seq_rounds=0,
                     per_seq=[[] for _ in range(n)])      # per sequence: (tree rows, accepted) of each of its rounds
        draft_trees = [DraftTrees(draft_sets[i]) for i in range(n)]
        while not all(done):
            active = [i for i in range(n) if not done[i]]
            blocks, trees = [], []
            for i in active:
                t, e, d = draft_trees[i].tree(out[i], self.n_window, pend[i], self.max_packed)
                blocks.append(t), trees.append((e, d))
                stats["plain_steps"] += int(len(t) == 1)
                stats["rows"] += len(t)
            self.eng.verify([slots[i] for i in active], blocks, self.mode, log_tau=self.log_tau, trees=trees)
            self.eng.commit()
            alpha, bonus, status, stop = self.eng.read_acceptance(len(active), stop_rows=True)
            if status:
                raise RuntimeError(f"SpecDecoder: device status {status}")
            for j, i in enumerate(active):
                # the accepted path: from the root down to the stop node
                path = np.empty(int(alpha[j]), dtype=np.int32)
                B.hsd_tree_path(blocks[j], trees[j][0], int(stop[j]), len(path), path)
                path = path.tolist()
                out[i].extend(path)
                out[i].append(int(bonus[j]))
                pend[i] = int(bonus[j])
                stats["accepted"] += int(alpha[j])
                stats["seq_rounds"] += 1
                stats["per_seq"][i].append((len(blocks[j]), int(alpha[j])))
                if len(out[i]) >= n_tokens[i] or (eos is not None and eos in path + [int(bonus[j])]):
                    done[i] = True
            stats["rounds"] += 1
        res = []
        for i in range(n):
            seq = out[i][: n_tokens[i]]
            if eos is not None and eos in seq:
                seq = seq[: seq.index(eos) + 1]
            res.append(np.asarray(seq, dtype=np.int32))
        return res, stats
