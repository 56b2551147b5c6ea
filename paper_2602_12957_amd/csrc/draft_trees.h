// Host side of decoupled verification (paper Section 3.2, Eq. 5-7), native because a round of a few regions spends as long
// here as on the GPU otherwise: match the reference window against a sequence's draft set, cut the candidates at the depth
// whose packed tree fits the cap, and pack them.  The definitions are match_candidates and cap_candidates of specdecode.py
// and pack_prefix_tree of runtime.py; this is the three in one pass over the candidates, one level of the tree at a time,
// which never builds what the cap would cut.  8 regions with two drafts of 128 tokens, 20 rounds: 10 ms in Python.
#pragma once

#include <cstdint>
#include <vector>

namespace hsd {

struct DraftSet {
  std::vector<int64_t> tokens;
  std::vector<int64_t> begin;   // n_drafts + 1 offsets into tokens
};

class DraftTree {
 public:
  // Nodes in level order; children of a node in the order in which their tokens first appear among the candidates.
  std::vector<int64_t> token;
  std::vector<int32_t> parent, depth, row, size;

  void build(const DraftSet &ds, const int64_t *window, int n_window, int64_t pending, int64_t max_packed) {
    struct Cand {
      const int64_t *t;
      int64_t n;
      int32_t node;
    };
    std::vector<Cand> cands;
    for (size_t d = 0; d + 1 < ds.begin.size(); ++d) {
      const int64_t *t = ds.tokens.data() + ds.begin[d];
      const int64_t n = ds.begin[d + 1] - ds.begin[d];
      if (n_window == 0) {
        if (n > 0) cands.push_back({t, n, 0});
        continue;
      }
      for (int64_t j = 0; j + n_window < n; ++j) {   // (an occurrence at the very end has no suffix)
        int k = 0;
        while (k < n_window && t[j + k] == window[k]) ++k;
        if (k == n_window) cands.push_back({t + j + n_window, n - j - n_window, 0});
      }
    }
    add(pending, -1, 0);
    for (int64_t k = 0;; ++k) {   // the level of depth k + 1
      const size_t level0 = token.size();
      bool over = false;
      for (Cand &c : cands) {
        if (c.n <= k) continue;
        int32_t child = first_[c.node];
        while (child >= 0 && token[child] != c.t[k]) child = next_[child];
        if (child < 0) {
          if (k > 0 && static_cast<int64_t>(token.size()) + 1 > max_packed) {
            over = true;   // this level does not fit: the cut is at the level before
            break;
          }
          child = add(c.t[k], c.node, static_cast<int32_t>(k + 1));
        }
        c.node = child;
      }
      if (over) {
        token.resize(level0), parent.resize(level0), depth.resize(level0);
        break;
      }
      if (token.size() == level0) break;   // no candidate is this long
    }
    // sizes of the subtrees, then pre-order rows: a child comes after the subtrees of its elder siblings
    const size_t n = token.size();
    size.assign(n, 1), row.assign(n, 0);
    for (size_t v = n; v-- > 1;) size[parent[v]] += size[v];
    std::vector<int32_t> used(n, 1);   // rows of a node's subtree given out so far
    for (size_t v = 1; v < n; ++v) {
      row[v] = row[parent[v]] + used[parent[v]];
      used[parent[v]] += size[v];
    }
  }

 private:
  std::vector<int32_t> first_, last_, next_;   // child lists; of a level that was cut off they are not looked at again
  int32_t add(int64_t t, int32_t p, int32_t d) {
    const int32_t v = static_cast<int32_t>(token.size());
    token.push_back(t), parent.push_back(p), depth.push_back(d);
    first_.push_back(-1), last_.push_back(-1), next_.push_back(-1);
    if (p >= 0) {
      if (last_[p] < 0) first_[p] = v;
      else next_[last_[p]] = v;
      last_[p] = v;
    }
    return v;
  }
};

}  // namespace hsd
