// Check of the refit plan as the device reads it (refit_words in refit_plan.h), over
// trees of several shapes, built with the address and undefined-behaviour sanitizers by
// the CPU test suite: the plan carried out from its words alone gives every slot its box,
// and the words take no more memory than the arrays that a refit level by level needs (a
// word per record for its patch and one for its parent, a word per node for its parent and
// one for the list of nodes by depth).  Prints one line per case; exit status 1 on failure.

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <functional>
#include <random>
#include <string>
#include <vector>

#include "../../paper_1811_03510_amd/csrc/refit_plan.h"

namespace {

int g_failures = 0;

void check(bool ok, const std::string& what) {
  if (!ok) {
    std::printf("FAIL: %s\n", what.c_str());
    ++g_failures;
  }
}

struct Interval {
  float lo, hi;
};

// A tree over n records in depth-first order; split(b, e, depth) gives the first record
// of the right half.  Boxes are intervals, in the first component of the node's boxes.
struct Tree {
  std::vector<float> nodes;
  std::vector<int32_t> leaf_parent, node_parent;
  std::vector<Interval> records;
};

float* slot_of(std::vector<float>& nodes, int32_t slot) {
  return nodes.data() + 16 * (size_t)(slot >> 1) + ((slot & 1) ? 6 : 0);
}

Tree make_tree(uint32_t n, const std::function<uint32_t(uint32_t, uint32_t, uint32_t)>& split) {
  Tree t;
  std::mt19937 g(n);
  std::uniform_real_distribution<float> U(-100.0f, 100.0f);
  for (uint32_t k = 0; k < n; ++k) {
    const float x = U(g);
    t.records.push_back({x, x + 1.0f});
  }
  const uint32_t n_nodes = n <= 1 ? n : n - 1;
  t.nodes.assign(16 * (size_t)n_nodes, 0.0f);
  t.leaf_parent.assign(n, -1);
  t.node_parent.assign(n_nodes, -1);
  auto put = [&](int32_t slot, const Interval& x, int32_t ref) {
    float* f = slot_of(t.nodes, slot);
    f[0] = x.lo;
    f[3] = x.hi;
    std::memcpy(t.nodes.data() + 16 * (size_t)(slot >> 1) + 12 + (slot & 1), &ref, 4);
  };
  std::function<Interval(uint32_t, uint32_t, uint32_t, uint32_t)> build = [&](uint32_t b, uint32_t e, uint32_t node,
                                                                              uint32_t depth) {
    const uint32_t m = split(b, e, depth);
    const uint32_t child[2] = {node + 1, node + (m - b)}, from[2] = {b, m}, to[2] = {m, e};
    Interval both{1e30f, -1e30f};
    for (uint32_t s = 0; s < 2; ++s) {
      const int32_t slot = (int32_t)(node << 1 | s);
      Interval x;
      if (to[s] - from[s] == 1) {
        t.leaf_parent[from[s]] = slot;
        x = t.records[from[s]];
        put(slot, x, ~(int32_t)from[s]);
      } else {
        t.node_parent[child[s]] = slot;
        x = build(from[s], to[s], child[s], depth + 1);
        put(slot, x, (int32_t)child[s]);
      }
      both = {std::min(both.lo, x.lo), std::max(both.hi, x.hi)};
    }
    return both;
  };
  if (n == 1) {
    put(0, t.records[0], ~0);
    put(1, t.records[0], ~0);
    t.leaf_parent[0] = 0;
  } else if (n > 1) {
    build(0, n, 0, 0);
  }
  return t;
}

void verify(const std::string& name, const Tree& t, uint32_t cap0, uint32_t cap1, bool limit) {
  const int before = g_failures;
  const uint32_t n = (uint32_t)t.leaf_parent.size(), n_nodes = (uint32_t)t.node_parent.size();
  const ccs::RefitPlan plan = ccs::plan_refit(t.nodes, t.leaf_parent, t.node_parent, cap0, cap1);
  const ccs::RefitWords w = ccs::refit_words(plan, t.leaf_parent, t.node_parent);
  if (limit) check(w.words.size() <= 2 * (size_t)n + 2 * (size_t)n_nodes, name + ": no more memory than level by level");
  check(w.one_block == (n <= cap0), name + ": one block");
  auto word = [&](size_t at, size_t k) { return w.words.at(at + k); };
  auto link = [&](size_t at, size_t k) { return (int32_t)w.words.at(at + k); };
  std::vector<float> nodes = t.nodes;  // boxes cleared, references kept
  for (size_t k = 0; k < n_nodes; ++k) std::fill(nodes.begin() + 16 * k, nodes.begin() + 16 * k + 12, 0.0f);
  auto store = [&](int32_t slot, const Interval& x) {
    float* f = slot_of(nodes, slot);
    f[0] = x.lo;
    f[3] = x.hi;
  };
  std::mt19937 g(n + cap0);
  for (size_t q = 0; q < plan.passes.size(); ++q)
    for (uint32_t b = plan.passes[q].first_block; b < plan.passes[q].first_block + plan.passes[q].n_blocks; ++b) {
      uint32_t i0 = 0, i1 = n, n0 = 0, n1 = n_nodes;
      if (!w.one_block) {
        i0 = word(w.block_items, b);
        i1 = word(w.block_items, b + 1);
        n0 = word(w.block_nodes, b);
        n1 = word(w.block_nodes, b + 1);
      }
      std::vector<uint32_t> order;
      for (uint32_t k = i0; k < i1; ++k) order.push_back(k);
      std::shuffle(order.begin(), order.end(), g);
      std::vector<int> arrived(n1 - n0, 0);
      for (const uint32_t k : order) {
        Interval x;
        if (q == 0) {
          x = t.records[k];
        } else {
          const float* f = slot_of(nodes, link(w.item_slot, k - n));
          x = {f[0], f[3]};
        }
        int32_t up = link(w.item_up, k);
        if (n == 1) {
          store(0, x);
          store(1, x);
        } else if (up < 0) {
          check(q == 0, name + ": an item without a parent in its block is a record");
          store(~up, x);
        } else {
          for (;;) {
            const uint32_t j = (uint32_t)up >> 1;
            check(j < n1 - n0, name + ": parent inside the block");
            const uint32_t id = word(w.node_id, n0 + j);
            store((int32_t)(id << 1 | (uint32_t)(up & 1)), x);
            if (arrived.at(j)++ == 0) break;
            const float *l = slot_of(nodes, (int32_t)(id << 1)), *r = slot_of(nodes, (int32_t)(id << 1 | 1u));
            x = {std::min(l[0], r[0]), std::max(l[3], r[3])};
            up = link(w.node_up, n0 + j);
            if (up < 0) {
              check((up == ccs::kRefitTop) == (id == 0), name + ": only the root has no slot");
              if (up != ccs::kRefitTop) store(~up, x);
              break;
            }
          }
        }
      }
    }
  check(nodes.empty() || std::memcmp(nodes.data(), t.nodes.data(), nodes.size() * sizeof(float)) == 0, name + ": every slot's box");
  std::printf("%s %s: n=%u passes=%zu words=%zu\n", g_failures == before ? "ok" : "FAILED", name.c_str(), n,
              plan.passes.size(), w.words.size());
}

}  // namespace

int main() {
  auto middle = [](uint32_t b, uint32_t e, uint32_t) { return b + (e - b) / 2; };
  std::mt19937 g(3);
  auto any = [&](uint32_t b, uint32_t e, uint32_t) { return b + 1 + (uint32_t)(g() % (e - b - 1)); };
  // one record off until 65 are left, with a halving every `every` levels: the most roots
  auto comb = [](uint32_t every) {
    return [every](uint32_t b, uint32_t e, uint32_t depth) {
      return e - b <= 65 || depth % every == 0 ? b + (e - b) / 2 : (depth & 1) != 0 ? b + 1 : e - 1;
    };
  };
  for (uint32_t n : {0u, 1u, 2u, 3u, 4u, 7u, 63u, 64u, 65u, 66u, 129u, 512u, 1000u, 70000u}) {
    verify("halves", make_tree(n, middle), 64, 1024, true);
    verify("anywhere", make_tree(n, any), 64, 1024, true);
    verify("halves, small blocks", make_tree(n, middle), 2, 3, false);
    verify("anywhere, small blocks", make_tree(n, any), 2, 2, false);
  }
  for (uint32_t every : {2u, 5u, 20u}) {
    verify("combs", make_tree(60, comb(every)), 64, 1024, true);
    verify("combs", make_tree(3000, comb(every)), 64, 1024, true);
    verify("combs", make_tree(50000, comb(every)), 64, 1024, true);
  }
  std::printf("%d failure(s)\n", g_failures);
  return g_failures ? 1 : 0;
}
