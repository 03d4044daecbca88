// Check of the refit's work plan (refit_plan.h) over BVHs of several shapes, built
// with the address and undefined-behaviour sanitizers by the CPU test suite: every
// block within its capacity, pass 0 covering the records in order, every node in
// exactly one block, and the plan carried out (each block's items in a shuffled
// order, the second child to reach a node going on) gives every slot the builder's
// box from slots that hold nothing.  Prints one line per case; exit status 1 on failure.

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "../../paper_1811_03510_amd/csrc/bvh_build.h"
#include "../../paper_1811_03510_amd/csrc/refit_plan.h"

namespace {

int g_failures = 0;

void check(bool ok, const std::string& what) {
  if (!ok) {
    std::printf("FAIL: %s\n", what.c_str());
    ++g_failures;
  }
}

struct Box {
  float v[6];
};

Box join(const Box& a, const Box& b) {
  Box r;
  for (int k = 0; k < 3; ++k) {
    r.v[k] = std::min(a.v[k], b.v[k]);
    r.v[3 + k] = std::max(a.v[3 + k], b.v[3 + k]);
  }
  return r;
}

void verify(const std::string& name, uint32_t n, uint32_t sah_depth, uint32_t cap0, uint32_t cap1, bool line) {
  const int before = g_failures;
  std::mt19937 g(n * 31 + cap0);
  std::uniform_real_distribution<float> U(-100.0f, 100.0f);
  std::vector<ccs::BuildBox> in(n);
  for (uint32_t k = 0; k < n; ++k)
    for (int a = 0; a < 3; ++a) {
      // a line of boxes with geometrically growing gaps makes a lopsided tree
      in[k].lo[a] = line ? (a == 0 ? std::ldexp(1.0f, (int)(k % 120) - 60) : 0.0f) : U(g);
      in[k].hi[a] = in[k].lo[a] + 0.5f;
    }
  const ccs::BvhOutput o = ccs::build_bvh(in, sah_depth, 4);
  const ccs::RefitPlan p = ccs::plan_refit(o.nodes, o.leaf_parent, o.node_parent, cap0, cap1);
  std::vector<float> nodes = o.nodes;  // boxes cleared, references kept
  for (size_t k = 0; k < nodes.size() / 16; ++k) std::fill(nodes.begin() + 16 * k, nodes.begin() + 16 * k + 12, 1e30f);
  auto slot = [&](int32_t s) { return nodes.data() + 16 * (size_t)(s >> 1) + ((s & 1) ? 6 : 0); };
  std::vector<int> seen(o.node_parent.size(), 0);
  for (size_t q = 0; q < p.passes.size(); ++q) {
    const ccs::RefitPass& pass = p.passes[q];
    check(pass.n_blocks > 0, name + ": a pass has blocks");
    for (uint32_t b = pass.first_block; b < pass.first_block + pass.n_blocks; ++b) {
      const uint32_t i0 = p.block_items[b], i1 = p.block_items[b + 1], n0 = p.block_nodes[b], n1 = p.block_nodes[b + 1];
      const uint32_t cap = q == 0 ? cap0 : cap1;
      check(i1 > i0 && i1 - i0 <= cap && n1 - n0 <= cap, name + ": block within its capacity");
      std::vector<uint32_t> order;
      for (uint32_t k = i0; k < i1; ++k) order.push_back(k);
      std::shuffle(order.begin(), order.end(), g);
      std::vector<int> arrived(n1 - n0, 0);
      for (uint32_t k : order) {
        Box x;
        if (q == 0) {
          check(k < n, name + ": items of pass 0 are the records");
          const ccs::BuildBox& bb = in[o.perm[k]];
          for (int a = 0; a < 3; ++a) {
            x.v[a] = bb.lo[a];
            x.v[3 + a] = bb.hi[a];
          }
          if (n == 1) std::memcpy(slot(1), x.v, sizeof x.v);
          std::memcpy(slot(o.leaf_parent[k]), x.v, sizeof x.v);
        } else {
          std::memcpy(x.v, slot(p.item_slot[k - n]), sizeof x.v);
        }
        for (int32_t link = p.item_up[k]; link >= 0;) {
          const uint32_t j = n0 + ((uint32_t)link >> 1);
          check(j < n1, name + ": parent inside the block");
          const uint32_t id = p.node_id[j];
          std::memcpy(slot((int32_t)(id << 1 | (uint32_t)(link & 1))), x.v, sizeof x.v);
          if (arrived[j - n0]++ == 0) break;
          seen[id]++;
          Box l, r;
          std::memcpy(l.v, slot((int32_t)(id << 1)), sizeof l.v);
          std::memcpy(r.v, slot((int32_t)(id << 1 | 1u)), sizeof r.v);
          x = join(l, r);
          link = p.node_up[j];
          if (link < 0 && o.node_parent[id] >= 0) std::memcpy(slot(o.node_parent[id]), x.v, sizeof x.v);
        }
      }
    }
  }
  if (n > 0) check(p.block_items[p.passes[0].first_block + p.passes[0].n_blocks] == n, name + ": pass 0 covers the records");
  bool once = true;
  for (int c : seen) once = once && c == (n == 1 ? 0 : 1);
  check(once, name + ": every node completed exactly once");
  check(nodes.empty() || std::memcmp(nodes.data(), o.nodes.data(), nodes.size() * sizeof(float)) == 0,
        name + ": the builder's boxes");
  std::printf("%s %s: n=%u depth=%u passes=%zu\n", g_failures == before ? "ok" : "FAILED", name.c_str(), n, o.max_depth,
              p.passes.size());
}

}  // namespace

int main() {
  for (uint32_t n : {0u, 1u, 2u, 3u, 63u, 64u, 65u, 66u, 129u, 512u, 1000u, 70000u}) {
    verify("random", n, 40, 64, 1024, false);
    verify("random, small blocks", n, 40, 2, 3, false);
  }
  verify("lopsided", 120, 47, 64, 1024, true);
  verify("lopsided, small blocks", 120, 47, 2, 2, true);
  verify("lopsided, many", 5000, 35, 64, 1024, true);
  std::printf("%d failure(s)\n", g_failures);
  return g_failures ? 1 : 0;
}
