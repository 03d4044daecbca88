#include "refit_plan.h"

#include <cstddef>
#include <cstring>
#include <utility>

namespace ccs {

RefitPlan plan_refit(const std::vector<float>& nodes, const std::vector<int32_t>& leaf_parent,
                     const std::vector<int32_t>& node_parent, uint32_t cap0, uint32_t cap1) {
  RefitPlan plan;
  const uint32_t n_nodes = (uint32_t)node_parent.size(), n = (uint32_t)leaf_parent.size();
  if (n == 0) return plan;
  auto child = [&](int32_t slot) {
    int32_t c;
    std::memcpy(&c, nodes.data() + 16 * (size_t)(slot >> 1) + 12 + (slot & 1), 4);
    return c;
  };
  std::vector<uint32_t> count(n_nodes, 0);   // items of the current pass below a node
  std::vector<uint8_t> item(2 * (size_t)n_nodes, 0);  // from pass 1 on: the slot's box is an item
  std::vector<int32_t> local(n_nodes);       // a node's index in its block
  for (uint32_t r = 0; r < n; ++r) count[(uint32_t)leaf_parent[r] >> 1]++;
  for (uint32_t k = n_nodes; k-- > 1;) count[(uint32_t)node_parent[k] >> 1] += count[k];  // children follow parents
  plan.item_up.reserve(n + n / 16);
  plan.node_id.reserve(n_nodes);
  plan.node_up.reserve(n_nodes);
  std::vector<uint32_t> live;                // nodes no treelet holds yet, parents first
  std::vector<int32_t> next, above, stack;   // slots
  for (bool done = false; !done;) {
    const bool records = plan.passes.empty();
    const uint32_t cap = records ? cap0 : cap1;
    for (size_t q = live.size(); q-- > 0;) {
      const uint32_t k = live[q];
      count[k] = 0;
      for (int32_t slot = (int32_t)(2 * k); slot < (int32_t)(2 * k + 2); ++slot)
        count[k] += item[(size_t)slot] ? 1u : count[(size_t)child(slot)];
    }
    live.clear();
    next.clear();
    RefitPass pass;
    pass.first_block = (uint32_t)plan.block_items.size();
    uint32_t in_block = cap;  // full: the first item opens a block
    auto room = [&](uint32_t items) {
      if (in_block + items > cap) {
        plan.block_items.push_back((uint32_t)plan.item_up.size());
        plan.block_nodes.push_back((uint32_t)plan.node_id.size());
        ++pass.n_blocks;
        in_block = 0;
      }
      in_block += items;
    };
    auto add_node = [&](uint32_t k, int32_t up) {
      local[k] = (int32_t)((uint32_t)plan.node_id.size() - plan.block_nodes.back());
      plan.node_id.push_back(k);
      plan.node_up.push_back(up);
    };
    auto link = [&](int32_t slot) { return local[(size_t)(slot >> 1)] << 1 | (slot & 1); };  // within the block
    above.assign(1, -1);  // walked from the root (-1), left before right
    while (!above.empty()) {
      const int32_t slot = above.back();
      above.pop_back();
      const int32_t ref = slot < 0 ? 0 : child(slot);
      if (slot >= 0 && (records ? ref < 0 : item[(size_t)slot] != 0)) {  // an item above every treelet
        if (records) {  // its box still has to reach its slot
          room(1);
          plan.item_up.push_back(-1);
        }
        next.push_back(slot);
        continue;
      }
      const uint32_t node = (uint32_t)ref, size = count[node];
      if (size > cap) {
        live.push_back(node);
        above.push_back((int32_t)(node << 1 | 1u));
        above.push_back((int32_t)(node << 1));
        continue;
      }
      room(size);
      add_node(node, -1);
      if (records) {  // depth first: the subtree's nodes and records are two runs
        for (uint32_t k = node + 1; k + 1 < node + size; ++k) add_node(k, link(node_parent[k]));
        for (uint32_t q = 0; q < size; ++q) plan.item_up.push_back(link(leaf_parent[plan.item_up.size()]));
      } else {
        stack.assign({(int32_t)(node << 1 | 1u), (int32_t)(node << 1)});
        while (!stack.empty()) {
          const int32_t s = stack.back();
          stack.pop_back();
          if (item[(size_t)s]) {
            plan.item_up.push_back(link(s));
            plan.item_slot.push_back(s);
            continue;
          }
          const uint32_t k = (uint32_t)child(s);
          add_node(k, link(s));
          stack.push_back((int32_t)(k << 1 | 1u));
          stack.push_back((int32_t)(k << 1));
        }
      }
      if (slot < 0)
        done = true;
      else
        next.push_back(slot);
    }
    // an end value behind the pass's blocks
    plan.block_items.push_back((uint32_t)plan.item_up.size());
    plan.block_nodes.push_back((uint32_t)plan.node_id.size());
    plan.passes.push_back(pass);
    for (const int32_t s : next) item[(size_t)s] = 1;  // what lies below them is not looked at again
  }
  return plan;
}

RefitWords refit_words(const RefitPlan& plan, const std::vector<int32_t>& leaf_parent,
                       const std::vector<int32_t>& node_parent) {
  RefitWords r;
  r.one_block = plan.passes.size() <= 1 && (plan.passes.empty() || plan.passes[0].n_blocks == 1);
  const size_t table = r.one_block ? 0 : plan.block_items.size();
  r.words.reserve(2 * table + plan.item_up.size() + plan.item_slot.size() + 2 * plan.node_id.size());
  auto put = [&](const auto& v, size_t count) {
    const size_t at = r.words.size();
    r.words.insert(r.words.end(), v.begin(), v.begin() + (std::ptrdiff_t)count);
    return at;
  };
  r.block_items = put(plan.block_items, table);
  r.block_nodes = put(plan.block_nodes, table);
  r.node_id = put(plan.node_id, plan.node_id.size());
  r.node_up = put(plan.node_up, plan.node_up.size());
  r.item_up = put(plan.item_up, plan.item_up.size());
  r.item_slot = put(plan.item_slot, plan.item_slot.size());
  for (size_t k = 0; k < plan.node_up.size(); ++k)
    if (plan.node_up[k] < 0) {
      const int32_t slot = node_parent[plan.node_id[k]];
      r.words[r.node_up + k] = (uint32_t)(slot < 0 ? kRefitTop : ~slot);
    }
  for (size_t k = 0; k < plan.item_up.size(); ++k)
    if (plan.item_up[k] < 0) r.words[r.item_up + k] = (uint32_t)~leaf_parent[k];  // a record above every treelet
  return r;
}

}  // namespace ccs
