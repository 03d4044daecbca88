#include "refit_plan.h"

#include <cstring>
#include <utility>

namespace ccs {

RefitPlan plan_refit(const std::vector<float>& nodes, const std::vector<int32_t>& leaf_parent,
                     const std::vector<int32_t>& node_parent, uint32_t cap0, uint32_t cap1) {
  RefitPlan plan;
  const uint32_t n_nodes = (uint32_t)node_parent.size(), n = (uint32_t)leaf_parent.size();
  if (n == 0) return plan;
  auto child = [&](uint32_t node, int side) {
    int32_t c;
    std::memcpy(&c, nodes.data() + 16 * (size_t)node + 12 + side, 4);
    return c;
  };
  // item[slot]: the slot's box is an item of the current pass; count[node]: items below it
  std::vector<uint8_t> item(2 * (size_t)n_nodes, 0);
  std::vector<uint32_t> count(n_nodes, 0);
  std::vector<int32_t> local(n_nodes, -1);  // a node's index in its block
  for (uint32_t r = 0; r < n; ++r) item[(size_t)leaf_parent[r]] = 1;
  if (n == 1) item[1] = 0;  // a lone record fills both slots of the root: one item
  std::vector<std::pair<int32_t, int32_t>> stack;  // (slot, its parent's index in the block or -1)
  std::vector<uint32_t> live(n_nodes);  // nodes no treelet holds yet, parents first
  for (uint32_t k = 0; k < n_nodes; ++k) live[k] = k;
  for (bool done = false; !done;) {
    const bool records = plan.passes.empty();
    const uint32_t cap = records ? cap0 : cap1;
    for (size_t q = live.size(); q-- > 0;) {
      const uint32_t k = live[q];
      uint32_t c = 0;
      for (int side = 0; side < 2; ++side) {
        const size_t slot = 2 * (size_t)k + (size_t)side;
        const int32_t ch = child(k, side);
        c += item[slot] ? 1u : ch >= 0 ? count[(size_t)ch] : 0u;
      }
      count[k] = c;
    }
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
    auto add_item = [&](int32_t slot, int32_t up) {
      plan.item_up.push_back(up);
      plan.item_slot.push_back(slot);
    };
    std::vector<int32_t> next;    // slots that are items of the next pass
    live.clear();
    // walk from the root, left before right; -1 stands for the root itself
    std::vector<int32_t> above = {-1};
    while (!above.empty()) {
      const int32_t slot = above.back();
      above.pop_back();
      if (slot >= 0 && item[(size_t)slot]) {  // an item above every treelet
        if (records) {  // its box still has to reach its slot
          room(1);
          add_item(slot, -1);
        }
        next.push_back(slot);
        continue;
      }
      const uint32_t node = slot < 0 ? 0u : (uint32_t)child((uint32_t)slot >> 1, slot & 1);
      if (count[node] > cap) {
        live.push_back(node);
        above.push_back((int32_t)(node << 1 | 1u));
        above.push_back((int32_t)(node << 1));
        continue;
      }
      room(count[node]);
      const uint32_t base = plan.block_nodes.back();
      auto add_node = [&](uint32_t k, int32_t up) {
        local[k] = (int32_t)((uint32_t)plan.node_id.size() - base);
        plan.node_id.push_back(k);
        plan.node_up.push_back(up);
        stack.emplace_back((int32_t)(k << 1 | 1u), local[k]);
        stack.emplace_back((int32_t)(k << 1), local[k]);
      };
      add_node(node, -1);
      while (!stack.empty()) {
        const auto [s, parent] = stack.back();
        stack.pop_back();
        const int32_t link = parent << 1 | (s & 1);
        if (item[(size_t)s])
          add_item(s, link);
        else if (child((uint32_t)s >> 1, s & 1) >= 0)
          add_node((uint32_t)child((uint32_t)s >> 1, s & 1), link);
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

}  // namespace ccs
