// Work plan of the BVH refit: which workgroup unions which node boxes, in a few
// passes instead of one launch per level.
//
// Pass 0 covers the patch records: every maximal subtree of at most `cap0` records
// is a treelet, consecutive treelets share a workgroup's `cap0` places (70 % of them
// filled on the object fields; taking subtrees apart to fill 90 % made the first pass
// no faster and the second one slower), and a record whose parent lies above every
// treelet only fills its slot.  The treelets'
// root slots and those records are the items of pass 1, whose treelets hold at most
// `cap1` items, and so on until one treelet holds the root.  Inside a workgroup a
// thread starts at its item and climbs: the second child to arrive at a node unions
// the two boxes and goes on, the first one stops.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace ccs {

// Slots and links are (node << 1 | side).
struct RefitPass {
  uint32_t first_block = 0, n_blocks = 0;  // in block_items / block_nodes
};

struct RefitPlan {
  std::vector<RefitPass> passes;
  // per block, and one end value after each pass's last block
  std::vector<uint32_t> block_items;  // first item: item k < n of pass 0 is record k
  std::vector<uint32_t> block_nodes;  // first entry of node_id / node_up
  std::vector<int32_t> item_up;       // item -> link to its parent among the block's nodes, -1: outside the block
  std::vector<int32_t> item_slot;     // item k >= n -> the slot that holds its box, at k - n
  std::vector<uint32_t> node_id;      // node of a block -> node of the BVH
  std::vector<int32_t> node_up;       // node of a block -> link to its parent in the block, -1: a treelet's root
};

// The plan as the device reads it, one array of words.  A link that leaves its block is
// the slot it goes to, as ~slot, so that the device needs no parents of nodes and records
// besides (with them a scene held more memory than with a list of nodes by depth):
// 12 bytes a patch, 8 a treelet and 8 a block.  A single block needs no table:
// it holds every record and every node, in order.
constexpr int32_t kRefitTop = INT32_MIN;  // in node_up: the root of the BVH
struct RefitWords {
  std::vector<uint32_t> words;
  bool one_block = true;
  size_t block_items = 0, block_nodes = 0, node_id = 0, node_up = 0, item_up = 0, item_slot = 0;  // where each begins
};

RefitWords refit_words(const RefitPlan& plan, const std::vector<int32_t>& leaf_parent,
                       const std::vector<int32_t>& node_parent);

// nodes: 16 floats per node, the children's references as bits at 12 and 13 (>= 0
// node, < 0 record ~child), in depth-first order (left child = node + 1); leaf_parent
// and node_parent as the builder gives them.
RefitPlan plan_refit(const std::vector<float>& nodes, const std::vector<int32_t>& leaf_parent,
                     const std::vector<int32_t>& node_parent, uint32_t cap0, uint32_t cap1);

}  // namespace ccs
