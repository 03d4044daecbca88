#include "scene_host.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>

#include "../../include/ccs.h"
#include "beside.h"
#include "record.h"

namespace ccs {

HostScene make_host_scene(const std::vector<float>& cp, const std::vector<uint8_t>& types, uint32_t stack, int threads,
                          uint32_t refit_cap0, uint32_t refit_cap1) {
  HostScene s;
  const uint32_t n = (uint32_t)types.size();
  // patch boxes (hull of 16 or 20 points); the fp32 anchors are their centres
  std::vector<BuildBox> boxes(n);
  for (uint32_t k = 0; k < n; ++k) {
    const float* p = cp.data() + 60 * (size_t)k;
    const int np = types[k] == CCS_GREGORY ? 20 : 16;
    BuildBox& b = boxes[k];
    for (int a = 0; a < 3; ++a) b.lo[a] = b.hi[a] = p[a];
    for (int q = 1; q < np; ++q)
      for (int a = 0; a < 3; ++a) {
        b.lo[a] = std::fmin(b.lo[a], p[3 * q + a]);
        b.hi[a] = std::fmax(b.hi[a], p[3 * q + a]);
      }
  }
  uint32_t log2n = 0;
  while ((1ull << log2n) < (uint64_t)std::max<uint32_t>(n, 1)) ++log2n;
  const uint32_t sah_depth = (uint32_t)std::max<int>(8, (int)stack - 1 - (int)log2n);
  s.bvh = build_bvh(boxes, sah_depth, threads);
  if (n > 0 && s.bvh.max_depth >= stack) return s;

  // records in leaf order
  auto records = [&]() {
    s.recs.assign((size_t)n * kRecFloats, 0.0f);
    s.inv_perm.resize(n);
    for (int a = 0; a < 3; ++a) {
      s.lo[a] = n ? INFINITY : 0.0f;
      s.hi[a] = n ? -INFINITY : 0.0f;
    }
    for (uint32_t r = 0; r < n; ++r) {
      const uint32_t k = s.bvh.perm[r];
      s.inv_perm[k] = r;
      const float* p = cp.data() + 60 * (size_t)k;
      float* q = s.recs.data() + (size_t)r * kRecFloats;
      const BuildBox& b = boxes[k];
      float anc[3];
      for (int a = 0; a < 3; ++a) {
        anc[a] = 0.5f * (b.lo[a] + b.hi[a]);
        s.lo[a] = std::fmin(s.lo[a], b.lo[a]);
        s.hi[a] = std::fmax(s.hi[a], b.hi[a]);
      }
      for (int sl = 0; sl < 16; ++sl)
        for (int a = 0; a < 3; ++a) q[16 * a + sl] = p[3 * sl + a] - anc[a];
      for (int sl = 16; sl < 20; ++sl)
        for (int a = 0; a < 3; ++a) q[48 + 4 * a + (sl - 16)] = p[3 * sl + a] - anc[a];
      q[60] = anc[0];
      q[61] = anc[1];
      q[62] = anc[2];
      const uint32_t meta = k | (types[k] == CCS_GREGORY ? kGregoryBit : 0u);
      std::memcpy(q + 63, &meta, 4);
    }
  };
  auto plan = [&]() {
    RefitPlan p = plan_refit(s.bvh.nodes, s.bvh.leaf_parent, s.bvh.node_parent, refit_cap0, refit_cap1);
    s.refit = refit_words(p, s.bvh.leaf_parent, s.bvh.node_parent);
    s.refit_passes = std::move(p.passes);
  };
  // of a large scene beside each other (the plan takes 26 ms for 1M patches)
  if (n >= (1u << 15)) {
    beside(plan, records);
  } else {
    plan();
    records();
  }
  return s;
}

}  // namespace ccs
