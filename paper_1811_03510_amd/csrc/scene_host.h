// The host side of scene creation: hierarchy, patch records and refit plan of validated
// patches.  Needs no GPU.
#pragma once

#include <cstdint>
#include <vector>

#include "bvh_build.h"
#include "refit_plan.h"

namespace ccs {

struct HostScene {
  BvhOutput bvh;
  std::vector<RefitPass> refit_passes;  // empty, as what follows, when the BVH is too deep
  RefitWords refit;
  std::vector<float> recs;              // kRecFloats per patch, in leaf order, in world frames
  std::vector<uint32_t> inv_perm;       // input patch index -> record
  float lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};  // scene bounds
};

// cp: 60 floats per patch; types: a tag per patch; stack: the depth that the BVH has to
// stay below (the caller refuses a deeper one).  Throws std::bad_alloc, with every thread
// it started ended.
HostScene make_host_scene(const std::vector<float>& cp, const std::vector<uint8_t>& types, uint32_t stack, int threads,
                          uint32_t refit_cap0, uint32_t refit_cap1);

}  // namespace ccs
