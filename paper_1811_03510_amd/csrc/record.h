// Constants of a patch record and of patch ids, for host and device code (the record's
// layout is described in patch_math.h).
#pragma once

#include <cstdint>

namespace ccs {

constexpr int kRecFloats = 64;
constexpr uint32_t kGregoryBit = 0x80000000u;
constexpr uint32_t kIdMask = 0x7FFFFFFFu;
constexpr uint32_t kNoHit = 0xFFFFFFFFu;

}  // namespace ccs
