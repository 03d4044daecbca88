// Kernels of the learned child ordering that share the intersection kernel's
// arithmetic: trace recording (policy inputs at the nodes on the path to each
// ray's reported leaf), stand-alone inference, and packing of the network into
// matrix-core operand fragments.  Compiled with the intersection kernel's
// floating-point flags so that inputs are formed exactly as during traversal.

#include <algorithm>

#include "ccs_internal.h"
#include "patch_math.h"
#include "policy.h"

namespace ccs {

// Per (ray, level k): the node of depth 2k holding the ray's reported leaf.  Its
// grid is recomputed for its domain (crop, or Alg. 2 on a Gregory patch), split
// along u, and both halves are slab-tested (without a cap); when both are met
// the node is a decision of the policy and the record gets
// its inputs and, as label, the grandchild holding the leaf.  Otherwise (and
// for rays that missed) the label is 255 and the inputs are zero.
//
// Bound by vector issue: about 1000 instructions per node, 64 B written.  Where the nodes
// fill the chip, a block takes 64 rays: a lane per ray maps it into its patch's frame
// once (87 instructions, 49 of them FP64), then the nodes of the rays that hit are dealt to
// the block's lanes, so that none stands idle for a ray that missed, and the rows of those
// are cleared.
// 65,537 rays at depth 12, 59 % of them hits: 31 -> 25 us; 300,000 rays on 50 objects
// 96 -> 80 us.  Blocks of 32 rays (28 us) or of 512 threads, Gregory patches behind the
// Bezier ones, and clearing the rows without a decision (93 % of the hits' rows)
// coalesced, gain nothing further.

// A ray as its reported patch's nodes see it: origin, tmin and reciprocal direction in the
// frame that the patch is subdivided in, the direction as the network sees it, and the
// patch's record with its Gregory bit.
struct RecordRay {
  float o[3], tmin, i[3], d[3];
  uint32_t rec;
};

__device__ __forceinline__ RecordRay record_ray(const DeviceScene& s, uint32_t slot, const float4& ro,
                                                const float4& rd) {
  RecordRay q;
  const float4 meta = reinterpret_cast<const float4*>(s.recs + (size_t)slot * kRecFloats)[15];
  q.rec = slot | (__float_as_uint(meta.w) & kGregoryBit);
  float pt0;  // unused: no cap here
  float dxp = rd.x, dyp = rd.y, dzp = rd.z;  // direction in the frame the patch is subdivided in
  if (!s.frames) patch_frame(meta, ro.x, ro.y, ro.z, rd.x, rd.y, rd.z, ro.w, q.o[0], q.o[1], q.o[2], q.tmin, pt0);
  if (s.frames) {
    const float4* fr = s.frames + 3 * (size_t)slot;
    const float4 r0 = fr[0], r1 = fr[1], r2 = fr[2];
    patch_frame_rows(meta, r0, r1, r2, ro.x, ro.y, ro.z, rd.x, rd.y, rd.z, ro.w, q.o[0], q.o[1], q.o[2], dxp, dyp,
                     dzp, q.tmin, pt0);
#pragma unroll
    for (int a = 0; a < 3; ++a) q.o[a] += r0.w;  // the box pad, as in the intersection kernel
  }
  // reciprocals rounded back to a direction, exactly as the intersection kernel sees it
  q.i[0] = safe_inv(dxp);
  q.i[1] = safe_inv(dyp);
  q.i[2] = safe_inv(dzp);
  q.d[0] = s.frames ? __builtin_amdgcn_rcpf(q.i[0]) : rd.x;
  q.d[1] = s.frames ? __builtin_amdgcn_rcpf(q.i[1]) : rd.y;
  q.d[2] = s.frames ? __builtin_amdgcn_rcpf(q.i[2]) : rd.z;
  return q;
}

// Level k of the ray q, whose reported leaf is at (u, v): the network's inputs (zero where
// there is no decision) and the label.
__device__ __forceinline__ uint32_t record_node(const DeviceScene& s, const RecordRay& q, float u, float v, uint32_t k,
                                                uint32_t L, float f[16]) {
  const uint32_t slot = q.rec & kIdMask;
  const bool greg = (q.rec & kGregoryBit) != 0;
  // the reported (u, v) is a leaf centre (2i + 1) 2^-(L+1): scaling by 2^L is exact
  const float scale = __uint_as_float((127u + L) << 23);
  const uint32_t iu = (uint32_t)(u * scale), iv = (uint32_t)(v * scale);
  const float size = __uint_as_float((127u - k) << 23);
  const float u0 = (float)(iu >> (L - k)) * size, v0 = (float)(iv >> (L - k)) * size;
  PatchPts P;
  load_grid(s.recs + (size_t)slot * kRecFloats, P, greg);
  float qx[4][4], qy[4][4], qz[4][4], dx, dy, dz;
  calc_points_and_d(P, greg, u0, u0 + size, v0, v0 + size, qx, qy, qz, dx, dy, dz);
  if (s.frames) {
    const float pad2 = 2.0f * s.frames[3 * (size_t)slot].w;
    dx += pad2;
    dy += pad2;
    dz += pad2;
  }
  Grid G;
  orient(qx, false, G.x);
  orient(qy, false, G.y);
  orient(qz, false, G.z);
  Row7 e[4];
  SlabPair sp = {q.tmin, __builtin_inff(), q.tmin, __builtin_inff()};
  split_fold(G.x, q.o[0], q.i[0], dx, e, sp);
  split_fold(G.y, q.o[1], q.i[1], dy, e, sp);
  split_fold(G.z, q.o[2], q.i[2], dz, e, sp);
  // no cap: the reported hit lies on the boxes' boundary as often as not, and a
  // capped test there would turn on rounding
  const bool ha = sp.na <= widen_far(sp.fa), hb = sp.nb <= widen_far(sp.fb);
#pragma unroll
  for (int i = 0; i < 16; ++i) f[i] = 0.0f;
  if (!(ha && hb)) return 255u;
  const float sx[4] = {qx[0][0], qx[3][0], qx[0][3], qx[3][3]};
  const float sy[4] = {qy[0][0], qy[3][0], qy[0][3], qy[3][3]};
  const float sz[4] = {qz[0][0], qz[3][0], qz[0][3], qz[3][3]};
  policy_features(policy_raw(sx, sy, sz, 0u, sp), q.o[0], q.o[1], q.o[2], q.d[0], q.d[1], q.d[2], (int)(2 * k), (int)L,
                  greg, f);
  return 2u * ((iu >> (L - 1 - k)) & 1u) + ((iv >> (L - 1 - k)) & 1u);
}

__device__ __forceinline__ void record_row(float* feats, uint8_t* labels, uint64_t idx, const float f[16],
                                           uint32_t label) {
  float4* o = reinterpret_cast<float4*>(feats + idx * 16);
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = make_float4(f[4 * i], f[4 * i + 1], f[4 * i + 2], f[4 * i + 3]);
  labels[idx] = (uint8_t)label;
}

// Few nodes: a lane for each, from the hit to the row, with no exchange between lanes.
// What it waits for is one chain of loads; the barrier of the other form adds to that.
__global__ __launch_bounds__(64) void k_record_nodes(DeviceScene s, const ccs_ray* __restrict__ rays,
                                                     const ccs_hit* __restrict__ hits, uint32_t n,
                                                     float* __restrict__ feats, uint8_t* __restrict__ labels) {
  const uint32_t L = (uint32_t)s.leaf_depth;
  const uint64_t idx = (uint64_t)blockIdx.x * 64 + threadIdx.x;
  if (idx >= (uint64_t)n * L) return;
  const uint32_t r = (uint32_t)(idx / L), k = (uint32_t)(idx % L);
  const float4 h = reinterpret_cast<const float4*>(hits)[r];
  const uint32_t id = __float_as_uint(h.y);
  float f[16];
  uint32_t label = 255u;
  if (id < s.n_patches) {
    const float4* r4 = reinterpret_cast<const float4*>(rays + r);
    const float4 ro = r4[0], rd = r4[1];
    const uint32_t slot = s.inv_perm[id];
    label = record_node(s, record_ray(s, slot, ro, rd), h.z, h.w, k, L, f);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = 0.0f;
  }
  record_row(feats, labels, idx, f, label);
}

constexpr int kRecordBlock = 256, kRecordRays = 64;  // a lane of the first wave per ray
__global__ __launch_bounds__(kRecordBlock) void k_record(DeviceScene s, const ccs_ray* __restrict__ rays,
                                                         const ccs_hit* __restrict__ hits, uint32_t n,
                                                         float* __restrict__ feats, uint8_t* __restrict__ labels) {
  // of the k-th ray that hit: its RecordRay, its leaf and its place in the block
  __shared__ float s_o[3][kRecordRays], s_tmin[kRecordRays], s_i[3][kRecordRays], s_d[3][kRecordRays], s_uv[2][kRecordRays];
  __shared__ uint32_t s_rec[kRecordRays], s_hit[kRecordRays], s_miss[kRecordRays], s_hits;
  const uint32_t L = (uint32_t)s.leaf_depth;
  const uint32_t ray0 = blockIdx.x * kRecordRays, here = min((uint32_t)kRecordRays, n - ray0);
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x, r = ray0 + lane;
    float4 h = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    uint32_t id = ~0u;
    if (lane < here) {
      h = reinterpret_cast<const float4*>(hits)[r];
      id = __float_as_uint(h.y);
    }
    const bool hit = lane < here && id < s.n_patches;
    const uint64_t m = __ballot(hit);
    const uint32_t at = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) s_hits = (uint32_t)__popcll(m);
    if (hit) {
      const float4* r4 = reinterpret_cast<const float4*>(rays + r);
      const float4 ro = r4[0], rd = r4[1];
      const uint32_t slot = s.inv_perm[id];
      const RecordRay q = record_ray(s, slot, ro, rd);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s_o[a][at] = q.o[a];
        s_i[a][at] = q.i[a];
        s_d[a][at] = q.d[a];
      }
      s_tmin[at] = q.tmin;
      s_uv[0][at] = h.z;
      s_uv[1][at] = h.w;
      s_rec[at] = q.rec;
      s_hit[at] = lane;
    } else if (lane < here) {
      s_miss[lane - at] = lane;
    }
  }
  __syncthreads();
  const uint32_t n_hits = s_hits;
  for (uint32_t t = threadIdx.x; t < n_hits * L; t += kRecordBlock) {
    const uint32_t at = t / L, k = t - at * L;
    RecordRay q;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      q.o[a] = s_o[a][at];
      q.i[a] = s_i[a][at];
      q.d[a] = s_d[a][at];
    }
    q.tmin = s_tmin[at];
    q.rec = s_rec[at];
    float f[16];
    const uint32_t label = record_node(s, q, s_uv[0][at], s_uv[1][at], k, L, f);
    record_row(feats, labels, (uint64_t)(ray0 + s_hit[at]) * L + k, f, label);
  }
  for (uint32_t t = threadIdx.x; t < (here - n_hits) * 4 * L; t += kRecordBlock) {
    const uint32_t q = t / (4 * L), w = t - q * 4 * L;
    const uint64_t idx = (uint64_t)(ray0 + s_miss[q]) * L;
    reinterpret_cast<float4*>(feats)[idx * 4 + w] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if ((w & 3u) == 0) labels[idx + w / 4] = 255;
  }
}

// Lane `lane`'s four values of weight tile 0..7 (tile < kPolicyWTiles) or bias tile
// 0..4 of the network's operand fragments (layout in policy.h).
__device__ __forceinline__ void fragment(const float* __restrict__ th, int tile, int lane, float v[4]) {
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = 4 * g + i;
    if (tile < 2)
      v[i] = th[kPolicyW1 + (16 * tile + r) * 16 + k];
    else if (tile < 6)
      v[i] = th[kPolicyW2 + (16 * ((tile - 2) >> 1) + r) * 32 + 16 * ((tile - 2) & 1) + k];
    else if (tile < kPolicyWTiles)
      v[i] = r < 4 ? th[kPolicyW3 + r * 32 + 16 * (tile - 6) + k] : 0.0f;
    else if (tile < kPolicyWTiles + 2)
      v[i] = th[kPolicyB1 + 16 * (tile - kPolicyWTiles) + k];
    else if (tile < kPolicyWTiles + 4)
      v[i] = th[kPolicyB2 + 16 * (tile - kPolicyWTiles - 2) + k];
    else
      v[i] = k < 4 ? th[kPolicyB3 + k] : 0.0f;
  }
}

// Network inference for n input rows, with the intersection kernel's arithmetic
// (policy_tile).  Bound by memory: 64 B read and 16 B written per row.  A wave reads
// the operand fragments once, from the parameters themselves (no packed copy, whose
// launch and temporaries cost as much as the inference of 100,000 rows), keeps them
// in registers and runs over tiles of 16 rows; a lane's 16-byte load of a tile is its
// matrix operand, a wave's load 1 KB in a row, four tiles in flight.  786,444 rows:
// 27 us and 9 us of packing -> 19.4 us.
constexpr int kInferWaves = 4, kInferTiles = 4;
__global__ __launch_bounds__(64 * kInferWaves) void k_policy_infer(const float* __restrict__ th,
                                                                   const float* __restrict__ x, uint32_t n,
                                                                   float* __restrict__ z) {
  const int lane = threadIdx.x & 63;
  uint2 w[kPolicyWTiles];
  float4 b[kPolicyBTiles];
#pragma unroll
  for (int t = 0; t < kPolicyWTiles; ++t) {
    float v[4];
    fragment(th, t, lane, v);
    w[t] = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
  }
#pragma unroll
  for (int t = 0; t < kPolicyBTiles; ++t) {
    float v[4];
    fragment(th, kPolicyWTiles + t, lane, v);
    b[t] = make_float4(v[0], v[1], v[2], v[3]);
  }
  const uint64_t step = (uint64_t)gridDim.x * kInferWaves * (16 * kInferTiles);
  for (uint64_t row0 = ((uint64_t)blockIdx.x * kInferWaves + (threadIdx.x >> 6)) * (16 * kInferTiles); row0 < n;
       row0 += step) {
    float4 f[kInferTiles];
#pragma unroll
    for (int t = 0; t < kInferTiles; ++t) {
      const uint64_t row = row0 + 16 * t + (lane & 15);
      f[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (row < n) f[t] = reinterpret_cast<const float4*>(x)[4 * row + (lane >> 4)];
    }
#pragma unroll
    for (int t = 0; t < kInferTiles; ++t) {
      const uint2 xv = make_uint2(bf16_pair(f[t].x, f[t].y), bf16_pair(f[t].z, f[t].w));
      const f32x4 lg = policy_tile([&](int k) { return w[k]; }, [&](int k) { return b[k]; }, as_bf16x4(xv));
      const uint64_t row = row0 + 16 * t + lane;
      if (lane < 16 && row < n) reinterpret_cast<float4*>(z)[row] = make_float4(lg[0], lg[1], lg[2], lg[3]);
    }
  }
}

// Operand fragments from the fp32 parameters (layout in policy.h).  Thread
// (tile, lane); weights rounded to bfloat16, biases kept in fp32.
__global__ __launch_bounds__(64) void k_policy_pack(const float* __restrict__ th, uint2* __restrict__ w,
                                                    float4* __restrict__ b) {
  const int tile = blockIdx.x, lane = threadIdx.x;
  float v[4];
  fragment(th, tile, lane, v);
  if (tile < kPolicyWTiles)
    w[tile * 64 + lane] = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
  else
    b[(tile - kPolicyWTiles) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
}

hipError_t launch_policy_pack(const float* params, uint2* w, float4* b, hipStream_t stream) {
  hipLaunchKernelGGL(k_policy_pack, dim3(kPolicyWTiles + kPolicyBTiles), dim3(64), 0, stream, params, w, b);
  return hipGetLastError();
}

hipError_t launch_policy_infer(const float* params, const float* x, uint32_t n, float* z, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  constexpr uint64_t kRows = 16 * kInferTiles * kInferWaves;
  constexpr uint64_t kBlocks = 1024;  // at most 16 waves per CU of 256, each reading the fragments once
  const uint32_t grid = (uint32_t)std::min<uint64_t>(kBlocks, (n + kRows - 1) / kRows);
  hipLaunchKernelGGL(k_policy_infer, dim3(grid), dim3(64 * kInferWaves), 0, stream, params, x, n, z);
  return hipGetLastError();
}

hipError_t launch_record(const DeviceScene& s, const ccs_ray* rays, const ccs_hit* hits, uint32_t n, float* feats,
                         uint8_t* labels, hipStream_t stream) {
  if (n == 0 || s.leaf_depth == 0) return hipSuccess;
  // Blocks of 64 rays from 160 rays per CU on (40,960): with fewer, some CUs get one block
  // more than others.  Above 16 levels a block goes round its lanes five times, and it takes
  // 240; below four levels its nodes do not fill them.  A lane per node against blocks, us:
  // 8,300 rays at depth 12 7.4, 11.3 and 41,700 19.8, 18.4; 10,000 on 50 objects 7.6, 11.2,
  // 40,000 17.9, 17.8 and 120,000 39.2, 34.9; depth 20 30,000 rays 22.4, 25.4, 60,000 37.1,
  // 35.3; depth 1 100,000 rays 7.5, 10.4, 2,000,000 71.5, 107.6; depth 4 50,000 11.5, 10.5.
  // (Blocks of 16 rays in between gained 5 % on one torus and lost 5 % on 50 objects.)
  const uint32_t L = (uint32_t)s.leaf_depth;
  if (L < 4 || n <= (L <= 16 ? 160u : 240u) * s.n_cus) {
    hipLaunchKernelGGL(k_record_nodes, dim3((uint32_t)(((uint64_t)n * L + 63) / 64)), dim3(64), 0, stream, s, rays,
                       hits, n, feats, labels);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_record, dim3((n + kRecordRays - 1) / kRecordRays), dim3(kRecordBlock), 0, stream, s, rays, hits,
                     n, feats, labels);
  return hipGetLastError();
}

}  // namespace ccs
