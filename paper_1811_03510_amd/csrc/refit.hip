// Refit of an existing scene to moved control points (animation playback).
// Topology is kept; anchors stay at their create-time values.
//
//   k_refit_patches  four lanes per patch record: lane j reads the four grid points
//                    4j .. 4j + 3 (three 16-byte loads) and the P^v point 16 + j,
//                    writes their coordinates to the anchored record as three
//                    16-byte and three 4-byte stores, and the patch's hull box, the
//                    quad's union, starts the workgroup's climb over its treelets;
//   k_refit_boxes    the same climb from the boxes that the launch before it left in
//                    its items' slots, up to the root (refit_plan.h).
// A climb needs no other workgroup: the second child to reach a node (a counter in
// LDS) unions the boxes and goes on.  Launch boundaries order the passes, so no
// thread waits on another and no device-wide fence is needed (each XCD's L2 is
// written back at kernel end).  A launch per BVH level instead spent 2 to 5 us on
// each level: refits of 512, 200,000 and 1,000,000 patches take 9.8, 45 and 202 us
// against 27.5 (11 launches), 91 (26) and 287 us.  What bounds them now is a chain
// of latencies per workgroup (its item range, the records' last words, points, stores, climb): without
// the stores 200,000 patches take 41 us, without the climb 41, with the points in
// record order 45; with the frame in each of a patch's lanes, 48.
// With patch-local frames the per-patch pass also recomputes each patch's frame and
// stores the record in it.  Compiled without
// floating-point contraction, so every refit of the same points gives the same bits.

#include "ccs_internal.h"
#include "patch_math.h"

namespace ccs {

constexpr int kRefitBlock = 4 * kRefitCap0;

__device__ __forceinline__ void write_child_box(float4* nodes, int node, int side, const float lo[3],
                                                const float hi[3]) {
  float* f = reinterpret_cast<float*>(nodes + 4 * (size_t)node);
  const int base = side ? 6 : 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f[base + k] = lo[k];
    f[base + 3 + k] = hi[k];
  }
}

// Nodes of a workgroup's treelets while it climbs.
template <int kNodes>
struct Treelets {
  float box[kNodes][12];  // both children's lo and hi, laid out as in a node
  uint32_t arrived[kNodes];
  uint32_t id[kNodes];
  int32_t up[kNodes];

  // The block's nodes, by all its threads; a barrier must follow.
  __device__ __forceinline__ void load(const RefitDev& p, uint32_t begin, uint32_t count) {
    for (uint32_t k = threadIdx.x; k < count; k += blockDim.x) {
      arrived[k] = 0;
      id[k] = p.node_id[begin + k];
      up[k] = p.node_up[begin + k];
    }
  }

  // From an item whose box is (lo, hi) and whose parent in the block is `link`.
  __device__ __forceinline__ void climb(float4* nodes, int32_t link, float lo[3], float hi[3]) {
    while (true) {
      const uint32_t k = (uint32_t)link >> 1;
      float* own = box[k] + ((link & 1) ? 6 : 0);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        own[a] = lo[a];
        own[3 + a] = hi[a];
      }
      __threadfence_block();  // the box before the count
      if (atomicAdd(&arrived[k], 1u) == 0u) return;
      __threadfence_block();
      const float4* b = reinterpret_cast<const float4*>(box[k]);
      const float4 x = b[0], y = b[1], z = b[2];
      float4* nd = nodes + 4 * (size_t)id[k];
      nd[0] = x;
      nd[1] = y;
      nd[2] = z;
      lo[0] = fminf(x.x, y.z);
      lo[1] = fminf(x.y, y.w);
      lo[2] = fminf(x.z, z.x);
      hi[0] = fmaxf(x.w, z.y);
      hi[1] = fmaxf(y.x, z.z);
      hi[2] = fmaxf(y.y, z.w);
      link = up[k];
      if (link < 0) {  // a treelet's root: its box goes to its slot, for the next pass
        if (link != kRefitTop) write_child_box(nodes, ~link >> 1, ~link & 1, lo, hi);
        return;
      }
    }
  }
};

template <int kCtrl>
__device__ __forceinline__ float quad(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kCtrl, 0xF, 0xF, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;
__device__ __forceinline__ float quad_lo(float x) {
  x = fminf(x, quad<kXor1>(x));
  return fminf(x, quad<kXor2>(x));
}
__device__ __forceinline__ float quad_hi(float x) {
  x = fmaxf(x, quad<kXor1>(x));
  return fmaxf(x, quad<kXor2>(x));
}

// Rows of a patch's frame, in double: r0 = unit(p30 - p00), r1 = unit of (p03 - p00)
// without its r0 part, r2 = r0 x r1; the identity for a degenerate u or v edge.
// Rows are stored in fp32 and the anchored points are mapped by the stored rows
// (in double, rounded once), so that rays mapped by the same rows see exactly
// the mapped patch.
__device__ __forceinline__ void patch_rows(const float p00[3], const float p30[3], const float p03[3], float rf[9]) {
  double eu[3], ev[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    eu[a] = (double)p30[a] - (double)p00[a];
    ev[a] = (double)p03[a] - (double)p00[a];
  }
  const double lu = sqrt(eu[0] * eu[0] + eu[1] * eu[1] + eu[2] * eu[2]);
  const double lv = sqrt(ev[0] * ev[0] + ev[1] * ev[1] + ev[2] * ev[2]);
  double m[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
  if (lu > 0.0 && lv > 0.0) {
    const double iu = 1.0 / lu;
    const double r0[3] = {iu * eu[0], iu * eu[1], iu * eu[2]};
    const double dv = ev[0] * r0[0] + ev[1] * r0[1] + ev[2] * r0[2];
    const double w[3] = {ev[0] - dv * r0[0], ev[1] - dv * r0[1], ev[2] - dv * r0[2]};
    const double lw = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
    if (lw > 1e-9 * lv) {
      const double iw = 1.0 / lw;
      const double r1[3] = {iw * w[0], iw * w[1], iw * w[2]};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        m[a] = r0[a];
        m[3 + a] = r1[a];
      }
      m[6] = r0[1] * r1[2] - r0[2] * r1[1];
      m[7] = r0[2] * r1[0] - r0[0] * r1[2];
      m[8] = r0[0] * r1[1] - r0[1] * r1[0];
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) rf[k] = (float)m[k];
}

__global__ __launch_bounds__(kRefitBlock) void k_refit_patches(DeviceScene s, const float* __restrict__ cp) {
  __shared__ __align__(16) Treelets<kRefitCap0> tree;
  __shared__ float rows[kRefitCap0][9];
  uint32_t first = 0, end = s.n_patches, nodes0 = 0, nodes1 = s.n_nodes;
  if (s.refit.block_items) {
    first = s.refit.block_items[blockIdx.x];
    end = s.refit.block_items[blockIdx.x + 1];
    nodes0 = s.refit.block_nodes[blockIdx.x];
    nodes1 = s.refit.block_nodes[blockIdx.x + 1];
  }
  tree.load(s.refit, nodes0, nodes1 - nodes0);
  // the frames' rows, a lane per patch of the first wave (their roots and divisions
  // in each of a patch's four lanes would double the kernel's instructions)
  if (s.frames && threadIdx.x < kRefitCap0 && first + threadIdx.x < end) {
    const uint32_t meta = __float_as_uint(s.recs[(size_t)(first + threadIdx.x) * kRecFloats + 63]);
    const float* src = cp + (size_t)(meta & kIdMask) * 60;
    patch_rows(src, src + 9, src + 36, rows[threadIdx.x]);
  }
  __syncthreads();
  const uint32_t r = first + threadIdx.x / 4;
  const int j = threadIdx.x & 3;
  if (r >= end) return;
  float* rec = s.recs + (size_t)r * kRecFloats;
  const float4 meta = reinterpret_cast<const float4*>(rec)[15];  // anchor xyz, meta bits: unchanged
  const bool greg = (__float_as_uint(meta.w) & kGregoryBit) != 0;
  const float* src = cp + (size_t)(__float_as_uint(meta.w) & kIdMask) * 60;  // 240 B, 16-B aligned
  float p[5][3];                                   // grid points 4j .. 4j + 3, then P^v point 16 + j
  {
    const float4* g = reinterpret_cast<const float4*>(src) + 3 * j;
    const float4 a = g[0], b = g[1], c = g[2];
    p[0][0] = a.x; p[0][1] = a.y; p[0][2] = a.z;
    p[1][0] = a.w; p[1][1] = b.x; p[1][2] = b.y;
    p[2][0] = b.z; p[2][1] = b.w; p[2][2] = c.x;
    p[3][0] = c.y; p[3][1] = c.z; p[3][2] = c.w;
#pragma unroll
    for (int a2 = 0; a2 < 3; ++a2) p[4][a2] = src[48 + 3 * j + a2];
  }
  float lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = fminf(fminf(p[0][a], p[1][a]), fminf(p[2][a], p[3][a]));
    hi[a] = fmaxf(fmaxf(p[0][a], p[1][a]), fmaxf(p[2][a], p[3][a]));
    lo[a] = quad_lo(greg ? fminf(lo[a], p[4][a]) : lo[a]);  // a Bezier patch's hull is that of its 16 points
    hi[a] = quad_hi(greg ? fmaxf(hi[a], p[4][a]) : hi[a]);
  }
  const float anc[3] = {meta.x, meta.y, meta.z};
  float out[5][3];
  if (s.frames) {
    float rf[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) rf[a][b] = rows[threadIdx.x / 4][3 * a + b];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const double q[3] = {(double)p[k][0] - (double)anc[0], (double)p[k][1] - (double)anc[1],
                           (double)p[k][2] - (double)anc[2]};
#pragma unroll
      for (int a = 0; a < 3; ++a)
        out[k][a] = (float)((double)rf[a][0] * q[0] + (double)rf[a][1] * q[1] + (double)rf[a][2] * q[2]);
    }
    // gap-closing pad (Sec. 3.4): 2^-19 of the patch's largest extent in its frame;
    // every subdivision box of the patch is grown by it on all sides
    float ext = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float l = fminf(fminf(out[0][a], out[1][a]), fminf(out[2][a], out[3][a]));
      float h = fmaxf(fmaxf(out[0][a], out[1][a]), fmaxf(out[2][a], out[3][a]));
      l = quad_lo(greg ? fminf(l, out[4][a]) : l);
      h = quad_hi(greg ? fmaxf(h, out[4][a]) : h);
      ext = fmaxf(ext, h - l);
    }
    const float pad = ldexpf(ext, -19);
    if (j < 3) {  // lane j stores row j
      const float4 row = make_float4(j == 0 ? rf[0][0] : j == 1 ? rf[1][0] : rf[2][0],
                                     j == 0 ? rf[0][1] : j == 1 ? rf[1][1] : rf[2][1],
                                     j == 0 ? rf[0][2] : j == 1 ? rf[1][2] : rf[2][2], j == 0 ? pad : 0.0f);
      s.frames[3 * (size_t)r + j] = row;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
      for (int a = 0; a < 3; ++a) out[k][a] = p[k][a] - anc[a];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    reinterpret_cast<float4*>(rec)[4 * a + j] = make_float4(out[0][a], out[1][a], out[2][a], out[3][a]);
    rec[48 + 4 * a + j] = out[4][a];
  }
  if (j != 0) return;
  float4* nodes = const_cast<float4*>(s.nodes);
  const int32_t up = s.refit.item_up[r];
  if (s.n_patches == 1) {  // a lone patch occupies both slots of the root
    write_child_box(nodes, 0, 0, lo, hi);
    write_child_box(nodes, 0, 1, lo, hi);
  } else if (up < 0) {
    write_child_box(nodes, ~up >> 1, ~up & 1, lo, hi);
  } else {
    tree.climb(nodes, up, lo, hi);
  }
}

__global__ __launch_bounds__(kRefitCap1) void k_refit_boxes(float4* __restrict__ nodes, RefitDev plan,
                                                            uint32_t first_block, uint32_t n_records) {
  __shared__ __align__(16) Treelets<kRefitCap1> tree;
  const uint32_t block = first_block + blockIdx.x;
  const uint32_t first = plan.block_items[block], end = plan.block_items[block + 1];
  const uint32_t nodes0 = plan.block_nodes[block];
  tree.load(plan, nodes0, plan.block_nodes[block + 1] - nodes0);
  __syncthreads();
  const uint32_t k = first + threadIdx.x;
  if (k >= end) return;
  const int32_t slot = plan.item_slot[k - n_records];
  const float* f = reinterpret_cast<const float*>(nodes + 4 * (size_t)(slot >> 1)) + ((slot & 1) ? 6 : 0);
  float lo[3] = {f[0], f[1], f[2]}, hi[3] = {f[3], f[4], f[5]};
  tree.climb(nodes, plan.item_up[k], lo, hi);
}

hipError_t launch_refit(const DeviceScene& s, const float* cp_world, const std::vector<RefitPass>& passes,
                        hipStream_t stream) {
  for (size_t k = 0; k < passes.size(); ++k) {
    const dim3 grid(passes[k].n_blocks);
    if (k == 0)
      hipLaunchKernelGGL(k_refit_patches, grid, dim3(kRefitBlock), 0, stream, s, cp_world);
    else
      hipLaunchKernelGGL(k_refit_boxes, grid, dim3(kRefitCap1), 0, stream, const_cast<float4*>(s.nodes),
                         s.refit, passes[k].first_block, s.n_patches);
  }
  return hipGetLastError();
}

}  // namespace ccs
