// One ray on sixteen lanes: the intersection kernel's traversal, subdivision step
// and grid recompute with a ray's arithmetic spread over a group of 16 lanes (a
// DPP row), four rays to a wave.
//
// Why: with one ray per lane a subdivision step is ~340 vector instructions and a
// recompute ~430, issued at one per six cycles (all that one wave issues), so a single
// ray advances a Gregory level every 1.9 us however empty the machine is, and a launch
// lasts at least as long as its heaviest ray (up to ~1700 steps and recomputes on a
// grazing ray, where the mean is 40).  Spread over 16 lanes the same step is ~140
// instructions and the recompute ~220, without a memory access (the record stays in
// registers): 0.94 us per Gregory level.  With all 64 lanes on one ray, below, it is
// 0.47 us.  Per ray this issues several times as many instructions, so it is used only
// where lanes would idle: for the last rays of a wave (a small launch runs a wave per ray
// from the start).
//
// Lane l of a group: b = l & 3, q = l >> 2, component c = min(q, 2) (q = 3 repeats
// z, so that a reduction over the four quads is one over the three components).
// Lane (c, b) holds row b of component c of the working grid, G_c[a][b] for
// a = 0..3 along the next split's axis; every other value of a ray is the same on
// all its 16 lanes.  Rows are reduced within a quad (quad_perm), components across
// quads (row rotations by 4 and 8), and the grid is transposed within each quad
// after a split.
//
// Every value is formed by the operations of the one-lane kernel in its order
// (minima and maxima are exact in any order), so a ray's result has the same bits
// on either path, and a ray can move from one to the other between two steps.
#pragma once

#include "ccs_internal.h"
#include "patch_math.h"
#include "policy.h"
#include "ray_valid.h"

namespace ccs {

constexpr int kGroupLanes = 16;
constexpr int kGroupsPerWave = 64 / kGroupLanes;
// Node visits of a traversing group between two passes over the other groups' steps.
constexpr int kGroupNodeSteps = 4;

template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kCtrl, 0xF, 0xF, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kQuadLane1 = 0x55, kQuadLane2 = 0xAA;
constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128;

__device__ __forceinline__ float quad_min(float x) {
  x = fminf(x, dpp<kQuadXor1>(x));
  return fminf(x, dpp<kQuadXor2>(x));
}
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, dpp<kQuadXor1>(x));
  return fmaxf(x, dpp<kQuadXor2>(x));
}
__device__ __forceinline__ float across_min(float x) {
  x = fminf(x, dpp<kRowRor4>(x));
  return fminf(x, dpp<kRowRor8>(x));
}
__device__ __forceinline__ float across_max(float x) {
  x = fmaxf(x, dpp<kRowRor4>(x));
  return fmaxf(x, dpp<kRowRor8>(x));
}

// 4x4 transpose over a quad: lane b's h[k] becomes lane k's h[b].
__device__ __forceinline__ void quad_transpose(float h[4], bool b0, bool b1) {
  const float s0 = dpp<kQuadXor1>(b0 ? h[0] : h[1]), s1 = dpp<kQuadXor1>(b0 ? h[2] : h[3]);
  const float t0 = b0 ? s0 : h[0], t1 = b0 ? h[1] : s0, t2 = b0 ? s1 : h[2], t3 = b0 ? h[3] : s1;
  const float r0 = dpp<kQuadXor2>(b1 ? t0 : t2), r1 = dpp<kQuadXor2>(b1 ? t1 : t3);
  h[0] = b1 ? r0 : t0;
  h[1] = b1 ? r1 : t1;
  h[2] = b1 ? t2 : r0;
  h[3] = b1 ? t3 : r1;
}

// What a group does next (a group that waits for a ray is kGroupFree).
enum GroupMode : int {
  kGroupFree = 0, kGroupWalk = 1, kGroupStep = 2, kGroupGrid = 3, kGroupDead = 4,
  kGroupDecide = 5  // learned order: waits for the network
};

template <typename CodeT>
struct GroupRay {
  int mode;
  uint32_t rid;
  const float4* nodes;   // the ray's frame
  const float* recs;
  const float4* frames;  // nullptr: world frame
  float ox, oy, oz, dx, dy, dz, tmin;  // world ray
  float wo, wi;                        // its origin and reciprocal direction, component c
  float best_t, hu, hv;
  uint32_t best_id;
  int cur, sp;
  // current patch
  float po, pi, dd;  // component c of the patch-frame origin, reciprocal direction, displacement (with the pad)
  float ptmin, pt0, pad2;
  uint32_t rec_idx, pmeta;
  CodeT code, trail;
  int depth;
  uint32_t mirror;
  float u0, v0;  // lower corner of the current domain
  float p[4];    // the record's points (i, j = b) of component c
  float pv[2];   // P^v of the inner points (1, j) and (2, j) of component c, j = 2 for b = 2, else 1
  float g[4];    // the working grid's row
  uint32_t vpref;  // learned order: the v-half to take at the next split, as in the one-lane kernel
};

struct GroupLane {
  int b, c;
  bool b0, b1, j2;
  __device__ __forceinline__ explicit GroupLane(int lane) {
    b = lane & 3;
    const int q = (lane >> 2) & 3;
    c = q < 2 ? q : 2;
    b0 = (b & 1) != 0;
    b1 = (b & 2) != 0;
    j2 = b == 2;
  }
  __device__ __forceinline__ float pick(float x, float y, float z) const { return c == 0 ? x : c == 1 ? y : z; }
};

// Lower corner of the domain of a path code.
template <typename CodeT>
__device__ __forceinline__ void group_corner(GroupRay<CodeT>& r, float leaf_scale) {
  r.u0 = (float)compact_even(r.code >> 1) * leaf_scale;
  r.v0 = (float)compact_even(r.code) * leaf_scale;
}

// The current patch's record into the lanes' registers.
template <typename CodeT>
__device__ __forceinline__ void group_load_record(GroupRay<CodeT>& r, const GroupLane& ln) {
  const float* rec = r.recs + (size_t)r.rec_idx * kRecFloats;
  const float4 x = reinterpret_cast<const float4*>(rec)[4 * ln.c + ln.b];
  const float2 v = reinterpret_cast<const float2*>(rec + 48)[2 * ln.c + (ln.j2 ? 1 : 0)];
  r.p[0] = x.x;
  r.p[1] = x.y;
  r.p[2] = x.z;
  r.p[3] = x.w;
  r.pv[0] = v.x;
  r.pv[1] = v.y;
}

// World ray of a group from its two words.
template <typename CodeT>
__device__ __forceinline__ void group_set_ray(GroupRay<CodeT>& r, const GroupLane& ln, const float4& ro,
                                              const float4& rd) {
  r.ox = ro.x;
  r.oy = ro.y;
  r.oz = ro.z;
  r.tmin = ro.w;
  r.dx = rd.x;
  r.dy = rd.y;
  r.dz = rd.z;
  r.wo = ln.pick(ro.x, ro.y, ro.z);
  r.wi = safe_inv(ln.pick(rd.x, rd.y, rd.z));
}

// Candidate patch: Alg. 3 set up at the root, as the one-lane kernel does it.
template <typename CodeT>
__device__ __forceinline__ void group_candidate(GroupRay<CodeT>& r, const GroupLane& ln) {
  r.rec_idx = (uint32_t)(~r.cur);
  const float4 meta = reinterpret_cast<const float4*>(r.recs + (size_t)r.rec_idx * kRecFloats)[15];
  group_load_record(r, ln);
  r.pmeta = __float_as_uint(meta.w);
  const float qx = meta.x - r.ox, qy = meta.y - r.oy, qz = meta.z - r.oz;
  r.pt0 = (qx * r.dx + qy * r.dy + qz * r.dz) * __builtin_amdgcn_rcpf(r.dx * r.dx + r.dy * r.dy + r.dz * r.dz);
  const double ax = fma((double)r.pt0, (double)r.dx, (double)r.ox - (double)meta.x);
  const double ay = fma((double)r.pt0, (double)r.dy, (double)r.oy - (double)meta.y);
  const double az = fma((double)r.pt0, (double)r.dz, (double)r.oz - (double)meta.z);
  r.ptmin = (float)((double)r.tmin - (double)r.pt0);
  if (r.frames) {
    const float4* fr = r.frames + 3 * (size_t)r.rec_idx;
    const float4 row = fr[ln.c];
    const float pad = reinterpret_cast<const float*>(fr)[3];
    const double ex = r.dx, ey = r.dy, ez = r.dz;
    r.po = (float)fma((double)row.z, az, fma((double)row.y, ay, (double)row.x * ax));
    r.pi = safe_inv((float)fma((double)row.z, ez, fma((double)row.y, ey, (double)row.x * ex)));
    r.po += pad;  // boxes grown by the pad: the low planes through the origin, the high ones through dd
    r.pad2 = 2.0f * pad;
  } else {
    r.po = ln.c == 0 ? (float)ax : ln.c == 1 ? (float)ay : (float)az;
    r.pi = r.wi;
    r.pad2 = 0.0f;
  }
  r.code = r.trail = 0;
  r.mirror = 0;
  r.depth = 0;
  r.u0 = r.v0 = 0.0f;
  if (r.pmeta & kGregoryBit) {
    r.mode = kGroupGrid;
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a) r.g[a] = r.p[a];
    r.dd = r.pad2;
    r.mode = kGroupStep;
  }
}

// The children of a BVH node and the distances at which their boxes are entered (+inf:
// missed); lane (c, b) tests component c of child b & 1.
template <typename CodeT>
__device__ __forceinline__ int2 group_children(const GroupRay<CodeT>& r, const GroupLane& ln, int node, float& t0,
                                               float& t1) {
  const float* nd = reinterpret_cast<const float*>(r.nodes + 4 * (size_t)node);
  const int at = (ln.b0 ? 6 : 0) + ln.c;
  const float lo = nd[at], hi = nd[at + 3];
  const int2 ch = *reinterpret_cast<const int2*>(nd + 12);
  const float capw = r.best_t + fabsf(r.best_t) * 0x1p-21f;
  const float x0 = (lo - r.wo) * r.wi, x1 = (hi - r.wo) * r.wi;
  const float nr = fmaxf(across_max(fminf(x0, x1)), r.tmin);
  const float fr = fminf(widen_far(across_min(fmaxf(x0, x1))), capw);
  const float own = nr <= fr ? nr : __builtin_inff();
  const float other = dpp<kQuadXor1>(own);
  t0 = ln.b0 ? other : own;
  t1 = ln.b0 ? own : other;
  return ch;
}

// One BVH node.  The node stack of the ray is stack[kStride * level].  Returns false
// when the ray is done.
template <int kStride, typename CodeT>
__device__ __forceinline__ bool group_node(GroupRay<CodeT>& r, const GroupLane& ln, int* stack) {
  float t0, t1;
  const int2 ch = group_children(r, ln, r.cur, t0, t1);
  const bool h0 = t0 != __builtin_inff(), h1 = t1 != __builtin_inff();
  if (h0 && h1) {
    const bool first1 = t1 < t0;
    if (r.sp < (int)kMaxBvhDepth) {  // always holds: the host rejects deeper BVHs
      stack[r.sp * kStride] = first1 ? ch.x : ch.y;
      ++r.sp;
    }
    r.cur = first1 ? ch.y : ch.x;
  } else if (h0 || h1) {
    r.cur = h0 ? ch.x : ch.y;
  } else if (r.sp > 0) {
    --r.sp;
    r.cur = stack[r.sp * kStride];
  } else {
    return false;
  }
  return true;
}

// The current domain's grid (and Gregory displacement): Alg. 2 and the crop of
// calc_component, one column j = b of the points per lane for the u pass, one
// row i = b for the v pass.
// kGregory: 0 a Bezier patch, 2 a Gregory patch, 1 as its meta word says.
template <int kGregory, typename CodeT>
__device__ __forceinline__ void group_grid(GroupRay<CodeT>& r, const GroupLane& ln) {
  const float su = __uint_as_float((uint32_t)(127 - ((r.depth + 1) >> 1)) << 23);
  const float sv = __uint_as_float((uint32_t)(127 - (r.depth >> 1)) << 23);
  const float u0 = r.u0, u1 = u0 + su, v0 = r.v0, v1 = v0 + sv;
  float p0 = r.p[0], p1 = r.p[1], p2 = r.p[2], p3 = r.p[3], d = 0.0f;
  if (kGregory == 2 || (kGregory == 1 && (r.pmeta & kGregoryBit))) {
    const bool inner = ln.b0 != ln.b1;  // j = 1 or 2
    const float wv1 = wbar1(v0, v1), wv2 = wbar2(v0, v1), wv = ln.j2 ? wv2 : wv1;
    const float dvl = ln.j2 ? 1.0f - v1 : v0, dvh = ln.j2 ? 1.0f - v0 : v1;
    float w[2], s[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float dul = i == 0 ? u0 : 1.0f - u1, duh = i == 0 ? u1 : 1.0f - u0;
      const float lam_lo = dul * __builtin_amdgcn_rcpf(dul + dvh), lam_hi = duh * __builtin_amdgcn_rcpf(duh + dvl);
      w[i] = (i == 0 ? wbar1(u0, u1) : wbar2(u0, u1)) * wv;
      const float x = i == 0 ? p1 : p2, e = x - r.pv[i];
      const float A = fmaf(lam_lo, e, r.pv[i]), B = fmaf(lam_hi, e, r.pv[i]);
      const float m = inner ? fminf(A, B) : x;
      if (i == 0)
        p1 = m;
      else
        p2 = m;
      s[i] = fabsf(A - B);
    }
    // the displacement's sum in the order (1,1), (2,1), (1,2), (2,2)
    d = fmaf(dpp<kQuadLane1>(w[0]), dpp<kQuadLane1>(s[0]), d);
    d = fmaf(dpp<kQuadLane1>(w[1]), dpp<kQuadLane1>(s[1]), d);
    d = fmaf(dpp<kQuadLane2>(w[0]), dpp<kQuadLane2>(s[0]), d);
    d = fmaf(dpp<kQuadLane2>(w[1]), dpp<kQuadLane2>(s[1]), d);
  }
  const Crop4 mu = crop_matrix(u0, u1), mv = crop_matrix(v0, v1);
  float h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    h[i] = fmaf(mu.m[i][3], p3, fmaf(mu.m[i][2], p2, fmaf(mu.m[i][1], p1, mu.m[i][0] * p0)));
  quad_transpose(h, ln.b0, ln.b1);
  float q[4], qt[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    q[j] = fmaf(mv.m[j][3], h[3], fmaf(mv.m[j][2], h[2], fmaf(mv.m[j][1], h[1], mv.m[j][0] * h[0])));
    qt[j] = q[j];
  }
  quad_transpose(qt, ln.b0, ln.b1);
  const bool along_v = (r.depth & 1) != 0;  // the split runs along v: row i = b over j as it is
#pragma unroll
  for (int a = 0; a < 4; ++a) r.g[a] = along_v ? q[a] : qt[a];
  r.dd = d + r.pad2;
  r.mirror = 0;
  r.mode = kGroupStep;
}

// Both halves of the working grid: the points of the lane's row, and entry, exit and
// hit of the halves in storage order, against the best distance so far.
struct GroupSplit {
  Row7 e;
  float ta, xa, tb, xb;
  bool hit_a, hit_b;
};

template <typename CodeT>
__device__ __forceinline__ GroupSplit group_split(const GroupRay<CodeT>& r) {
  GroupSplit h;
  h.e = casteljau_half(r.g[0], r.g[1], r.g[2], r.g[3]);
  const Row7& e = h.e;
  const float la = quad_min(fminf(fminf(fminf(e.v[0], e.v[1]), e.v[2]), e.v[3]));
  const float ha = quad_max(fmaxf(fmaxf(fmaxf(e.v[0], e.v[1]), e.v[2]), e.v[3]));
  const float lb = quad_min(fminf(fminf(fminf(e.v[3], e.v[4]), e.v[5]), e.v[6]));
  const float hb = quad_max(fmaxf(fmaxf(fmaxf(e.v[3], e.v[4]), e.v[5]), e.v[6]));
  const float a0 = (la - r.po) * r.pi, a1 = (ha + r.dd - r.po) * r.pi;
  const float b0 = (lb - r.po) * r.pi, b1 = (hb + r.dd - r.po) * r.pi;
  h.ta = fmaxf(across_max(fminf(a0, a1)), r.ptmin);
  h.xa = across_min(fmaxf(a0, a1));
  h.tb = fmaxf(across_max(fminf(b0, b1)), r.ptmin);
  h.xb = across_min(fmaxf(b0, b1));
  const float cap = (r.best_t - r.pt0) + (fabsf(r.best_t) + fabsf(r.pt0)) * 0x1p-22f;
  h.hit_a = h.ta <= fminf(widen_far(h.xa), cap);
  h.hit_b = h.tb <= fminf(widen_far(h.xb), cap);
  return h;
}

// A leaf entered at distance tf with path code lc, recorded when it is the best.
template <typename CodeT>
__device__ __forceinline__ bool group_leaf(GroupRay<CodeT>& r, float tf, CodeT lc, float leaf_scale) {
  const uint32_t pid = r.pmeta & kIdMask;
  if (!(tf < r.best_t || (tf == r.best_t && pid < r.best_id))) return false;
  r.best_t = tf;
  r.best_id = pid;
  r.hu = (float)(2u * compact_even(lc >> 1) + 1u) * (0.5f * leaf_scale);
  r.hv = (float)(2u * compact_even(lc) + 1u) * (0.5f * leaf_scale);
  return true;
}

// One subdivision step.  Returns false when the patch is finished (the caller
// takes the next candidate from the stack or ends the ray).  Learned order: a split
// along u where both halves are hit leaves the node's corners and slab results in
// the group's 16 words at `feat` and its mirror bits in `mirror0`, and waits for
// the network.
template <bool kLearned, typename CodeT>
__device__ __forceinline__ bool group_step(GroupRay<CodeT>& r, const GroupLane& ln, int L2, float leaf_scale,
                                           uint32_t* feat, uint32_t& mirror0) {
  const GroupSplit h = group_split(r);
  const Row7& e = h.e;
  const float ta = h.ta, xa = h.xa, tb = h.tb, xb = h.xb;
  const bool hit_a = h.hit_a, hit_b = h.hit_b;
  const int axis = r.depth & 1;
  const bool mir = ((r.mirror >> axis) & 1u) != 0;
  const bool h_lo = mir ? hit_b : hit_a, h_up = mir ? hit_a : hit_b;
  const float t_lo = mir ? tb : ta, t_up = mir ? ta : tb;
  bool go_up = h_up && (!h_lo || t_up < t_lo);
  const CodeT bit = (CodeT)1 << (L2 - 1 - r.depth);
  bool decide = false;
  if (kLearned) {
    if ((r.vpref & 1u) && axis == 1 && hit_a && hit_b && r.depth != L2 - 1) go_up = (r.vpref & 2u) != 0;
    r.vpref = 0;
    decide = axis == 0 && hit_a && hit_b;
  }
  const bool second = go_up != mir;
  if (hit_a || hit_b) {
    if (r.depth != L2 - 1) {
      if (kLearned && decide) {
        // the layout of policy_store_node: component c's corners (0,0), (3,0), (0,3), (3,3)
        // at 4c, then the slab results
        if (ln.b0 == ln.b1) {
          float* o = reinterpret_cast<float*>(feat) + 4 * ln.c + (ln.b0 ? 2 : 0);
          o[0] = e.v[0];
          o[1] = e.v[6];
        }
        reinterpret_cast<float4*>(feat)[3] = make_float4(ta, xa, tb, xb);
        mirror0 = r.mirror;
      }
      r.g[0] = second ? e.v[6] : e.v[0];
      r.g[1] = second ? e.v[5] : e.v[1];
      r.g[2] = second ? e.v[4] : e.v[2];
      r.g[3] = e.v[3];
      quad_transpose(r.g, ln.b0, ln.b1);
      if (hit_a && hit_b) r.trail |= bit;
      if (go_up) {
        r.code |= bit;
        const float half = __uint_as_float((uint32_t)(126 - (r.depth >> 1)) << 23);
        r.u0 += axis ? 0.0f : half;
        r.v0 += axis ? half : 0.0f;
      }
      if (second) r.mirror ^= 1u << axis;
      r.depth++;
      if (r.pmeta & kGregoryBit) r.mode = kGroupGrid;
      if (kLearned && decide) r.mode = kGroupDecide;
      return true;
    }
    group_leaf(r, r.pt0 + (go_up ? t_up : t_lo), (CodeT)(r.code | (go_up ? bit : (CodeT)0)), leaf_scale);
  }
  if (r.trail == 0) return false;
  const int k = sizeof(CodeT) == 8 ? __builtin_ctzll((uint64_t)r.trail) : __builtin_ctz((uint32_t)r.trail);
  const CodeT tb_bit = (CodeT)1 << k;
  r.trail ^= tb_bit;
  r.code = (r.code ^ tb_bit) & ~(tb_bit - 1);
  r.depth = L2 - k;
  group_corner(r, leaf_scale);
  r.mode = kGroupGrid;
  return true;
}

// Learned order: the network for the groups that wait for it, by the whole wave.
// feats: 16 words per group.
template <typename CodeT>
__device__ __forceinline__ void group_decide(GroupRay<CodeT>& r, const PolicyDev& policy, uint32_t* feats,
                                             uint32_t mirror0, int L2, int lane, float leaf_scale) {
  const uint64_t waiting = __ballot(r.mode == kGroupDecide);
  if (waiting == 0) return;
  const int group = lane / kGroupLanes, base = lane & ~(kGroupLanes - 1);
  // the components' values from the group's three quads
  const float fd = r.frames ? __builtin_amdgcn_rcpf(r.pi) : 0.0f;
  const float px = __shfl(r.po, base), py = __shfl(r.po, base + 4), pz = __shfl(r.po, base + 8);
  const float fx = __shfl(fd, base), fy = __shfl(fd, base + 4), fz = __shfl(fd, base + 8);
  if (r.mode == kGroupDecide) {
    float f[16];
    policy_features(policy_load_node(feats, group, mirror0), px, py, pz, r.frames ? fx : r.dx, r.frames ? fy : r.dy,
                    r.frames ? fz : r.dz, r.depth - 1, L2 / 2, (r.pmeta & kGregoryBit) != 0, f);
    policy_store_inputs<16>(feats, group, f);
  }
  // a network input row per waiting group (16 columns of a tile, of which four are read)
  uint64_t need = 0;
#pragma unroll
  for (int g = 0; g < kGroupsPerWave; ++g) need |= ((waiting >> (kGroupLanes * g)) & 1ull) << g;
  policy_wave<16>(policy, feats, need, lane);
  if (r.mode == kGroupDecide) {
    const float4 lg = reinterpret_cast<const float4*>(feats)[4 * group];
    const uint32_t top = policy_top(lg.x, lg.y, lg.z, lg.w);
    const CodeT bit = (CodeT)1 << (L2 - r.depth);  // path bit of the u-split just taken
    r.vpref = 1u | ((top & 1u) << 1);
    if (((top >> 1) != 0) != ((r.code & bit) != 0)) {
      r.code ^= bit;  // the other u-half first; the trail bit keeps the closest-first one pending
      group_corner(r, leaf_scale);
      r.mode = kGroupGrid;
    } else {
      r.mode = (r.pmeta & kGregoryBit) ? kGroupGrid : kGroupStep;
    }
  }
}

// ------------------------------------------------------------ one ray to a wave
// When a wave holds a single ray, all four groups carry it and its control state is
// the wave's: path, trail and stack live in scalar registers and every decision is a
// scalar branch (a Bezier step then issues ~130 instructions instead of ~240).  On a
// Gregory patch, whose grids depend on the domain alone, the groups expand four
// nodes at once: the current one, its two children and the nearest pending sibling
// (at a leaf's parent the three nearest); what the traversal does next is looked up
// among them.  Nothing is used that was tested against another best distance.
// Heaviest rays of three scenes alone, on 16 lanes -> on 64: torus 175 -> 98 us, its
// leaf depth 18 792 -> 405 us, world frames 1092 -> 790 us.
//
// A node is one word here: its path code with a marker bit below the last split's
// (bit L2-1-depth, the bit its own split would own).
template <typename T>
__device__ __forceinline__ T uniform(T x) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "words");
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
  for (uint32_t k = 0; k < sizeof(T) / 4; ++k) w[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[k]);
  __builtin_memcpy(&x, w, sizeof(T));
  return x;
}

// Whether a condition that is the same in all lanes holds, as a scalar.
__device__ __forceinline__ bool wave_is(bool x) { return __ballot(x) != 0; }

template <typename CodeT>
__device__ __forceinline__ CodeT lowest(CodeT x) { return x & (CodeT)(0 - x); }

// The sibling pending at the lowest bit of `trail` (not 0).
template <typename CodeT>
__device__ __forceinline__ CodeT pending(CodeT node, CodeT trail) {
  const CodeT bit = lowest(trail);
  return ((node ^ bit) & ~(CodeT)(bit - 1)) | (CodeT)(bit >> 1);
}

// Path code, depth and domain corner of a node into r.
template <typename CodeT>
__device__ __forceinline__ void solo_domain(GroupRay<CodeT>& r, CodeT node, int L2, float leaf_scale) {
  r.code = node & (CodeT)(node - 1);
  const int k = sizeof(CodeT) == 8 ? __builtin_ctzll((uint64_t)node) : __builtin_ctz((uint32_t)node);
  r.depth = L2 - 1 - k;
  group_corner(r, leaf_scale);
}

// Gregory patch: from `node`, whose grid is due, as far as one expansion reaches.
// Returns false when the patch is finished.
template <typename CodeT>
__device__ __forceinline__ bool solo_expand(GroupRay<CodeT>& r, const GroupLane& ln, CodeT& node, CodeT& trail, int L2,
                                            float leaf_scale, int lane) {
  CodeT n1 = 0, n2 = 0, n3 = 0;  // 0 is no node
  {
    CodeT left = trail;
    auto next = [&]() {
      CodeT p = 0;
      if (left != 0) {
        p = pending(node, left);
        left &= left - 1;
      }
      return p;
    };
    const CodeT bit = lowest(node);
    if (bit != 1) {
      n1 = (node ^ bit) | (CodeT)(bit >> 1);
      n2 = node | (CodeT)(bit >> 1);
    } else {
      n1 = next();
      n2 = next();
    }
    n3 = next();
  }
  const int group = lane / kGroupLanes;
  CodeT own = group == 0 ? node : group == 1 ? n1 : group == 2 ? n2 : n3;
  own = own != 0 ? own : node;
  solo_domain(r, own, L2, leaf_scale);
  group_grid<2>(r, ln);
  const GroupSplit h = group_split(r);  // a fresh grid: the lower half is stored first
  const bool up = h.hit_b && (!h.hit_a || h.tb < h.ta);
  const float tf = r.pt0 + (up ? h.tb : h.ta);
  const int seen = (h.hit_a ? 1 : 0) | (h.hit_b ? 2 : 0) | (up ? 4 : 0);
  const int s0 = __builtin_amdgcn_readlane(seen, 0), s1 = __builtin_amdgcn_readlane(seen, kGroupLanes),
            s2 = __builtin_amdgcn_readlane(seen, 2 * kGroupLanes), s3 = __builtin_amdgcn_readlane(seen, 3 * kGroupLanes);
  int see = s0;
  for (;;) {
    const CodeT bit = lowest(node);
    bool better = false;
    if ((see & 3) != 0) {
      if (bit != 1) {
        trail |= (see & 3) == 3 ? bit : (CodeT)0;
        node = ((see & 4) ? node : (CodeT)(node ^ bit)) | (CodeT)(bit >> 1);
        see = node == n1 ? s1 : node == n2 ? s2 : node == n3 ? s3 : -1;
        if (see < 0) return true;
        continue;
      }
      const int at = node == n1 ? 1 : node == n2 ? 2 : node == n3 ? 3 : 0;
      const float t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tf), kGroupLanes * at));
      better = wave_is(group_leaf(r, t, (CodeT)((node ^ bit) | ((see & 4) ? 1 : 0)), leaf_scale));
    }
    if (trail == 0) return false;
    node = pending(node, trail);
    trail &= trail - 1;
    see = node == n1 ? s1 : node == n2 ? s2 : node == n3 ? s3 : -1;
    if (see < 0 || better) return true;  // after a record the other nodes' tests are out of date
  }
}

// The current patch of a wave's ray, whose grid is due or in r.g with r.mirror, to its end.
template <typename CodeT>
__device__ __forceinline__ void solo_patch(GroupRay<CodeT>& r, const GroupLane& ln, int L2, float leaf_scale, int lane) {
  CodeT trail = uniform(r.trail);
  CodeT node = uniform(r.code) | (CodeT)1 << (L2 - 1 - uniform(r.depth));
  bool due = uniform(r.mode) == kGroupGrid;
  const int axis = uniform(r.depth) & 1;
  // mirror bit of the next split's axis and of the other one: every descent swaps them
  uint32_t m0 = (uniform(r.mirror) >> axis) & 1u, m1 = (uniform(r.mirror) >> (axis ^ 1)) & 1u;
  const bool gregory = (uniform(r.pmeta) & kGregoryBit) != 0;
  for (;;) {
    if (due) {
      if (gregory) {
        if (!solo_expand(r, ln, node, trail, L2, leaf_scale, lane)) return;
        continue;
      }
      solo_domain(r, node, L2, leaf_scale);
      group_grid<0>(r, ln);
      m0 = m1 = 0;
    }
    const GroupSplit h = group_split(r);
    const bool mir = m0 != 0;
    const bool h_lo = mir ? h.hit_b : h.hit_a, h_up = mir ? h.hit_a : h.hit_b;
    const float t_lo = mir ? h.tb : h.ta, t_up = mir ? h.ta : h.tb;
    const bool go_up = h_up && (!h_lo || t_up < t_lo);
    const int see = uniform((h_lo ? 1 : 0) | (h_up ? 2 : 0) | (go_up ? 4 : 0));
    const CodeT bit = lowest(node);
    if ((see & 3) != 0) {
      if (bit != 1) {
        const bool second = ((see >> 2) & 1) != (int)m0;
        r.g[0] = second ? h.e.v[6] : h.e.v[0];
        r.g[1] = second ? h.e.v[5] : h.e.v[1];
        r.g[2] = second ? h.e.v[4] : h.e.v[2];
        r.g[3] = h.e.v[3];
        quad_transpose(r.g, ln.b0, ln.b1);
        const uint32_t m = m0 ^ (second ? 1u : 0u);
        m0 = m1;
        m1 = m;
        trail |= (see & 3) == 3 ? bit : (CodeT)0;
        node = ((see & 4) ? node : (CodeT)(node ^ bit)) | (CodeT)(bit >> 1);
        due = gregory;
        continue;
      }
      group_leaf(r, r.pt0 + (go_up ? t_up : t_lo), (CodeT)((node ^ bit) | ((see & 4) ? 1 : 0)), leaf_scale);
    }
    if (trail == 0) return;
    node = pending(node, trail);
    trail &= trail - 1;
    due = true;
  }
}

// The same in the learned order, a node at a time: the next node depends on the
// network's answer.  feats: 16 words for each of the 16 columns of a network tile, of
// which the ray takes the first.
template <typename CodeT>
__device__ __forceinline__ void solo_patch_learned(GroupRay<CodeT>& r, const GroupLane& ln, const PolicyDev& policy,
                                                   uint32_t* feats, int L2, float leaf_scale, int lane) {
  CodeT trail = uniform(r.trail);
  CodeT node = uniform(r.code) | (CodeT)1 << (L2 - 1 - uniform(r.depth));
  bool due = uniform(r.mode) == kGroupGrid;
  uint32_t vpref = uniform(r.vpref);
  r.vpref = 0;
  const int axis = uniform(r.depth) & 1;
  uint32_t m0 = (uniform(r.mirror) >> axis) & 1u, m1 = (uniform(r.mirror) >> (axis ^ 1)) & 1u;
  const bool gregory = (uniform(r.pmeta) & kGregoryBit) != 0;
  for (;;) {
    if (due) {
      solo_domain(r, node, L2, leaf_scale);
      if (gregory)
        group_grid<2>(r, ln);
      else
        group_grid<0>(r, ln);
      m0 = m1 = 0;
    }
    const GroupSplit h = group_split(r);
    const bool mir = m0 != 0;
    const bool h_lo = mir ? h.hit_b : h.hit_a, h_up = mir ? h.hit_a : h.hit_b;
    const float t_lo = mir ? h.tb : h.ta, t_up = mir ? h.ta : h.tb;
    const bool closer_up = h_up && (!h_lo || t_up < t_lo);
    int see = uniform((h_lo ? 1 : 0) | (h_up ? 2 : 0) | (closer_up ? 4 : 0));
    const CodeT bit = lowest(node);
    const bool along_u = (bit & (CodeT)0x5555555555555555ull) == 0, both = (see & 3) == 3;
    if ((vpref & 1u) && !along_u && both && bit != 1) see = 3 | (int)((vpref & 2u) << 1);
    vpref = 0;
    if ((see & 3) != 0) {
      if (bit != 1) {
        const bool decide = along_u && both;
        if (decide && lane < kGroupLanes) {  // as in group_step
          if (ln.b0 == ln.b1) {
            float* o = reinterpret_cast<float*>(feats) + 4 * ln.c + (ln.b0 ? 2 : 0);
            o[0] = h.e.v[0];
            o[1] = h.e.v[6];
          }
          reinterpret_cast<float4*>(feats)[3] = make_float4(h.ta, h.xa, h.tb, h.xb);
        }
        const uint32_t mirror0 = m0 | (m1 << 1);
        const bool second = ((see >> 2) & 1) != (int)m0;
        r.g[0] = second ? h.e.v[6] : h.e.v[0];
        r.g[1] = second ? h.e.v[5] : h.e.v[1];
        r.g[2] = second ? h.e.v[4] : h.e.v[2];
        r.g[3] = h.e.v[3];
        quad_transpose(r.g, ln.b0, ln.b1);
        const uint32_t m = m0 ^ (second ? 1u : 0u);
        m0 = m1;
        m1 = m;
        trail |= both ? bit : (CodeT)0;
        node = ((see & 4) ? node : (CodeT)(node ^ bit)) | (CodeT)(bit >> 1);
        due = gregory;
        if (decide) {
          const int k = sizeof(CodeT) == 8 ? __builtin_ctzll((uint64_t)bit) : __builtin_ctz((uint32_t)bit);
          const float fd = r.frames ? __builtin_amdgcn_rcpf(r.pi) : 0.0f;
          const float px = __shfl(r.po, 0), py = __shfl(r.po, 4), pz = __shfl(r.po, 8);
          const float fx = __shfl(fd, 0), fy = __shfl(fd, 4), fz = __shfl(fd, 8);
          float f[16];
          policy_features(policy_load_node(feats, 0, mirror0), px, py, pz, r.frames ? fx : r.dx, r.frames ? fy : r.dy,
                          r.frames ? fz : r.dz, L2 - 1 - k, L2 / 2, gregory, f);
          policy_store_inputs<16>(feats, 0, f);
          policy_wave<16>(policy, feats, 1ull, lane);
          const float4 lg = reinterpret_cast<const float4*>(feats)[0];
          const uint32_t top = uniform(policy_top(lg.x, lg.y, lg.z, lg.w));
          vpref = 1u | ((top & 1u) << 1);
          if ((int)(top >> 1) != ((see >> 2) & 1)) {
            node ^= bit;  // the other u-half first; the trail bit keeps the closest-first one pending
            due = true;
          }
        }
        continue;
      }
      group_leaf(r, r.pt0 + ((see & 4) ? t_up : t_lo), (CodeT)((node ^ bit) | ((see & 4) ? 1 : 0)), leaf_scale);
    }
    if (trail == 0) return;
    node = pending(node, trail);
    trail &= trail - 1;
    due = true;
  }
}

// Every group's lanes take the words of the lanes of the group that starts at `first`.
template <typename T>
__device__ __forceinline__ void spread(T& x, int first, int lane) {
  static_assert(sizeof(T) % 4 == 0, "words");
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
  for (uint32_t k = 0; k < sizeof(T) / 4; ++k)
    w[k] = (uint32_t)__shfl((int)w[k], first + (lane & (kGroupLanes - 1)));
  __builtin_memcpy(&x, w, sizeof(T));
}

}  // namespace ccs
