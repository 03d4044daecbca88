// Stream compaction of ray arrays: the rays the intersection kernel traces
// (its validity test, below) are copied in input order to a dense array with
// their input indices, so that a path tracer's later bounce levels, where most
// pixels' paths have ended (Sec. 4: a bounce of a missed ray is inactive), are
// traced without cycling through their inactive rays.
//
// The order is the input order, so the result is deterministic.  The test of a traced
// ray is the intersection kernel's own (ray_valid.h), and this file is compiled with
// that kernel's floating-point flags (denormals flushed), so both decide alike.
//
// Up to 2,097,152 rays: two launches over the same split of the rays: a run of 256 k
// consecutive rays per wave, k the smallest that leaves at most kCompactBlocks blocks
// of four waves, all resident at once.  The first counts each run's active rays; the
// second adds up the counts before its own (at most 8192 words, read by every block;
// a scan of its own in one workgroup took 4 to 30 us) and copies.  Bound by memory:
// 32 B read per ray, twice, and 36 B written per active ray, 5.0 TB/s of the 5.1 TB/s
// that a copy reaches.  A lane loads half a ray, so that a wave's load is 1 KB in a
// row (its neighbour's half comes by a lane exchange), and four such loads are in
// flight.  The second launch walks each run backwards, beginning with what the first
// one read last (2 % faster than forwards).  30 % of 921,600 rays take 17.0 us, of
// 184,000 16.3 -> 12.8 us.  1024 or 4096 blocks and 2 or 8 loads in flight are no faster
// at any size.
//
// More rays: one pass over them (k_compact_tiles, below), after a launch that clears its
// words.  The sizes at which the forms change are those of 256 CUs.

#include "ccs_internal.h"
#include "ray_valid.h"

namespace ccs {

constexpr int kCompactBlock = 256;
constexpr int kCompactWaves = kCompactBlock / 64;
constexpr uint32_t kCompactBlocks = 2048;  // eight per CU
constexpr uint32_t kCompactUnit = 256;     // rays of a wave's run: a multiple of this (a work word per run)
constexpr int kCompactLoads = 4;           // loads in flight: 32 rays each
constexpr int kTileWaves = 16, kTileBlock = 64 * kTileWaves;
constexpr int kTileLoads = 16;  // loads in flight, and halves of rays a lane holds
constexpr uint32_t kTileRays = 32u * kTileLoads * kTileWaves;  // 8192
// One pass from the size on at which every CU has more than one tile, up to what the
// 30 bits of a tile's word can count: 4,000,000 rays (30 % active) 60 -> 55 us and
// 8,294,399 rays 123 -> 100 us, but 921,600 rays 17 -> 21 us.
constexpr uint32_t kTilesFrom = 256u * kTileRays + 1u, kTilesTo = (1u << 30) - 1u;

// The value of lane ^ 1 (its bits, moved within a quad).  It passes through an empty
// asm statement: the optimizer, which sees that it comes from an integer, would turn
// the comparison of a direction with zero into one of bits, and a denormal direction,
// zero to the intersection kernel, would count as traced.
__device__ __forceinline__ float neighbour(float x) {
  float y = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
  asm volatile("" : "+v"(y));
  return y;
}

// Loads 16-byte halves of kLoads times 32 rays from `first` on and
// returns which of them are traced (both lanes of a ray say the same).
template <int kLoads>
__device__ __forceinline__ void load_halves(const float4* __restrict__ half, uint32_t first, uint32_t end, int lane,
                                            float4 own[kLoads], bool act[kLoads]) {
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const uint32_t at = 32u * q + (uint32_t)(lane >> 1);
    own[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // a zero direction: not traced
    if (at < end - first) own[q] = half[2 * ((size_t)first + at) + (lane & 1)];
  }
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    float4 o;  // the other half, from the neighbouring lane
    o.x = neighbour(own[q].x);
    o.y = neighbour(own[q].y);
    o.z = neighbour(own[q].z);
    o.w = neighbour(own[q].w);
    act[q] = (lane & 1) ? ray_traced(o, own[q]) : ray_traced(own[q], o);
  }
}

// Active rays of each run: work[1 + run].
__global__ __launch_bounds__(kCompactBlock) void k_compact_count(const ccs_ray* __restrict__ rays, uint32_t n,
                                                                 uint32_t run_rays, uint32_t* __restrict__ work) {
  const int lane = threadIdx.x & 63;
  const uint32_t run = blockIdx.x * kCompactWaves + (threadIdx.x >> 6);
  const uint64_t begin = (uint64_t)run * run_rays;
  if (begin >= n) return;
  const uint32_t end = (uint32_t)min((uint64_t)n, begin + run_rays);
  const float4* half = reinterpret_cast<const float4*>(rays);
  uint32_t c = 0;
  for (uint64_t i = begin; i < end; i += 32u * kCompactLoads) {
    float4 own[kCompactLoads];
    bool act[kCompactLoads];
    load_halves<kCompactLoads>(half, (uint32_t)i, end, lane, own, act);
#pragma unroll
    for (int q = 0; q < kCompactLoads; ++q) c += (uint32_t)__popcll(__ballot(act[q]));
  }
  if (lane == 0) work[1 + run] = c / 2u;
}

// Active ray i goes to out[actives before its run + its rank in the run].  The count
// of all rays is written by the wave of the last run.
__global__ __launch_bounds__(kCompactBlock) void k_compact_scatter(const ccs_ray* __restrict__ rays, uint32_t n,
                                                                   uint32_t run_rays, uint32_t* __restrict__ work,
                                                                   ccs_ray* __restrict__ out,
                                                                   uint32_t* __restrict__ index) {
  __shared__ uint32_t s_wave[kCompactWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t first = blockIdx.x * kCompactWaves, run = first + wave;
  uint32_t before = 0;
  for (uint32_t k = threadIdx.x; k < first; k += kCompactBlock) before += work[1 + k];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) before += (uint32_t)__shfl_xor((int)before, d);
  if (lane == 0) s_wave[wave] = before;
  __syncthreads();
  const uint64_t begin = (uint64_t)run * run_rays;
  if (begin >= n) return;
  uint32_t pos = 0;  // one past the place of the last active ray not yet copied
#pragma unroll
  for (int w = 0; w < kCompactWaves; ++w) pos += s_wave[w];
  for (int w = 0; w <= wave; ++w) pos += work[1 + first + w];
  const uint32_t end = (uint32_t)min((uint64_t)n, begin + run_rays);
  if (end == n && lane == 0) work[0] = pos;
  const float4* half = reinterpret_cast<const float4*>(rays);
  float4* out_half = reinterpret_cast<float4*>(out);
  constexpr uint32_t kStep = 32u * kCompactLoads;
  for (uint32_t left = (uint32_t)(((end - begin) + kStep - 1) / kStep); left-- > 0;) {
    const uint32_t i = (uint32_t)begin + left * kStep;
    float4 own[kCompactLoads];
    bool act[kCompactLoads];
    load_halves<kCompactLoads>(half, i, end, lane, own, act);
#pragma unroll
    for (int q = kCompactLoads - 1; q >= 0; --q) {
      const uint64_t m = __ballot(act[q]);
      pos -= (uint32_t)__popcll(m) / 2u;
      if (act[q]) {
        const uint32_t at = pos + (uint32_t)__popcll(m & ((1ull << (lane & ~1)) - 1ull)) / 2u;
        out_half[2 * (size_t)at + (lane & 1)] = own[q];
        if ((lane & 1) == 0) index[at] = i + 32u * q + (uint32_t)(lane >> 1);
      }
    }
  }
}

// One pass over tiles of kTileRays consecutive rays, a tile per block, which holds
// its rays in registers while it learns how many active rays lie before them
// (decoupled look-back, Merrill and Garland 2016), so that every ray is read once.
// Tiles are taken by a ticket: every tile before a block's own is held by a block that
// has started, and a block publishes its own count before it waits, so every wait
// ends.  A tile's word holds its count (kCount) and later the count of all rays up to
// its end (kUpto); value and flag are one word, read and written at device scope.
// Bound by the chain of these words, 6.6 ns a tile (tiles of 2048, 4096 and 8192 rays
// take 120, 107 and 100 us for 8,294,399 rays, 30 % of them active), and by a block's
// load and store phases, which only other CUs' overlap: 355 MB at 3.55 TB/s, against
// 620 MB at 5.0 TB/s of the two launches.  All waves looking back together, 512 or
// 1024 tiles at a time, is slower (103 to 115 us), as are two words a tile.
__global__ void k_compact_reset(uint32_t* __restrict__ work, uint32_t words) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) work[1 + i] = 0u;
}

__device__ __forceinline__ uint32_t peek(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void post(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kTileBlock) void k_compact_tiles(const ccs_ray* __restrict__ rays, uint32_t n,
                                                              uint32_t tiles, uint32_t* __restrict__ work,
                                                              ccs_ray* __restrict__ out,
                                                              uint32_t* __restrict__ index) {
  constexpr uint32_t kUpto = 0x80000000u, kCount = 0x40000000u;
  __shared__ uint32_t s_tile, s_before, s_wave[kTileWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* state = work + 2;
  if (threadIdx.x == 0) s_tile = atomicAdd(work + 1, 1u);
  __syncthreads();
  const uint32_t tile = s_tile;
  const uint64_t begin = (uint64_t)tile * kTileRays + (uint64_t)wave * (32u * kTileLoads);
  const uint32_t end = (uint32_t)min((uint64_t)n, begin + 32u * kTileLoads);
  float4 own[kTileLoads];
  bool act[kTileLoads];
  uint32_t c = 0;
  if (begin < n) {
    load_halves<kTileLoads>(reinterpret_cast<const float4*>(rays), (uint32_t)begin, end, lane, own, act);
#pragma unroll
    for (int q = 0; q < kTileLoads; ++q) c += (uint32_t)__popcll(__ballot(act[q])) / 2u;
  }
  if (lane == 0) s_wave[wave] = c;
  __syncthreads();
  if (wave == 0) {
    uint32_t total = 0, before = 0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) total += s_wave[w];
    if (tile != 0) {
      if (lane == 0) post(state + tile, total | kCount);
      for (uint32_t last = tile;;) {  // lane k looks at tile last - 1 - k
        const uint32_t x = (uint32_t)lane < last ? peek(state + (last - 1u - (uint32_t)lane)) : kUpto;
        const uint64_t mu = __ballot((x & kUpto) != 0), mk = __ballot((x & kCount) != 0);
        const int stop = mu != 0 ? __ffsll((unsigned long long)mu) - 1 : 64;  // the nearest tile with its sum
        const uint64_t need = stop >= 64 ? ~0ull : (1ull << stop) - 1ull;
        if ((mk & need) != need) {
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        uint32_t v = lane <= stop ? x & ~(kUpto | kCount) : 0u;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) v += (uint32_t)__shfl_xor((int)v, d);
        before += v;
        if (stop < 64) break;
        last -= 64u;
      }
    }
    if (lane == 0) {
      post(state + tile, (before + total) | kUpto);
      s_before = before;
      if (tile == tiles - 1u) work[0] = before + total;
    }
  }
  __syncthreads();
  if (begin >= n) return;
  uint32_t pos = s_before;
  for (int w = 0; w < wave; ++w) pos += s_wave[w];
  float4* out_half = reinterpret_cast<float4*>(out);
#pragma unroll
  for (int q = 0; q < kTileLoads; ++q) {
    const uint64_t m = __ballot(act[q]);
    if (act[q]) {
      const uint32_t at = pos + (uint32_t)__popcll(m & ((1ull << (lane & ~1)) - 1ull)) / 2u;
      out_half[2 * (size_t)at + (lane & 1)] = own[q];
      if ((lane & 1) == 0) index[at] = (uint32_t)begin + 32u * q + (uint32_t)(lane >> 1);
    }
    pos += (uint32_t)__popcll(m) / 2u;
  }
}

__global__ void k_compact_empty(uint32_t* work) { work[0] = 0u; }

hipError_t launch_compact_rays(const ccs_ray* rays, uint32_t n, ccs_ray* out, uint32_t* index, uint32_t* work,
                               hipStream_t stream) {
  if (n == 0) {
    hipLaunchKernelGGL(k_compact_empty, dim3(1), dim3(1), 0, stream, work);
    return hipGetLastError();
  }
  if (n >= kTilesFrom && n <= kTilesTo) {
    const uint32_t tiles = (uint32_t)(((uint64_t)n + kTileRays - 1) / kTileRays), words = 1u + tiles;
    hipLaunchKernelGGL(k_compact_reset, dim3((words + 255u) / 256u), dim3(256), 0, stream, work, words);
    hipLaunchKernelGGL(k_compact_tiles, dim3(tiles), dim3(kTileBlock), 0, stream, rays, n, tiles, work, out, index);
    return hipGetLastError();
  }
  constexpr uint64_t kPerBlock = (uint64_t)kCompactUnit * kCompactWaves;
  const uint32_t per_run = (uint32_t)((n + kPerBlock * kCompactBlocks - 1) / (kPerBlock * kCompactBlocks));
  const uint32_t run_rays = kCompactUnit * per_run;
  const uint32_t nb = (uint32_t)((n + kPerBlock * per_run - 1) / (kPerBlock * per_run));
  hipLaunchKernelGGL(k_compact_count, dim3(nb), dim3(kCompactBlock), 0, stream, rays, n, run_rays, work);
  hipLaunchKernelGGL(k_compact_scatter, dim3(nb), dim3(kCompactBlock), 0, stream, rays, n, run_rays, work, out, index);
  return hipGetLastError();
}

}  // namespace ccs
