// What the batched kernels share: the search for a tile's stream, and descriptors as kernel arguments.
#pragma once

#include <hip/hip_runtime.h>

#include <cstring>

#include "gmm_frame.hpp"
#include "gmm_internal.hpp"

namespace rgbd {

// The stream of tile t: the last entry of `first` (n entries, first[0] = 0, increasing) that is
// <= t. A binary search in scalar registers: its loads hit the scalar cache that every block of
// the CU reads `first` through, which a tile map of one word per tile does not (64 streams, fp32:
// 312 us per launch either way), and a wave-wide probe of all entries at once, one vector load,
// waits longer (321 us).
__device__ __forceinline__ uint32_t find_stream(const uint32_t* __restrict__ first, uint32_t n, uint32_t t) {
  uint32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (first[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// What differs from stream to stream of a descriptor. Streams of one call nearly always share the
// model constants; sent once per launch, they let the 4 KB of a kernel's arguments carry 32
// streams, where whole descriptors fill them with 16.
struct PackEntry {
  uint32_t npix, width, mode;
  uint32_t dense;  // bit 0 rgb_dense, bit 1 depth_dense
  const uint8_t* rgb;
  int64_t rgb_pitch;
  const uint16_t* depth;
  int64_t depth_pitch;
  void* st_rgb;
  void* st_depth;
  uint8_t* fstate;
  uint64_t* fg_rgb;
  uint64_t* fg_depth;
  uint64_t* fused;
  uint64_t* wave_bytes;
};

struct PackArgs {
  PackEntry e[kPackPerLaunch];
  uint32_t first[kPackPerLaunch];
  ModelConsts kc, kd;
  uint32_t base;   // index of e[0] in the tables
  uint32_t count;  // entries used
};
static_assert(sizeof(PackArgs) + 2 * sizeof(void*) <= 4096, "kernel arguments");

inline bool same_consts(const FrameArgs& a, const FrameArgs& b) {
  return std::memcmp(&a.kc, &b.kc, sizeof(ModelConsts)) == 0 && std::memcmp(&a.kd, &b.kd, sizeof(ModelConsts)) == 0;
}

inline PackEntry pack_entry(const FrameArgs& a) {
  return PackEntry{static_cast<uint32_t>(a.npix), static_cast<uint32_t>(a.width), static_cast<uint32_t>(a.mode),
                   (a.rgb_dense ? 1u : 0u) | (a.depth_dense ? 2u : 0u), a.rgb, a.rgb_pitch, a.depth, a.depth_pitch,
                   a.st_rgb, a.st_depth, a.fstate, a.fg_rgb, a.fg_depth, a.fused, a.wave_bytes};
}

// Streams [0, n) of `a`, all with the same constants, n <= kPackPerLaunch (`first` may be NULL).
inline PackArgs pack_args(const FrameArgs* a, const uint32_t* first, int32_t n, uint32_t base) {
  PackArgs p{};
  p.base = base;
  p.count = static_cast<uint32_t>(n);
  p.kc = a[0].kc;
  p.kd = a[0].kd;
  for (int32_t i = 0; i < n; ++i) {
    p.e[i] = pack_entry(a[i]);
    if (first) p.first[i] = first[i];
  }
  return p;
}

__device__ __forceinline__ FrameArgs unpack_entry(const PackArgs& p, uint32_t i) {
  const PackEntry e = p.e[i];
  FrameArgs a{};
  a.npix = e.npix;
  a.tiles64 = (e.npix + kWave - 1) / kWave;
  a.width = static_cast<int32_t>(e.width);
  a.rgb_dense = static_cast<int32_t>(e.dense & 1u);
  a.depth_dense = static_cast<int32_t>(e.dense >> 1);
  a.rgb = e.rgb;
  a.rgb_pitch = e.rgb_pitch;
  a.depth = e.depth;
  a.depth_pitch = e.depth_pitch;
  a.st_rgb = e.st_rgb;
  a.st_depth = e.st_depth;
  a.fstate = e.fstate;
  a.fg_rgb = e.fg_rgb;
  a.fg_depth = e.fg_depth;
  a.fused = e.fused;
  a.kc = p.kc;
  a.kd = p.kd;
  a.mode = static_cast<int32_t>(e.mode);
  a.wave_bytes = e.wave_bytes;
  return a;
}

}  // namespace rgbd
