// State I/O: the device layout of a handle's state to and from the canonical float64 layout
// (gmm_read_state, gmm_write_state), converted on the device.
//
// A value's place in the device layout is affine in its pixel's tile and lane (ValueMap), so one
// lane per canonical element moves it: canonical elements are contiguous (a wave reads or writes
// 512 B), the state side is 4- or 2-byte pieces at the row's or the suffix's lane stride, merged
// in the caches. What bounds the call is the host side: the canonical state (336 B per pixel of a
// paired stream at M = 5) crosses the link and is written to pageable memory. The elements go
// through one static device buffer, kChunk at a time, so a call allocates nothing and cannot run
// out of device memory; ~8 MB is where the pageable copies stop getting faster (26 MB to the host
// in 1.5 ms and from it in 0.96 ms, in pieces of 4 MB or more; 1.6 and 0.99 ms in pieces of 1 MB).
// The conversion used to run on one host thread, value by value: a write, a frame and a read of a 320x240
// paired stream (M = 5, fp32) took 49.5 ms; it takes 3.1 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "gmm.h"
#include "gmm_internal.hpp"

namespace rgbd {

constexpr uint32_t kChunk = 1u << 20;  // canonical elements in the buffer
static __device__ __align__(256) double io_buffer[kChunk];

// Value k (parameter-major, rank within) of pixel p lies at base + (p / 64) tile + (p % 64) lane.
struct ValueMap {
  uint32_t base, tile, lane;
};
constexpr uint32_t kMaxValues = 6 * 5;  // (C + 2) M at most: four channels, M = 5

struct BlockMap {
  ValueMap v[kMaxValues];
  uint32_t npix;
  uint32_t first_weight;  // k of the first weight: (C + 1) M
  uint32_t scale;         // byte offset of the scale plane (scaled form)
  float dk[4];            // ModelConsts::dk, for the hole factor
};

static BlockMap block_map(const gmm_handle* h, uint32_t C, const ModelConsts& k) {
  const uint32_t M = static_cast<uint32_t>(h->cfg.M), es = static_cast<uint32_t>(h->esize);
  const TileLayout L = tile_layout(M, C, es);
  BlockMap b{};
  for (uint32_t i = 0; i < (C + 2) * M; ++i) {
    const uint32_t v = value_index(i / M, i % M, M, C, es);
    b.v[i].base = static_cast<uint32_t>(state_value_offset(v, 0, h->tiles64, M, C, es));
    if (v >= L.nf) {
      b.v[i].tile = 64u * L.sb;
      b.v[i].lane = L.sb;
    } else {
      uint32_t c = 0;
      while (L.first[c + 1] <= v) ++c;
      b.v[i].tile = 64u * L.hot;
      b.v[i].lane = L.width[c];
    }
  }
  b.npix = static_cast<uint32_t>(h->npix);
  b.first_weight = (C + 1) * M;
  b.scale = scaled_weights(es) ? static_cast<uint32_t>(state_scale_offset(0, h->tiles64, M, C, es)) : 0u;
  for (int i = 0; i < 4; ++i) b.dk[i] = k.dk[i];
  return b;
}

__device__ __forceinline__ uint32_t value_at(const BlockMap& b, uint32_t k, uint32_t p) {
  const ValueMap m = b.v[k];
  return m.base + (p >> 6) * m.tile + (p & 63u) * m.lane;
}

// A finite or infinite double to a 16-bit binary format of `frac` fraction bits and exponent bias
// `bias`, to nearest with ties to even in one rounding (a conversion through fp32 would round
// twice); magnitudes that round past the largest finite value become infinite.
__device__ __forceinline__ uint32_t round_to_16(uint64_t u, int frac, int bias) {
  const uint32_t sign = static_cast<uint32_t>(u >> 63) << 15;
  const int e = static_cast<int>((u >> 52) & 0x7FFu) - 1023;
  const uint64_t m = (u & 0xFFFFFFFFFFFFFull) | (1ull << 52);
  const uint32_t inf = (2u * static_cast<uint32_t>(bias) + 1u) << frac;
  const int emin = 1 - bias;
  const int shift = 52 - frac + (e < emin ? emin - e : 0);
  uint32_t r = 0;
  if (shift <= 53) r = static_cast<uint32_t>((m + ((1ull << (shift - 1)) - 1u) + ((m >> shift) & 1u)) >> shift);
  // a normal number's implicit bit adds one to the exponent field, as does a carry out of the fraction
  const uint32_t field = e < emin ? 0u : static_cast<uint32_t>(min(e, bias + 1) - emin) << frac;
  return sign | min(r + field, inf);
}

template <typename S> struct Canonical;
template <> struct Canonical<float> {
  static __device__ __forceinline__ double get(const uint8_t* at) { return *reinterpret_cast<const float*>(at); }
  static __device__ __forceinline__ void put(uint8_t* at, double v) { *reinterpret_cast<float*>(at) = static_cast<float>(v); }
};
template <> struct Canonical<f16s> {
  static __device__ __forceinline__ double get(const uint8_t* at) {
    return static_cast<double>(*reinterpret_cast<const _Float16*>(at));
  }
  static __device__ __forceinline__ void put(uint8_t* at, double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const bool nan = (u & 0x7FFFFFFFFFFFFFFFull) > 0x7FF0000000000000ull;  // stored as a zero of its sign
    *reinterpret_cast<uint16_t*>(at) = static_cast<uint16_t>(nan ? (u >> 63) << 15 : round_to_16(u, 10, 15));
  }
};
template <> struct Canonical<bf16s> {
  static __device__ __forceinline__ double get(const uint8_t* at) {
    return __builtin_bit_cast(float, static_cast<uint32_t>(*reinterpret_cast<const uint16_t*>(at)) << 16);
  }
  static __device__ __forceinline__ void put(uint8_t* at, double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const bool nan = (u & 0x7FFFFFFFFFFFFFFFull) > 0x7FF0000000000000ull;  // quiet, the payload's high bits kept
    *reinterpret_cast<uint16_t*>(at) =
        static_cast<uint16_t>(nan ? ((u >> 48) & 0x8000u) | 0x7FC0u | ((u >> 45) & 0x3Fu) : round_to_16(u, 7, 127));
  }
};

// Canonical elements [e0, e0 + count) of a block into the buffer. Scaled weights come out as the
// pixel's effective scale (the tile's scale times its hole factor, one fp32 product as the frame
// kernels form it) times the scaled weight, a product of two floats and exact in double.
template <typename S>
__global__ void __launch_bounds__(kBlock) unpack_kernel(const uint8_t* __restrict__ block, const uint8_t* __restrict__ flags,
                                                        BlockMap b, double* __restrict__ out, uint32_t e0, uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t e = e0 + i, k = e / b.npix, p = e - k * b.npix;
  double v = Canonical<S>::get(block + value_at(b, k, p));
  if constexpr (kScaled<S>) {
    if (k >= b.first_weight) {
      float g = *reinterpret_cast<const float*>(block + b.scale + 4u * (p >> 6));
      if (flags) g = g * hole_factor(flags[p] >> kHoleShift, b.dk);
      v *= static_cast<double>(g);
    }
  }
  out[i] = v;
}

template <typename S>
__global__ void __launch_bounds__(kBlock) pack_state_kernel(uint8_t* __restrict__ block, BlockMap b,
                                                            const double* __restrict__ in, uint32_t e0, uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t e = e0 + i, k = e / b.npix, p = e - k * b.npix;
  Canonical<S>::put(block + value_at(b, k, p), in[i]);
}

__global__ void __launch_bounds__(kBlock) unit_scale_kernel(float* __restrict__ scale, uint32_t tiles64) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < tiles64) scale[i] = 1.f;
}

// List 1 elements [e0, e0 + count): the fused bit of every pixel, then its counter.
__global__ void __launch_bounds__(kBlock) unpack_fuse_kernel(const uint8_t* __restrict__ flags, uint32_t npix,
                                                             double* __restrict__ out, uint32_t e0, uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t e = e0 + i;
  const int v = e < npix ? (flags[e] >> 3) & 1 : static_cast<int>(flags[e - npix] & 7u) - 3;
  out[i] = static_cast<double>(v);
}

// Flags of `count` pixels from their fused bits (in[0 ..)) and counters (in[count ..)); no holes counted.
__global__ void __launch_bounds__(kBlock) pack_fuse_kernel(uint8_t* __restrict__ flags, const double* __restrict__ in,
                                                           uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  flags[i] = static_cast<uint8_t>((static_cast<int>(in[count + i]) + 3) | (static_cast<int>(in[i]) << 3));
}

static inline dim3 blocks_for(uint32_t n) { return dim3((n + kBlock - 1) / kBlock); }

template <typename S>
static hipError_t launch_unpack(const void* block, const uint8_t* flags, const BlockMap& b, double* out, uint32_t e0,
                                uint32_t count, hipStream_t s) {
  unpack_kernel<S><<<blocks_for(count), dim3(kBlock), 0, s>>>(static_cast<const uint8_t*>(block), flags, b, out, e0, count);
  return hipGetLastError();
}

template <typename S>
static hipError_t launch_pack(void* block, const BlockMap& b, const double* in, uint32_t e0, uint32_t count, hipStream_t s) {
  pack_state_kernel<S><<<blocks_for(count), dim3(kBlock), 0, s>>>(static_cast<uint8_t*>(block), b, in, e0, count);
  return hipGetLastError();
}

// The buffer of the current device and the lock of its users. A call holds the lock until its
// stream has drained; it synchronises the stream once before taking it, so that it never waits
// for other work with the lock held.
constexpr int kLocks = 64;
static std::mutex g_io_mu[kLocks];

static hipError_t io_address(double** p) {
  void* a = nullptr;
  const hipError_t e = hipGetSymbolAddress(&a, HIP_SYMBOL(io_buffer));
  *p = static_cast<double*>(a);
  return e == hipSuccess && a == nullptr ? hipErrorInvalidSymbol : e;
}

// One model of a handle: its state block and the shape of its canonical block.
struct Model {
  void* st;
  uint32_t C;
  const ModelConsts* k;
  const uint8_t* flags;  // the pixels' hole counts (depth), or none
};

static int models_of(const gmm_handle* h, Model (&m)[2]) {
  int n = 0;
  if (has_rgb(h)) m[n++] = Model{h->st_rgb, is_augmented(h) ? 4u : 3u, &h->kc, nullptr};
  if (sep_depth(h)) m[n++] = Model{h->st_depth, 1u, &h->kd, h->fstate};
  return n;
}

}  // namespace rgbd

using namespace rgbd;

extern "C" {

gmm_status gmm_read_state(gmm_handle* h, double* host_out, void* stream) {
  if (!h || !host_out) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  DeviceGuard g(h->cfg.device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the handle's device");
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "state copy to host");
  std::lock_guard<std::mutex> lk(g_io_mu[h->cfg.device % kLocks]);
  double* buf = nullptr;
  e = io_address(&buf);
  if (e != hipSuccess) return hip_fail(e, "address of the state I/O buffer");
  const uint32_t n = static_cast<uint32_t>(h->npix), M = static_cast<uint32_t>(h->cfg.M);
  double* o = host_out;
  Model models[2];
  const int nm = models_of(h, models);
  for (int i = 0; i < nm; ++i) {
    const Model& m = models[i];
    const BlockMap b = block_map(h, m.C, *m.k);
    const uint32_t total = (m.C + 2) * M * n;  // < 2^32: the block's bytes are below 2^31
    for (uint32_t e0 = 0; e0 < total && e == hipSuccess; e0 += kChunk) {
      const uint32_t count = std::min(kChunk, total - e0);
      switch (h->cfg.state_dtype) {
        case GMM_F32: e = launch_unpack<float>(m.st, m.flags, b, buf, e0, count, s); break;
        case GMM_F16: e = launch_unpack<f16s>(m.st, m.flags, b, buf, e0, count, s); break;
        default: e = launch_unpack<bf16s>(m.st, m.flags, b, buf, e0, count, s); break;
      }
      if (e == hipSuccess) e = hipMemcpyAsync(o + e0, buf, sizeof(double) * count, hipMemcpyDeviceToHost, s);
    }
    o += total;
  }
  if (sep_both(h)) {
    for (uint32_t e0 = 0; e0 < 2 * n && e == hipSuccess; e0 += kChunk) {
      const uint32_t count = std::min(kChunk, 2 * n - e0);
      unpack_fuse_kernel<<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate, n, buf, e0, count);
      e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(o + e0, buf, sizeof(double) * count, hipMemcpyDeviceToHost, s);
    }
  }
  const hipError_t es = hipStreamSynchronize(s);  // on an error too: nothing may still use the buffer
  if (e == hipSuccess) e = es;
  if (e != hipSuccess) return hip_fail(e, "state copy to host");
  return GMM_OK;
}

gmm_status gmm_write_state(gmm_handle* h, const double* host_in, void* stream) {
  if (!h || !host_in) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  const uint32_t n = static_cast<uint32_t>(h->npix), M = static_cast<uint32_t>(h->cfg.M);
  Model models[2];
  const int nm = models_of(h, models);
  size_t params = 0;
  for (int i = 0; i < nm; ++i) params += static_cast<size_t>(models[i].C + 2) * M * n;
  const double* fuse_in = host_in + params;
  if (sep_both(h)) {  // no early exit and no call: the loop vectorises
    int bad_bit = 0, bad_count = 0;
    for (uint32_t i = 0; i < n; ++i) {
      const double I = fuse_in[i], c = fuse_in[static_cast<size_t>(n) + i];
      const double r = c >= -3.0 && c <= 3.0 ? c : 0.5;  // 0.5: not an integer
      bad_bit |= !(I == 0.0 || I == 1.0);
      bad_count |= r != static_cast<double>(static_cast<int>(r));
    }
    if (bad_bit) return fail(GMM_ERR_INVALID_ARG, "fusion bit I must be 0 or 1");
    if (bad_count) return fail(GMM_ERR_INVALID_ARG, "fusion counter cpt must be an integer in [-3, 3]");
  }
  DeviceGuard g(h->cfg.device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the handle's device");
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "state copy to device");
  std::lock_guard<std::mutex> lk(g_io_mu[h->cfg.device % kLocks]);
  double* buf = nullptr;
  e = io_address(&buf);
  if (e != hipSuccess) return hip_fail(e, "address of the state I/O buffer");
  const double* in = host_in;
  for (int i = 0; i < nm; ++i) {
    const Model& m = models[i];
    const BlockMap b = block_map(h, m.C, *m.k);
    const uint32_t total = (m.C + 2) * M * n;
    for (uint32_t e0 = 0; e0 < total && e == hipSuccess; e0 += kChunk) {
      const uint32_t count = std::min(kChunk, total - e0);
      e = hipMemcpyAsync(buf, in + e0, sizeof(double) * count, hipMemcpyHostToDevice, s);
      if (e != hipSuccess) break;
      switch (h->cfg.state_dtype) {
        case GMM_F32: e = launch_pack<float>(m.st, b, buf, e0, count, s); break;
        case GMM_F16: e = launch_pack<f16s>(m.st, b, buf, e0, count, s); break;
        default: e = launch_pack<bf16s>(m.st, b, buf, e0, count, s); break;
      }
    }
    in += total;
    if (e == hipSuccess && scaled_weights(static_cast<uint32_t>(h->esize))) {  // the weights as written: scale 1
      unit_scale_kernel<<<blocks_for(h->tiles64), dim3(kBlock), 0, s>>>(
          reinterpret_cast<float*>(static_cast<uint8_t*>(m.st) + b.scale), h->tiles64);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = launch_rekey(m.st, h->cfg.state_dtype, h->tiles64, h->cfg.M, static_cast<int>(m.C), s);
  }
  // the flags: List 1 state where there is one, no holes counted
  if (e == hipSuccess && sep_depth(h)) e = launch_fill_u8(h->fstate, kFuseInit, static_cast<int64_t>(h->fuse_bytes), s);
  if (sep_both(h)) {
    constexpr uint32_t half = kChunk / 2;
    for (uint32_t p0 = 0; p0 < n && e == hipSuccess; p0 += half) {
      const uint32_t count = std::min(half, n - p0);
      e = hipMemcpyAsync(buf, fuse_in + p0, sizeof(double) * count, hipMemcpyHostToDevice, s);
      if (e == hipSuccess)
        e = hipMemcpyAsync(buf + count, fuse_in + static_cast<size_t>(n) + p0, sizeof(double) * count, hipMemcpyHostToDevice, s);
      if (e != hipSuccess) break;
      pack_fuse_kernel<<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate + p0, buf, count);
      e = hipGetLastError();
    }
  }
  const hipError_t es = hipStreamSynchronize(s);  // on an error too: nothing may still use the buffer
  if (e == hipSuccess) e = es;
  if (e != hipSuccess) return hip_fail(e, "state copy to device");
  h->last_stream = s;
  return GMM_OK;
}

}  // extern "C"
