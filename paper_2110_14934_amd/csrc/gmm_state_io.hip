// State I/O: the device layout of a handle's state to and from the canonical float64 layout
// (gmm_read_state, gmm_write_state), converted on the device.
//
// A value's place in the device layout is affine in its pixel's tile and lane (ValueMap), so one
// lane per canonical element moves it: canonical elements are contiguous (a wave reads or writes
// 512 B), the state side is 4- or 2-byte pieces at the row's or the suffix's lane stride, merged
// in the caches. What bounds the call is the host side: the canonical state (336 B per pixel of a
// paired stream at M = 5) crosses the link and is written to pageable memory. The elements go
// through a static device buffer, a piece at a time, so a call allocates nothing and cannot run out of
// device memory. A call alone has 8 MB of it, where the pageable copies stop getting faster: a write
// and a read of a 320x240 paired stream (M = 5, fp32; 25.8 MB each way) take 2.53 ms, in pieces of 4 MB
// 2.74. The conversion used to run on one host thread, value by value: with a frame between them they
// took 49.5 ms and take 2.6.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <condition_variable>
#include <mutex>

#include "gmm.h"
#include "gmm_internal.hpp"

namespace rgbd {

constexpr uint32_t kSegment = 1u << 17;  // canonical elements
constexpr uint32_t kSegments = 16;
static __device__ __align__(256) double io_buffer[kSegments * kSegment];

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

// List 1 elements: the fused bits (BIT) or the counters of pixels [p0, p0 + count).
template <bool BIT>
__global__ void __launch_bounds__(kBlock) unpack_fuse_kernel(const uint8_t* __restrict__ flags, double* __restrict__ out,
                                                             uint32_t p0, uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t f = flags[p0 + i];
  out[i] = static_cast<double>(BIT ? static_cast<int>((f >> 3) & 1u) : static_cast<int>(f & 7u) - 3);
}

template <bool BIT>
__global__ void __launch_bounds__(kBlock) pack_fuse_kernel(uint8_t* __restrict__ flags, const double* __restrict__ in,
                                                           uint32_t p0, uint32_t count) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count) return;
  const uint32_t f = flags[p0 + i];
  const int v = static_cast<int>(in[i]);
  flags[p0 + i] = static_cast<uint8_t>(BIT ? (f & ~8u) | static_cast<uint32_t>(v) << 3 : (f & ~7u) | static_cast<uint32_t>(v + 3));
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

// A call's part of the current device's buffer: adjacent segments, as many as its `elements` fill, but
// at most half of those that are free, given back when the call ends. A call synchronises its stream
// before it takes them, so that it never waits for other work while others wait for it, and again
// before it gives them back. A call waits only when all segments are taken. 16 threads, a write and a
// read of a 64x48 state each: 0.77 ms; 3.9 with one buffer and a lock, 2.4 when each converted on the
// host. Of a 640x480 state: 59, 229 and 268 ms.
constexpr int kDevices = 64;
struct Segments {
  std::mutex mu;
  std::condition_variable given_back;
  uint32_t used = 0;  // a bit per segment
};
static Segments g_io[kDevices];

class IoSegments {
 public:
  IoSegments(int device, uint64_t elements) : io_(g_io[device % kDevices]) {
    constexpr uint32_t kAll = (1u << kSegments) - 1u;
    std::unique_lock<std::mutex> lk(io_.mu);
    io_.given_back.wait(lk, [&] { return io_.used != kAll; });
    const uint32_t half = std::max(1, __builtin_popcount(kAll & ~io_.used) / 2);
    for (uint32_t n = static_cast<uint32_t>(std::min<uint64_t>(half, (elements + kSegment - 1) / kSegment)); mask_ == 0; --n)
      for (uint32_t at = 0; at + n <= kSegments && mask_ == 0; ++at) {
        const uint32_t m = ((1u << n) - 1u) << at;
        if (io_.used & m) continue;
        mask_ = m;
        first_ = at;
        count_ = n;
      }
    io_.used |= mask_;
  }
  ~IoSegments() {
    {
      std::lock_guard<std::mutex> lk(io_.mu);
      io_.used &= ~mask_;
    }
    io_.given_back.notify_all();
  }
  IoSegments(const IoSegments&) = delete;
  IoSegments& operator=(const IoSegments&) = delete;
  double* in(double* buffer) const { return buffer + static_cast<size_t>(first_) * kSegment; }
  uint32_t elements() const { return count_ * kSegment; }

 private:
  Segments& io_;
  uint32_t mask_ = 0, first_ = 0, count_ = 0;
};

static hipError_t io_address(double** p) {
  void* a = nullptr;
  const hipError_t e = hipGetSymbolAddress(&a, HIP_SYMBOL(io_buffer));
  *p = static_cast<double*>(a);
  return e == hipSuccess && a == nullptr ? hipErrorInvalidSymbol : e;
}

// A part of a handle's canonical state: a model's block, or the fused bits or the counters of List 1.
struct Part {
  enum Kind { kModel, kBits, kCounters } kind;
  uint64_t count;  // elements
  void* st;        // a model's state block and the rest of it
  uint32_t C;
  const ModelConsts* k;
  const uint8_t* flags;  // the pixels' hole counts (depth), or none
  BlockMap map;
};
constexpr int kMaxParts = 4;

// The parts of a handle's canonical state, in its order.
static int parts_of(const gmm_handle* h, Part (&p)[kMaxParts]) {
  const uint64_t n = static_cast<uint64_t>(h->npix), M = static_cast<uint64_t>(h->cfg.M);
  int c = 0;
  const auto model = [&](void* st, uint32_t C, const ModelConsts& k, const uint8_t* flags) {
    p[c++] = Part{Part::kModel, (C + 2) * M * n, st, C, &k, flags, block_map(h, C, k)};
  };
  if (has_rgb(h)) model(h->st_rgb, is_augmented(h) ? 4u : 3u, h->kc, nullptr);
  if (sep_depth(h)) model(h->st_depth, 1u, h->kd, h->fstate);
  if (sep_both(h)) {
    p[c++] = Part{Part::kBits, n, nullptr, 0, nullptr, nullptr, {}};
    p[c++] = Part{Part::kCounters, n, nullptr, 0, nullptr, nullptr, {}};
  }
  return c;
}

static uint64_t elements_of(const Part* p, int n) {
  uint64_t total = 0;
  for (int i = 0; i < n; ++i) total += p[i].count;
  return total;
}

// Elements [e0, e0 + count) of a part into `out`.
static hipError_t unpack_part(const gmm_handle* h, const Part& p, double* out, uint32_t e0, uint32_t count, hipStream_t s) {
  if (p.kind == Part::kModel) {
    switch (h->cfg.state_dtype) {
      case GMM_F32: return launch_unpack<float>(p.st, p.flags, p.map, out, e0, count, s);
      case GMM_F16: return launch_unpack<f16s>(p.st, p.flags, p.map, out, e0, count, s);
      default: return launch_unpack<bf16s>(p.st, p.flags, p.map, out, e0, count, s);
    }
  }
  if (p.kind == Part::kBits)
    unpack_fuse_kernel<true><<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate, out, e0, count);
  else
    unpack_fuse_kernel<false><<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate, out, e0, count);
  return hipGetLastError();
}

static hipError_t pack_part(const gmm_handle* h, const Part& p, const double* in, uint32_t e0, uint32_t count, hipStream_t s) {
  if (p.kind == Part::kModel) {
    switch (h->cfg.state_dtype) {
      case GMM_F32: return launch_pack<float>(p.st, p.map, in, e0, count, s);
      case GMM_F16: return launch_pack<f16s>(p.st, p.map, in, e0, count, s);
      default: return launch_pack<bf16s>(p.st, p.map, in, e0, count, s);
    }
  }
  if (p.kind == Part::kBits)
    pack_fuse_kernel<true><<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate, in, e0, count);
  else
    pack_fuse_kernel<false><<<blocks_for(count), dim3(kBlock), 0, s>>>(h->fstate, in, e0, count);
  return hipGetLastError();
}

// fn(part, first element in the part, element in the piece, count) for every part that elements
// [e0, e0 + count) of the canonical state touch; stops at the first error.
template <typename F>
static hipError_t each_part(const Part* p, int n, uint64_t e0, uint64_t count, F fn) {
  hipError_t e = hipSuccess;
  uint64_t at = 0;
  for (int i = 0; i < n && e == hipSuccess; at += p[i].count, ++i) {
    const uint64_t a = std::max(at, e0), b = std::min(at + p[i].count, e0 + count);
    if (a < b) e = fn(p[i], static_cast<uint32_t>(a - at), static_cast<size_t>(a - e0), static_cast<uint32_t>(b - a));
  }
  return e;
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
  double* buf = nullptr;
  e = io_address(&buf);
  if (e != hipSuccess) return hip_fail(e, "address of the state I/O buffer");
  Part parts[kMaxParts];
  const int n = parts_of(h, parts);
  const uint64_t total = elements_of(parts, n);
  const IoSegments io(h->cfg.device, total);
  buf = io.in(buf);
  for (uint64_t e0 = 0; e0 < total && e == hipSuccess; e0 += io.elements()) {
    const uint64_t count = std::min<uint64_t>(io.elements(), total - e0);
    e = each_part(parts, n, e0, count, [&](const Part& p, uint32_t at, size_t to, uint32_t c) {
      return unpack_part(h, p, buf + to, at, c, s);
    });
    if (e == hipSuccess) e = hipMemcpyAsync(host_out + e0, buf, sizeof(double) * count, hipMemcpyDeviceToHost, s);
  }
  const hipError_t es = hipStreamSynchronize(s);  // on an error too: nothing may still use the buffer
  if (e == hipSuccess) e = es;
  if (e != hipSuccess) return hip_fail(e, "state copy to host");
  return GMM_OK;
}

gmm_status gmm_write_state(gmm_handle* h, const double* host_in, void* stream) {
  if (!h || !host_in) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  Part parts[kMaxParts];
  const int n = parts_of(h, parts);
  const uint64_t total = elements_of(parts, n);
  if (sep_both(h)) {  // no early exit and no call: the loop vectorises
    const size_t npix = static_cast<size_t>(h->npix);
    const double* fuse_in = host_in + (total - 2 * npix);
    int bad_bit = 0, bad_count = 0;
    for (size_t i = 0; i < npix; ++i) {
      const double I = fuse_in[i], c = fuse_in[npix + i];
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
  double* buf = nullptr;
  e = io_address(&buf);
  if (e != hipSuccess) return hip_fail(e, "address of the state I/O buffer");
  const IoSegments io(h->cfg.device, total);
  buf = io.in(buf);
  // no holes counted; List 1 state, where there is one, with the elements below
  if (sep_depth(h)) e = launch_fill_u8(h->fstate, kFuseInit, static_cast<int64_t>(h->fuse_bytes), s);
  for (uint64_t e0 = 0; e0 < total && e == hipSuccess; e0 += io.elements()) {
    const uint64_t count = std::min<uint64_t>(io.elements(), total - e0);
    e = hipMemcpyAsync(buf, host_in + e0, sizeof(double) * count, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = each_part(parts, n, e0, count, [&](const Part& p, uint32_t at, size_t from, uint32_t c) {
        return pack_part(h, p, buf + from, at, c, s);
      });
  }
  for (int i = 0; i < n && e == hipSuccess; ++i) {
    const Part& p = parts[i];
    if (p.kind != Part::kModel) continue;
    if (scaled_weights(static_cast<uint32_t>(h->esize))) {  // the weights as written: scale 1
      unit_scale_kernel<<<blocks_for(h->tiles64), dim3(kBlock), 0, s>>>(
          reinterpret_cast<float*>(static_cast<uint8_t*>(p.st) + p.map.scale), h->tiles64);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = launch_rekey(p.st, h->cfg.state_dtype, h->tiles64, h->cfg.M, static_cast<int>(p.C), s);
  }
  const hipError_t es = hipStreamSynchronize(s);  // on an error too: nothing may still use the buffer
  if (e == hipSuccess) e = es;
  if (e != hipSuccess) return hip_fail(e, "state copy to device");
  h->last_stream = s;
  return GMM_OK;
}

}  // extern "C"
