// Batched launch for callers that cannot allocate device memory: gmm_batch_apply_static.
//
// gmm_batch_apply keeps each batch's stream descriptors and first tiles in device memory that
// gmm_batch_create allocates. This entry point takes the handles directly and keeps the same
// per-call tables in one file-scope device array instead (`scratch`, below): the descriptors of
// up to kStaticMaxStreams streams and each stream's first tile. They reach the device as kernel
// arguments (pack_descriptors), so no host buffer has to outlive the call, and the batched kernel
// runs on them, so results are bit-identical to gmm_batch_apply.
//
// The array is one per device and shared by every call on that device: calls that overlap on one
// device (different streams, or different host threads without ordering) race on it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "gmm.h"
#include "gmm_batch.hpp"
#include "gmm_internal.hpp"

namespace rgbd {

constexpr int kStaticMaxStreams = GMM_STATIC_MAX_STREAMS;
constexpr size_t kTableBytes = static_cast<size_t>(kStaticMaxStreams) * sizeof(FrameArgs);
constexpr size_t kScratchBytes = (kTableBytes + kStaticMaxStreams * sizeof(uint32_t) + 255) / 256 * 256;
static_assert(kTableBytes % 256 == 0, "the first-tile array starts 256-byte aligned");

// [descriptors: kStaticMaxStreams x FrameArgs][first tile of each stream: kStaticMaxStreams x u32]
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

// The batched kernel on descriptors in its own arguments: one launch instead of two where they fit,
// which saves the pack kernel and the gap behind it. 256 threads a block, one block per piece, no
// byte counting.
template <int M, typename S, int CP>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(M <= 3 ? 6 : 5))) batch_args_kernel(
    PackArgs p, uint32_t tile_px, uint32_t piece_shift) {
  __shared__ uint32_t lds[kWavesPerBlock][48];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const uint32_t b = blockIdx.x, t = b >> piece_shift, piece_px = tile_px >> piece_shift;
  const uint32_t s = find_stream(p.first, p.count, t);
  const FrameArgs a = unpack_entry(p, s);
  const uint32_t t0 = (t - p.first[s]) * tile_px + (b & ((1u << piece_shift) - 1u)) * piece_px;
  process_tile<M, S, kBlock, CP, false>(a, t0, piece_px, lane, lds[wv]);
}

template <int M, typename S>
static hipError_t launch_args_ms(const PackArgs& p, const BatchLaunch& l, hipStream_t s) {
  if (l.stream)
    batch_args_kernel<M, S, kStream><<<dim3(l.grid), dim3(kBlock), l.lds, s>>>(p, l.tile_px, l.piece_shift);
  else
    batch_args_kernel<M, S, kCached><<<dim3(l.grid), dim3(kBlock), l.lds, s>>>(p, l.tile_px, l.piece_shift);
  return hipGetLastError();
}

template <typename S>
static hipError_t launch_args_s(int M, const PackArgs& p, const BatchLaunch& l, hipStream_t s) {
  switch (M) {
    case 1: return launch_args_ms<1, S>(p, l, s);
    case 2: return launch_args_ms<2, S>(p, l, s);
    case 3: return launch_args_ms<3, S>(p, l, s);
    case 4: return launch_args_ms<4, S>(p, l, s);
    case 5: return launch_args_ms<5, S>(p, l, s);
    default: return hipErrorInvalidValue;
  }
}

bool fits_args(const FrameArgs* a, const BatchLaunch& l) {
  if (l.n_streams > static_cast<uint32_t>(kPackPerLaunch) || l.measure || l.block != kBlock ||
      l.grid != l.n_pieces)
    return false;
  for (uint32_t i = 1; i < l.n_streams; ++i)
    if (!same_consts(a[0], a[i])) return false;
  return true;
}

hipError_t launch_batch_args(int M, int dtype, const FrameArgs* a, const uint32_t* first, const BatchLaunch& l,
                             hipStream_t s) {
  const PackArgs p = pack_args(a, first, static_cast<int32_t>(l.n_streams), 0);
  switch (dtype) {
    case GMM_F32: return launch_args_s<float>(M, p, l, s);
    case GMM_F16: return launch_args_s<f16s>(M, p, l, s);
    case GMM_BF16: return launch_args_s<bf16s>(M, p, l, s);
    default: return hipErrorInvalidValue;
  }
}

// Per device: the device address of `scratch` (from hipGetSymbolAddress, taken once with the
// device current; the array's name in host code is not a device address) and the CU count.
constexpr int kMaxDevices = 64;
static std::mutex g_static_mu;
static bool g_static_ready[kMaxDevices];
static uint8_t* g_scratch_ptr[kMaxDevices];
static int g_static_cus[kMaxDevices];

static gmm_status static_setup(int dev, uint8_t** ptr, int* cus) {
  if (dev < 0 || dev >= kMaxDevices) return fail(GMM_ERR_INVALID_ARG, "device ordinal out of range");
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ready[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress of the static scratch array");
    if (p == nullptr) return fail(GMM_ERR_DEVICE, "hipGetSymbolAddress returned NULL for the scratch array");
    int n = 0;
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "CU count");
    g_scratch_ptr[dev] = static_cast<uint8_t*>(p);
    g_static_cus[dev] = n;
    g_static_ready[dev] = true;
  }
  *ptr = g_scratch_ptr[dev];
  *cus = g_static_cus[dev];
  return GMM_OK;
}

}  // namespace rgbd

using namespace rgbd;

extern "C" gmm_status gmm_batch_apply_static(gmm_handle* const* handles, int32_t n, const gmm_stream_io* io,
                                             const gmm_batch_tuning* tuning, void* stream) {
  if (n < 1 || n > kStaticMaxStreams)
    return fail(GMM_ERR_INVALID_ARG, "n must be in 1.." + std::to_string(kStaticMaxStreams) +
                                         " (the size of the static descriptor table)");
  if (!handles || !io) return fail(GMM_ERR_INVALID_ARG, "NULL handles or io");
  const gmm_batch_tuning t = tuning ? *tuning : kDefaultTuning;
  if (t.block_threads != 256 && t.block_threads != 512)
    return fail(GMM_ERR_INVALID_ARG, "block_threads must be 256 or 512");
  if (t.tile_pixels < t.block_threads || t.tile_pixels % t.block_threads || t.tile_pixels > 64 * t.block_threads)
    return fail(GMM_ERR_INVALID_ARG, "tile_pixels must be a multiple of block_threads, at most 64x it");
  if (t.blocks_per_cu < 1 || t.blocks_per_cu > 32) return fail(GMM_ERR_INVALID_ARG, "blocks_per_cu must be in 1..32");
  // every handle once (a handle twice would race inside the launch): sorted copy on the stack
  const gmm_handle* sorted[kStaticMaxStreams];
  for (int32_t i = 0; i < n; ++i) {
    const gmm_handle* h = handles[i];
    if (!h) return fail(GMM_ERR_INVALID_ARG, "NULL handle");
    if (is_augmented(h)) return fail(GMM_ERR_UNSUPPORTED, "augmented handles run one at a time");
    if (h->cfg.device != handles[0]->cfg.device || h->cfg.M != handles[0]->cfg.M ||
        h->cfg.state_dtype != handles[0]->cfg.state_dtype)
      return fail(GMM_ERR_INVALID_ARG, "all handles need the same device, M and state dtype");
    sorted[i] = h;
  }
  std::sort(sorted, sorted + n);
  for (int32_t i = 1; i < n; ++i)
    if (sorted[i] == sorted[i - 1]) return fail(GMM_ERR_INVALID_ARG, "a handle appears twice");
  uint64_t total = 0, pixels = 0;
  for (int32_t i = 0; i < n; ++i) {
    gmm_handle* h = handles[i];
    const gmm_stream_io& s = io[i];
    gmm_status st = check_frame_args(h, s.rgb, s.rgb_pitch_bytes, s.depth, s.depth_pitch_bytes, s.fg_rgb, s.fg_depth);
    if (st != GMM_OK) {
      set_error("stream " + std::to_string(i) + ": " + gmm_last_error());
      return st;
    }
    if (s.fused) {
      if (!has_both(h)) return fail(GMM_ERR_STATE, "stream " + std::to_string(i) + ": fusion needs both modalities");
      if (reinterpret_cast<uintptr_t>(s.fused) % 8)
        return fail(GMM_ERR_INVALID_ARG, "stream " + std::to_string(i) + ": fused mask not 8-byte aligned");
    }
    total += (static_cast<uint64_t>(h->npix) + t.tile_pixels - 1) / t.tile_pixels;
    pixels += static_cast<uint64_t>(h->npix);
  }
  if (total >= (1ull << 31)) return fail(GMM_ERR_INVALID_ARG, "too many tiles in one launch");
  const int dev = handles[0]->cfg.device;
  DeviceGuard g(dev);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the handles' device");
  uint8_t* base = nullptr;
  int cus = 0;
  gmm_status st = static_setup(dev, &base, &cus);
  if (st != GMM_OK) return st;
  FrameArgs* table = reinterpret_cast<FrameArgs*>(base);
  uint32_t* first = reinterpret_cast<uint32_t*>(base + kTableBytes);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e = hipSuccess;
  uint32_t next_first = 0;
  BatchLaunch l = batch_launch(t, static_cast<uint32_t>(total), pixels, cus);
  l.table = table;
  l.first = first;
  l.n_streams = static_cast<uint32_t>(n);
  l.stream = streams_rows(handles, static_cast<size_t>(n));
  bool packed = true;
  for (int32_t b = 0; b < n && e == hipSuccess; b += kPackPerLaunch) {
    FrameArgs a[kPackPerLaunch];
    uint32_t f[kPackPerLaunch];
    const int32_t count = std::min(kPackPerLaunch, n - b);
    for (int32_t i = 0; i < count; ++i) {
      gmm_handle* h = handles[b + i];
      const gmm_stream_io& s = io[b + i];
      a[i] = frame_args(h, s.rgb, s.rgb_pitch_bytes, s.depth, s.depth_pitch_bytes, s.fg_rgb, s.fg_depth, s.fused);
      l.measure = l.measure || a[i].wave_bytes != nullptr;
      f[i] = next_first;
      next_first += static_cast<uint32_t>((h->npix + t.tile_pixels - 1) / t.tile_pixels);
    }
    if (count == n && fits_args(a, l)) {
      packed = false;
      e = launch_batch_args(handles[0]->cfg.M, handles[0]->cfg.state_dtype, a, f, l, hs);
    } else {
      e = pack_descriptors(a, f, count, table + b, first + b, hs);
    }
  }
  if (e == hipSuccess && packed) e = launch_batch(handles[0]->cfg.M, handles[0]->cfg.state_dtype, l, hs);
  if (e != hipSuccess) return hip_fail(e, "static batch kernel launch");
  for (int32_t i = 0; i < n; ++i) handles[i]->last_stream = hs;
  return GMM_OK;
}
