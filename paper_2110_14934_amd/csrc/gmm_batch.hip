// Batched path: every stream of a batch advances one frame in ONE launch.
//
// Work is cut into tiles of `tile_pixels` consecutive pixels of one stream (a multiple of the
// block size, so tiles start on mask-word boundaries). Per-stream kernel arguments (frame and mask
// pointers, state blocks, constants) live in a device descriptor table with one slot per prepared
// frame-set, each stream's first tile in an array beside it that a block searches for the stream
// of its tile. The per-pixel body is the one
// the single-stream kernel uses (process_pixel), so results are bit-identical to one launch per
// stream.
//
// A launch reads only device memory prepared earlier (descriptor slot, first tiles): it allocates
// nothing and synchronises nothing, so it can be captured into a hipGraph and replayed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <sstream>
#include <string>
#include <tuple>
#include <vector>

#include "gmm.h"
#include "gmm_batch.hpp"
#include "gmm_frame.hpp"
#include "gmm_internal.hpp"

namespace rgbd {

// Five waves per SIMD, six at M <= 3: the body fits them without spilling (checked at build time by
// the tests). At M = 3 in fp32 it would have five, at 82 registers: 24 streams of 160x120 8.74 us with
// five and 8.40 with six, 4 VGA streams 16.3 and 15.9, 96 VGA streams 410 and 394. At M = 1 and 2 and in
// 16-bit state it has six or more anyway, and nothing changes (96 VGA streams, M = 2, fp32: 399 us).
// A block takes one piece of a tile (tile_px >> piece_shift pixels) and the grid usually has a
// block for every piece (batch_launch below); a smaller grid walks the pieces b, b+G, b+2G, ...
// CP: the cache policy of the rows (kCached or kStream; streams_rows).
// MEASURE: the body that adds each wave's state bytes to the streams' traffic records; the launch
// takes it (with kStream) only when a stream of the batch has one, so the common body never forms
// the counts.
template <int M, typename S, int BLOCK, int CP, bool MEASURE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(M <= 3 ? 6 : 5))) batch_kernel(const FrameArgs* __restrict__ table,
                                                      const uint32_t* __restrict__ first, uint32_t n_streams,
                                                      uint32_t n_pieces, uint32_t tile_px, uint32_t piece_shift) {
  __shared__ uint32_t lds[BLOCK / kWave][48];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const uint32_t piece_px = tile_px >> piece_shift, part_mask = (1u << piece_shift) - 1u;
  for (uint32_t b = blockIdx.x; b < n_pieces; b += gridDim.x) {
    const uint32_t t = b >> piece_shift;
    const uint32_t s = find_stream(first, n_streams, t);
    const FrameArgs a = table[s];
    const uint32_t t0 = (t - first[s]) * tile_px + (b & part_mask) * piece_px;
    process_tile<M, S, BLOCK, CP, MEASURE>(a, t0, piece_px, lane, lds[wv]);
  }
}

template <int M, typename S, int CP, bool MEASURE>
static hipError_t launch_batch_mscm(const BatchLaunch& l, hipStream_t s) {
  const dim3 grid(l.grid);
  if (l.block == 256)
    batch_kernel<M, S, 256, CP, MEASURE><<<grid, dim3(256), l.lds, s>>>(l.table, l.first, l.n_streams, l.n_pieces, l.tile_px, l.piece_shift);
  else if (l.block == 512)
    batch_kernel<M, S, 512, CP, MEASURE><<<grid, dim3(512), l.lds, s>>>(l.table, l.first, l.n_streams, l.n_pieces, l.tile_px, l.piece_shift);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int M, typename S>
static hipError_t launch_batch_ms(const BatchLaunch& l, hipStream_t s) {
  if (l.measure) return launch_batch_mscm<M, S, kStream, true>(l, s);
  return l.stream ? launch_batch_mscm<M, S, kStream, false>(l, s) : launch_batch_mscm<M, S, kCached, false>(l, s);
}

template <typename S>
static hipError_t launch_batch_s(int M, const BatchLaunch& l, hipStream_t s) {
  switch (M) {
    case 1: return launch_batch_ms<1, S>(l, s);
    case 2: return launch_batch_ms<2, S>(l, s);
    case 3: return launch_batch_ms<3, S>(l, s);
    case 4: return launch_batch_ms<4, S>(l, s);
    case 5: return launch_batch_ms<5, S>(l, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch(int M, int dtype, const BatchLaunch& l, hipStream_t s) {
  switch (dtype) {
    case GMM_F32: return launch_batch_s<float>(M, l, s);
    case GMM_F16: return launch_batch_s<f16s>(M, l, s);
    case GMM_BF16: return launch_batch_s<bf16s>(M, l, s);
    default: return hipErrorInvalidValue;
  }
}

// Grid: with as many blocks per CU as a CU can hold (2048 threads) or more, one block per piece:
// the dispatcher then hands the next piece to whichever CU is free, where blocks walking fixed
// pieces wait for the slowest (64 uneven fp32 streams, M = 5: 360 us walking 1024-pixel tiles with 8 blocks per
// CU, 315 us one block per tile). Fewer blocks per CU walk.
// Pieces: a launch of the default shape, which leaves it to the library (is_open), cuts the default tiles of 1024 pixels into
// pieces of 512, or of 256 when all pixels together are few (kSmallBatchPixels): larger pieces
// spread a block's start (the search, the descriptor) over more pixels, smaller ones leave a
// shorter chain in each wave and an evener end. Pieces of 256 / 512 / 1024 pixels: 64 uneven fp32
// streams (29 M pixels) 338 / 312 / 318 us, 32 VGA fp16 streams (9.8 M pixels) 145 / 140 / 147
// us. Where the line lies, in rows that stay in the caches: 6 VGA streams (1.8 M) M = 5 fp32 24.6 / 23.2 /
// 24.4, fp16 21.8 / 21.9 / 23.3, M = 3 fp32 22.9 / 22.9 / 25.4; 4 VGA (1.2 M) M = 5 fp32 17.0 / 16.6 / 16.7,
// M = 3 fp32 16.1 / 15.7 / 15.7, fp16 13.3 / 12.8 / 13.8; 3 VGA (0.9 M) M = 5 fp32 13.6 / 13.3 / 13.2, fp16 12.8 /
// 13.3 / 13.6, M = 3 fp32 12.8 / 13.6 / 13.0; 2 of 320x240 (0.15 M) M = 5 fp32 5.0 / 6.1 / 8.8, M = 3 fp16 4.2 /
// 5.0 / 7.0.
constexpr uint64_t kSmallBatchPixels = uint64_t(1) << 20;
constexpr uint32_t kMaxGrid = 1u << 22;  // blocks, so that grid x block stays below 2^32 threads

BatchLaunch batch_launch(const gmm_batch_tuning& t, uint32_t n_tiles, uint64_t pixels, int cu_count) {
  BatchLaunch l{};
  l.block = t.block_threads;
  l.tile_px = static_cast<uint32_t>(t.tile_pixels);
  l.piece_shift = !is_open(t) || n_tiles >= (1u << 28) ? 0u : (pixels < kSmallBatchPixels ? 2u : 1u);
  l.n_pieces = n_tiles << l.piece_shift;
  const uint32_t want = walks(t) ? static_cast<uint32_t>(t.blocks_per_cu) * static_cast<uint32_t>(cu_count) : kMaxGrid;
  l.grid = std::max(1u, std::min(want, l.n_pieces));
  return l;
}

// Ticks that read frames over the host link (gmm_exec_launch) keep the caller's blocks per CU by what
// a CU has room for, not by a grid of walking blocks: the dispatcher then gives the next piece to the
// CU that is free, where a walking block whose loads come back late holds up all its pieces. The room
// is LDS: each block reserves so much that no more than `blocks` fit. Ticks of 32 VGA fp16 streams and
// of 16 fp32 ones with 4 blocks of 256 threads per CU: 1169 and 614 us walking, 1069 and 552 us so.
void limit_residency(BatchLaunch& l, uint32_t blocks) {
  constexpr uint32_t kLdsPerCu = 160u << 10, kGrain = 1280;
  const uint32_t own = static_cast<uint32_t>(l.block) / kWave * 48u * 4u;
  l.grid = std::min(kMaxGrid, l.n_pieces);
  l.lds = (kLdsPerCu / (blocks + 1) / kGrain + 1) * kGrain - own;
}

struct PackWholeArgs {
  FrameArgs a[kPackPerLaunch / 2];
  uint32_t first[kPackPerLaunch / 2];
  uint32_t base, count;
};
static_assert(sizeof(PackWholeArgs) + 2 * sizeof(void*) <= 4096, "kernel arguments");

// A launch costs its latency (~1.7 us on the GPU, ~3.5 us of the caller's time), so what counts is
// how many there are: 24 small streams take one (three of 8 whole descriptors before: 25.2 -> 21.4
// us a static call). `first` may be NULL.
__global__ void __launch_bounds__(64) pack_kernel(PackArgs p, FrameArgs* __restrict__ table,
                                                  uint32_t* __restrict__ first) {
  const uint32_t i = threadIdx.x;
  if (i >= p.count) return;
  table[p.base + i] = unpack_entry(p, i);
  if (first) first[p.base + i] = p.first[i];
}

__global__ void __launch_bounds__(64) pack_whole_kernel(PackWholeArgs p, FrameArgs* __restrict__ table,
                                                        uint32_t* __restrict__ first) {
  const uint32_t i = threadIdx.x;
  if (i >= p.count) return;
  table[p.base + i] = p.a[i];
  if (first) first[p.base + i] = p.first[i];
}

hipError_t pack_descriptors(const FrameArgs* a, const uint32_t* first, int32_t n, FrameArgs* d_table, uint32_t* d_first,
                            hipStream_t s) {
  hipError_t e = hipSuccess;
  for (int32_t b = 0; b < n && e == hipSuccess;) {
    int32_t same = 1;  // streams from b on with b's constants
    while (same < kPackPerLaunch && b + same < n && same_consts(a[b], a[b + same]))
      ++same;
    if (same >= kPackPerLaunch / 2 || b + same == n) {
      pack_kernel<<<1, 64, 0, s>>>(pack_args(a + b, first ? first + b : nullptr, same, static_cast<uint32_t>(b)), d_table, d_first);
      b += same;
    } else {
      PackWholeArgs p{};
      p.base = static_cast<uint32_t>(b);
      p.count = static_cast<uint32_t>(std::min(kPackPerLaunch / 2, n - b));
      for (uint32_t i = 0; i < p.count; ++i) {
        p.a[i] = a[b + static_cast<int32_t>(i)];
        if (first) p.first[i] = first[b + static_cast<int32_t>(i)];
      }
      pack_whole_kernel<<<1, 64, 0, s>>>(p, d_table, d_first);
      b += static_cast<int32_t>(p.count);
    }
    e = hipGetLastError();
  }
  return e;
}

// Tunings found by the autotuner, per (device, M, dtype, stream mix), for this process.
static std::mutex g_tune_mu;
static std::map<std::string, std::pair<gmm_batch_tuning, double>> g_tune_cache;

}  // namespace rgbd

using namespace rgbd;

struct gmm_batch {
  int device = 0;
  int M = 0;
  int dtype = 0;
  int cu_count = 0;
  std::vector<gmm_handle*> handles;
  int n_slots = 0;
  FrameArgs* d_table = nullptr;              // n_slots x n descriptors
  std::vector<FrameArgs*> h_staging;         // pinned, one per slot (n > kPackStreams)
  std::vector<hipEvent_t> staging_done;      // last upload from each staging buffer
  std::vector<uint8_t> slot_ready;
  std::vector<uint8_t> slot_measure;         // a stream of the slot's descriptors has a traffic record
  uint32_t* d_first_tile = nullptr;
  uint32_t n_tiles = 0;
  uint64_t pixels = 0;                       // of one frame of every stream
  gmm_batch_tuning tuning = kDefaultTuning;
  hipStream_t last_stream = nullptr;
};

static size_t n_streams(const gmm_batch* b) { return b->handles.size(); }

static gmm_status validate_tuning(const gmm_batch_tuning* t) {
  if (!t) return fail(GMM_ERR_INVALID_ARG, "tuning is NULL");
  if (t->block_threads != 256 && t->block_threads != 512)
    return fail(GMM_ERR_INVALID_ARG, "block_threads must be 256 or 512");
  if (t->tile_pixels < t->block_threads || t->tile_pixels % t->block_threads ||
      t->tile_pixels > 64 * t->block_threads)
    return fail(GMM_ERR_INVALID_ARG, "tile_pixels must be a multiple of block_threads, at most 64x it");
  if (t->blocks_per_cu < 1 || t->blocks_per_cu > 32) return fail(GMM_ERR_INVALID_ARG, "blocks_per_cu must be in 1..32");
  return GMM_OK;
}

static uint32_t count_tiles(const gmm_batch* b, uint32_t tile_px) {
  uint64_t total = 0;
  for (const auto* h : b->handles) total += (static_cast<uint64_t>(h->npix) + tile_px - 1) / tile_px;
  return static_cast<uint32_t>(std::min<uint64_t>(total, UINT32_MAX));
}

// First tiles for tile size `tile_px` (synchronous; not for use under capture).
static gmm_status build_tiles(gmm_batch* b, uint32_t tile_px) {
  std::vector<uint32_t> first(n_streams(b));
  uint64_t total = 0;
  b->pixels = 0;
  for (size_t i = 0; i < n_streams(b); ++i) {
    first[i] = static_cast<uint32_t>(total);
    total += (static_cast<uint64_t>(b->handles[i]->npix) + tile_px - 1) / tile_px;
    b->pixels += static_cast<uint64_t>(b->handles[i]->npix);
  }
  if (total >= (1ull << 31)) return fail(GMM_ERR_INVALID_ARG, "too many tiles in one batch");
  const hipError_t e = hipMemcpy(b->d_first_tile, first.data(), first.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "first tile upload");
  b->n_tiles = static_cast<uint32_t>(total);
  return GMM_OK;
}

static gmm_status apply_tuning(gmm_batch* b, const gmm_batch_tuning& t) {
  if (t.tile_pixels != b->tuning.tile_pixels || b->n_tiles == 0) {
    gmm_status st = build_tiles(b, static_cast<uint32_t>(t.tile_pixels));
    if (st != GMM_OK) return st;
  }
  b->tuning = t;
  return GMM_OK;
}

static hipError_t run_slot(gmm_batch* b, int slot, hipStream_t s) {
  BatchLaunch l = batch_launch(b->tuning, b->n_tiles, b->pixels, b->cu_count);
  l.table = b->d_table + static_cast<size_t>(slot) * n_streams(b);
  l.first = b->d_first_tile;
  l.n_streams = static_cast<uint32_t>(n_streams(b));
  l.measure = b->slot_measure[slot] != 0;
  l.stream = streams_rows(b->handles.data(), n_streams(b));
  return launch_batch(b->M, b->dtype, l, s);
}

static void free_batch(gmm_batch* b) {
  for (auto* p : b->h_staging)
    if (p) (void)hipHostFree(p);
  for (auto ev : b->staging_done)
    if (ev) (void)hipEventDestroy(ev);
  if (b->d_table) (void)hipFree(b->d_table);
  if (b->d_first_tile) (void)hipFree(b->d_first_tile);
  delete b;
}

static std::string mix_key(const gmm_batch* b) {
  hipDeviceProp_t prop;
  std::ostringstream k;
  if (hipGetDeviceProperties(&prop, b->device) == hipSuccess) k << prop.gcnArchName << "/" << prop.multiProcessorCount;
  k << "|M" << b->M << "|d" << b->dtype;
  std::vector<std::string> parts;
  for (auto* h : b->handles) {
    std::ostringstream s;
    s << h->cfg.width << "x" << h->cfg.height << "m" << h->cfg.modalities;
    parts.push_back(s.str());
  }
  std::sort(parts.begin(), parts.end());
  for (auto& p : parts) k << "|" << p;
  return k.str();
}

extern "C" {

gmm_status gmm_batch_create(gmm_handle* const* handles, int32_t n, int32_t n_slots, gmm_batch** out) {
  if (!out) return fail(GMM_ERR_INVALID_ARG, "out is NULL");
  if (!handles || n <= 0) return fail(GMM_ERR_INVALID_ARG, "a batch needs at least one handle");
  if (n_slots < 1 || n_slots > 4096) return fail(GMM_ERR_INVALID_ARG, "n_slots must be in 1..4096");
  std::set<const gmm_handle*> seen;
  for (int32_t i = 0; i < n; ++i) {
    const gmm_handle* h = handles[i];
    if (!h) return fail(GMM_ERR_INVALID_ARG, "NULL handle in batch");
    if (!seen.insert(h).second) return fail(GMM_ERR_INVALID_ARG, "a handle appears twice in the batch");
    if (is_augmented(h)) return fail(GMM_ERR_UNSUPPORTED, "augmented handles run one at a time");
    if (h->cfg.device != handles[0]->cfg.device || h->cfg.M != handles[0]->cfg.M ||
        h->cfg.state_dtype != handles[0]->cfg.state_dtype)
      return fail(GMM_ERR_INVALID_ARG, "all handles of a batch need the same device, M and state dtype");
  }
  gmm_batch* b = new (std::nothrow) gmm_batch();
  if (!b) return fail(GMM_ERR_OUT_OF_MEMORY, "host allocation of the batch failed");
  b->handles.assign(handles, handles + n);
  b->device = handles[0]->cfg.device;
  b->M = handles[0]->cfg.M;
  b->dtype = handles[0]->cfg.state_dtype;
  b->n_slots = n_slots;
  DeviceGuard g(b->device);
  if (!g.ok()) {
    delete b;
    return fail(GMM_ERR_DEVICE, "cannot select the handles' device");
  }
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, b->device);
  if (e != hipSuccess) {
    delete b;
    return hip_fail(e, "hipGetDeviceProperties");
  }
  b->cu_count = prop.multiProcessorCount;
  const size_t tbytes = static_cast<size_t>(n_slots) * n * sizeof(FrameArgs);
  e = hipMalloc(&b->d_table, tbytes);
  if (e == hipSuccess) e = hipMalloc(&b->d_first_tile, static_cast<size_t>(n) * sizeof(uint32_t));
  if (e != hipSuccess) {
    free_batch(b);
    return fail(GMM_ERR_OUT_OF_MEMORY, "device allocation of the batch tables failed");
  }
  const bool pack = n_streams(b) <= kPackStreams;
  b->h_staging.assign(pack ? 0 : n_slots, nullptr);
  b->staging_done.assign(pack ? 0 : n_slots, nullptr);
  b->slot_ready.assign(n_slots, 0);
  b->slot_measure.assign(n_slots, 0);
  for (size_t s = 0; s < b->h_staging.size(); ++s) {
    e = hipHostMalloc(reinterpret_cast<void**>(&b->h_staging[s]), static_cast<size_t>(n) * sizeof(FrameArgs),
                      hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&b->staging_done[s], hipEventDisableTiming);
    if (e != hipSuccess) {
      free_batch(b);
      return fail(GMM_ERR_OUT_OF_MEMORY, "pinned staging allocation failed");
    }
  }
  gmm_status st = build_tiles(b, static_cast<uint32_t>(b->tuning.tile_pixels));
  if (st != GMM_OK) {
    free_batch(b);
    return st;
  }
  *out = b;
  return GMM_OK;
}

gmm_status gmm_batch_destroy(gmm_batch* b) {
  if (!b) return GMM_OK;
  gmm_status st = GMM_OK;
  {
    DeviceGuard g(b->device);
    hipError_t e = hipStreamSynchronize(b->last_stream);
    if (e != hipSuccess) st = hip_fail(e, "hipStreamSynchronize in batch destroy");
    for (auto ev : b->staging_done) (void)hipEventSynchronize(ev);
    free_batch(b);
  }
  return st;
}

gmm_status gmm_batch_set_tuning(gmm_batch* b, const gmm_batch_tuning* t) {
  if (!b) return fail(GMM_ERR_INVALID_ARG, "batch is NULL");
  gmm_status st = validate_tuning(t);
  if (st != GMM_OK) return st;
  DeviceGuard g(b->device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the batch's device");
  (void)hipStreamSynchronize(b->last_stream);  // the first tiles may be rebuilt
  return apply_tuning(b, *t);
}

gmm_status gmm_batch_get_tuning(const gmm_batch* b, gmm_batch_tuning* t) {
  if (!b || !t) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  *t = b->tuning;
  return GMM_OK;
}

gmm_status gmm_batch_set_frames(gmm_batch* b, int32_t slot, const gmm_stream_io* io, void* stream) {
  if (!b || !io) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  if (slot < 0 || slot >= b->n_slots) return fail(GMM_ERR_INVALID_ARG, "slot out of range");
  // validate every stream before touching anything
  for (size_t i = 0; i < n_streams(b); ++i) {
    gmm_handle* h = b->handles[i];
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
  }
  DeviceGuard g(b->device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the batch's device");
  const bool pack = n_streams(b) <= kPackStreams;
  hipError_t e = pack ? hipSuccess : hipEventSynchronize(b->staging_done[slot]);  // previous upload from this buffer
  if (e != hipSuccess) return hip_fail(e, "staging event");
  FrameArgs packed[kPackStreams];
  FrameArgs* host = pack ? packed : b->h_staging[slot];
  bool measure = false;
  for (size_t i = 0; i < n_streams(b); ++i) {
    const gmm_stream_io& s = io[i];
    host[i] = frame_args(b->handles[i], s.rgb, s.rgb_pitch_bytes, s.depth, s.depth_pitch_bytes, s.fg_rgb,
                         s.fg_depth, s.fused);
    measure = measure || host[i].wave_bytes != nullptr;
  }
  hipStream_t hs = static_cast<hipStream_t>(stream);
  FrameArgs* table = b->d_table + static_cast<size_t>(slot) * n_streams(b);
  if (pack) {
    e = pack_descriptors(host, nullptr, static_cast<int32_t>(n_streams(b)), table, nullptr, hs);
  } else {
    e = hipMemcpyAsync(table, host, n_streams(b) * sizeof(FrameArgs), hipMemcpyHostToDevice, hs);
    if (e == hipSuccess) e = hipEventRecord(b->staging_done[slot], hs);
  }
  if (e != hipSuccess) return hip_fail(e, "descriptor upload");
  b->slot_ready[slot] = 1;
  b->slot_measure[slot] = measure ? 1 : 0;
  b->last_stream = hs;
  return GMM_OK;
}

gmm_status gmm_batch_run(gmm_batch* b, int32_t slot, void* stream) {
  if (!b) return fail(GMM_ERR_INVALID_ARG, "batch is NULL");
  if (slot < 0 || slot >= b->n_slots) return fail(GMM_ERR_INVALID_ARG, "slot out of range");
  if (!b->slot_ready[slot]) return fail(GMM_ERR_STATE, "slot has no frames (call gmm_batch_set_frames first)");
  DeviceGuard g(b->device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the batch's device");
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipError_t e = run_slot(b, slot, hs);
  if (e != hipSuccess) return hip_fail(e, "batch kernel launch");
  b->last_stream = hs;
  for (auto* h : b->handles) h->last_stream = hs;
  return GMM_OK;
}

gmm_status gmm_batch_apply(gmm_batch* b, const gmm_stream_io* io, void* stream) {
  gmm_status st = gmm_batch_set_frames(b, 0, io, stream);
  if (st != GMM_OK) return st;
  return gmm_batch_run(b, 0, stream);
}

gmm_status gmm_batch_autotune(gmm_batch* b, int32_t slot, void* stream, gmm_batch_tuning* best_out,
                              double* best_ms_out) {
  if (!b) return fail(GMM_ERR_INVALID_ARG, "batch is NULL");
  if (slot < 0 || slot >= b->n_slots) return fail(GMM_ERR_INVALID_ARG, "slot out of range");
  if (!b->slot_ready[slot]) return fail(GMM_ERR_STATE, "slot has no frames (call gmm_batch_set_frames first)");
  DeviceGuard g(b->device);
  if (!g.ok()) return fail(GMM_ERR_DEVICE, "cannot select the batch's device");
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const std::string key = mix_key(b);
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune_cache.find(key);
    if (it != g_tune_cache.end()) {
      (void)hipStreamSynchronize(hs);
      gmm_status st = apply_tuning(b, it->second.first);
      if (st != GMM_OK) return st;
      if (best_out) *best_out = it->second.first;
      if (best_ms_out) *best_ms_out = it->second.second;
      return GMM_OK;
    }
  }
  // trial launches advance the streams: keep a copy of every state and put it back afterwards
  size_t total = 0;
  for (auto* h : b->handles) total += h->rgb_bytes + h->depth_bytes + h->fuse_bytes;
  void* backup = nullptr;
  hipError_t e = hipMalloc(&backup, total);
  if (e != hipSuccess) return fail(GMM_ERR_OUT_OF_MEMORY, "autotune state backup allocation failed");
  auto copy_states = [&](bool save) -> hipError_t {
    size_t off = 0;
    for (auto* h : b->handles) {
      const size_t nb = h->rgb_bytes + h->depth_bytes + h->fuse_bytes;
      char* bk = static_cast<char*>(backup) + off;
      hipError_t r = save ? hipMemcpyAsync(bk, h->mem, nb, hipMemcpyDeviceToDevice, hs)
                          : hipMemcpyAsync(h->mem, bk, nb, hipMemcpyDeviceToDevice, hs);
      if (r != hipSuccess) return r;
      off += nb;
    }
    return hipStreamSynchronize(hs);
  };
  e = copy_states(true);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  const gmm_batch_tuning start = b->tuning;
  gmm_batch_tuning best = start;
  double best_ms = 1e30;
  gmm_status st = GMM_OK;
  // every candidate is timed from the same saved state on the same frame-sets (`slot` and the
  // prepared slots after it, cyclically), so all see the same mix of pixels that keep their
  // top component and pixels that do not
  std::vector<int32_t> slots;
  for (int32_t i = 0; i < b->n_slots && slots.size() < 4; ++i) {
    const int32_t sl = (slot + i) % b->n_slots;
    if (b->slot_ready[sl]) slots.push_back(sl);
  }
  if (e == hipSuccess) {
    const int blocks[] = {256, 512};
    const int tile_mult[] = {1, 2, 4, 8, 16};
    const int per_cu[] = {2, 4, 8, 16};
    // candidates often come to the same launch (with 2048 threads a CU or more, one block per tile):
    // each launch is tried once, by threads, pixels per piece and blocks
    std::set<std::tuple<int, uint32_t, uint32_t>> tried;
    for (int bt : blocks) {
      for (int tm : tile_mult) {
        for (int pc : per_cu) {
          gmm_batch_tuning t{bt, bt * tm, pc};
          const BatchLaunch l = batch_launch(t, count_tiles(b, static_cast<uint32_t>(t.tile_pixels)), b->pixels, b->cu_count);
          if (!tried.insert({l.block, l.tile_px >> l.piece_shift, l.grid}).second) continue;
          st = apply_tuning(b, t);
          if (st != GMM_OK) break;
          e = run_slot(b, slot, hs);  // warm-up
          if (e == hipSuccess) e = copy_states(false);
          if (e == hipSuccess) e = hipEventRecord(e0, hs);
          const int reps = static_cast<int>(slots.size());
          for (int r = 0; r < reps && e == hipSuccess; ++r) e = run_slot(b, slots[r], hs);
          if (e == hipSuccess) e = hipEventRecord(e1, hs);
          if (e == hipSuccess) e = copy_states(false);
          if (e == hipSuccess) e = hipEventSynchronize(e1);
          float ms = 0.f;
          if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
          if (e != hipSuccess) break;
          const double avg = ms / reps;
          if (avg < best_ms) {
            best_ms = avg;
            best = t;
          }
        }
        if (e != hipSuccess || st != GMM_OK) break;
      }
      if (e != hipSuccess || st != GMM_OK) break;
    }
  }
  hipError_t er = copy_states(false);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(backup);
  if (e != hipSuccess) return hip_fail(e, "autotune trial");
  if (er != hipSuccess) return hip_fail(er, "autotune state restore");
  if (st != GMM_OK) return st;
  st = apply_tuning(b, best);
  if (st != GMM_OK) return st;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache[key] = {best, best_ms};
  }
  if (best_out) *best_out = best;
  if (best_ms_out) *best_ms_out = best_ms;
  b->last_stream = hs;
  return GMM_OK;
}

gmm_status gmm_batch_tiles(const gmm_batch* b, uint32_t* n_tiles) {
  if (!b || !n_tiles) return fail(GMM_ERR_INVALID_ARG, "NULL argument");
  *n_tiles = b->n_tiles;
  return GMM_OK;
}

}  // extern "C"
