// Host-side internals shared by the ABI layer and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "gmm.h"
#include "gmm_device.hpp"

namespace rgbd {

// Everything one frame-kernel launch needs for one stream.
struct FrameArgs {
  int64_t npix;
  uint32_t tiles64;        // 64-pixel tiles of the state layout (ceil(npix / 64))
  uint32_t pad0_;
  int32_t width;
  int32_t rgb_dense;       // rgb rows are contiguous (pitch == 3*width) and 4-byte aligned
  int32_t depth_dense;     // depth rows are contiguous (pitch == 2*width)
  const uint8_t* rgb;
  int64_t rgb_pitch;
  const uint16_t* depth;
  int64_t depth_pitch;
  void* st_rgb;            // colour state block: 5*M values per pixel (four-channel variant: 6*M), plus rank
                           // 1's key and one scale per tile in the fp32 form
  void* st_depth;          // depth state block: 3*M values per pixel (and the same extras)
  uint8_t* fstate;         // List 1 state bytes
  uint64_t* fg_rgb;
  uint64_t* fg_depth;
  uint64_t* fused;
  ModelConsts kc;          // colour constants
  ModelConsts kd;          // depth constants (the fields both modalities share equal kc's: depth_consts)
  int32_t mode;            // kModeRGB | kModeDepth | kModeFuse bits of this stream
  int32_t pad_;
  uint64_t* wave_bytes;    // optional: per-wave running total of state bytes moved (measurement)
};

enum FrameMode : int { kModeRGB = 1, kModeDepth = 2, kModeFuse = 4, kModeAug = 8 };

// Launchers (return hipSuccess or the launch error).
// `stream`: the kernel's rows take the non-temporal cache policy (kStream), for streams
// whose rows cannot stay in the last-level cache between frames (streams_rows).
hipError_t launch_frame(const FrameArgs& a, int M, int dtype, int mode, bool stream, hipStream_t s);
hipError_t launch_fuse(const uint64_t* fr, const uint64_t* fd, uint64_t* out, uint8_t* fstate,
                       int64_t npix, hipStream_t s);
hipError_t launch_init(void* st, int dtype, uint32_t tiles64, int M, int C, float var0, hipStream_t s);
// Rank 1's key of every pixel from the stored values (scaled form; a no-op otherwise).
hipError_t launch_rekey(void* st, int dtype, uint32_t tiles64, int M, int C, hipStream_t s);
hipError_t launch_fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s);

bool frame_variant_compiled(int M, int dtype);
// One launch of the batched kernel: the streams' descriptors and first tiles (device memory) and
// the launch shape.
struct BatchLaunch {
  const FrameArgs* table;
  const uint32_t* first;  // first tile of each stream, increasing from 0
  uint32_t n_streams;
  uint32_t n_pieces;      // tiles << piece_shift
  uint32_t tile_px;       // pixels per tile
  uint32_t piece_shift;   // a tile is 2^piece_shift pieces, one block each
  uint32_t grid;
  int block;              // threads per block
  uint32_t lds = 0;       // bytes of LDS a block reserves beyond its own use (limit_residency)
  bool measure;           // some descriptor has a traffic record (wave_bytes): the kernel that counts bytes runs
  bool stream;            // streams_rows of the streams
};
constexpr gmm_batch_tuning kDefaultTuning{256, 1024, 8};
// Whether a tuning leaves the shape to the library: the default does, whether a caller set it or not,
// so that setting the tuning that was read back changes nothing.
inline bool is_open(const gmm_batch_tuning& t) {
  return t.block_threads == kDefaultTuning.block_threads && t.tile_pixels == kDefaultTuning.tile_pixels &&
         t.blocks_per_cu == kDefaultTuning.blocks_per_cu;
}
// Whether a tuning has fewer blocks per CU than a CU holds (2048 threads): its blocks walk tiles.
inline bool walks(const gmm_batch_tuning& t) { return t.blocks_per_cu * t.block_threads < 2048; }
// The launch shape for a tuning.
BatchLaunch batch_launch(const gmm_batch_tuning& t, uint32_t n_tiles, uint64_t pixels, int cu_count);
// One block per piece for `l`, with at most `blocks` of them on a CU at a time.
void limit_residency(BatchLaunch& l, uint32_t blocks);
hipError_t launch_batch(int M, int dtype, const BatchLaunch& l, hipStream_t s);
// Descriptors (and first tiles, unless NULL) of n streams to the device as kernel arguments, up to
// kPackPerLaunch streams with equal model constants per launch, half as many with mixed ones.
constexpr int kPackPerLaunch = 32;
hipError_t pack_descriptors(const FrameArgs* a, const uint32_t* first, int32_t n, FrameArgs* d_table, uint32_t* d_first,
                            hipStream_t s);
// Launches that need no table afterwards (the static call, ticks) carry the descriptors of up to
// kPackPerLaunch streams with equal constants in the batched kernel's own arguments; fits_args says
// whether `l` may. 24 small streams 21.8 -> 18.1 us a static call.
bool fits_args(const FrameArgs* a, const BatchLaunch& l);
hipError_t launch_batch_args(int M, int dtype, const FrameArgs* a, const uint32_t* first, const BatchLaunch& l,
                             hipStream_t s);
// Up to this many streams a batch's or a tick's descriptors go that way, above it in one copy from
// page-locked memory. gmm_batch_apply on small streams, arguments against copy: 1 stream 8.9 and
// 14.6 us, 32 streams 13.9 and 17.3 us, 33 streams (a second launch) 18.2 and 17.2 us.
constexpr size_t kPackStreams = kPackPerLaunch;

inline size_t dtype_size(int dtype) { return dtype == GMM_F32 ? 4 : 2; }

void set_error(const std::string& msg);
gmm_status fail(gmm_status st, const std::string& msg);
gmm_status hip_fail(hipError_t e, const char* what);

// Switches to a device for the duration of a call, restoring the caller's.
class DeviceGuard {
 public:
  explicit DeviceGuard(int dev) {
    ok_ = hipGetDevice(&prev_) == hipSuccess;
    if (ok_ && prev_ != dev) ok_ = hipSetDevice(dev) == hipSuccess;
    switched_ = ok_ && prev_ != dev;
  }
  ~DeviceGuard() {
    if (switched_) (void)hipSetDevice(prev_);
  }
  bool ok() const { return ok_; }

 private:
  int prev_ = 0;
  bool ok_ = false;
  bool switched_ = false;
};

}  // namespace rgbd

struct gmm_handle {  // the library's per-stream object (opaque in gmm.h)
  gmm_config cfg;
  int64_t npix = 0;
  uint32_t tiles64 = 0;     // 64-pixel tiles of the state layout
  size_t esize = 0;         // bytes per stored value
  size_t rgb_bytes = 0;     // colour block
  size_t depth_bytes = 0;   // depth block
  size_t fuse_bytes = 0;    // List 1 state bytes (padded)
  void* mem = nullptr;      // device state: [colour][depth][fusion]
  bool owns_mem = false;    // allocated by gmm_create (else provided by the caller)
  uint64_t* wave_bytes = nullptr;  // optional per-wave traffic record (gmm_set_traffic_record)
  void* st_rgb = nullptr;
  void* st_depth = nullptr;
  uint8_t* fstate = nullptr;
  hipStream_t last_stream = nullptr;
  size_t hot = 0;           // bytes that every frame touches: hot rows, frames and flags
  uint64_t touched = 0;     // hot bytes that the device's launches had gone through after its last frame (streams_rows)
  rgbd::ModelConsts kc{}, kd{};
};

inline bool has_rgb(const gmm_handle* h) { return (h->cfg.modalities & GMM_RGB) != 0; }
inline bool has_depth(const gmm_handle* h) { return (h->cfg.modalities & GMM_DEPTH) != 0; }
inline bool has_both(const gmm_handle* h) { return has_rgb(h) && has_depth(h); }
// the four-channel (R, G, B, depth byte) variant: one mixture, no separate models, no fusion
inline bool is_augmented(const gmm_handle* h) { return h->cfg.variant == GMM_AUGMENTED; }
// the per-modality separate models of the method (colour block, depth block, List 1 state)
inline bool sep_rgb(const gmm_handle* h) { return has_rgb(h) && !is_augmented(h); }
inline bool sep_depth(const gmm_handle* h) { return has_depth(h) && !is_augmented(h); }
inline bool sep_both(const gmm_handle* h) { return has_both(h) && !is_augmented(h); }

namespace rgbd {
// Validation and kernel arguments of one stream's frame (shared by the plain and batched paths).
gmm_status check_frame_args(gmm_handle* h, const uint8_t* rgb, int64_t rgb_pitch, const uint16_t* depth,
                            int64_t depth_pitch, uint64_t* fg_rgb, uint64_t* fg_depth);
FrameArgs frame_args(gmm_handle* h, const uint8_t* rgb, int64_t rgb_pitch, const uint16_t* depth,
                     int64_t depth_pitch, uint64_t* fg_rgb, uint64_t* fg_depth, uint64_t* fused);
// A validated handle with its sizes and constants, no device memory yet.
gmm_status new_handle(const gmm_config* cfg, gmm_handle** out);
// Point the handle's state at `mem` (state_bytes(h) bytes, 256-byte aligned).
void place_state(gmm_handle* h, void* mem);
// Enqueue the initial (all components empty) state on `s`.
hipError_t init_state(gmm_handle* h, hipStream_t s);
size_t state_bytes(const gmm_handle* h);
// Whether a launch that advances these `n` streams of one device by one frame streams their rows;
// notes the launch. Rows kept in the last-level cache (256 MB) are there for a stream's next frame
// only if less than that has gone through it since: what counts is the hot bytes of all launches on
// the device between two frames of a stream, its own included, however they are divided into
// streams, batches and ticks. A stream's first frame counts its launch alone, and a captured launch
// keeps the policy of its capture (its replays are not seen). The launch takes the policy that is right
// for the larger part of its bytes. The line lies below the cache's size, since
// masks and the suffixes of some pixels go through it too. Rows kept against rows streamed, us a call,
// every stream with frames of its own: a 2560x1600 paired fp32 stream (188 MB) 51.7 and 53.2, 2400x1800
// (199 MB) 57.2 and 56.1, 2560x1920 (226 MB) 67.2 and 63.5; one batch of VGA fp32 streams, 12 (170 MB)
// 54.7 and 56.4, 14 (198 MB) 68.2 and 65.4, 16 (226 MB) 77.9 and 73.0, of 16 fp16 ones (206 MB) 73.1 and
// 67.5; single streams in turn, two of 1920x1080 (191 MB) 28.7 and 29.0, five of 1280x720 (212 MB) 15.5
// and 15.2, 13 VGA (184 MB) 7.6 and 7.7, 18 (254 MB) 8.0 and 7.7; batches in turn, two of 7 VGA streams
// (198 MB) 34.5 and 35.8, two of 8 (226 MB) 39.7 and 39.1, two of 9 fp16 ones (232 MB) 41.4 and 39.7. Far
// beyond it: eight 1920x1080 fp32 streams in turn 34.4 and 29.1.
constexpr size_t kStreamHotBytes = size_t(184) << 20;
bool streams_rows(gmm_handle* const* h, size_t n);
}  // namespace rgbd
