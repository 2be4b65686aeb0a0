// Confusion counts of two bit-packed masks (the quantities of Eqs. 1-3, Sec. V.A).
//
// One lane per mask word: popcounts of pred & truth, pred and truth over the valid bits (TN
// follows from the pixel count), reduced across the wave with cross-lane adds and across the block
// through LDS. What bounds a call is launches and latency, not the masks' bytes (77 KB for a VGA
// pair), so masks up to kOneBlockWords are counted by one block that writes the four counts
// itself; larger ones by many blocks that add to counts which a first tiny kernel clears.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gmm.h"
#include "gmm_internal.hpp"

namespace rgbd {

__global__ void __launch_bounds__(4) clear_counts_kernel(unsigned long long* counts) {
  if (threadIdx.x < 4) counts[threadIdx.x] = 0ull;
}

// Set bits of (pred & truth, pred, truth) that one wave counts. 32 bits hold them for any mask that fits
// a device: a mask is cut over 8192 waves, so that one reaches 2^32 bits past 2^39 words (4 TB). Sums
// over waves take 64 bits.
struct Ones {
  uint32_t both, pred, truth;
};

__device__ __forceinline__ Ones wave_sum(Ones v) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    v.both += __shfl_xor(v.both, d, kWave);
    v.pred += __shfl_xor(v.pred, d, kWave);
    v.truth += __shfl_xor(v.truth, d, kWave);
  }
  return v;
}

// Words first, first + step, ... of the masks, eight in flight.
__device__ __forceinline__ Ones count_words(const uint64_t* __restrict__ pred, const uint64_t* __restrict__ truth,
                                            uint64_t first, uint64_t step, uint64_t nwords, uint64_t last_valid) {
  Ones o{0, 0, 0};
  constexpr uint32_t U = 4;
  for (uint64_t w = first; w < nwords; w += U * step) {
    uint64_t p[U], t[U];
#pragma unroll
    for (uint32_t j = 0; j < U; ++j) {
      const uint64_t at = w + j * step;
      p[j] = at < nwords ? pred[at] : 0ull;
      t[j] = at < nwords ? truth[at] : 0ull;
    }
#pragma unroll
    for (uint32_t j = 0; j < U; ++j) {
      const uint64_t valid = w + j * step == nwords - 1 ? last_valid : ~0ull;
      o.both += __popcll(p[j] & t[j] & valid);
      o.pred += __popcll(p[j] & valid);
      o.truth += __popcll(t[j] & valid);
    }
  }
  return o;
}

constexpr int kCountBlock = 1024;

template <bool ALONE>
__global__ void __launch_bounds__(kCountBlock) confusion_kernel(const uint64_t* __restrict__ pred,
                                                          const uint64_t* __restrict__ truth, uint64_t npix,
                                                          uint64_t nwords, unsigned long long* __restrict__ counts) {
  constexpr int WAVES = kCountBlock / kWave;
  __shared__ Ones part[WAVES];
  const uint32_t rem = static_cast<uint32_t>(npix & 63u);
  const uint64_t last_valid = rem ? (1ull << rem) - 1ull : ~0ull;
  const Ones o = wave_sum(count_words(pred, truth, blockIdx.x * kCountBlock + threadIdx.x, gridDim.x * kCountBlock,
                                           nwords, last_valid));
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = o;
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint64_t both = 0, p = 0, t = 0;
  for (int i = 0; i < WAVES; ++i) {
    both += part[i].both;
    p += part[i].pred;
    t += part[i].truth;
  }
  if constexpr (ALONE) {
    counts[0] = both;
    counts[1] = p - both;
    counts[2] = npix + both - p - t;
    counts[3] = t - both;
  } else {  // the pixel count enters once; the sum is exact modulo 2^64
    atomicAdd(&counts[0], both);
    atomicAdd(&counts[1], p - both);
    atomicAdd(&counts[2], (blockIdx.x == 0 ? npix : 0ull) + both - p - t);
    atomicAdd(&counts[3], t - both);
  }
}

// One block, one launch up to kOneBlockWords: a VGA mask 3.5 us on the GPU and 4.0 us a call from
// Python, where clearing and counting in many blocks takes 4.7 and 6.6 us; 10^6 pixels 5.9 and 4.1
// against 4.9 and 6.6, a call in a loop being bound by the launches; a 1920x1080 mask 9.6 against 4.9
// on the GPU. Above it, blocks of kWordsPerBlock words: the adds of all blocks meet at one cache line,
// and 64 of them cost less than 1024 (3840x2160: 5.8 us, with a block per 256 words 28 us, and with an
// add for every wave besides 101 us).
constexpr uint64_t kOneBlockWords = 16384;
constexpr uint64_t kWordsPerBlock = 4096;

}  // namespace rgbd

using namespace rgbd;

extern "C" gmm_status gmm_mask_confusion(const uint64_t* pred, const uint64_t* truth, int64_t npix,
                                         uint64_t* counts, void* stream) {
  if (!pred || !truth || !counts) return fail(GMM_ERR_INVALID_ARG, "NULL mask or counts");
  if (npix <= 0) return fail(GMM_ERR_INVALID_ARG, "npix must be > 0");
  if ((reinterpret_cast<uintptr_t>(pred) | reinterpret_cast<uintptr_t>(truth) |
       reinterpret_cast<uintptr_t>(counts)) % 8)
    return fail(GMM_ERR_INVALID_ARG, "masks and counts must be 8-byte aligned");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint64_t n = static_cast<uint64_t>(npix);
  const uint64_t words = (n + 63) / 64;
  auto* c = reinterpret_cast<unsigned long long*>(counts);
  hipError_t e = hipSuccess;
  if (words <= kOneBlockWords) {
    confusion_kernel<true><<<1, dim3(kCountBlock), 0, s>>>(pred, truth, n, words, c);
    e = hipGetLastError();
  } else {
    const uint64_t blocks = std::min<uint64_t>((words + kWordsPerBlock - 1) / kWordsPerBlock, 512u);
    clear_counts_kernel<<<1, 4, 0, s>>>(c);
    e = hipGetLastError();
    if (e == hipSuccess) {
      confusion_kernel<false><<<dim3(static_cast<unsigned>(blocks)), dim3(kCountBlock), 0, s>>>(pred, truth, n, words, c);
      e = hipGetLastError();
    }
  }
  if (e != hipSuccess) return hip_fail(e, "confusion kernel launch");
  return GMM_OK;
}
