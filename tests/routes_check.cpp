// What the library asks of the HIP runtime, without a GPU: the program stands in for the runtime
// (its symbols come before libamdhip64's), remembers allocations, copies and launches, and runs no
// kernel. Each check drives the C ABI and looks at the launches and copies that a call made.
//
//   routes_check NAME...
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "gmm.h"

// ---- the stand-in runtime ----------------------------------------------------------------------

struct Region {
  size_t bytes;
  hipMemoryType type;
  unsigned flags;
};
struct Launch {
  std::string name;
  unsigned grid, block;
  size_t lds;
};

struct Runtime {
  std::mutex mu;
  std::map<const void*, std::string> kernels;
  std::map<uintptr_t, Region> regions;
  std::vector<Launch> launches;
  size_t h2d = 0, d2h = 0;  // asynchronous copies
  std::function<void(const void* dst, const void* src, size_t n)> on_copy;  // called by them, unlocked
  std::function<void()> on_sync;                                            // and by stream synchronisations
};
static Runtime& rt() {
  static Runtime r;
  return r;
}

static std::map<uintptr_t, Region>::iterator region_of(const void* p) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(p);
  auto it = rt().regions.upper_bound(a);
  if (it == rt().regions.begin()) return rt().regions.end();
  --it;
  return a < it->first + it->second.bytes ? it : rt().regions.end();
}

static hipError_t allocate(void** p, size_t n, hipMemoryType type, unsigned flags) {
  *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);
  if (!*p) return hipErrorOutOfMemory;
  std::lock_guard<std::mutex> lk(rt().mu);
  rt().regions[reinterpret_cast<uintptr_t>(*p)] = Region{n, type, flags};
  return hipSuccess;
}

static hipError_t release(void* p) {
  {
    std::lock_guard<std::mutex> lk(rt().mu);
    rt().regions.erase(reinterpret_cast<uintptr_t>(p));
  }
  std::free(p);
  return hipSuccess;
}

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
  rt().kernels[host] = st == 0 ? d : name;
  std::free(d);
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t n, int, int) {
  rt().regions[reinterpret_cast<uintptr_t>(var)] = Region{n, hipMemoryTypeDevice, 0};
}

static thread_local struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
} g_call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_call = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_call.grid;
  *b = g_call.block;
  *lds = g_call.lds;
  *s = g_call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t lds, hipStream_t) {
  std::lock_guard<std::mutex> lk(rt().mu);
  rt().launches.push_back(Launch{rt().kernels[f], g.x, b.x, lds});
  return hipSuccess;
}

hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* sym) { return *p = const_cast<void*>(sym), hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) { return allocate(p, n, hipMemoryTypeDevice, 0); }
hipError_t hipFree(void* p) { return release(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) { return allocate(p, n, hipMemoryTypeHost, flags); }
hipError_t hipHostFree(void* p) { return release(p); }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (rt().on_copy) rt().on_copy(dst, src, n);
  std::lock_guard<std::mutex> lk(rt().mu);
  (kind == hipMemcpyHostToDevice ? rt().h2d : rt().d2h) += kind == hipMemcpyDeviceToDevice ? 0 : 1;
  return hipSuccess;
}

hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::lock_guard<std::mutex> lk(rt().mu);
  std::memset(a, 0, sizeof *a);
  const auto it = region_of(p);
  a->type = it == rt().regions.end() ? hipMemoryTypeUnregistered : it->second.type;
  a->device = it == rt().regions.end() ? -2 : 0;
  if (it == rt().regions.end()) return hipSuccess;
  a->devicePointer = const_cast<void*>(p);
  a->hostPointer = it->second.type == hipMemoryTypeHost ? a->devicePointer : nullptr;
  a->allocationFlags = it->second.flags;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* n, hipDeviceptr_t p) {
  std::lock_guard<std::mutex> lk(rt().mu);
  const auto it = region_of(p);
  if (it == rt().regions.end()) return hipErrorNotFound;
  *base = reinterpret_cast<hipDeviceptr_t>(it->first);
  *n = it->second.bytes;
  return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t* e) { return *e = reinterpret_cast<hipEvent_t>(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = reinterpret_cast<hipStream_t>(1), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  if (rt().on_sync) rt().on_sync();
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

}  // extern "C"

// ---- what the checks share ---------------------------------------------------------------------

static int g_bad = 0;
#define EXPECT(cond)                                                   \
  do {                                                                 \
    if (!(cond)) std::printf("line %d: %s\n", __LINE__, #cond), ++g_bad; \
  } while (0)
#define OK(call) EXPECT((call) == GMM_OK)

static gmm_handle* handle(int w, int h, int modalities = GMM_RGB | GMM_DEPTH, int M = 5, int dtype = GMM_F32) {
  gmm_config c;
  OK(gmm_config_default(&c, w, h, modalities, M));
  c.state_dtype = dtype;
  gmm_handle* g = nullptr;
  OK(gmm_create(&c, &g));
  return g;
}

// Page-locked host memory.
static uint8_t* pinned(size_t n, unsigned flags = 0) {
  void* p = nullptr;
  (void)hipHostMalloc(&p, n, flags);
  return static_cast<uint8_t*>(p);
}

struct Counts {
  size_t h2d, d2h;
};

static size_t host_allocations() {
  size_t n = 0;
  for (const auto& r : rt().regions) n += r.second.type == hipMemoryTypeHost;
  return n;
}

// One tick of an executor, waited for: the copies of frames and masks it made.
static Counts tick(gmm_exec* x, const std::vector<gmm_exec_item>& items) {
  const Counts before{rt().h2d, rt().d2h};
  OK(gmm_exec_launch(x, items.data(), static_cast<int32_t>(items.size()), nullptr));
  OK(gmm_exec_drain(x));
  return Counts{rt().h2d - before.h2d, rt().d2h - before.d2h};
}

// ---- checks ------------------------------------------------------------------------------------

// A frame is used in place only if all of it lies in one page-locked allocation: its ends may lie in
// two with memory between them that the GPU cannot read.
static void gap() {
  constexpr int W = 320, H = 240;
  constexpr size_t n = size_t(W) * H * 3;
  gmm_exec* x = nullptr;
  OK(gmm_exec_create(0, 2, &x));
  gmm_handle* h = handle(W, H, GMM_RGB);
  OK(gmm_exec_attach(x, h, nullptr));
  uint8_t* whole = pinned(n + 8192);
  uint64_t* mask = reinterpret_cast<uint64_t*>(pinned(W * H / 8));
  std::vector<gmm_exec_item> it{{h, whole, nullptr, mask, nullptr, nullptr}};
  EXPECT(tick(x, it).h2d == 0);
  // the same memory as two page-locked regions with an ordinary page between them
  rt().regions.erase(reinterpret_cast<uintptr_t>(whole));
  rt().regions[reinterpret_cast<uintptr_t>(whole)] = Region{4096, hipMemoryTypeHost, 0};
  rt().regions[reinterpret_cast<uintptr_t>(whole) + 8192] = Region{n, hipMemoryTypeHost, 0};
  EXPECT(tick(x, it).h2d == 1);
  it[0].host_rgb = whole + 8192;  // inside the second region
  EXPECT(tick(x, it).h2d == 0);
  it[0].host_rgb = whole + 8196;  // its last bytes past the region's end
  EXPECT(tick(x, it).h2d == 1);
  // a mask with such a gap goes through the device arena
  it[0].host_rgb = whole + 8192;
  it[0].host_fg_rgb = reinterpret_cast<uint64_t*>(whole);
  EXPECT(tick(x, it).d2h == 1);
  OK(gmm_exec_destroy(x));
  OK(gmm_destroy(h));
}

// Only memory known to be coherent between host and device is used in place; every other kind of
// page-locked memory is copied.
static void coherence() {
  constexpr int W = 64, H = 64;
  constexpr size_t n = size_t(W) * H * 3;
  gmm_exec* x = nullptr;
  OK(gmm_exec_create(0, 2, &x));
  gmm_handle* h = handle(W, H, GMM_RGB);
  OK(gmm_exec_attach(x, h, nullptr));
  const struct {
    unsigned flags;
    bool in_place;
  } kinds[] = {
      {hipHostMallocDefault, true},
      {hipHostMallocCoherent, true},
      {hipHostMallocCoherent | hipHostMallocPortable, true},
      {hipHostMallocCoherent | hipHostMallocMapped, true},
      {hipHostMallocNonCoherent, false},
      {hipHostMallocPortable, false},
      {hipHostMallocMapped, false},
      {hipHostMallocWriteCombined, false},
      {hipExtHostRegisterCoarseGrained, false},  // also hipHostRegisterReadOnly, which a mask must not be written to
      {hipHostMallocCoherent | hipExtHostRegisterCoarseGrained, false},
  };
  for (const auto& k : kinds) {
    uint8_t* frame = pinned(n, k.flags);
    uint64_t* mask = reinterpret_cast<uint64_t*>(pinned(W * H / 8, k.flags));
    const Counts c = tick(x, {{h, frame, nullptr, mask, nullptr, nullptr}});
    if (c.h2d != (k.in_place ? 0u : 1u) || c.d2h != (k.in_place ? 0u : 1u))
      std::printf("flags %#x: %zu frames and %zu masks copied\n", k.flags, c.h2d, c.d2h), ++g_bad;
  }
  OK(gmm_exec_destroy(x));
  OK(gmm_destroy(h));
}

// Masks that share memory with a frame or another mask of the tick are delivered after the kernel, in
// the order of the items, as if every frame had been copied in first: they are not written in place.
static void overlap() {
  constexpr int W = 64, H = 64;
  constexpr size_t px = size_t(W) * H, words = px / 64;
  gmm_exec* x = nullptr;
  OK(gmm_exec_create(0, 2, &x));
  gmm_handle* h[2] = {handle(W, H), handle(W, H)};
  for (auto* g : h) OK(gmm_exec_attach(x, g, nullptr));
  uint8_t* rgb[2] = {pinned(px * 3), pinned(px * 3)};
  uint16_t* depth[2] = {reinterpret_cast<uint16_t*>(pinned(px * 2)), reinterpret_cast<uint16_t*>(pinned(px * 2))};
  uint64_t* m = reinterpret_cast<uint64_t*>(pinned(6 * words * 8));
  const std::vector<gmm_exec_item> apart{{h[0], rgb[0], depth[0], m, m + words, m + 2 * words},
                                         {h[1], rgb[1], depth[1], m + 3 * words, m + 4 * words, m + 5 * words}};
  EXPECT(tick(x, apart).d2h == 0);
  std::vector<gmm_exec_item> it = apart;
  it[0].host_fg_rgb = reinterpret_cast<uint64_t*>(rgb[0]);  // over its own colour frame
  EXPECT(tick(x, it).d2h == 1);
  it = apart;
  it[0].host_fused = reinterpret_cast<uint64_t*>(depth[1]) + 3;  // inside another stream's depth frame
  EXPECT(tick(x, it).d2h == 1);
  it = apart;
  it[1].host_fg_depth = it[1].host_fg_rgb;  // one buffer for two masks
  EXPECT(tick(x, it).d2h == 1);
  it = apart;
  it[1].host_fused = m + words - 1;  // across the end of one mask and the start of the next
  EXPECT(tick(x, it).d2h == 1);
  it = apart;
  it[1].host_rgb = rgb[0];  // frames may share memory: nothing writes them
  it[1].host_depth = reinterpret_cast<uint16_t*>(rgb[0] + 2);
  EXPECT(tick(x, it).d2h == 0);
  it[1].host_depth = depth[1];
  it[0].host_fg_rgb = reinterpret_cast<uint64_t*>(rgb[0] + 8);  // a mask in a frame that two streams share
  EXPECT(tick(x, it).d2h == 1);
  EXPECT(tick(x, apart).d2h == 0);
  OK(gmm_exec_destroy(x));
  for (auto* g : h) OK(gmm_destroy(g));
}

// The policy (CP) of the last frame or batched launch: 0 rows kept in the caches, 2 rows streamed.
static int policy() {
  for (size_t i = rt().launches.size(); i-- > 0;) {
    const std::string k = rt().launches[i].name.substr(0, rt().launches[i].name.find('('));
    const size_t last = k.rfind(',');
    if (k.find("batch_kernel<") != std::string::npos)  // <M, S, BLOCK, CP, MEASURE>
      return std::atoi(k.c_str() + k.rfind(',', last - 1) + 1);
    if (k.find("batch_args_kernel<") != std::string::npos || k.find("frame_kernel<") != std::string::npos)
      return std::atoi(k.c_str() + last + 1);  // <..., CP>
  }
  return -1;
}

// A stream may be detached after its handle has gone: the handle is a key then, its memory is not
// read, and the executor's other streams are served as if it had never been there.
static void detach() {
  constexpr int W = 64, H = 64;
  gmm_exec* x = nullptr;
  OK(gmm_exec_create(0, 2, &x));
  gmm_handle *gone = handle(W, H, GMM_RGB), *h = handle(W, H, GMM_RGB);
  OK(gmm_exec_attach(x, h, nullptr));
  OK(gmm_exec_attach(x, gone, nullptr));
  OK(gmm_destroy(gone));
  gmm_handle* other = handle(1024, 1024, GMM_RGB);  // most likely in the memory of the first
  const size_t before = rt().regions.size();
  OK(gmm_exec_detach(x, gone));
  EXPECT(rt().regions.size() == before - 1);  // its frame slots
  EXPECT(gmm_exec_detach(x, gone) == GMM_ERR_INVALID_ARG);
  uint8_t* frame = pinned(W * H * 3);
  (void)tick(x, {{h, frame, nullptr, reinterpret_cast<uint64_t*>(pinned(W * H / 8)), nullptr, nullptr}});
  EXPECT(policy() == 0);  // one small stream stays in the caches
  OK(gmm_exec_destroy(x));
  OK(gmm_destroy(h));
  OK(gmm_destroy(other));
}

// Setting the shape that a batch reports changes nothing; the static call takes the default shape and
// no shape for the same thing.
static void round_trip() {
  gmm_handle* h[2] = {handle(640, 480), handle(320, 240)};
  void* mem = nullptr;
  (void)hipMalloc(&mem, 1 << 21);
  uint8_t* d = static_cast<uint8_t*>(mem);
  uint64_t* m = reinterpret_cast<uint64_t*>(mem);
  const gmm_stream_io io[2] = {{d, 1920, reinterpret_cast<uint16_t*>(d), 1280, m, m + 4800, nullptr},
                               {d, 960, reinterpret_cast<uint16_t*>(d), 640, m + 9600, m + 10800, nullptr}};
  gmm_batch* b = nullptr;
  OK(gmm_batch_create(h, 2, 1, &b));
  const auto shape = [&] {
    OK(gmm_batch_apply(b, io, nullptr));
    return rt().launches.back();
  };
  const auto same = [](const Launch& x, const Launch& y) { return x.name == y.name && x.grid == y.grid && x.block == y.block; };
  gmm_batch_tuning t{};
  const Launch first = shape();
  OK(gmm_batch_get_tuning(b, &t));
  OK(gmm_batch_set_tuning(b, &t));
  EXPECT(same(shape(), first));
  const gmm_batch_tuning other{512, 2048, 1};
  OK(gmm_batch_set_tuning(b, &other));
  const Launch walking = shape();
  EXPECT(walking.block == 512 && walking.grid == 150 + 38);  // a block per tile, fewer than CUs
  OK(gmm_batch_set_tuning(b, &t));
  EXPECT(same(shape(), first));
  OK(gmm_batch_apply_static(h, 2, io, nullptr, nullptr));
  const Launch open = rt().launches.back();
  OK(gmm_batch_apply_static(h, 2, io, &t, nullptr));
  EXPECT(same(rt().launches.back(), open));
  OK(gmm_batch_destroy(b));
  for (auto* g : h) OK(gmm_destroy(g));
}

// A launch shape set on an executor holds for ticks that read page-locked frames too: its threads and
// tiles as they are, its blocks per CU as the number that a CU has LDS for.
static void exec_tuning() {
  constexpr int W = 1024, H = 1024;
  constexpr size_t px = size_t(W) * H, kLdsPerCu = 160 << 10;
  gmm_exec* x = nullptr;
  OK(gmm_exec_create(0, 2, &x));
  gmm_handle* h = handle(W, H);
  OK(gmm_exec_attach(x, h, nullptr));
  uint64_t* m = reinterpret_cast<uint64_t*>(pinned(3 * px / 8));
  uint8_t* rgb = pinned(px * 3);
  uint16_t* depth = reinterpret_cast<uint16_t*>(pinned(px * 2));
  const std::vector<gmm_exec_item> it{{h, rgb, depth, m, m + px / 64, m + 2 * (px / 64)}};
  for (int threads : {256, 512})
    for (int tiles : {1, 4})
      for (int per_cu = 1; per_cu <= 32; ++per_cu) {
        const gmm_batch_tuning t{threads, threads * tiles, per_cu};
        if (threads == 256 && tiles == 4 && per_cu == 8) continue;  // the default
        OK(gmm_exec_set_tuning(x, &t));
        const Counts n = tick(x, it);
        const Launch& l = rt().launches.back();
        const size_t own = static_cast<size_t>(threads) / 64 * 192;
        const bool shaped = l.block == static_cast<unsigned>(threads) && l.grid == px / t.tile_pixels;
        const bool held = per_cu * threads >= 2048 ? l.lds == 0 : kLdsPerCu / (l.lds + own) == static_cast<size_t>(per_cu);
        if (!shaped || !held || n.h2d || n.d2h)
          std::printf("{%d, %d, %d}: %u blocks of %u threads, %zu bytes of LDS, %zu frames copied\n", threads, t.tile_pixels,
                      per_cu, l.grid, l.block, l.lds, n.h2d), ++g_bad;
      }
  // frames that are copied leave the kernel's blocks walking, as a batch's do
  const gmm_batch_tuning t{256, 1024, 2};
  OK(gmm_exec_set_tuning(x, &t));
  std::vector<uint8_t> c(px * 3);
  std::vector<uint16_t> d(px);
  const Counts n = tick(x, {{h, c.data(), d.data(), m, nullptr, nullptr}});
  EXPECT(n.h2d == 2 && rt().launches.back().grid == 512 && rt().launches.back().lds == 0);
  OK(gmm_exec_destroy(x));
  OK(gmm_destroy(h));
}

// A tick that waits for the host link leaves most of every CU to other work: two blocks of 256 threads
// on a CU, a quarter of its LDS free, where they keep the link busy (`blocks`: 0 where they do not).
static void residency() {
  constexpr size_t kLdsPerCu = 160 << 10;
  const auto check = [&](int w, int h, int modalities, const std::vector<int>& counts, size_t blocks) {
    const size_t px = static_cast<size_t>(w) * h;
    gmm_exec* x = nullptr;
    OK(gmm_exec_create(0, 2, &x));
    std::vector<gmm_handle*> g;
    std::vector<gmm_exec_item> in_place, copied;
    std::vector<uint8_t> rgb(px * 3);
    std::vector<uint16_t> depth(px);
    uint8_t* p = pinned(px * 3);
    for (int n : counts) {
      while (static_cast<int>(g.size()) < n) {
        g.push_back(handle(w, h, modalities));
        OK(gmm_exec_attach(x, g.back(), nullptr));
        const bool c = modalities & GMM_RGB, d = modalities & GMM_DEPTH;
        in_place.push_back({g.back(), c ? p : nullptr, d ? reinterpret_cast<uint16_t*>(p) : nullptr, nullptr, nullptr, nullptr});
        copied.push_back({g.back(), c ? rgb.data() : nullptr, d ? depth.data() : nullptr, nullptr, nullptr, nullptr});
      }
      (void)tick(x, in_place);
      const Launch l = rt().launches.back();
      const size_t fit = kLdsPerCu / (l.lds + 768);
      const bool brief = n * px < (1 << 20);  // over before anyone waits long
      const bool full = brief || blocks == 0;
      if (l.block != 256 || l.grid != n * px / (brief ? 256 : 512) ||
          (full ? l.lds != 0 : fit != blocks || kLdsPerCu - fit * (l.lds + 768) < kLdsPerCu / 4))
        std::printf("%d of %dx%d (%d): %u blocks of %u threads, %zu bytes of LDS\n", n, w, h, modalities, l.grid, l.block, l.lds), ++g_bad;
      (void)tick(x, copied);
      EXPECT(rt().launches.back().lds == 0);
    }
    OK(gmm_exec_destroy(x));
    for (auto* q : g) OK(gmm_destroy(q));
  };
  // up to 32 streams' descriptors travel with the kernel, more in a table
  check(512, 256, GMM_RGB | GMM_DEPTH, {1, 7, 8, 32, 40}, 2);
  check(512, 256, GMM_DEPTH, {7, 8, 40}, 2);
  check(512, 256, GMM_RGB, {7, 8, 40}, 0);
  check(1024, 1024, GMM_RGB | GMM_DEPTH, {1, 2}, 2);
}

// Rows are kept in the last-level cache if they are still there when the stream's next frame comes
// (less than 184 MiB has gone through it): what other launches on the device go through in between
// counts, whatever they belong to.
static void cache_policy() {
  constexpr int W = 640, H = 480;  // 307200 pixels, 46 hot bytes each: 14.1 MB
  void* mem = nullptr;
  (void)hipMalloc(&mem, 1 << 21);
  uint8_t* d = static_cast<uint8_t*>(mem);
  uint64_t* m = reinterpret_cast<uint64_t*>(mem);
  const gmm_stream_io io{d, 3 * W, reinterpret_cast<uint16_t*>(d), 2 * W, m, m + 4800, nullptr};
  const std::vector<gmm_stream_io> ios(40, io);
  std::vector<gmm_handle*> h;
  for (int i = 0; i < 40; ++i) h.push_back(handle(W, H));
  const auto frame = [&](gmm_handle* g) {
    OK(gmm_apply_frame(g, d, 3 * W, reinterpret_cast<uint16_t*>(d), 2 * W, m, m + 4800, nullptr));
    return policy();
  };
  // single streams: 13 in turn stay in the cache (184 MB), 24 do not, one of them alone does again
  for (int i = 0; i < 26; ++i) EXPECT(frame(h[i % 13]) == 0);
  for (int i = 0; i < 72; ++i) EXPECT(frame(h[i % 24]) == 2 || i < 24);
  for (int i = 0; i < 4; ++i) EXPECT(frame(h[23]) == 0);
  // one batch of 13, of 14; two of 6 in turn, four of 8 in turn, by either batched call
  const auto batches = [&](int count, int each, bool fixed) {
    std::vector<gmm_batch*> b(count);
    int last = -1;
    for (int i = 0; i < count; ++i) OK(gmm_batch_create(h.data() + i * each, each, 1, &b[i]));
    for (int t = 0; t < 3; ++t)
      for (int i = 0; i < count; ++i) {
        if (fixed) OK(gmm_batch_apply_static(h.data() + i * each, each, ios.data(), nullptr, nullptr));
        else OK(gmm_batch_apply(b[i], ios.data(), nullptr));
        last = policy();
      }
    for (auto* x : b) OK(gmm_batch_destroy(x));
    return last;
  };
  for (bool fixed : {false, true}) {
    EXPECT(batches(1, 13, fixed) == 0);
    EXPECT(batches(1, 14, fixed) == 2);
    EXPECT(batches(2, 6, fixed) == 0);
    EXPECT(batches(4, 8, fixed) == 2);
  }
  // a frame of a stream larger than the cache, between two frames of a small one, makes the small one's
  // rows stream, in every state type and by every call
  gmm_handle* big = handle(3072, 2048);
  for (int dtype : {GMM_F32, GMM_F16, GMM_BF16}) {
    std::vector<gmm_handle*> g;
    for (int i = 0; i < 6; ++i) g.push_back(handle(64, 48, GMM_RGB | GMM_DEPTH, 5, dtype));
    const std::vector<gmm_stream_io> small(6, {d, 3 * 64, reinterpret_cast<uint16_t*>(d), 2 * 64, m, m + 48, nullptr});
    const std::vector<std::function<void()>> calls = {
        [&] { OK(gmm_apply_frame(g[0], d, 192, reinterpret_cast<uint16_t*>(d), 128, m, m + 48, nullptr)); },
        [&] { OK(gmm_batch_apply_static(g.data(), 6, small.data(), nullptr, nullptr)); }};
    for (const auto& call : calls) {
      call();
      call();
      EXPECT(policy() == 0);
      OK(gmm_apply_frame(big, d, 3 * 3072, reinterpret_cast<uint16_t*>(d), 2 * 3072, m, m, nullptr));
      EXPECT(policy() == 2);
      call();
      EXPECT(policy() == 2);
    }
    for (auto* q : g) OK(gmm_destroy(q));
  }
  OK(gmm_destroy(big));
  // two executors, 12 streams each, each stream in turn; then one stream of them alone
  gmm_exec* x[2] = {};
  for (auto& e : x) OK(gmm_exec_create(0, 2, &e));
  for (int i = 0; i < 24; ++i) OK(gmm_exec_attach(x[i % 2], h[i], nullptr));
  uint8_t* rgb = pinned(W * H * 3);
  uint16_t* depth = reinterpret_cast<uint16_t*>(pinned(W * H * 2));
  for (int i = 0; i < 72; ++i) {
    (void)tick(x[i % 2], {{h[i % 24], rgb, depth, nullptr, nullptr, nullptr}});
    EXPECT(i < 24 || policy() == 2);
  }
  for (int i = 0; i < 4; ++i) {
    (void)tick(x[1], {{h[23], rgb, depth, nullptr, nullptr, nullptr}});
    EXPECT(policy() == 0);
  }
  for (auto* e : x) OK(gmm_exec_destroy(e));
  for (auto* g : h) OK(gmm_destroy(g));
}

// Reads and writes of states on one device run side by side, each in memory of its own.
static void state_io() {
  std::mutex mu;
  std::condition_variable cv;
  constexpr int kCalls = 24;
  const int sizes[][2] = {{64, 48}, {160, 120}, {320, 240}, {17, 13}};
  std::vector<gmm_handle*> h;
  std::vector<std::vector<double>> host(kCalls);
  for (int i = 0; i < kCalls; ++i) {
    h.push_back(handle(sizes[i % 4][0], sizes[i % 4][1], GMM_RGB | GMM_DEPTH, 5, i % 2 ? GMM_F16 : GMM_F32));
    size_t n = 0;
    OK(gmm_state_size(h[i], &n));
    host[i].assign(n, 0.0);
  }
  // a call whose copy takes its time does not hold up another one
  bool open = false, done = false;
  std::thread::id slow;
  rt().on_copy = [&](const void*, const void*, size_t) {
    std::unique_lock<std::mutex> lk(mu);
    if (std::this_thread::get_id() == slow) cv.wait(lk, [&] { return open; });
  };
  std::thread a([&] {
    {
      std::lock_guard<std::mutex> lk(mu);
      slow = std::this_thread::get_id();
    }
    cv.notify_all();
    OK(gmm_read_state(h[2], host[2].data(), nullptr));
  });
  std::this_thread::sleep_for(std::chrono::milliseconds(50));
  std::thread b([&] {
    OK(gmm_write_state(h[0], host[0].data(), nullptr));
    OK(gmm_read_state(h[0], host[0].data(), nullptr));
    std::lock_guard<std::mutex> lk(mu);
    done = true;
    cv.notify_all();
  });
  {
    std::unique_lock<std::mutex> lk(mu);
    EXPECT(cv.wait_for(lk, std::chrono::seconds(5), [&] { return done; }));
    open = true;
  }
  cv.notify_all();
  a.join();
  b.join();
  // what calls at the same time copy from and to the device never overlaps, until they have drained
  std::map<std::thread::id, std::pair<const char*, const char*>> busy;
  int overlaps = 0, most = 0;
  rt().on_copy = [&](const void* dst, const void* src, size_t n) {
    {
      std::lock_guard<std::mutex> lk(mu);
      const bool read = std::any_of(host.begin(), host.end(), [&](const std::vector<double>& v) {
        return dst >= v.data() && dst < v.data() + v.size();
      });
      const char* p = static_cast<const char*>(read ? src : dst);
      for (const auto& o : busy) overlaps += o.first != std::this_thread::get_id() && p < o.second.second && o.second.first < p + n;
      busy[std::this_thread::get_id()] = {p, p + n};
      most = std::max(most, static_cast<int>(busy.size()));
    }
    std::this_thread::sleep_for(std::chrono::milliseconds(2));
  };
  rt().on_sync = [&] {
    std::lock_guard<std::mutex> lk(mu);
    busy.erase(std::this_thread::get_id());
  };
  std::vector<std::thread> calls;
  for (int i = 0; i < kCalls; ++i)
    calls.emplace_back([&, i] {
      OK(gmm_read_state(h[i], host[i].data(), nullptr));
      OK(gmm_write_state(h[i], host[i].data(), nullptr));
    });
  for (auto& t : calls) t.join();
  EXPECT(overlaps == 0);
  EXPECT(most > 4);
  rt().on_copy = nullptr;
  rt().on_sync = nullptr;
  for (auto* g : h) OK(gmm_destroy(g));
}

// The autotuner times every launch once: candidates that come to the same blocks on the same pixels
// are one.
static void autotune() {
  void* mem = nullptr;
  (void)hipMalloc(&mem, 1 << 23);
  uint8_t* d = static_cast<uint8_t*>(mem);
  uint64_t* m = reinterpret_cast<uint64_t*>(mem);
  const auto trials = [&](int w, int h, int n) {
    std::vector<gmm_handle*> g;
    for (int i = 0; i < n; ++i) g.push_back(handle(w, h));
    const std::vector<gmm_stream_io> io(n, {d, 3 * w, reinterpret_cast<uint16_t*>(d), 2 * w, m, m, nullptr});
    gmm_batch* b = nullptr;
    OK(gmm_batch_create(g.data(), n, 1, &b));
    OK(gmm_batch_set_frames(b, 0, io.data(), nullptr));
    const size_t before = rt().launches.size();
    gmm_batch_tuning best{};
    OK(gmm_batch_autotune(b, 0, nullptr, &best, nullptr));
    const size_t made = rt().launches.size() - before;
    gmm_batch_tuning now{};
    OK(gmm_batch_get_tuning(b, &now));
    EXPECT(std::memcmp(&now, &best, sizeof now) == 0);
    OK(gmm_batch_destroy(b));
    for (auto* x : g) OK(gmm_destroy(x));
    return made / 2;  // a warm-up and a timed launch each
  };
  // 256 threads: 2 or 4 blocks a CU walk, more are a block per tile; 512: 2 walk. Five tile sizes each.
  EXPECT(trials(1920, 1080, 16) == 15 + 10);
  // so few pixels that every tile has a block whatever the blocks per CU: the five tile sizes are left
  EXPECT(trials(64, 64, 2) == 5 + 5);
}

// A batch has page-locked staging memory only where descriptors are copied from it: above 32 streams.
static void staging() {
  std::vector<gmm_handle*> h;
  for (int i = 0; i < 33; ++i) h.push_back(handle(64, 48, GMM_RGB));
  for (int n : {1, 32, 33}) {
    const size_t before = host_allocations();
    gmm_batch* b = nullptr;
    OK(gmm_batch_create(h.data(), n, 3, &b));
    EXPECT(host_allocations() - before == (n > 32 ? 3u : 0u));
    void* mem = nullptr;
    (void)hipMalloc(&mem, 1 << 16);
    const std::vector<gmm_stream_io> io(n, {static_cast<uint8_t*>(mem), 3 * 64, nullptr, 0, static_cast<uint64_t*>(mem), nullptr, nullptr});
    const size_t copies = rt().h2d;
    for (int slot = 0; slot < 3; ++slot) {
      OK(gmm_batch_set_frames(b, slot, io.data(), nullptr));
      OK(gmm_batch_run(b, slot, nullptr));
    }
    EXPECT(rt().h2d - copies == (n > 32 ? 3u : 0u));
    OK(gmm_batch_destroy(b));
    EXPECT(host_allocations() == before);
  }
  for (auto* g : h) OK(gmm_destroy(g));
}

int main(int argc, char** argv) {
  const std::map<std::string, std::function<void()>> checks = {
      {"gap", gap},
      {"coherence", coherence},
      {"overlap", overlap},
      {"detach", detach},
      {"round_trip", round_trip},
      {"exec_tuning", exec_tuning},
      {"residency", residency},
      {"cache_policy", cache_policy},
      {"state_io", state_io},
      {"autotune", autotune},
      {"staging", staging},
  };
  for (int i = 1; i < argc; ++i) {
    const auto it = checks.find(argv[i]);
    if (it == checks.end()) return std::printf("no check %s\n", argv[i]), 2;
    it->second();
  }
  std::printf(g_bad ? "%d failed\n" : "routes ok\n", g_bad);
  return g_bad ? 1 : 0;
}
