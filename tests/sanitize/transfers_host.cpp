// The host side of loads, layered loads and stores on a stand-in for the HIP
// runtime, meant to be built with AddressSanitizer and
// UndefinedBehaviorSanitizer.
//
// Test infrastructure only: it links the product's ea_api.cpp and
// ea_tier_meta.cpp with the few runtime calls they make, done synchronously
// on host memory, and a plain C++ piece copy in the kernel's place.  Device
// memory can be made to run out and every allocation is counted.  Calls of
// more pages than fit the kernel arguments must give the right pages with and
// without device memory for their index arrays, must leave no error behind
// for the caller's next runtime call, and must allocate nothing once a plain
// load of as many pages has run.  Caches of few layers, whose calls the copy to
// device memory would only make longer, must make none.  Scale words must
// arrive whether units move their own or groups of eight, which is chosen by
// direction and piece size.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <iterator>
#include <numeric>
#include <map>
#include <random>
#include <vector>

#include "ea.h"
#include "ea_internal.hpp"

namespace {

bool g_no_device_memory = false;
int64_t g_allocations = 0;
hipError_t g_last = hipSuccess;
std::map<const uint8_t *, size_t> g_device;  // live device allocations and their sizes
int64_t g_from_device = 0;  // copies whose index arrays lie in device memory
int32_t g_scale_layers = 0;  // of the last copy

hipError_t done(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}

bool in_device(const void *p) {
  const uint8_t *b = static_cast<const uint8_t *>(p);
  auto it = g_device.upper_bound(b);
  return it != g_device.begin() && b < std::prev(it)->first + std::prev(it)->second;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 8;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  ++g_allocations;
  if (g_no_device_memory) return done(hipErrorOutOfMemory);
  *p = std::malloc(n);
  g_device[static_cast<uint8_t *>(*p)] = n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  g_device.erase(static_cast<uint8_t *>(p));
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  ++g_allocations;
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace ea {
hipError_t probe_xcd_round_robin(int, bool *ok) { *ok = true; return hipSuccess; }
hipError_t launch_layer_checksum(const uint8_t *, const uint8_t *, int64_t, int64_t, int32_t,
                                 const int32_t *, int32_t, uint64_t *, hipStream_t) {
  return hipSuccess;
}
// The pieces and scale words of layers [begin, begin + count), as the kernel
// takes them: entry i is page i % C of its slot.
hipError_t launch_piece_copy(const PieceCopy &a, const InlineIdx *inl, const ArgPages *, int dir,
                             int, int64_t, hipStream_t) {
  if (inl == nullptr && in_device(a.pages) && in_device(a.slot_idx)) ++g_from_device;
  g_scale_layers = a.scale_layers;
  const auto move = [dir](uint8_t *cache, uint8_t *slot, int64_t n) {
    std::memcpy(dir == kToSlots ? slot : cache, dir == kToSlots ? cache : slot, (size_t)n);
  };
  for (int64_t i = 0; i < a.n; ++i) {
    const int64_t page = inl ? inl->pages[i] : a.pages[i];
    uint8_t *slot = a.slots + (inl ? inl->slots[i] : a.slot_idx[i]) * a.slot_bytes;
    for (int64_t l = a.layer_begin; l < a.layer_begin + a.layer_count; ++l) {
      const int64_t at = l * a.chunk + i % a.chunk;
      move(a.cache + (l * a.num_pages + page) * a.piece_bytes, slot + at * a.piece_bytes,
           a.piece_bytes);
      if (a.scales == nullptr || l % a.scale_layers != 0) continue;
      for (int64_t k = 0; k < a.scale_layers && l + k < a.num_layers; ++k)
        move(a.scales + ((l + k) * a.num_pages + page) * 8,
             slot + a.payload_bytes + (at + k * a.chunk) * 8, 8);
    }
  }
  return hipSuccess;
}
}  // namespace ea

namespace {

[[noreturn]] void fail(const char *what, int64_t n) {
  std::fprintf(stderr, "WRONG: %s (%lld pages)\n", what, (long long)n);
  std::exit(1);
}

constexpr int32_t kPages = 9000;
constexpr int64_t kPiece = 2 * 16 * 1 * 1 * 1;

struct Rig {
  int32_t layers;
  std::vector<uint8_t> kv;
  ea_cache *cache = nullptr;
  ea_tier *tier = nullptr;
  uint8_t *host = nullptr;
  std::vector<hipEvent_t> events;
  std::mt19937 r;

  Rig(unsigned seed, int32_t L) : layers(L), kv((size_t)(L * kPages * kPiece)), r(seed) {
    const ea_cache_desc d = [&] {
      ea_cache_desc x{};
      x.base = kv.data();
      x.num_pages = kPages;
      x.num_layers = layers;
      x.page_tokens = 16;
      x.num_kv_heads = 1;
      x.head_dim = 1;
      x.elem_bytes = 1;
      return x;
    }();
    if (ea_cache_create(&d, &cache) != EA_OK) fail("cache", 0);
    if (ea_tier_create(cache, kPages * layers * kPiece, -1, &tier) != EA_OK) fail("tier", 0);
    ea_tier_info info;
    if (ea_tier_get_info(tier, &info) != EA_OK) fail("info", 0);
    host = static_cast<uint8_t *>(info.host_base);
    for (int64_t i = 0; i < info.capacity_slots * info.slot_bytes; ++i) host[i] = (uint8_t)r();
    for (int l = 0; l < layers; ++l) {
      hipEvent_t e;
      (void)hipEventCreate(&e);
      events.push_back(e);
    }
  }
  ~Rig() {
    if (ea_tier_destroy(tier) != EA_OK || ea_cache_destroy(cache) != EA_OK) fail("destroy", 0);
    for (hipEvent_t e : events) (void)hipEventDestroy(e);
  }

  void load(int32_t n, bool layered) {
    std::vector<int64_t> slots(kPages);
    std::vector<int32_t> pages(kPages);
    std::iota(slots.begin(), slots.end(), 0);
    std::iota(pages.begin(), pages.end(), 0);
    std::shuffle(slots.begin(), slots.end(), r);
    std::shuffle(pages.begin(), pages.end(), r);
    std::vector<uint8_t> want = kv;
    for (int32_t i = 0; i < n; ++i)
      for (int64_t l = 0; l < layers; ++l)
        std::memcpy(&want[(size_t)((l * kPages + pages[i]) * kPiece)],
                    host + (slots[i] * layers + l) * kPiece, kPiece);
    const int rc = layered ? ea_load_blocks_layered(tier, cache, slots.data(), pages.data(), n,
                                                    nullptr, events.data(), layers)
                           : ea_load_blocks(tier, cache, slots.data(), pages.data(), n, nullptr);
    if (rc != EA_OK) fail(layered ? "layered load refused" : "load refused", n);
    if (kv != want) fail("pages differ", n);
    if (hipGetLastError() != hipSuccess) fail("an error is left behind", n);
  }
};

// Pages and scale words through store, load and layered load, and the group
// of layers whose words move together each way.
void scale_words(int32_t layers, int32_t head_dim, int32_t chunk, int32_t n, int32_t group_out,
                 int32_t group_in) {
  const int64_t piece = 32 * (int64_t)head_dim, pages = 3 * n * chunk;
  std::vector<uint8_t> kv((size_t)(layers * pages * piece)), sc((size_t)(layers * pages * 8));
  std::mt19937 r((unsigned)(layers * 131 + head_dim + chunk));
  for (auto &b : kv) b = (uint8_t)r();
  for (auto &b : sc) b = (uint8_t)r();
  ea_cache_desc d{};
  d.base = kv.data();
  d.scale_base = sc.data();
  d.num_pages = (int32_t)pages;
  d.num_layers = layers;
  d.page_tokens = 16;
  d.num_kv_heads = 1;
  d.head_dim = head_dim;
  d.elem_bytes = 1;
  ea_cache *cache = nullptr;
  ea_tier *tier = nullptr;
  if (ea_cache_create(&d, &cache) != EA_OK) fail("cache", n);
  const int64_t slot = layers * chunk * piece + (layers * chunk * 8 + 255) / 256 * 256;
  if (ea_tier_create_chunked(cache, chunk, n * slot, -1, &tier) != EA_OK) fail("tier", n);
  std::vector<hipEvent_t> events((size_t)layers);
  for (auto &e : events) (void)hipEventCreate(&e);
  std::vector<int64_t> slots((size_t)n);
  std::vector<int32_t> ids((size_t)pages);
  std::iota(slots.begin(), slots.end(), 0);
  std::iota(ids.begin(), ids.end(), 0);
  std::shuffle(slots.begin(), slots.end(), r);
  std::shuffle(ids.begin(), ids.end(), r);
  const int32_t m = n * chunk;
  std::vector<uint8_t> want = kv, want_sc = sc;
  for (int32_t i = 0; i < 2 * m; ++i)
    for (int64_t l = 0; l < layers; ++l) {
      const int64_t from = l * pages + ids[i % m], to = l * pages + ids[m + i];
      std::memcpy(&want[to * piece], &kv[from * piece], (size_t)piece);
      std::memcpy(&want_sc[to * 8], &sc[from * 8], 8);
    }
  if (ea_store_blocks(cache, tier, ids.data(), slots.data(), nullptr, n, nullptr) != EA_OK)
    fail("store", n);
  if (g_scale_layers != group_out) fail("group of the store", head_dim);
  if (ea_load_blocks(tier, cache, slots.data(), ids.data() + m, n, nullptr) != EA_OK)
    fail("load", n);
  if (g_scale_layers != group_in) fail("group of the load", head_dim);
  if (ea_load_blocks_layered(tier, cache, slots.data(), ids.data() + 2 * m, n, nullptr,
                             events.data(), layers) != EA_OK)
    fail("layered load", n);
  if (g_scale_layers != group_in) fail("group of the layered load", head_dim);
  if (kv != want || sc != want_sc) fail("pages or scales differ", n);
  for (auto &e : events) (void)hipEventDestroy(e);
  if (ea_tier_destroy(tier) != EA_OK || ea_cache_destroy(cache) != EA_OK) fail("destroy", n);
}

}  // namespace

int main() {
  {  // device memory at hand: the layers' copies read the indices from it
    Rig g(1, 9);
    for (int32_t n : {1, 32, 33, 40, 4096}) {
      const int64_t before = g_from_device;
      g.load(n, true);
      if ((n > 32 ? g.layers : 0) != g_from_device - before) fail("indices not on the device", n);
    }
    g.load(5000, true);  // the ring grows
    for (int k = 0; k < 6; ++k) g.load(4100 + k, true);
  }
  {  // none left, from the first call on, and again once the ring grows
    Rig g(2, 8);
    g_no_device_memory = true;
    for (int32_t n : {33, 40, 4096, 4097}) g.load(n, true);
    g.load(5000, false);
    g_no_device_memory = false;
    g.load(8000, true);
    g_no_device_memory = true;
    g.load(9000, true);
    g_no_device_memory = false;
  }
  for (int32_t layers : {2, 7, 8}) {
    // a plain load has made the ring: layered loads of any size in it allocate
    // nothing, and a few layers read the ring itself
    Rig g(3, layers);
    g.load(40, false);
    const int64_t allocations = g_allocations, before = g_from_device;
    for (int32_t n : {33, 40, 4096}) g.load(n, true);
    if (g_allocations != allocations) fail("allocated again", 40);
    if (g_from_device != before + (layers >= 8 ? 3 * layers : 0)) fail("indices copied", layers);
  }
  // layers around the groups' ends; one page per slot, and chunks, whose words
  // are not neighbours
  for (int32_t layers : {1, 7, 8, 9, 17})
    for (int32_t n : {3, 40}) {
      scale_words(layers, 65, 1, n, 8, 8);
      scale_words(layers, 2, 16, n, 1, 1);
    }
  // stores of pieces of 2,048 bytes and the next larger ones, around 5 MiB
  scale_words(17, 64, 1, 200, 8, 8);
  scale_words(17, 65, 1, 148, 8, 8);
  scale_words(17, 65, 1, 149, 1, 8);
  if (!g_device.empty()) fail("device memory left", 0);
  std::puts("ok");
  return 0;
}
