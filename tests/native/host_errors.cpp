// What plora_batch_begin leaves behind when a HIP call of it fails, how a batch's image travels and which items its lists
// hold, on the CPU against the stand-in HIP runtime (fake_hip.*).  One check per name given on the command line.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "fake_hip.h"
#include "plora.h"
#include "plora_internal.h"

#define CHECK(c) do { if (!(c)) { std::printf("CHECK failed at line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

namespace {
int g_image_launches = 0;             // images sent by a kernel
int g_image_fault_in = 0;             // > 0: that many launches from now, one is queued and reports an error all the same
int g_image_checks = 0;               // image kernels that have run
hipStream_t g_image_stream = nullptr; // stream of the last one
long g_fused_runs = 0;
int g_items[2][4];                    // [op][kind]: records that the launches read
int g_shrink_mode = -1, g_shrink_lone = 0, g_shrink_shared = 0;  // of the last launch
std::vector<std::pair<int, std::vector<int32_t>>> g_rest;  // cooperative expand launches: an item's rank, and the head of the page table it gives
}  // namespace

namespace plora {
void count_items(int op, const LaunchArgs& a, hipStream_t st) {
  fakehip::enqueue_kernel(st, [=] {
    for (int i = 0; i < a.n_items; ++i)
      if (a.items[i].kind >= 0) { CHECK((a.items[i].kind & 0xff) < 4); ++g_items[op][a.items[i].kind & 0xff]; }
  });
}
hipError_t launch_shrink(int dtype, const LaunchArgs& a, const SlotPtrs&, int, int mode, hipStream_t st, hipEvent_t, hipEvent_t) {
  g_shrink_mode = mode;
  g_shrink_lone = a.n_lone;
  if (a.n_lone > 0)  // single records of matrix-core items (or padding), then whole blocks without
    fakehip::enqueue_kernel(st, [=] {
      CHECK(a.n_items >= a.n_lone && (a.n_items - a.n_lone) % 4 == 0);
      for (int i = 0; i < a.n_items; ++i) CHECK(a.items[i].kind == -1 || ((a.items[i].kind & 0xff) > 0) == (i < a.n_lone));
      CHECK(dtype != PLORA_F32);
      for (int i = 0; i < a.n_lone; ++i) CHECK(a.items[i].kind == -1 || (a.items[i].kind & 0xff) == 1);
    });
  g_shrink_shared = a.slot_fastest;
  if (mode == kModeShrinkPanel)  // block i runs on XCD i % 8, whatever the slots: the row panels of a token tile on one of them
    fakehip::enqueue_kernel(st, [=] {
      std::map<int, int> xcd;  // of a tile, by its first token
      for (int i = 0; i < a.n_items; i += 4)
        if ((a.items[i].kind & 0xff) == 2) CHECK(xcd.emplace(a.items[i].tok[0], i / 4 % kXcds).first->second == i / 4 % kXcds);
    });
  count_items(0, a, st);
  return hipSuccess;
}
hipError_t launch_expand(int, const LaunchArgs& a, const SlotPtrs&, int, int, int mode, hipStream_t st, hipEvent_t, hipEvent_t) {
  count_items(1, a, st);
  if (mode == kModeCoop)
    fakehip::enqueue_kernel(st, [=] {
      for (int i = 0; i < a.n_items; ++i) {
        CHECK(!(a.items[i].kind & kItemContig));
        g_rest.push_back({a.items[i].rank, std::vector<int32_t>(a.pt + a.items[i].pt_off, a.pt + a.items[i].pt_off + a.items[i].rank)});
      }
    });
  return hipSuccess;
}
hipError_t launch_scatter(const uint8_t*, uint8_t*, int, uint64_t, const int32_t*, uint32_t, hipStream_t) { return hipSuccess; }
// When the stream reaches it, the page-locked image has to be what it was when the kernel was queued.
hipError_t launch_copy_image(const void* src, void* dst, size_t bytes, hipStream_t st) {
  auto then = std::make_shared<std::vector<uint8_t>>((const uint8_t*)src, (const uint8_t*)src + bytes);
  fakehip::enqueue_kernel(st, [=] {
    CHECK(std::memcmp(src, then->data(), bytes) == 0);
    std::memcpy(dst, src, bytes);
    ++g_image_checks;
  });
  ++g_image_launches;
  g_image_stream = st;
  if (g_image_fault_in > 0 && --g_image_fault_in == 0) return hipErrorUnknown;
  return hipSuccess;
}
// The one-launch form's counters have to be clear when a batch object's first launch runs.
hipError_t launch_delta_queue(int, const FusedArgs& f, const FusedPtrs&, hipStream_t st, hipEvent_t, hipEvent_t) {
  const uint32_t* queue = f.queue;
  fakehip::enqueue_kernel(st, [=] {
    for (int i = 0; i < kQueueWords; ++i) CHECK(queue[i] == 0);
    ++g_fused_runs;
  });
  return hipSuccess;
}
uint64_t static_scratch_bytes() { return 0; }
hipError_t static_scratch(void**) { return hipErrorNotSupported; }
}  // namespace plora

namespace {
struct Fixture {
  plora_pool* p = nullptr;
  hipStream_t st = nullptr, other = nullptr, copy = nullptr;
  void *blob = nullptr, *x = nullptr, *v = nullptr, *y = nullptr;
  explicit Fixture(int dtype = PLORA_BF16) {
    const int32_t d_in[1] = {64}, d_out[1] = {32};
    plora_layout lay{1, d_in, d_out, dtype, 4, 16};
    CHECK(plora_pool_create(4096, 16, &lay, nullptr, 0, &p) == PLORA_OK);
    for (auto* s : {&st, &other, &copy}) CHECK(hipStreamCreateWithFlags(s, hipStreamNonBlocking) == hipSuccess);
    CHECK(hipHostMalloc(&blob, plora_adapter_bytes(p, 16), 0) == hipSuccess);
    for (void** q : {&x, &v, &y}) CHECK(hipMalloc(q, 1 << 16) == hipSuccess);
    for (int i = 0; i < 3; ++i) CHECK(plora_load_adapter(p, i, 16, 1.f, blob, copy, nullptr, nullptr) == PLORA_OK);
    fakehip::drain();
  }
  ~Fixture() {
    CHECK(plora_pool_destroy(p) == PLORA_OK);
    CHECK(hipHostFree(blob) == hipSuccess);
    for (void* q : {x, v, y}) CHECK(hipFree(q) == hipSuccess);
    for (hipStream_t s : {st, other, copy}) CHECK(hipStreamDestroy(s) == hipSuccess);
  }
  // one batch of n tokens of adapter a on stream s, begun and ended (nothing runs); the begin's result
  int batch(int a, int n, hipStream_t s) {
    std::vector<int32_t> t2a(n, a);
    plora_batch* b = nullptr;
    const int rc = plora_batch_begin(p, t2a.data(), n, s, &b);
    if (rc == PLORA_OK) CHECK(plora_batch_end(p, b) == PLORA_OK);
    return rc;
  }
  // the same with its delta, run to the end: g_items says what the lists held
  void delta(const std::vector<int32_t>& t2a) {
    plora_batch* b = nullptr;
    const void* xs = x;
    float* vs = (float*)v;
    void* ys = y;
    std::memset(g_items, 0, sizeof(g_items));
    CHECK(plora_batch_begin(p, t2a.data(), (int32_t)t2a.size(), st, &b) == PLORA_OK);
    CHECK(plora_delta(p, b, 0, 1, &xs, &vs, &ys, st) == PLORA_OK);
    CHECK(plora_batch_end(p, b) == PLORA_OK);
    fakehip::drain();
  }
  void recycled() {  // a batch object whose first image has passed
    CHECK(plora_pool_set_option(p, "batches_per_marker", 1) == PLORA_OK);
    CHECK(batch(0, 8, st) == PLORA_OK);
    fakehip::drain();
    g_image_launches = g_image_checks = 0;
  }
};

// A begin that fails after its image was queued must not hand the image's buffers to the next batch.
void image_in_flight() {
  for (int how = 0; how < 3; ++how) {
    Fixture f;
    f.recycled();
    if (how == 0) g_image_fault_in = 1;  // the launch itself is reported as failed
    if (how == 1) {                      // the wait for an adapter that is still loading fails
      CHECK(plora_load_adapter(f.p, 3, 16, 1.f, f.blob, f.copy, nullptr, nullptr) == PLORA_OK);
      fakehip::fail_wait_in(1);
    }
    if (how < 2) CHECK(f.batch(how == 1 ? 3 : 1, 8, f.st) == PLORA_ERR_HIP);
    if (how == 2) {  // an image for the side stream (the first of a second object), and the wait for it fails
      int32_t t2a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      plora_batch* open = nullptr;
      CHECK(plora_batch_begin(f.p, t2a, 8, f.st, &open) == PLORA_OK);  // holds the recycled object
      fakehip::fail_wait_in(1);
      CHECK(f.batch(1, 8, f.st) == PLORA_ERR_HIP);
      CHECK(plora_batch_end(f.p, open) == PLORA_OK);
    }
    g_image_fault_in = 0;
    fakehip::fail_wait_in(0);
    // more batches, also with larger images and on another stream, while the first image still waits
    for (int k = 0; k < 4; ++k) CHECK(f.batch(2, 5 + 400 * k, k % 2 ? f.other : f.st) == PLORA_OK);
    fakehip::drain();
    CHECK(g_image_checks == g_image_launches && (how == 2 || g_image_launches >= 1));
    CHECK(f.batch(2, 16, f.st) == PLORA_OK);  // and the objects come back into use
    fakehip::drain();
  }
}

// An error that the caller has not looked at is still there after a begin, whichever way the image goes.
void callers_error() {
  Fixture f;
  CHECK(plora_pool_set_option(f.p, "batches_per_marker", 1) == PLORA_OK);
  struct { int n; bool capturing; int kernels; } way[] = {{8, false, 0}, {8, false, 1}, {60000, false, 0}, {8, true, 0}};
  for (auto& w : way) {  // the first of an object, a small one by kernel, one over the limit, one on a stream under capture
    fakehip::set_capturing(f.st, w.capturing);
    g_image_launches = 0;
    fakehip::set_last_error(hipErrorInvalidDevice);
    CHECK(f.batch(0, w.n, f.st) == PLORA_OK);
    CHECK(hipGetLastError() == hipErrorInvalidDevice);
    CHECK(g_image_launches == w.kernels);
    fakehip::set_capturing(f.st, false);
    fakehip::drain();
  }
}

// A batch object whose counters could not be cleared at first clears them later, and always ahead of its first launch.
void counters_cleared() {
  for (int how = 0; how < 2; ++how) {
    Fixture f;
    CHECK(plora_pool_set_option(f.p, "fused_max_tasks", 1 << 20) == PLORA_OK);
    if (how == 0) fakehip::fail_memset_in(1);
    if (how == 1) fakehip::fail_wait_in(1);  // the batch stream's wait for the image, behind the clearing
    CHECK(f.batch(0, 8, f.st) == PLORA_ERR_HIP);
    fakehip::fail_memset_in(0);
    fakehip::fail_wait_in(0);
    g_fused_runs = 0;
    for (int k = 0; k < 3; ++k) {
      std::vector<int32_t> t2a(8, k);
      plora_batch* b = nullptr;
      const void* x = f.x;
      float* v = (float*)f.v;
      void* y = f.y;
      CHECK(plora_batch_begin(f.p, t2a.data(), 8, f.st, &b) == PLORA_OK);
      CHECK(plora_delta(f.p, b, 0, 1, &x, &v, &y, f.st) == PLORA_OK);
      CHECK(plora_batch_end(f.p, b) == PLORA_OK);
      while (fakehip::step(f.st)) {}  // the batch stream as far as it gets without the others
    }
    fakehip::drain();
    CHECK(g_fused_runs == 3);
  }
}

// fp32 pools: an explicit threshold holds as it is given, for each operation by itself; unset, the library's own.
void fp32_thresholds() {
  struct { int shrink, expand; int64_t tokens; bool mfma_s, mfma_e; } want[] = {
    {-1, -1, 31, false, false}, {-1, -1, 32, false, true},  // (a lone group is too little for the shrink's)
    {1, -1, 8, true, false},    {-1, 1, 8, false, true},
    {32, -1, 31, false, false}, {32, -1, 32, true, true},  {16, -1, 16, true, false},
    {-1, 40, 39, false, false}, {-1, 40, 40, false, true}, {0, 0, 48, false, false},
  };
  for (auto& w : want) {
    Fixture f(PLORA_F32);
    for (const char* k : {"coop_max_workgroups_shrink", "coop_max_workgroups_expand"}) CHECK(plora_pool_set_option(f.p, k, 0) == PLORA_OK);
    if (w.shrink >= 0) CHECK(plora_pool_set_option(f.p, "mfma_min_tokens", w.shrink) == PLORA_OK);
    if (w.expand >= 0) CHECK(plora_pool_set_option(f.p, "mfma_min_tokens_expand", w.expand) == PLORA_OK);
    f.delta(std::vector<int32_t>((size_t)w.tokens, 0));
    std::printf("thresholds %d %d, %d tokens: %d and %d matrix-core items\n", w.shrink, w.expand, (int)w.tokens, g_items[0][1], g_items[1][1]);
    CHECK((g_items[0][1] > 0) == w.mfma_s && (g_items[0][0] > 0) == !w.mfma_s);
    CHECK((g_items[1][1] > 0) == w.mfma_e && (g_items[1][0] > 0) == !w.mfma_e);
  }
}

// A prefill shrink takes panel items as such where they fill the GPU and cuts them where they do not.
void panel_route() {
  enum { kPanel, kCut, kCoop, kOther };
  struct { int rank, tiles, slots, distinct_x, limit, route; } want[] = {
    {64, 47, 4, 2, 32, kCut},  {64, 48, 4, 2, 32, kPanel}, {16, 48, 4, 2, 32, kPanel},
    {64, 255, 1, 1, 32, kCut}, {64, 256, 1, 1, 32, kPanel}, {16, 256, 1, 1, 32, kCut},
    {64, 63, 4, 4, 32, kCut},  {64, 64, 4, 4, 32, kPanel},  {16, 64, 4, 4, 32, kCut},
    {64, 1, 1, 1, 0, kPanel},  {16, 300, 8, 1, -1, kOther},           {64, 31, 4, 1, 32, kOther},
    {128, 190, 1, 1, 32, kCut},          {128, 192, 1, 1, 32, kPanel},          {128, 192, 8, 8, 32, kPanel},         {16, 32, 1, 1, 32, kCoop},           {16, 40, 1, 1, 32, kCut},
  };
  for (auto& w : want) {
    const int n_slots = 8;
    const std::vector<int32_t> d(n_slots, 64);
    plora_layout lay{n_slots, d.data(), d.data(), PLORA_BF16, 2, 128};
    plora_pool* p = nullptr;
    CHECK(plora_pool_create(4096, 128, &lay, nullptr, 0, &p) == PLORA_OK);
    CHECK(plora_pool_set_option(p, "panel_min_tiles_shrink", w.limit) == PLORA_OK);
    hipStream_t st = nullptr;
    CHECK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess);
    void* blob = nullptr;
    CHECK(hipHostMalloc(&blob, plora_adapter_bytes(p, 128), 0) == hipSuccess);
    std::memset(blob, 0, plora_adapter_bytes(p, 128));
    CHECK(plora_load_adapter(p, 0, w.rank, 1.f, blob, st, nullptr, nullptr) == PLORA_OK);
    std::vector<int32_t> t2a((size_t)w.tiles * 64 / (w.rank > 64 ? 2 : 1), 0);
    if (w.route != kCoop) t2a.resize(t2a.size() + 5, 0), t2a[0] = -1;  // some tokens for items of other kinds
    plora_batch* b = nullptr;
    CHECK(plora_batch_begin(p, t2a.data(), (int32_t)t2a.size(), st, &b) == PLORA_OK);
    std::vector<const void*> x(n_slots);
    std::vector<float*> v(n_slots, (float*)0x1000);
    for (int q = 0; q < n_slots; ++q) x[q] = (const void*)(uintptr_t)(0x10000 + 256 * (q * w.distinct_x / w.slots));
    CHECK(plora_shrink(p, b, 0, w.slots, x.data(), v.data(), st) == PLORA_OK);
    CHECK(plora_batch_end(p, b) == PLORA_OK);
    fakehip::drain();
    std::printf("rank %d, %d tiles, %d slots reading %d x, limit %d: mode %d, %d single records\n", w.rank, w.tiles, w.slots, w.distinct_x, w.limit, g_shrink_mode,
                g_shrink_lone);
    const int route = g_shrink_mode == plora::kModeShrinkPanel ? kPanel : g_shrink_mode == plora::kModeCoop ? kCoop : g_shrink_lone > 0 ? kCut : kOther;
    CHECK(route == w.route);
    CHECK(route != kPanel || g_shrink_shared == (4 * (w.slots - w.distinct_x) >= w.slots));  // slots that read one x side by side
    CHECK(plora_pool_destroy(p) == PLORA_OK);
    CHECK(hipHostFree(blob) == hipSuccess && hipStreamDestroy(st) == hipSuccess);
  }
}

// The same for fp32 shrink: matrix-core items where they fill the GPU, vector-ALU blocks where they do not.
void fp32_route() {
  enum { kMatrix, kVector, kCoop };
  struct { int adapters, tokens, rank, slots, set, route, d_in = 64; } want[] = {
    {16, 64, 64, 1, -1, kVector}, {16, 64, 64, 2, -1, kVector}, {16, 64, 64, 3, -1, kMatrix}, {16, 64, 64, 1, 16, kCoop},
    {64, 16, 8, 2, -1, kCoop},    {64, 16, 8, 4, -1, kVector},  {64, 16, 32, 5, -1, kVector}, {64, 16, 32, 6, -1, kMatrix},
    {15, 64, 64, 8, -1, kVector},  // (60 items: not in the list)
    {32, 96, 16, 3, -1, kVector}, {32, 96, 16, 4, -1, kMatrix}, {32, 70, 16, 8, -1, kVector},  // (tiles that replace 16, and 12)
    {16, 256, 64, 1, -1, kMatrix},
    {64, 24, 16, 8, -1, kVector, 2040}, {64, 24, 16, 8, -1, kMatrix, 2048}, {64, 24, 16, 7, -1, kVector, 2048},  // (tiles that replace 12; slots kept apart)
  };
  for (auto& w : want) {
    const int n_slots = 8;
    const std::vector<int32_t> d_in(n_slots, w.d_in), d_out(n_slots, 64);
    plora_layout lay{n_slots, d_in.data(), d_out.data(), PLORA_F32, w.adapters, 64};
    plora_pool* p = nullptr;
    CHECK(plora_pool_create(65536, (8 + w.d_in / 64) * w.adapters, &lay, nullptr, 0, &p) == PLORA_OK);
    if (w.set >= 0) CHECK(plora_pool_set_option(p, "mfma_min_tokens", w.set) == PLORA_OK);
    hipStream_t st = nullptr;
    CHECK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess);
    void* blob = nullptr;
    CHECK(hipHostMalloc(&blob, plora_adapter_bytes(p, 64), 0) == hipSuccess);
    std::memset(blob, 0, plora_adapter_bytes(p, 64));
    std::vector<int32_t> t2a;
    for (int i = 0; i < w.adapters; ++i) {
      CHECK(plora_load_adapter(p, i, w.rank, 1.f, blob, st, nullptr, nullptr) == PLORA_OK);
      t2a.insert(t2a.end(), (size_t)w.tokens, i);
    }
    plora_batch* b = nullptr;
    std::memset(g_items, 0, sizeof(g_items));
    CHECK(plora_batch_begin(p, t2a.data(), (int32_t)t2a.size(), st, &b) == PLORA_OK);
    std::vector<const void*> x(n_slots, (const void*)0x10000);
    std::vector<float*> v(n_slots, (float*)0x1000);
    CHECK(plora_shrink(p, b, 0, w.slots, x.data(), v.data(), st) == PLORA_OK);
    CHECK(plora_batch_end(p, b) == PLORA_OK);
    fakehip::drain();
    std::printf("%d adapters, %d tokens each, rank %d, %d slots: mode %d, %d single records\n", w.adapters, w.tokens, w.rank, w.slots, g_shrink_mode, g_shrink_lone);
    const int route = g_shrink_mode == plora::kModeCoop ? kCoop : g_items[0][1] > 0 ? kMatrix : kVector;
    CHECK(route == w.route);
    CHECK(route != kVector || g_items[0][0] == w.adapters * ((w.tokens + 3) / 4) * w.rank / 8);
    CHECK(plora_pool_destroy(p) == PLORA_OK);
    CHECK(hipHostFree(blob) == hipSuccess && hipStreamDestroy(st) == hipSuccess);
  }
}
// What a panel batch has besides its 64-token blocks goes to the cooperative expand with the page tables of its own adapters, wherever
// those lie between the adapters of the blocks.
void rest_tables() {
  const int32_t d = 1024, ranks[5] = {40, 3, 64, 5, 7}, tokens[5] = {200, 3, 130, 4, 1};
  plora_layout lay{1, &d, &d, PLORA_BF16, 5, 64};
  plora_pool* p = nullptr;
  CHECK(plora_pool_create(4096, 128, &lay, nullptr, 0, &p) == PLORA_OK);  // a page per rank
  CHECK(plora_pool_set_option(p, "contig_fast_path", 0) == PLORA_OK);
  CHECK(plora_pool_set_option(p, "panel_min_blocks", 1) == PLORA_OK);
  hipStream_t st = nullptr;
  CHECK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess);
  void* blob = nullptr;
  CHECK(hipHostMalloc(&blob, plora_adapter_bytes(p, 64), 0) == hipSuccess);
  std::memset(blob, 0, plora_adapter_bytes(p, 64));
  std::vector<int32_t> t2a;
  for (int i = 0; i < 5; ++i) {
    CHECK(plora_load_adapter(p, i, ranks[i], 1.f, blob, st, nullptr, nullptr) == PLORA_OK);
    t2a.insert(t2a.end(), (size_t)tokens[i], i);
  }
  plora_batch* b = nullptr;
  CHECK(plora_batch_begin(p, t2a.data(), (int32_t)t2a.size(), st, &b) == PLORA_OK);
  const float* v = (const float*)0x1000;
  void* y = (void*)0x10000;
  g_rest.clear();
  CHECK(plora_expand(p, b, 0, 1, &v, &y, st) == PLORA_OK);
  CHECK(plora_batch_end(p, b) == PLORA_OK);
  fakehip::drain();
  CHECK(g_rest.size() == 3);  // adapters 4, 3 and 1, longest first
  for (int k = 0; k < 3; ++k) {
    const int i = k == 0 ? 4 : k == 1 ? 3 : 1;
    const int32_t* pt = nullptr;
    uint32_t n = 0;
    CHECK(plora_adapter_pages(p, i, &pt, &n) == PLORA_OK && n == (uint32_t)ranks[i]);
    CHECK(g_rest[k].first == ranks[i] && g_rest[k].second == std::vector<int32_t>(pt, pt + n));
  }
  CHECK(plora_pool_destroy(p) == PLORA_OK);
  CHECK(hipHostFree(blob) == hipSuccess && hipStreamDestroy(st) == hipSuccess);
}
}  // namespace

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    const std::string name = argv[i];
    if (name == "image_in_flight") image_in_flight();
    else if (name == "callers_error") callers_error();
    else if (name == "counters_cleared") counters_cleared();
    else if (name == "fp32_thresholds") fp32_thresholds();
    else if (name == "panel_route") panel_route();
    else if (name == "fp32_route") fp32_route();
    else if (name == "rest_tables") rest_tables();
    else return 2;
    std::printf("%s OK\n", name.c_str());
  }
  return 0;
}
