// Host side of the library on a stand-in for the HIP runtime: this program
// defines the runtime functions that liblv.so calls (its definitions come
// before the real ones in symbol lookup), with two devices, memory that is only
// reserved, kernels that do nothing, and a log of what was called.  It checks
// what no single GPU can show safely: which device a destruction waits for,
// what orders streams after an error, launch sizes at the limits of the sizes
// that are accepted, and how much device memory a call takes.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <string>
#include <vector>

#include "lv.h"

namespace {

struct Dim3 {
  uint32_t x, y, z;
};
enum Kind { kLaunch, kSync, kRecord, kWait, kMemset, kMalloc };
struct Op {
  Kind kind;
  std::string name;  // kernel
  void* p;           // stream, event or memory
  void* stream;
  uint64_t size;     // threads in the grid, or bytes
  uint64_t launched; // the largest grid dimension in threads
  int device;
  const void* arg0;
};

std::vector<Op>& ops() {
  static std::vector<Op> v;
  return v;
}
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<void*, size_t>& blocks() {
  static std::map<void*, size_t> m;
  return m;
}
int g_device = 0;
uint64_t g_bytes = 0, g_peak = 0;
uint64_t fail_size = 0;  // allocations of this many bytes fail after fail_skip of them
int fail_skip = 0;
std::string fail_after;  // the launch of this kernel leaves an error
int g_error = 0;
Dim3 c_grid, c_block;
size_t c_shmem;
void* c_stream;

int get(void** p, size_t bytes) {
  if (fail_size && bytes == fail_size && fail_skip-- <= 0) return 2;  // out of memory
  *p = mmap(nullptr, bytes ? bytes : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) return 2;
  blocks()[*p] = bytes ? bytes : 1;
  g_bytes += bytes;
  if (g_bytes > g_peak) g_peak = g_bytes;
  ops().push_back({kMalloc, "", *p, nullptr, bytes, 0, g_device, nullptr});
  return 0;
}
int put(void* p) {
  auto it = blocks().find(p);
  if (it == blocks().end()) return 1;
  g_bytes -= it->second;
  munmap(p, it->second);
  blocks().erase(it);
  return 0;
}

}  // namespace

extern "C" {
typedef void* stream_t;
typedef void* event_t;

void** __hipRegisterFatBinary(const void*) {
  static void* m = nullptr;
  return &m;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shmem, stream_t s) {
  c_grid = g, c_block = b, c_shmem = shmem, c_stream = s;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shmem, stream_t* s) {
  *g = c_grid, *b = c_block, *shmem = c_shmem, *s = c_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t, stream_t s) {
  const std::string& name = kernels()[f];
  const uint64_t x = (uint64_t)g.x * b.x, y = (uint64_t)g.y * b.y, z = (uint64_t)g.z * b.z;
  const uint64_t most = x > y ? (x > z ? x : z) : (y > z ? y : z);
  ops().push_back({kLaunch, name, nullptr, s, x * y * z, most, g_device, args ? *(const void**)args[0] : nullptr});
  // the runtime refuses empty grids and dimensions of 2^32 threads or more
  if (most >= (1ull << 32) || x * y * z == 0) g_error = 9;
  if (!fail_after.empty() && name.find(fail_after) != std::string::npos) g_error = 719;
  return g_error;
}
int hipGetLastError() {
  const int e = g_error;
  g_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "error"; }
int hipGetDevice(int* d) {
  *d = g_device;
  return 0;
}
int hipSetDevice(int d) {
  g_device = d;
  return 0;
}
int hipDeviceSynchronize() {
  ops().push_back({kSync, "", nullptr, nullptr, 0, 0, g_device, nullptr});
  return 0;
}
int hipStreamSynchronize(stream_t) { return 0; }
int hipStreamWaitEvent(stream_t s, event_t e, unsigned) {
  ops().push_back({kWait, "", e, s, 0, 0, g_device, nullptr});
  return 0;
}
int hipStreamCreateWithFlags(stream_t* s, unsigned) {
  *s = malloc(1);
  return 0;
}
int hipStreamDestroy(stream_t s) {
  free(s);
  return 0;
}
int hipEventCreate(event_t* e) {
  *e = malloc(1);
  return 0;
}
int hipEventCreateWithFlags(event_t* e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(event_t e) {
  free(e);
  return 0;
}
int hipEventRecord(event_t e, stream_t s) {
  ops().push_back({kRecord, "", e, s, 0, 0, g_device, nullptr});
  return 0;
}
int hipEventSynchronize(event_t) { return 0; }
int hipEventElapsedTime(float* t, event_t, event_t) {
  *t = 0;
  return 0;
}
int hipMalloc(void** p, size_t n) { return get(p, n); }
int hipMallocAsync(void** p, size_t n, stream_t) { return get(p, n); }
int hipFree(void* p) { return put(p); }
int hipFreeAsync(void* p, stream_t) { return put(p); }
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(n ? n : 1, 1);
  return 0;
}
int hipHostFree(void* p) {
  free(p);
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static char buf[4096 * 4];
  *p = buf;
  return 0;
}
int hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = (size_t)288 << 30;
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) {
  if (kind != 3) memcpy(d, s, n);  // device to device: nothing reads it
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, stream_t) { return hipMemcpy(d, s, n, kind); }
int hipMemsetAsync(void* p, int, size_t n, stream_t s) {
  ops().push_back({kMemset, "", p, s, n, 0, g_device, nullptr});
  return 0;
}
}  // extern "C"

namespace {

#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      fprintf(stderr, "line %d: %s (%s)\n", __LINE__, #c, lv_last_error()); \
      exit(1);                                                          \
    }                                                                   \
  } while (0)

void* const S1 = reinterpret_cast<void*>(0x1000);
void* const S2 = reinterpret_cast<void*>(0x2000);

void* device_mem(size_t bytes) {
  void* p = nullptr;
  CHECK(get(&p, bytes) == 0);
  return p;
}

lv_scene* make_scene(int64_t n, void* s) {
  float* x = static_cast<float*>(device_mem(16 * (size_t)n));
  lv_scene* sc = nullptr;
  CHECK(lv_scene_create(x, x, x, x, n, nullptr, s, &sc) == LV_OK);
  return sc;
}

// n rows, `deg` edges each, all to column 0
lv_graph* make_graph(int n, int deg, void* s) {
  int32_t* rp = static_cast<int32_t*>(device_mem(4 * (size_t)(n + 1)));
  int32_t* col = static_cast<int32_t*>(device_mem(4 * (size_t)n * deg + 4));
  for (int i = 0; i <= n && deg; i++) rp[i] = i * deg;  // reserved memory is 0
  lv_graph* g = nullptr;
  CHECK(lv_graph_create_csr(n, (int64_t)n * deg, rp, col, col, LV_F32, s, &g) == LV_OK);
  return g;
}

// A graph is destroyed while another device is current: its own device is
// waited for before its buffers go to the cache, and the current one is kept.
void destroy_on_other_device() {
  g_device = 1;
  lv_graph* g = make_graph(100, 3, S1);
  float* x = static_cast<float*>(device_mem(4 * 100 * 8));
  CHECK(lv_diffuse(nullptr, g, x, LV_F32, 8, 2, x + 400, S1) == LV_OK);
  g_device = 0;
  const size_t at = ops().size();
  CHECK(lv_graph_destroy(g) == LV_OK);
  bool waited = false;
  for (size_t i = at; i < ops().size(); i++) waited = waited || (ops()[i].kind == kSync && ops()[i].device == 1);
  CHECK(waited);
  CHECK(g_device == 0);
}

// Calls on one graph share its buffers, also where a call fails half-way: what it
// has queued is ordered before the next call on another stream.
void order_after_failed_diffusion() {
  for (int launch = 0; launch < 2; launch++) {
    lv_scene* sc = make_scene(100, S1);
    lv_graph* g = make_graph(100, 3, S1);
    float* x = static_cast<float*>(device_mem(4 * 100 * 16));
    if (launch) {
      fail_after = "spmm";
    } else {  // the third buffer of the signal's size: after the graph's order is queued
      fail_size = 4 * 800 + 4 * 800 / 8 + 256;
      fail_skip = 2;
    }
    CHECK(lv_diffuse(sc, g, x, LV_F32, 8, 2, x + 800, S1) == (launch ? LV_ERR_DEVICE : LV_ERR_OUT_OF_MEMORY));
    fail_size = 0;
    fail_after.clear();
    void* event = nullptr;
    int queued = 0;
    for (const Op& o : ops()) {
      if (o.kind == kLaunch && o.stream == S1) queued++, event = nullptr;
      if (o.kind == kRecord && o.stream == S1) event = o.p;
    }
    CHECK(queued > 0);
    CHECK(event);
    const size_t at = ops().size();
    CHECK(lv_diffuse(sc, g, x, LV_F32, 4, 2, x + 800, S2) == LV_OK);
    bool waits = false;
    for (size_t i = at; i < ops().size() && ops()[i].kind != kLaunch; i++)
      waits = waits || (ops()[i].kind == kWait && ops()[i].stream == S2 && ops()[i].p == event);
    CHECK(waits);
    ops().clear();
    CHECK(lv_graph_destroy(g) == LV_OK && lv_scene_destroy(sc) == LV_OK && lv_release_scratch(nullptr, 1) == LV_OK);
  }
}

// Threads of all launches of a kernel; no launch since op `at` is refused.
uint64_t threads_of(const char* kernel, size_t at) {
  uint64_t sum = 0;
  for (size_t i = at; i < ops().size(); i++) {
    if (ops()[i].kind != kLaunch) continue;
    if (ops()[i].launched >= (1ull << 32)) fprintf(stderr, "%s\n", ops()[i].name.c_str());
    CHECK(ops()[i].launched < (1ull << 32));
    if (ops()[i].name.find(kernel) != std::string::npos) sum += ops()[i].size;
  }
  return sum;
}

// 2^28 edges with 16 lanes each (more than 128 channels).
void edge_weight_launches() {
  const int64_t n = 1 << 24, k = 16;
  lv_scene* sc = make_scene(n, S1);
  float* f = static_cast<float*>(device_mem(4 * (size_t)n * 129));
  lv_graph* g = nullptr;
  const size_t at = ops().size();
  const lv_status st = lv_graph_build_knn(sc, f, 129, (int)k, nullptr, S1, &g);
  CHECK(threads_of("edge_weights", at) >= (uint64_t)(n * k * 16));
  CHECK(st == LV_OK);
}

// The locality order of 2^28 rows, 16 lanes each.
void graph_order_launches() {
  const int n = 1 << 28;
  lv_scene* sc = make_scene(n, S1);
  lv_graph* g = make_graph(n, 0, S1);
  float* x = static_cast<float*>(device_mem(8 * (size_t)n));
  const size_t at = ops().size();
  const lv_status st = lv_diffuse(sc, g, x, LV_F32, 1, 1, x + n, S1);
  CHECK(threads_of("permute_csr", at) >= 16 * ((uint64_t)n + 1));
  CHECK(st == LV_OK);
}

// 2048 views of 1920x1080 in one group of more than 32 channels: two waves for
// each of 67M quadrants.
void uplift_launches() {
  const int m = 2048, D = 33, n = 10;
  lv_scene* sc = make_scene(n, S1);
  lv_camera cam = {{1, 0, 0, 0, 1, 0, 0, 0, 1}, {0, 0, 0}, 1000, 1000, 960, 540, 0.01f, 1920, 1080, 0};
  std::vector<lv_camera> cams(m, cam);
  std::vector<const void*> maps(m, device_mem(64));
  float* out = static_cast<float*>(device_mem(4 * n * D + 4 * (size_t)m * D));
  const size_t at = ops().size();
  const lv_status st = lv_uplift(sc, cams.data(), m, maps.data(), LV_FP8_E4M3, out + n * D, D, out, nullptr, S1);
  CHECK(threads_of("blend_wide", at) >= (uint64_t)m * 120 * 68 * 4 * 64);
  CHECK(st == LV_OK);
}

// The device memory of a diffusion does not grow with its steps.
void diffusion_memory() {
  const int n = 64, D = 64;
  lv_graph* g = make_graph(n, 2, S1);
  float* x = static_cast<float*>(device_mem(8 * n * D));
  g_peak = g_bytes;
  const uint64_t held = g_bytes;
  CHECK(lv_diffuse(nullptr, g, x, LV_F32, D, 100000, x + n * D, S1) == LV_OK);
  CHECK(g_peak - held < (4 << 20));
}

// The scratch of a graph build stays with the stream up to the scratch budget
// (16 GiB on this card) and is given back above it.
void graph_scratch() {
  for (int64_t n : {(int64_t)1 << 20, (int64_t)1 << 25}) {
    lv_scene* sc = make_scene(n, S1);
    float* f = static_cast<float*>(device_mem(4 * (size_t)n));
    lv_graph* g = nullptr;
    g_peak = g_bytes;
    const uint64_t held = g_bytes;
    CHECK(lv_graph_build_knn(sc, f, 1, 16, nullptr, S1, &g) == LV_OK);
    CHECK(g_peak - held >= 800 * (uint64_t)n);
    CHECK(g_bytes - held <= ((uint64_t)18 << 30));
    CHECK((g_bytes - held >= 800 * (uint64_t)n) == (n == 1 << 20));
    CHECK(lv_graph_destroy(g) == LV_OK && lv_scene_destroy(sc) == LV_OK && lv_release_scratch(S1, 0) == LV_OK);
  }
}

}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> tests = {
      {"destroy_on_other_device", destroy_on_other_device},
      {"order_after_failed_diffusion", order_after_failed_diffusion},
      {"edge_weight_launches", edge_weight_launches},
      {"graph_order_launches", graph_order_launches},
      {"uplift_launches", uplift_launches},
      {"diffusion_memory", diffusion_memory},
      {"graph_scratch", graph_scratch},
  };
  CHECK(argc == 2 && tests.count(argv[1]));
  tests.at(argv[1])();
  printf("ok\n");
  return 0;
}
