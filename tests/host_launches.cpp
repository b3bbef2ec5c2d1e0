// What the library enqueues, seen from the host: this program stands in for
// the HIP runtime calls that libpark.so makes (a symbol of the executable comes
// before the runtime's), records every kernel launch and runs no device code,
// so no GPU is needed.  It also stands in for getenv, whose answers a check can
// change from one read to the next.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "park.h"

extern "C" char** environ;

// ---------------------------------------------------------------- stand-ins
static std::map<const void*, std::string>& kernel_names() {  // (used before main)
  static std::map<const void*, std::string> names;
  return names;
}

struct Launch {
  std::string name;  // mangled kernel name
  bool lds_ok;       // its dynamic LDS is within 64 KB or what this device was told
  dim3 grid;
};
static std::vector<Launch> launches;
static std::map<std::string, std::vector<std::string>> env_script;  // answers, the last one repeated
static std::map<std::string, int> env_reads;
static int device = 0;
static int attribute_failures = 0;  // hipFuncSetAttribute calls that will fail
static std::map<std::pair<int, const void*>, size_t> lds_allowed;  // per device and kernel

static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} config;

extern "C" {

char* getenv(const char* name) {
  const auto it = env_script.find(name);
  if (it != env_script.end()) {
    const int k = env_reads[name]++;
    const auto& a = it->second;
    const std::string& v = a[k < (int)a.size() ? k : (int)a.size() - 1];
    return v.empty() ? nullptr : const_cast<char*>(v.c_str());
  }
  const size_t n = std::strlen(name);
  for (char** e = environ; e && *e; ++e)
    if (!std::strncmp(*e, name, n) && (*e)[n] == '=') return *e + n + 1;
  return nullptr;
}

void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  kernel_names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t lds, hipStream_t) {
  const auto it = lds_allowed.find({device, f});
  launches.push_back({kernel_names()[f], lds <= (it == lds_allowed.end() ? 65536u : it->second),
                      grid});
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = device;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int bytes) {
  if (attribute_failures > 0) return --attribute_failures, hipErrorUnknown;
  lds_allowed[{device, f}] = bytes;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)(uintptr_t)64;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)(uintptr_t)128;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

}  // extern "C"

// ------------------------------------------------------------------- checks
static int failures = 0;

#define EXPECT(cond)                                                          \
  do {                                                                        \
    if (!(cond)) {                                                            \
      std::fprintf(stderr, "%s:%d: failed: %s\n", __FILE__, __LINE__, #cond); \
      ++failures;                                                             \
    }                                                                         \
  } while (0)

static void* const FAKE = (void*)(uintptr_t)(1u << 20);  // 256-byte aligned, never read

static int count(const char* kernel) {
  int n = 0;
  for (const Launch& l : launches) n += l.name.find(kernel) != std::string::npos;
  return n;
}

static park_status cluster(int N, int C, int T, int H = 2, int dim = 128,
                           int metric = PARK_METRIC_QRKC, size_t ws_bytes = (size_t)1 << 40,
                           int dtype = PARK_BF16) {
  const park_dims d = {H, N, dim, dtype};
  launches.clear();
  return park_cluster_keys(FAKE, FAKE, &d, C, T, 0, 1, metric, 0.05, 1e-6, 1e-12, nullptr,
                           (int32_t*)FAKE, (int32_t*)FAKE, nullptr, nullptr, FAKE, ws_bytes, nullptr);
}

// A workspace for CQ and CK serves the clustering of either side.
static void workspace_of_unequal_sides() {
  struct { int H, N, CQ, CK, d, dtype; } cases[] = {{1, 4096, 16, 64, 64, PARK_F32},
                                                    {3, 6001, 1, 2048, 128, PARK_BF16},
                                                    {40, 75600, 295, 1182, 128, PARK_BF16},
                                                    {2, 4096, 600, 32, 64, PARK_BF16},
                                                    {2, 4096, 256, 256, 128, PARK_BF16}};
  for (const auto& c : cases) {
    const park_dims d = {c.H, c.N, c.d, c.dtype};
    size_t bytes = 0;
    EXPECT(park_workspace_size(&d, c.CQ, c.CK, &bytes) == PARK_OK);
    for (int C : {c.CQ, c.CK})
      EXPECT(cluster(c.N, C, 2, c.H, c.d, PARK_METRIC_QRKC, bytes, c.dtype) == PARK_OK);
  }
}

// The options of the candidate filter hold for a whole k-means: its rounds read
// what the setup and the rounds before them left.
static void kmeans_options() {
  const int T = 6;
  // the filter switched on or off between any two reads
  for (int flip = 1; flip < 10; ++flip)
    for (const char* first : {"", "0"}) {
      std::vector<std::string> a(flip, first);
      a.push_back(*first ? "" : "0");
      env_script["PARK_KMEANS_FILTER"] = a;
      env_reads.clear();
      EXPECT(cluster(4096, 600, T) == PARK_OK);
      const int setup = count("k_xnorm"), rounds = count("k_cand"), dense = count("k_assign_fast");
      EXPECT(rounds + dense == T);
      EXPECT(setup ? rounds == T - 1 : rounds == 0);
    }
  env_script.clear();
  // the radii: of the second round only, or of all from the second on
  for (int flip = 1; flip < 10; ++flip) {
    std::vector<std::string> a(flip, "");
    a.push_back("1");
    env_script["PARK_KFILTER_EXACT_RADIUS"] = a;
    env_reads.clear();
    EXPECT(cluster(4096, 600, T) == PARK_OK);
    const int radii = count("k_radius");
    EXPECT(radii == 1 || radii == T - 1);
  }
  env_script.clear();
}

// The counting sort takes four wavefronts on tiles of 1024 tokens, eight on 2048,
// and of larger ones sixteen up to 256 workgroups and eight beyond; no histogram
// pass for heads of one tile.
static void sort_routes() {
  struct { int H, N, nw, hist; } cases[] = {{1, 300, 8, 0},     {1, 2048, 8, 0},   {1, 2049, 16, 0},
                                            {1, 4096, 16, 0},   {1, 4097, 4, 2},   {1, 8192, 4, 2},
                                            {1, 8193, 8, 2},    {256, 4096, 16, 0}, {257, 4096, 8, 0},
                                            {1, 65536, 8, 2},   {1, 65537, 16, 2}, {16, 65537, 8, 2},
                                            {24, 119056, 8, 2}, {3, 119056, 16, 2}};
  for (const auto& c : cases) {
    EXPECT(cluster(c.N, 300, 2, c.H) == PARK_OK);
    EXPECT(count(("k_sort_scatterILi" + std::to_string(c.nw) + "E").c_str()) == 2);
    EXPECT(count("k_sort_scatter") == 2 && count("k_sort_hist") == c.hist);
  }
}

// Without a metric the centroids' preparation uses 1024 threads on small grids,
// with one the four wavefronts per 64 columns that its product is laid out for.
static void prep_routes() {
  struct { int H, C, d, metric; const char* kernel; } cases[] = {
      {1, 128, 128, PARK_METRIC_EUCLID, "k_prepILi128ELi1024E"},
      {1, 128, 64, PARK_METRIC_EUCLID, "k_prepILi64ELi1024E"},
      {32, 256, 128, PARK_METRIC_EUCLID, "k_prepILi128ELi512E"},
      {32, 256, 64, PARK_METRIC_EUCLID, "k_prepILi64ELi256E"},
      {1, 128, 128, PARK_METRIC_QRKC, "k_prepILi128ELi512E"},
      {1, 128, 64, PARK_METRIC_QRKC, "k_prepILi64ELi256E"}};
  for (const auto& c : cases) {
    EXPECT(cluster(4096, c.C, 3, c.H, c.d, c.metric) == PARK_OK);
    EXPECT(count("k_prep") == 3 && count(c.kernel) == 3);
  }
}

// The refinement against every centroid takes small clusterings of 64-dimension
// heads only: its work grows with the listed tokens times all centroids.
static void refine_routes() {
  struct { int H, N, C, d, all; } cases[] = {
      {1, 4096, 64, 64, 1},   {12, 17019, 266, 64, 1},  {8, 32768, 511, 64, 1},
      {24, 8136, 266, 64, 1},
      {8, 32769, 511, 64, 0}, {24, 30000, 133, 64, 0},  {40, 64521, 64, 64, 0},
      {1, 4096, 64, 128, 0},  {12, 17019, 512, 64, 0}};
  for (const auto& c : cases) {
    EXPECT(cluster(c.N, c.C, 3, c.H, c.d) == PARK_OK);
    EXPECT(count("k_refine_all") == (c.all ? 3 : 0));
    EXPECT(count("k_refine_cand") == (c.all ? 0 : 3));
    for (const Launch& l : launches)  // chunks of one rank side by side, whatever the chunks a head has
      if (l.name.find("k_refine_all") != std::string::npos) EXPECT((int)l.grid.x == c.H);
  }
}

static park_status attention(int dtype, int d) {
  const park_dims dims = {1, 4096, d, dtype};
  launches.clear();
  return park_block_sparse_attn(FAKE, FAKE, FAKE, (int32_t*)FAKE, (int32_t*)FAKE, (int32_t*)FAKE,
                                (int32_t*)FAKE, (int32_t*)FAKE, &dims, 64, 2048, FAKE, PARK_F32,
                                nullptr, FAKE, (size_t)1 << 40, nullptr);
}

// A kernel with more than 64 KB of dynamic LDS is allowed it on every device it
// runs on, and a failure to allow it is no answer for later calls.
static void lds_reservations() {
  auto all_ok = [] {
    for (const Launch& l : launches)
      if (!l.lds_ok) {
        std::fprintf(stderr, "device %d: %s\n", device, l.name.c_str());
        return false;
      }
    return true;
  };
  lds_allowed.clear();
  for (device = 0; device < 3; ++device) {
    attribute_failures = 1;
    EXPECT(cluster(4096, 2048, 2) == PARK_ERR_HIP);
    EXPECT(attribute_failures == 0);
    EXPECT(cluster(4096, 2048, 2) == PARK_OK && all_ok());
    for (int d : {64, 128}) {
      attribute_failures = 1;
      EXPECT(attention(PARK_BF16, d) == PARK_ERR_HIP);
      EXPECT(attention(PARK_BF16, d) == PARK_OK && all_ok());
    }
    EXPECT(attention(PARK_F32, 128) == PARK_OK && all_ok());
  }
  device = 0;
}

int main() {
  lds_reservations();
  workspace_of_unequal_sides();
  kmeans_options();
  refine_routes();
  prep_routes();
  sort_routes();
  if (failures) {
    std::fprintf(stderr, "%d host check(s) failed\n", failures);
    return 1;
  }
  std::printf("host launch checks passed\n");
  return 0;
}
