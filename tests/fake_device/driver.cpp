// Host code of libimloc on a machine without a GPU: this program defines the HIP
// calls that the library makes, so that a context can be made and the launches
// that a call would do are looked at instead of done (test infrastructure:
// tests/test_fake_device.py).  Device memory is never touched: workspace and arrays
// are made-up addresses.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <map>

#include "imloc.h"

extern "C" int imloc_internal_lift_kept(imloc_ctx* ctx, int32_t* n);

struct Dim3 {
  uint32_t x, y, z;
};

namespace {
int fails = 0;
int launches = 0;
bool fail_host_malloc = false;
std::map<void*, size_t> host_blocks;
struct Config {
  Dim3 grid, block;
  size_t shmem;
  void* stream;
} config;
const char* what = "";

void check(bool ok, const char* text) {
  if (ok) return;
  std::printf("failed: %s (%s)\n", text, what);
  ++fails;
}

// limits of the device: hipDeviceAttributeMaxGridDimX, Y, Z and work-items in 32 bits
void look(Dim3 g, Dim3 b) {
  ++launches;
  const bool ok = g.x >= 1 && g.y >= 1 && g.z >= 1 && g.y <= 65536 && g.z <= 65536 &&
                  (uint64_t)g.x * b.x < (1ull << 32) && (uint64_t)b.x * b.y * b.z <= 1024;
  if (!ok) std::printf("grid %u %u %u block %u %u %u\n", g.x, g.y, g.z, b.x, b.y, b.z);
  check(ok, "launch within the limits of a grid");
}
}  // namespace

extern "C" {
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "made-up error"; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)(uintptr_t)(1 << 20); return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipEventCreate(void** e) { *e = (void*)8; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = (void*)8; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventQuery(void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) {
  if (fail_host_malloc) return 2;
  *p = std::calloc(1, n);
  host_blocks[*p] = n;
  return 0;
}
int hipHostFree(void* p) {  // stays mapped and says so: a later read is seen
  std::memset(p, 0x5a, host_blocks[p]);
  return 0;
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void* st) {
  config = Config{g, b, s, st};
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
  *g = config.grid;
  *b = config.block;
  *s = config.shmem;
  *st = config.stream;
  return 0;
}
int hipLaunchKernel(const void*, Dim3 g, Dim3 b, void**, size_t, void*) {
  look(g, b);
  return 0;
}
}  // extern "C"

int main(int argc, char** argv) {
  const char* test = argc > 1 ? argv[1] : "";
  imloc_ctx* ctx = nullptr;
  if (imloc_create(&ctx, 0, nullptr) != IMLOC_OK) return 2;
  imloc_set_workspace(ctx, (void*)(uintptr_t)(1 << 28), (size_t)1 << 46);
  float* a = (float*)(uintptr_t)(1 << 24);
  const imloc_corr corr{a, a, a, a, a, a};
  const imloc_camera K{500.0, 500.0, 320.0, 240.0};
  if (!std::strcmp(test, "grids")) {
    imloc_ransac_params p;
    imloc_paper_params(4.0, &p);
    p.fixed_samples = 8;
    p.batch = 8;
    imloc_pose pose;
    for (int64_t m : {int64_t(3), int64_t(10000), int64_t(65535) * 1024, int64_t(65536) * 1024, int64_t(2000000000)}) {
      what = "scoring subset";
      p.max_score_points = m;
      const int before = launches;
      check(imloc_lo_ransac_pnp(ctx, &corr, m + m / 16 + 1, &K, &p, &pose, nullptr, nullptr) >= 0, "call");
      check(launches > before + 4, "launches seen");
    }
    what = "starts";
    double* d = (double*)(uintptr_t)(1 << 24);
    for (int32_t np : {1, 4096, 65535})
      for (int64_t n : {int64_t(1), int64_t(20000), int64_t(2000000000)})
        check(imloc_local_optimize(ctx, &corr, n, &K, d, np, 4.0, 10, d, d, (int64_t*)d) == IMLOC_OK, "call");
    what = "matches";
    const imloc_matches m{a, a, a, a, a, (int32_t*)a};
    const imloc_corr_out o{a, a, a, a, a, a, (int32_t*)a};
    imloc_pose T{{1, 0, 0, 0, 1, 0, 0, 0, 1}, {0, 0, 0}};
    for (int64_t n : {1, 1024, 1025, 2000000000})
      check(imloc_lift(ctx, &m, n, a, 1, 480, 640, &K, &T, 1, 0.05f, &o, n, (int32_t*)a) == IMLOC_OK, "call");
  } else if (!std::strcmp(test, "kept")) {
    what = "staging that could not be replaced";
    fail_host_malloc = true;
    check(imloc_set_staging(ctx, 1 << 22) == IMLOC_EHIP, "set_staging fails");
    check(imloc_get_staging(ctx) == 0, "no staging");
    const imloc_corr_out o{a, a, a, a, a, a, (int32_t*)a};
    check(imloc_lift(ctx, nullptr, 0, nullptr, 0, 0, 0, nullptr, nullptr, 1, 0.f, &o, 0, (int32_t*)a) == IMLOC_OK,
          "a lift of no matches");
    int32_t n = -1;
    const int rc = imloc_internal_lift_kept(ctx, &n);
    check(rc != IMLOC_OK || n == 0, "the count of a lift is read from memory that is still there");
  } else if (!std::strcmp(test, "noalloc")) {
    // the largest batches of samples that the fixed array held when it was set
    // (per query: local optimisations, points, samples), and batches past it
    const struct { int32_t k; int64_t n, samples; bool fits; } q[] = {
        {32, 30111, 44246, true}, {32, 32768, 44135, true}, {8, 30721, 45141, true}, {1, 30721, 45415, true},
        {32, 25000, 44467, true}, {1, 30721, 46000, false}, {32, 32768, 46000, false}, {1, 200000, 46000, false}};
    imloc_ransac_params p;
    imloc_paper_params(4.0, &p);
    imloc_pose pose;
    for (const auto& e : q) {
      what = e.fits ? "fits" : "does not fit";
      p.max_score_points = 0;
      p.lo_top_k = e.k;
      p.fixed_samples = p.batch = e.samples;
      const int rc = imloc_lo_ransac_pnp_noalloc(ctx, &corr, e.n, &K, &p, &pose, nullptr, nullptr);
      check((rc == IMLOC_ENOMEM) == !e.fits, "query of the fixed array");
    }
    check(imloc_noalloc_max_bytes() == size_t(32) << 20, "limit");
  } else {
    return 3;
  }
  std::printf("%d failure(s)\n", fails);
  return fails != 0;
}
