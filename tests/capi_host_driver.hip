// Host side of the C ABI against a runtime without a device: this file
// defines the HIP calls and kernel launchers that cmflb_capi.hip uses, as
// counters over plain host memory, and `main` walks the library through one
// kind of calls (argv[1]) and prints what it asked of the runtime.  Host code
// only; nothing here launches a kernel.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../include/cmflb.h"
#include "../paper_2602_16486_amd/csrc/cmflb_internal.h"

extern "C" char __hip_fatbin[16];
char __hip_fatbin[16];

namespace {

// what a captured run of steps does when it is launched
struct Graph {
  int64_t *step = nullptr;
  int64_t by = 0;
};

constexpr size_t kDeviceBytes = (size_t)288 << 30;
uint64_t threads = 0;  // most threads of one step launch
int captures = 0, graph_launches = 0, execs = 0, direct_steps = 0, streams = 0, events = 0;
bool capturing = false;
Graph recorded;
size_t live = 0, most = 0, pinned = 0, most_pinned = 0;
std::map<void *, size_t> sizes, pins;
std::mutex mu;  // guards what calls from several threads count

#define CHECK(cond)                                                \
  do {                                                             \
    if (!(cond)) {                                                 \
      printf("line %d: %s (%s)\n", __LINE__, #cond, cmf_last_error()); \
      exit(1);                                                     \
    }                                                              \
  } while (0)

}  // namespace

// the allocation of this thread that fails (counted down; < 0: none)
thread_local int fail_at = -1;

void *operator new(size_t n) {
  if (fail_at >= 0 && fail_at-- == 0) throw std::bad_alloc();
  if (void *p = malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

extern "C" {
hipError_t hipStreamCreate(hipStream_t *s) {
  ++streams;
  *s = (hipStream_t)malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  --streams;
  free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  ++events;
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::lock_guard<std::mutex> lk(mu);
  --events;
  free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  std::lock_guard<std::mutex> lk(mu);
  if (live + n > kDeviceBytes) return hipErrorOutOfMemory;
  *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) return hipErrorOutOfMemory;
  const int keep = fail_at;
  fail_at = -1;  // only the library's allocations fail
  sizes[*p] = n;
  fail_at = keep;
  live += n;
  most = live > most ? live : most;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  std::lock_guard<std::mutex> lk(mu);
  live -= sizes.at(p);
  munmap(p, sizes.at(p));
  sizes.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  *p = malloc(n);
  const int keep = fail_at;
  fail_at = -1;
  pins[*p] = n;
  fail_at = keep;
  pinned += n;
  most_pinned = pinned > most_pinned ? pinned : most_pinned;
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  std::lock_guard<std::mutex> lk(mu);
  pinned -= pins.at(p);
  pins.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind != hipMemcpyDeviceToDevice) memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int *d) {
  *d = 1;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  ++captures;
  capturing = true;
  recorded = Graph{};
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  capturing = false;
  *g = (hipGraph_t)&recorded;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  ++execs;
  *e = (hipGraphExec_t)new Graph(recorded);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  --execs;
  delete (Graph *)e;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  ++graph_launches;
  const Graph *g = (const Graph *)e;
  *g->step += g->by;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t *, size_t *, hipDeviceptr_t) { return hipErrorInvalidValue; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *, const void *) { return hipErrorInvalidValue; }
hipfftResult hipfftDestroy(hipfftHandle) { return HIPFFT_SUCCESS; }
hipfftResult hipfftExecR2C(hipfftHandle, hipfftReal *, hipfftComplex *) { return HIPFFT_SUCCESS; }
hipfftResult hipfftPlan2d(hipfftHandle *, int, int, hipfftType) { return HIPFFT_SUCCESS; }
hipfftResult hipfftPlan3d(hipfftHandle *, int, int, int, hipfftType) { return HIPFFT_SUCCESS; }
hipfftResult hipfftPlanMany(hipfftHandle *, int, int *, int *, int, int, int *, int, int, hipfftType, int) {
  return HIPFFT_SUCCESS;
}
hipfftResult hipfftSetStream(hipfftHandle, hipStream_t) { return HIPFFT_SUCCESS; }
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}  // extern "C"

namespace cmf {
namespace {
hipError_t bump(int64_t *p, int64_t by) {
  if (capturing)
    recorded = Graph{p, by};
  else
    *p += by;
  return hipSuccess;
}
}  // namespace

hipError_t launch_step(int, int, bool, bool, int, const void *, const void *, void *, const int64_t *,
                       int, double *, int grid, int block, hipStream_t) {
  threads = (uint64_t)grid * block > threads ? (uint64_t)grid * block : threads;
  direct_steps += !capturing;
  return hipSuccess;
}
hipError_t launch_step_fused(int, bool, int, const void *, const void *, void *, const int64_t *, int,
                             int nsteps, double *, int64_t, hipStream_t) {
  direct_steps += nsteps;
  return hipSuccess;
}
hipError_t launch_ensemble_step(int, bool, const void *, const int32_t *, int, const void *, void *,
                                const int64_t *, int, double *, hipStream_t) {
  direct_steps += !capturing;
  return hipSuccess;
}
hipError_t launch_finalize(const double *, int, double *, double *, int, int64_t *step, int, int by,
                           double, bool, hipStream_t) {
  return by ? bump(step, by) : hipSuccess;
}
hipError_t launch_finalize_batch(const double *, int64_t, int, int, double *, double *, int,
                                 int64_t *step, int, int by, double, bool, hipStream_t) {
  return by ? bump(step, by) : hipSuccess;
}
hipError_t launch_ensemble_finalize(int, const void *, int, const double *, int64_t, int, double *, int,
                                    int64_t *step, int, int by, double *, bool, hipStream_t) {
  return by ? bump(step, by) : hipSuccess;
}
hipError_t launch_bump_step(int64_t *p, int64_t by, hipStream_t) { return bump(p, by); }
hipError_t launch_zero_i64(int64_t *p, int64_t n, hipStream_t) {
  memset(p, 0, 8 * n);
  return hipSuccess;
}
hipError_t launch_get_state(int q, int, const ConvParams &c, const void *, double *f, hipStream_t) {
  for (int64_t i = 0; i < (int64_t)q * c.nx * c.ny * c.nz; ++i) f[i] = (double)i;
  return hipSuccess;
}
#define UNUSED_LAUNCH(name, ...) \
  hipError_t name(__VA_ARGS__) { return hipSuccess; }
UNUSED_LAUNCH(launch_macro, int, int, const ConvParams &, const void *, double *, double *, hipStream_t)
UNUSED_LAUNCH(launch_macro, int, int, const ConvParams &, const void *, float *, float *, hipStream_t)
UNUSED_LAUNCH(launch_noise, int, int, uint32_t, uint32_t, uint32_t, uint64_t, int64_t, int64_t, double *, hipStream_t)
UNUSED_LAUNCH(launch_gather, int, int, const ConvParams &, const void *, const int64_t *, int64_t, double *, hipStream_t)
UNUSED_LAUNCH(launch_philox, const uint32_t *, int64_t, uint32_t, uint32_t, uint32_t *, hipStream_t)
UNUSED_LAUNCH(launch_init_eq, int, int, const ConvParams &, const double *, const double *, void *, hipStream_t)
UNUSED_LAUNCH(launch_set_i64, int64_t *, int64_t, hipStream_t)
UNUSED_LAUNCH(launch_macro_dev, int, int, const ConvParams &, const void *, float *, hipStream_t)
UNUSED_LAUNCH(launch_set_state, int, int, const ConvParams &, const double *, void *, hipStream_t)
UNUSED_LAUNCH(launch_sk_shells, int, int, int, int, int64_t, int32_t *, int32_t *, int64_t *, hipStream_t)
UNUSED_LAUNCH(launch_sk_segments, const double *, int64_t, int, int, int, int, const int32_t *, const int64_t *, double *, double *, hipStream_t)
UNUSED_LAUNCH(launch_sk_accumulate, const void *, int64_t, double, double *, hipStream_t)
UNUSED_LAUNCH(launch_vel_stats, int, int, const ConvParams &, const void *, double *, int, double, double *, VelState *, unsigned long long *, hipStream_t)
UNUSED_LAUNCH(launch_stream_copy, const void *, void *, size_t, hipStream_t)
}  // namespace cmf

namespace {

cmf_desc desc(int q, int nx, int ny, int nz, int storage) {
  cmf_desc d;
  memset(&d, 0, sizeof d);
  d.q = q, d.nx = nx, d.ny = ny, d.nz = nz, d.storage = storage;
  d.rho0 = 1.0, d.tau = 0.8, d.kT = 1e-4, d.seed = 1;
  return d;
}

// launch shapes and tiles changed again and again between runs long enough
// for captured graphs
void graphs() {
  const cmf_desc d = desc(27, 12, 14, 17, 1);
  cmf_lattice *L = nullptr;
  CHECK(cmf_create(&d, nullptr, &L) == CMF_OK);
  int64_t step = 0, want = 0;
  for (int r = 0; r < 6; ++r) {
    for (int n : {96, 33, 64, 7}) {
      CHECK(cmf_step(L, n) == CMF_OK);
      want += n;
    }
    CHECK(cmf_set_launch(L, 64 * (1 + r % 4), 100 + r) == CMF_OK);
  }
  cmf_launch shape;
  CHECK(cmf_get_launch(L, &shape) == CMF_OK && shape.block == 128);
  CHECK(cmf_get_step(L, &step) == CMF_OK && step == want);
  printf("lattice captures %d\n", captures);
  cmf_destroy(L);
  // shapes set before the first run keep the graphs
  captures = graph_launches = 0;
  CHECK(cmf_create(&d, nullptr, &L) == CMF_OK);
  CHECK(cmf_autotune(L, 2, nullptr, 0, nullptr) == CMF_OK && cmf_set_launch(L, 128, 77) == CMF_OK);
  for (int r = 0; r < 5; ++r) CHECK(cmf_step(L, 64) == CMF_OK);
  printf("tuned captures %d launches %d\n", captures, graph_launches);
  cmf_destroy(L);
  captures = 0;
  cmf_desc two[2] = {desc(27, 12, 14, 17, 1), desc(9, 30, 20, 1, 1)};
  cmf_ensemble *E = nullptr;
  CHECK(cmf_ensemble_create(two, 2, nullptr, &E) == CMF_OK);
  want = 0;
  for (int r = 0; r < 6; ++r) {
    for (int n : {96, 33, 64, 7}) {
      CHECK(cmf_ensemble_step(E, n) == CMF_OK);
      want += n;
    }
    CHECK(cmf_ensemble_set_tiles(E, 1 + r, 2) == CMF_OK);
  }
  CHECK(cmf_ensemble_get_step(E, &step) == CMF_OK && step == want);
  printf("ensemble captures %d\n", captures);
  cmf_ensemble_destroy(E);
}

// boxes with many more tiles than lanes are full of: what an untuned lattice
// and the tuner launch, and the device memory beside the populations
void shapes() {
  const int boxes[][4] = {{27, 1, 4096, 4096}, {27, 1, 8192, 8192}, {27, 3, 2048, 2048}, {19, 2, 4096, 2048},
                          {19, 1, 1 << 24, 1}, {9, 1, 1 << 25, 1}, {9, 2, 1 << 22, 1}, {27, 70, 512, 512},
                          {27, 256, 256, 256}, {27, 1024, 1024, 1024}, {9, 4096, 4096, 1}, {19, 50, 50, 50}};
  for (auto &b : boxes)
    for (int storage = 0; storage < 4; ++storage)
      for (uint32_t flags : {0u, CMF_FLAG_IN_PLACE}) {
        cmf_desc d = desc(b[0], b[1], b[2], b[3], storage);
        d.flags = flags;
        const size_t population = cmf_external_bytes(&d);
        if (!population || population > kDeviceBytes) continue;
        cmf_lattice *L = nullptr;
        threads = most = 0;
        CHECK(cmf_create(&d, nullptr, &L) == CMF_OK);
        CHECK(cmf_step(L, 9) == CMF_OK);
        cmf_launch s;
        CHECK(cmf_get_launch(L, &s) == CMF_OK);
        printf("box %d %d %d %d storage %d flags %u block %d grid %d threads %llu population %zu beside %zu",
               b[0], b[1], b[2], b[3], storage, flags, s.block, s.grid, (unsigned long long)threads,
               population, most - population);
        threads = 0;
        const int rc = cmf_autotune(L, 1, nullptr, 0, nullptr);
        // (a copy of the state has to fit as well)
        CHECK(rc == CMF_OK || (rc == CMF_ENOMEM && population + population / 2 > kDeviceBytes));
        printf(" tuner %llu\n", (unsigned long long)threads);
        cmf_destroy(L);
      }
}

// workgroup sizes of untuned lattices
void blocks() {
  const int boxes[][5] = {{9, 1030, 900, 1, 0}, {9, 1030, 900, 1, 1}, {9, 1290, 800, 1, 0}, {9, 600, 600, 1, 0},
                          {27, 64, 64, 1, 1}, {27, 32, 32, 32, 1}, {19, 12, 14, 17, 2}, {27, 36, 36, 36, 1},
                          {27, 50, 50, 50, 1}, {27, 256, 256, 256, 1}};
  for (auto &b : boxes) {
    const cmf_desc d = desc(b[0], b[1], b[2], b[3], b[4]);
    cmf_lattice *L = nullptr;
    cmf_launch s;
    CHECK(cmf_create(&d, nullptr, &L) == CMF_OK && cmf_get_launch(L, &s) == CMF_OK);
    printf("block %d %dx%dx%d %d %d\n", b[0], b[1], b[2], b[3], b[4], s.block);
    cmf_destroy(L);
  }
}

// populations of 14 MB fetched while one allocation after another fails
void allocations() {
  const cmf_desc d = desc(27, 40, 40, 40, 1);
  const int64_t n = 27 * 40 * 40 * 40;
  cmf_lattice *L = nullptr;
  CHECK(cmf_create(&d, nullptr, &L) == CMF_OK);
  std::vector<double> f(n);
  int failed = 0;
  for (int k = 0; k < 24; ++k) {
    for (auto &x : f) x = -1.0;
    fail_at = k;
    const int rc = cmf_get_populations(L, f.data());
    failed += fail_at < 0;
    fail_at = -1;
    CHECK(rc == CMF_OK);
    for (int64_t i = 0; i < n; ++i) CHECK(f[i] == (double)i);
  }
  printf("allocations failed %d\n", failed);
  cmf_destroy(L);
}

// many lattices and ensembles whose populations are fetched, in turn and by
// several threads at once
void pinned_memory() {
  cmf_desc d = desc(27, 40, 40, 40, 1);
  const int64_t n = 27 * 40 * 40 * 40;
  std::vector<cmf_lattice *> lats(40);
  auto fetch = [&](cmf_lattice *L) {
    std::vector<double> f(n, -1.0);
    CHECK(cmf_get_populations(L, f.data()) == CMF_OK);
    for (int64_t i = 0; i < n; ++i) CHECK(f[i] == (double)i);
  };
  for (auto &L : lats) {
    CHECK(cmf_create(&d, nullptr, &L) == CMF_OK);
    fetch(L);
  }
  cmf_ensemble *E = nullptr;
  CHECK(cmf_ensemble_create(&d, 1, nullptr, &E) == CMF_OK);
  std::vector<double> f(n);
  CHECK(cmf_ensemble_get_populations(E, 0, f.data()) == CMF_OK && f[n - 1] == (double)(n - 1));
  printf("pinned in turn %zu\n", most_pinned);
  std::vector<std::thread> threads;
  for (int t = 0; t < 10; ++t)
    threads.emplace_back([&, t] {
      for (int r = 0; r < 3; ++r)
        for (int k = t; k < 40; k += 10) fetch(lats[k]);
    });
  for (auto &t : threads) t.join();
  printf("pinned at once %zu\n", most_pinned);
  for (auto L : lats) cmf_destroy(L);
  cmf_ensemble_destroy(E);
  printf("pinned after %zu\n", pinned);
  CHECK(cmf_create(&d, nullptr, &lats[0]) == CMF_OK);
  fetch(lats[0]);
  cmf_destroy(lats[0]);
}

}  // namespace

int main(int argc, char **argv) {
  const char *what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "graphs")) graphs();
  if (!strcmp(what, "shapes")) shapes();
  if (!strcmp(what, "blocks")) blocks();
  if (!strcmp(what, "allocations")) allocations();
  if (!strcmp(what, "pinned")) pinned_memory();
  printf("left %d %d %d %zu %zu\n", execs, streams, events, live, pinned);
  return 0;
}
