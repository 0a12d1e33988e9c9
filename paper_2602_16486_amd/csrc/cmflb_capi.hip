// cmflb_capi.hip -- implementation of the C ABI declared in include/cmflb.h:
// lattice objects, the FP64 per-mode constants, launch geometry, captured
// step graphs and the statistics ring.
//
// Method: De Rosis & Zhou, "A fluctuating lattice Boltzmann formulation based
// on orthogonal central moments" (arXiv 2602.16486).
#include <math.h>
#include <stddef.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hipfft/hipfft.h>

#include <condition_variable>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/cmflb.h"
#include "cmflb_device.h"
#include "cmflb_internal.h"

using namespace cmf;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

#define HIP_TRY(call)                                                      \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess)                                                  \
      return fail(CMF_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)

constexpr double kCs2 = 1.0 / 3.0;
constexpr int kGraphSteps = 32;
// most steps whose statistics one forked reduction handles (lattices): the
// partial sums go to a ring of 2 K slots, K = kStatBatch, or fewer steps
// (down to 1) when the ring would exceed kStatRingBytes
constexpr int kStatBatch = 8;
constexpr size_t kStatRingBytes = (size_t)256 << 20, kEnsRingBytes = (size_t)16 << 20;
// most steps of a fused lattice (several steps per launch) per reduction
constexpr int kFusedSlots = 64;
constexpr size_t kFusedRingBytes = (size_t)8 << 20;
static_assert(kGraphSteps % kStatBatch == 0, "a captured run is whole batches");
// largest box whose structure-factor fields are transformed as one batch
constexpr int64_t kSkBatchSites = (int64_t)1 << 22;
// noise counters are distinct for steps below 2^56 (see site_normals)
constexpr int64_t kMaxStep = (int64_t)1 << 56;

// one-axis weights of the rest state: w(0) = 2/3, w(+-1) = 1/6; the D2Q9 and
// D3Q27 weights of Sec. 2.2 / 2.3 are their products (4/9, 1/9, 1/36 and
// 8/27, 2/27, 1/54, 1/216).
double axis_weight(int c) { return c == 0 ? 2.0 / 3.0 : 1.0 / 6.0; }
// one-axis norms sum_c w(c) P_p(c)^2 of P_0 = 1, P_1 = c, P_2 = c^2 - c_s^2
const double kAxisNorm[3] = {1.0, 1.0 / 3.0, 2.0 / 9.0};

template <class L>
void lattice_weights(double *w) {
  for (int i = 0; i < L::Q; ++i)
    w[i] = axis_weight(L::cx[i]) * axis_weight(L::cy[i]) *
           (L::D == 3 ? axis_weight(L::cz[i]) : 1.0);
}

// D3Q19 weights (Sec. 2.4): 1/3 at rest, 1/18 on the axes, 1/36 on the
// face diagonals
void d3q19_weights(double *w) {
  for (int i = 0; i < 19; ++i) w[i] = i == 0 ? 1.0 / 3.0 : (i <= 6 ? 1.0 / 18.0 : 1.0 / 36.0);
}

// the D3Q19 basis polynomials of Sec. 2.4 at c
void d3q19_basis(double x, double y, double z, double *P) {
  const double c2 = x * x + y * y + z * z;
  const double row[19] = {1.0, x, y, z, c2 - 1.0, 3.0 * x * x - c2, y * y - z * z, x * y, y * z,
                          x * z, x * (3.0 * c2 - 5.0), y * (3.0 * c2 - 5.0), z * (3.0 * c2 - 5.0),
                          x * (y * y - z * z), y * (z * z - x * x), z * (x * x - y * y),
                          3.0 * c2 * c2 - 6.0 * c2 + 1.0, (2.0 * c2 - 3.0) * (3.0 * x * x - c2),
                          (2.0 * c2 - 3.0) * (y * y - z * z)};
  for (int v = 0; v < 19; ++v) P[v] = row[v];
}

// b_v of the paper's orthogonal bases (Sec. 2.2 and 2.3): products of the
// one-axis norms; D2Q9 rows 3 and 4 are sums/differences of two orthogonal
// products and have norm 2/9 + 2/9.  D3Q19 (Sec. 2.4): sum_i w_i P_v(c_i)^2.
void mode_norms(int q, double *b) {
  if (q == 19) {
    double w[19];
    d3q19_weights(w);
    for (int v = 0; v < 19; ++v) b[v] = 0.0;
    for (int i = 0; i < 19; ++i) {
      double P[19];
      d3q19_basis(D3Q19::cx[i], D3Q19::cy[i], D3Q19::cz[i], P);
      for (int v = 0; v < 19; ++v) b[v] += w[i] * P[v] * P[v];
    }
  } else if (q == 27) {
    for (int v = 0; v < 27; ++v) {
      const int pos = D3Q27::mode_pos[v];
      b[v] = kAxisNorm[pos % 3] * kAxisNorm[(pos / 3) % 3] * kAxisNorm[pos / 9];
    }
  } else {
    const int px[9] = {0, 1, 0, -1, -1, 1, 2, 1, 2};
    const int py[9] = {0, 0, 1, -1, -1, 1, 1, 2, 2};
    for (int v = 0; v < 9; ++v)
      b[v] = px[v] < 0 ? 2.0 * kAxisNorm[2] * kAxisNorm[0]
                       : kAxisNorm[px[v]] * kAxisNorm[py[v]];
  }
}

// the compile-time sqrt(b_v) of the kernels against the norms computed here
bool sqrt_norms_consistent(int q) {
  double b[27];
  mode_norms(q, b);
  for (int v = 0; v < q; ++v) {
    const double s = q == 9 ? sqrt_norm<D2Q9>(v) : (q == 19 ? sqrt_norm<D3Q19>(v) : sqrt_norm<D3Q27>(v));
    if (fabs(s * s - b[v]) > 1e-14 * b[v]) return false;
  }
  return true;
}

bool is_omega_mode(int q, int v) {
  return q == 9 ? (v == 4 || v == 5) : (v >= 7 && v <= 9);
}

int first_noisy(int q) { return q == 9 ? 3 : 4; }

size_t storage_bytes(int storage) {
  switch (storage) {
    case kF64: return 8;
    case kF32: return 4;
    case kF16:
    case kBF16: return 2;
  }
  return 0;
}

int env_int(const char *name, int dflt) {
  const char *s = getenv(name);
  if (!s || !*s) return dflt;
  return atoi(s);
}

// env_int clamped to [lo, hi]
int env_int(const char *name, int dflt, int lo, int hi) {
  const int v = env_int(name, dflt);
  return v < lo ? lo : (v > hi ? hi : v);
}

}  // namespace

namespace {

// FP64 per-mode constants of one descriptor: rates, weights, mode noise
// factors amp_v = I~_v sqrt(Lambda_v (2 - Lambda_v) b_v) (eq. phi_general
// is phi_v = sqrt(rho kT / c_s^2) amp_v), storage scales.
struct ModeConstants {
  double lambda[27], w[27], amp[27];
  float scale[27];
  bool general;
};

void mode_constants(const cmf_desc *desc, ModeConstants &mc) {
  const int q = desc->q;
  const double omega = 1.0 / desc->tau;
  for (int v = 0; v < q; ++v)
    mc.lambda[v] = desc->lambda ? desc->lambda[v] : (is_omega_mode(q, v) ? omega : 1.0);
  mc.general = false;
  for (int v = first_noisy(q); v < q; ++v)
    if (!is_omega_mode(q, v) && mc.lambda[v] != 1.0) mc.general = true;
  double b[27];
  if (q == 9)
    lattice_weights<D2Q9>(mc.w);
  else if (q == 19)
    d3q19_weights(mc.w);
  else
    lattice_weights<D3Q27>(mc.w);
  mode_norms(q, b);
  for (int v = 0; v < q; ++v) {
    const double lv = mc.lambda[v];
    mc.amp[v] = v >= first_noisy(q) ? sqrt(lv * (2.0 - lv) * b[v]) : 0.0;
  }
  for (int i = 0; i < q; ++i) {
    if (desc->storage == kF16 || desc->storage == kBF16) {
      const double sigma = desc->kT > 0.0 ? sqrt(desc->rho0 * desc->kT * mc.w[i] / kCs2)
                                          : 1e-2 * mc.w[i];
      mc.scale[i] = (float)ldexp(1.0, (int)ceil(log2(sigma)));
    } else {
      mc.scale[i] = 1.0f;
    }
  }
}

// Captured runs of kGraphSteps steps: step j passes step offset j and runs
// on the caller's stream; the steps go in batches of K consecutive steps
// (K = the lattice's or ensemble's stat_batch, at most kStatBatch),
// step j writing its partial sums to slot j mod 2K; once a batch is done,
// one statistics reduction for all its steps runs on a second stream
// (default priority), overlapping the next batch; the first step of batch
// b + 2 waits for it (it reuses the slots); the step counter advances once,
// after the last reduction.  One fork per batch instead of one per step:
// the event records and waits between the streams cost microseconds each.
struct ForkedRun {
  hipStream_t aux = nullptr;
  hipEvent_t ev_step[kGraphSteps] = {};
  hipEvent_t ev_fin[kGraphSteps] = {};
  bool ready = false;
};

void forked_release(ForkedRun &F) {
  for (int j = 0; j < kGraphSteps; ++j) {
    if (F.ev_step[j]) (void)hipEventDestroy(F.ev_step[j]);
    if (F.ev_fin[j]) (void)hipEventDestroy(F.ev_fin[j]);
    F.ev_step[j] = F.ev_fin[j] = nullptr;
  }
  if (F.aux) (void)hipStreamDestroy(F.aux);
  F.aux = nullptr;
  F.ready = false;
}

int forked_init(ForkedRun &F) {
  if (F.ready) return CMF_OK;
  hipError_t e = hipStreamCreate(&F.aux);
  for (int j = 0; j < kGraphSteps && e == hipSuccess; ++j) {
    e = hipEventCreateWithFlags(&F.ev_step[j], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&F.ev_fin[j], hipEventDisableTiming);
  }
  if (e != hipSuccess) {
    forked_release(F);
    return fail(CMF_EHIP, "stream/event creation failed: %s", hipGetErrorString(e));
  }
  F.ready = true;
  return CMF_OK;
}

// Enqueue a run of n <= kGraphSteps steps in the forked form on stream s,
// in batches of K steps: step(j, stream) enqueues step j (step offset j,
// partial-sum slot j mod 2K); fin(j0, count, bump, stream) the statistics
// reduction of steps j0 .. j0 + count - 1 (only when `stats`), which then
// advances the step counter by bump, on the second stream; that of the last
// batch on s itself, which would only wait for it (one step with its
// statistics read by a following kernel, D2Q9 96 x 61: 45.4 -> 12.9 us with kSingleLevelRows); the
// step counter advances by n at the end.  Used inside a graph
// capture (runs of kGraphSteps) and directly (the remainder of a cmf_step
// call), so the statistics of direct steps overlap the next steps as well.
template <class StepFn, class FinFn>
hipError_t enqueue_forked(hipStream_t s, ForkedRun &F, bool stats, int K, int64_t *step_dev,
                          StepFn step, FinFn fin, int n) {
  hipError_t e = hipSuccess;
  const int nbatch = (n + K - 1) / K;
  for (int b = 0; b < nbatch && e == hipSuccess; ++b) {
    const int j0 = b * K, j1 = j0 + K < n ? j0 + K : n;
    if (stats && b >= 2) e = hipStreamWaitEvent(s, F.ev_fin[b - 2], 0);
    for (int j = j0; j < j1 && e == hipSuccess; ++j) e = step(j, s);
    if (e != hipSuccess) break;
    if (stats && b < nbatch - 1) {
      e = hipEventRecord(F.ev_step[b], s);
      if (e == hipSuccess) e = hipStreamWaitEvent(F.aux, F.ev_step[b], 0);
      if (e == hipSuccess) e = fin(j0, j1 - j0, 0, F.aux);
      if (e == hipSuccess) e = hipEventRecord(F.ev_fin[b], F.aux);
    } else if (stats) {
      if (b >= 1) e = hipStreamWaitEvent(s, F.ev_fin[b - 1], 0);
      if (e == hipSuccess) e = fin(j0, j1 - j0, n == 1 ? 1 : 0, s);
    }
  }
  if (e == hipSuccess && !(stats && n == 1)) e = launch_bump_step(step_dev, n, s);
  return e;
}

template <class StepFn, class FinFn>
int run_forked(hipStream_t s, ForkedRun &F, bool stats, int K, int64_t *step_dev, StepFn step,
               FinFn fin, int n) {
  if (n < 1 || n > kGraphSteps) return fail(CMF_EINVAL, "internal: forked run of %d steps", n);
  if (stats && n > K) {
    int rc = forked_init(F);
    if (rc != CMF_OK) return rc;
  }
  const hipError_t e = enqueue_forked(s, F, stats, K, step_dev, step, fin, n);
  if (e != hipSuccess) return fail(CMF_EHIP, "step launch failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

template <class StepFn, class FinFn>
int capture_forked(hipStream_t s, ForkedRun &F, bool stats, int K, int64_t *step_dev,
                   StepFn step, FinFn fin, hipGraphExec_t *out) {
  if (stats) {
    int rc = forked_init(F);
    if (rc != CMF_OK) return rc;
  }
  HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
  hipError_t e = enqueue_forked(s, F, stats, K, step_dev, step, fin, kGraphSteps);
  hipGraph_t g = nullptr;
  const hipError_t ec = hipStreamEndCapture(s, &g);
  if (e == hipSuccess) e = ec;
  if (e == hipSuccess) e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  if (g) (void)hipGraphDestroy(g);
  if (e != hipSuccess) return fail(CMF_EHIP, "graph capture failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

// The pinned chunks of large copies to the host (see fetch), of one device.
constexpr size_t kFetchChunk = (size_t)4 << 20;
constexpr int kFetchSlots = 6, kFetchThreads = 4;

struct FetchRing {
  char *pin = nullptr;
  int device = -1;
  hipEvent_t ready[kFetchSlots] = {};
  bool busy = false;  // guarded by the pool's mutex, as is `device` while not busy
  void release() {
    for (auto &e : ready) {
      if (e) (void)hipEventDestroy(e);
      e = nullptr;
    }
    if (pin) (void)hipHostFree(pin);
    pin = nullptr;
    device = -1;
  }
  bool init(int dev) {
    if (pin && device == dev) return true;
    release();
    bool ok = true;
    for (auto &e : ready) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipHostMalloc((void **)&pin, kFetchSlots * kFetchChunk, hipHostMallocDefault) == hipSuccess;
    if (ok) {
      device = dev;
    } else {
      (void)hipGetLastError();
      release();
    }
    return ok;
  }
};

// The rings of the process: one while copies come one after the other, up to
// kFetchRings while threads copy at the same time (further ones leave the
// copy to the runtime), freed once no lattice or ensemble that used them is
// left.  Pinned for each call instead, a ring took 0.3 ms of it, and 4 ms once
// three ensembles were asked in turn (54 MB 5.9 against 2.2 ms); kept by each
// lattice, a hundred of them held 2.4 GB.
constexpr int kFetchRings = 4;
struct FetchPool {
  std::mutex mu;
  FetchRing ring[kFetchRings];
  int users = 0;
};
FetchPool g_fetch;  // (frees nothing at exit, when the runtime may be gone)

// A lattice's or ensemble's part in the pool, from its first large copy on.
struct FetchUser {
  bool joined = false;
  FetchUser() = default;
  FetchUser(const FetchUser &) = delete;
  FetchUser &operator=(const FetchUser &) = delete;
  ~FetchUser() {
    if (!joined) return;
    std::lock_guard<std::mutex> lk(g_fetch.mu);
    if (--g_fetch.users == 0)
      for (auto &r : g_fetch.ring) r.release();
  }
  // a ring of the current device for one copy, or NULL
  FetchRing *take() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    FetchRing *got = nullptr;
    {
      std::lock_guard<std::mutex> lk(g_fetch.mu);
      if (!joined) ++g_fetch.users;
      joined = true;
      for (auto &r : g_fetch.ring)
        if (!r.busy && (!got || (got->device != dev && r.device == dev))) got = &r;
      if (got) got->busy = true;
    }
    if (got && !got->init(dev)) {
      give(got);
      got = nullptr;
    }
    return got;
  }
  void give(FetchRing *r) {
    std::lock_guard<std::mutex> lk(g_fetch.mu);
    r->busy = false;
  }
};

}  // namespace

struct cmf_lattice {
  cmf_desc desc;
  int q = 0;
  int storage = 0;
  bool general = false;
  bool nt_stores = true;  // population rows are whole cache lines
  bool in_place = false;  // AA streaming on one buffer (buf[1] == buf[0])
  bool own_stream = false;
  bool own_bufs = true;  // false: the population buffers belong to the caller
  hipStream_t stream = nullptr;
  int device = 0;
  int64_t N = 0;
  void *buf[2] = {nullptr, nullptr};
  int parity = 0;  // buf[parity] holds the state of the current step
  double *partials = nullptr;
  double *level2 = nullptr;
  int nparts = 0;
  int partials_cap = 0;    // partial rows per slot
  int partials_slots = 0;  // slots allocated (2 stat_batch needed)
  int stat_batch = 1;      // steps per forked statistics reduction
  bool shape_set = false;  // launch shape asked for (cmf_set_launch, environment)
  int fused = 0;           // several steps per launch: rows of a tile (0: single steps)
  int fused_slots = 0;     // partial-sum slots of its statistics
  int cus = 256;
  double *series = nullptr;
  int cap = 0;
  int64_t *step_dev = nullptr;
  int64_t read_step = 0;   // first step whose statistics were not returned
  int block = 256;
  int grid = 1;
  double lambda[27];
  double w[27];
  double amp[27];
  float scale[27];
  double mass0 = 0.0;
  StepParams<float> pf;
  StepParams<double> pd;
  ConvParams cp;
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  bool graphs_dropped = false;  // a new launch shape dropped captured graphs
  ForkedRun forked;
  FetchUser fetches;
  char *vel_ws = nullptr;  // velocity statistics: VelState, counts, block sums
  // structure factor
  int sk_nbins = 0;
  int64_t sk_M = 0, sk_samples = 0;
  float *sk_fields = nullptr;
  void *sk_F = nullptr;
  double *sk_acc = nullptr, *sk_out = nullptr;
  int32_t *sk_perm = nullptr;
  int64_t *sk_off = nullptr;
  int sk_batch = 4;  // fields per transform call
  hipfftHandle sk_plan = 0;
  bool sk_has_plan = false;
};

namespace {

// weight class |c_i|^2 of population i of a q-velocity lattice
int weight_class_of(int q, int i) {
  if (q == 9) return weight_class<D2Q9>(i);
  if (q == 19) return weight_class<D3Q19>(i);
  return weight_class<D3Q27>(i);
}

// per-class storage scales (and reciprocals) from the per-population ones.
// With 16-bit storage the tensor-product lattices (D2Q9, D3Q27) hand the
// stores 2^|c_i|^2 d*_i (their inverse one-axis maps skip the halvings), so
// the store scale of class k carries 2^-k: the stored values are the same.
void class_scales(int q, int storage, const float *scale, float *cs, float *ics) {
  const bool doubled = (storage == kF16 || storage == kBF16) && q != 19;
  for (int k = 0; k < 4; ++k) {
    cs[k] = 1.0f;
    ics[k] = doubled ? ldexpf(1.0f, -k) : 1.0f;
  }
  for (int i = 0; i < q; ++i) {
    const int k = weight_class_of(q, i);
    cs[k] = scale[i];
    ics[k] = doubled ? ldexpf(1.0f / scale[i], -k) : 1.0f / scale[i];
  }
}

// Tiles per z plane of a 3-D lattice whose tiles are runs of the plane's sites,
// 0 where they are parts of a row.  A step of a 3-D box issues for most of its
// time, and lanes beyond the end of a row issue like any other: a row of 50
// takes a wave of 64, one of 150 three.  Runs of sites leave no lane idle but
// those of a plane's last tile, for some 25 more address operations per site (a
// lane's row is a vector value).  us per step, rows -> runs: D3Q27 FP32 50^3
// 14.3 -> 12.0, 32 x 96 x 96 20.7 -> 17.5, 100^3 44.3 -> 40.8, FP16 100^3 40.0
// -> 34.6, FP64 50^3 20.6 -> 19.1; D3Q19 BF16 72 x 60 x 50 15.6 -> 11.9, FP32
// in place 150 x 144 x 160 98.7 -> 87.9.  Where rows waste less than kFlatGain
// the gain is within the noise or lost (D3Q27 FP32 120^3 76.3 -> 77.1, 250 x
// 120 x 90 110.6 -> 111.9).  D3Q27 in FP32 waits for HBM once a box has
// outgrown the last-level cache, and a tile that ends inside a 32-byte sector
// has its ends written in two parts: then only rows of whole sectors go in runs
// (200 x 200 x 160 278 -> 268; 150 x 144 x 160, 22 % idle lanes, 145.4 ->
// 147.1; narrower rows of split sectors, which idle more, were not measured and
// stay rows).
constexpr double kFlatGain = 1.1;
constexpr int64_t kFlatCached = (int64_t)1 << 21;  // sites
int flat_plane_tiles(const cmf_desc &d, int block) {
  const int64_t plane = (int64_t)d.nx * d.ny, b = (int64_t)storage_bytes(d.storage);
  if (d.q == 9 || d.nx < 2 || d.nx > 8192 || plane * d.q * b >= (int64_t)1 << 32) return 0;
  if (d.q == 27 && d.storage == kF32 && !(d.flags & CMF_FLAG_IN_PLACE) &&
      plane * d.nz > kFlatCached && d.nx * b % 32 != 0)
    return 0;
  const int64_t flat = (plane + block - 1) / block;
  const int64_t rows = (int64_t)((d.nx + block - 1) / block) * d.ny;
  return kFlatGain * flat <= rows ? (int)flat : 0;
}

// Tiles of a lattice with workgroups of `block` threads.
int tiles_for(const cmf_desc &d, int block) {
  const int flat = flat_plane_tiles(d, block);
  return (flat ? flat : (d.nx + block - 1) / block * d.ny) * d.nz;
}

// Step-kernel parameters of a lattice description with workgroups of
// `block` threads.
template <typename R>
void fill_params(const cmf_desc &d, const double *lambda, const double *amp, const float *scale,
                 int block, StepParams<R> &p) {
  memset(&p, 0, sizeof p);
  p.nx = d.nx;
  p.ny = d.ny;
  p.nz = d.nz;
  const int flat = flat_plane_tiles(d, block);
  p.nxb = flat ? flat : (d.nx + block - 1) / block;
  p.ntiles = tiles_for(d, block);
  p.flat = flat ? (uint32_t)(((uint64_t)1 << 32) / (uint32_t)d.nx + 1) : 0;
  p.noise = d.kT > 0.0 ? 1 : 0;
  p.ncx = (d.nx + kCell - 1) / kCell;
  p.rho0 = (R)d.rho0;
  for (int v = 0; v < d.q; ++v) {
    p.amp[v] = (R)amp[v];
    p.oml[v] = (R)(1.0 - lambda[v]);
    p.lam[v] = (R)lambda[v];
  }
  p.amp1 = (R)sqrt(d.kT / kCs2);
  class_scales(d.q, d.storage, scale, p.scale, p.iscale);
  p.key0 = (uint32_t)d.seed;
  p.key1 = (uint32_t)(d.seed >> 32);
  p.replica = d.replica;
}

template <typename R>
void fill_step_params(const cmf_lattice *L, const double *amp,
                      const float *scale, StepParams<R> &p) {
  fill_params(L->desc, L->lambda, amp, scale, L->block, p);
}

// tuned launch shapes of this process, keyed by device/lattice/storage/box
std::mutex g_tune_mu;
std::map<std::string, std::pair<int, int>> g_tuned;
bool g_tune_file_loaded = false;

std::string tune_key(const cmf_lattice *L) {
  char b[160];
  snprintf(b, sizeof b, "dev%d:q%d:s%d:g%d:%dx%dx%d%s", L->device, L->q, L->storage,
           L->general ? 1 : 0, L->desc.nx, L->desc.ny, L->desc.nz, L->in_place ? ":aa" : "");
  return b;
}

// launch shapes the step kernels support: block threads per workgroup a
// multiple of 64 up to 256 (the statistics reduction assumes it), grid >= 1
bool valid_launch(int block, int grid) {
  return (block == 64 || block == 128 || block == 192 || block == 256) && grid >= 1;
}

void load_tune_file_locked() {
  if (g_tune_file_loaded) return;
  g_tune_file_loaded = true;
  const char *path = getenv("CMFLB_TUNE_CACHE");
  if (!path || !*path) return;
  FILE *f = fopen(path, "r");
  if (!f) return;
  char key[160];
  int block, grid;
  double ms;
  // only shapes that cmf_set_launch would accept; other lines are skipped
  while (fscanf(f, "%159s %d %d %lf", key, &block, &grid, &ms) == 4)
    if (valid_launch(block, grid)) g_tuned[key] = {block, grid};
  fclose(f);
}

void remember_tuned(const cmf_lattice *L, int block, int grid, double ms) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  load_tune_file_locked();
  const std::string key = tune_key(L);
  g_tuned[key] = {block, grid};
  const char *path = getenv("CMFLB_TUNE_CACHE");
  if (path && *path) {
    FILE *f = fopen(path, "a");
    if (f) {
      fprintf(f, "%s %d %d %.6f\n", key.c_str(), block, grid, ms);
      fclose(f);
    }
  }
}

bool lookup_tuned(const cmf_lattice *L, int *block, int *grid) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  load_tune_file_locked();
  auto it = g_tuned.find(tune_key(L));
  if (it == g_tuned.end()) return false;
  *block = it->second.first;
  *grid = it->second.second;
  return true;
}

// Workgroup size of an untuned lattice: the one whose tiles cover the box with
// the fewest lanes, weighted by what a lane costs in a workgroup of that size
// (the start of a workgroup and its statistics are shared by its lanes).  One
// tile per workgroup, D3Q27 in tiles of a row, us per step at 64 / 128 / 192 / 256 threads: nx =
// 300 FP32 110 / 101 / 104 / 114, FP64 207 / 218 / 222 / 262; nx = 200 FP32 160 /
// 159 / 175 / 119, FP64 317 / 314 / 412 / 309; nx = 160 FP32 147 / 162 / 138; nx =
// 100 FP32 58 / 48.  D2Q9's cheaper sites leave more of a step to the
// workgroups, so that fewer idle lanes weigh less (64 / 128 / 256 threads: 1030 x
// 900 FP32 - / 19.4 / 17.2, FP64 without noise 25.2 / 24.9 / 23.6; 600 x 600 FP64
// - / 15.3 / 17.0; 770 x 1000 FP32 - / 15.8 / 16.8).  A 3-D box that 64-thread
// tiles cover with two per CU takes those: nothing queues, and a wave's latency
// is the step (64 / 256 threads, D3Q27 FP32 and FP64: 16^3 7.2 / 7.8 and 10.8 / 12.7,
// 32^3, 512 tiles, 7.4 / 7.8 and 11.8 / 13.4; 256 x 16 x 16, 1024 tiles, 9.4 / 8.8
// and 14.6 / 14.4).
int default_block(const cmf_desc &d, int cus) {
  const bool f64 = d.storage == kF64, d2 = d.q == 9;
  if (!d2 && tiles_for(d, 64) <= 2 * cus) return 64;
  const double cost[4] = {!f64 ? 1.35 : d2 ? 1.18 : 1.1, d2 ? 1.13 : f64 ? 1.05 : 1.1,
                          d2 ? 1.12 : 1.1, 1.0};
  int best = 0;
  double least = 0.0;
  for (int k = 0; k < 4; ++k) {
    const int b = 64 * (k + 1);
    const double c = (double)tiles_for(d, b) * b * cost[k];
    if (!best || c < least) {
      best = b;
      least = c;
    }
  }
  return best;
}

// Small D2Q9 boxes take several steps per launch (cmflb_step_fused.hip): the
// rows of a tile, 0 for a box that takes single steps.  The smallest tile with
// at most one workgroup per CU, else two: within a step a CU's time is that of
// the sites around its tile as well, so that more and smaller tiles cost less
// until they queue (FP32 us per step in tiles of 4 / 8 / 12 / 16 rows: 100^2
// 2.03 / 2.22 / 2.32 / 2.52, 200^2 3.38 / 3.28 / 2.64 / 2.78, 256^2 4.27 / 3.36
// / 3.57 / 2.88; single steps 5.99, 6.36, 6.43).  In FP64 two workgroups of 8
// rows or more do not fit into a CU's LDS (104 KB and more of 160) and run one
// after the other, which still saves time (300^2 8.2 against 9.7 of single steps
// in place).  Beyond two per CU the sites computed twice outweigh the launches saved (400 x 300, 475
// tiles of 16: 4.94 against 8.50; 700 x 500, 1408: 13.2 against 11.7; 512^2,
// 1024: FP32 9.2 against 10.3, FP16 9.5 against 8.1, FP64 20.6 against 15.2;
// all before the first and last step of a launch had code of their own, which
// takes 7-10 % off FP32 and 16-bit launches; the limit is the same for every
// storage and was not measured again since).  A launch shape that was asked for
// keeps single steps in that shape.  Boxes of this size keep their statistics
// in cell order whether or not they can take several steps (in-place streaming
// and edges up to kFusedSteps cannot).
int choose_tile_rows(const cmf_lattice *L) {
  const cmf_desc &d = L->desc;
  if (L->q != 9 || L->shape_set) return 0;
  const int64_t ncx = (d.nx + kCell - 1) / kCell;
  for (int per_cu = 1; per_cu <= 2; ++per_cu)
    for (int ty = 4; ty <= 16; ty += 4)
      if (ncx * ((d.ny + ty - 1) / ty) <= (int64_t)per_cu * L->cus) return ty;
  return 0;
}

int ntiles_for(const cmf_lattice *L, int block) { return tiles_for(L->desc, block); }

// the runtime launches grids of fewer than 2^32 threads
bool launchable(int64_t grid, int block) { return grid * block < (int64_t)1 << 32; }

// One tile per workgroup, as long as the grid is launchable and the two slots
// of partial sums that a lattice needs at least take kStatRingBytes or 1/64 of
// the populations: tiles of full wavefronts stay far below that (1024^3 D3Q27
// FP32: 0.8 GB beside 232), but a box of one or few sites per row has a tile
// per row (1 x 4096 x 4096: 3.2 GB beside 7.2).  Workgroups beyond the limit
// stride over the tiles instead.
int one_tile_grid(const cmf_lattice *L, int block) {
  const int64_t state = (int64_t)L->q * L->N * storage_bytes(L->storage) * (L->in_place ? 1 : 2);
  const int64_t bytes = state / 64 > (int64_t)kStatRingBytes ? state / 64 : (int64_t)kStatRingBytes;
  int64_t g = bytes / (2 * (int64_t)sizeof(double) * kPartStride);
  if (!launchable(g, block)) g = (((int64_t)1 << 32) - 1) / block;
  const int nt = ntiles_for(L, block);
  return g < nt ? (int)g : nt;
}

// Workgroups of an untuned lattice.  FP32 and FP64 3-D steps wait for memory:
// one tile per workgroup (D3Q27 FP32 / FP64 us per step against 2 per CU:
// 50^3 14.5 / - against 20.3, 100^3 48.3 / 131 against 77.3 / 231, 128^3 82.3 / 214
// against 128 / 366).  16-bit steps issue in every cycle and keep 16 workgroups
// per CU, which reduce their statistics once (256^3 418 against 444 one-tile).
// D2Q9: 1024 threads per CU below 2^22 sites (1000 x 700 FP32 15.0 against 16.4
// one-tile, FP64 28.7 against 30.9; 1500 x 633 18.1 against 19.7), then
// one-tile in FP32 (4096^2 219 against 236) and 16 per CU in FP64 (490 against
// 512 one-tile).
int default_grid(const cmf_lattice *L, int block) {
  if (storage_bytes(L->storage) == 2) return 16 * L->cus;
  if (L->q == 9 && L->N < ((int64_t)1 << 22)) return 4 * L->cus * (256 / block);
  if (L->q == 9 && L->storage == kF64) return 16 * L->cus;
  return one_tile_grid(L, block);
}

// Destroy the captured runs of a lattice or ensemble whose launch shape
// changes.  It captures no others: a program that replayed graphs, dropped
// them and captured them anew, shape after shape on one lattice, once aborted
// on the host with a corrupted heap, and the cause is not known.  Direct steps
// give the same bits (64^3 D3Q27 FP32: 16.4 us per step in graphs, 17.6
// direct).
template <class T>
void drop_graphs(T *L) {
  for (auto &g : L->graph)
    if (g) {
      (void)hipGraphExecDestroy(g);
      g = nullptr;
      L->graphs_dropped = true;
    }
}

// Apply a launch shape: step parameters, partials capacity, graphs.
int apply_launch(cmf_lattice *L, int block, int grid, const double *amp,
                 const float *scale) {
  // new parameters and buffers first: on failure the current shape stays
  const int block0 = L->block;
  L->block = block;
  StepParams<double> pd;
  StepParams<float> pf;
  fill_step_params(L, amp, scale, pd);
  fill_step_params(L, amp, scale, pf);
  L->block = block0;
  const int nt = pf.ntiles;
  const int rows = choose_tile_rows(L);
  const bool cells = rows > 0;
  const int fused = L->in_place || L->desc.nx <= kFusedSteps || L->desc.ny <= kFusedSteps ? 0 : rows;
  pd.cells = pf.cells = cells ? 1 : 0;
  const int g = cells ? pf.ncx * L->desc.ny : grid < nt ? grid : nt;
  const size_t slot_bytes = sizeof(double) * kPartStride * (size_t)g;
  int K = kStatBatch;
  while (K > 1 && 2 * (size_t)K * slot_bytes > kStatRingBytes) K /= 2;
  int slots = 2 * K;
  // more for launches of several steps, within kFusedRingBytes and the
  // second-level rows of kStatBatch steps of the largest grids
  const int nb = (g + kLevel2Threshold - 1) / kLevel2Threshold;
  if (fused)
    while (slots < kFusedSlots && 2 * (size_t)slots * slot_bytes <= kFusedRingBytes &&
           2 * slots * nb <= kStatBatch * kMaxLevel2)
      slots *= 2;
  if (g > L->partials_cap || slots > L->partials_slots) {
    double *parts = nullptr;
    if (hipMalloc((void **)&parts, (size_t)slots * slot_bytes) != hipSuccess)
      return fail(CMF_ENOMEM, "hipMalloc of the statistics partials failed");
    if (L->partials) (void)hipFree(L->partials);
    L->partials = parts;
    L->partials_cap = g;
    L->partials_slots = slots;
  }
  L->fused_slots = slots;
  L->stat_batch = K;
  L->block = block;
  L->pd = pd;
  L->pf = pf;
  L->fused = fused;
  L->grid = cells || grid > nt ? nt : grid;  // cell order: one workgroup per tile
  L->nparts = g;
  drop_graphs(L);
  return CMF_OK;
}

const void *step_params(const cmf_lattice *L) {
  return L->storage == kF64 ? (const void *)&L->pd : (const void *)&L->pf;
}

// partial-sum slot b (0 .. 2 stat_batch - 1) of the lattice
double *partials_buf(const cmf_lattice *L, int b) {
  return L->partials + (size_t)b * kPartStride * L->partials_cap;
}

// Streaming form of a step that starts from state parity b: the pull from
// buffer b into buffer 1 - b, or in place the even half of an AA pair from
// parity 0 (populations at their own sites) and the odd half from parity 1.
int stream_mode(const cmf_lattice *L, int b) {
  return !L->in_place ? kStreamPull : b == 0 ? kStreamAAEven : kStreamAAOdd;
}

// conversion parameters for the current state parity
ConvParams conv(const cmf_lattice *L) {
  ConvParams cp = L->cp;
  cp.layout = !L->in_place ? kLayoutPull : L->parity == 0 ? kLayoutNatural : kLayoutSwapped;
  return cp;
}

// the fused step from state parity b, step index *step_dev + off
hipError_t launch_lattice_step(const cmf_lattice *L, int b, int off, double *partials,
                               hipStream_t s) {
  return launch_step(L->q, L->storage, L->general, L->nt_stores, stream_mode(L, b), step_params(L),
                     L->buf[b], L->buf[b ^ 1], L->step_dev, off, partials, L->grid, L->block, s);
}

// One direct step: the fused kernel, then its statistics and the step
// counter on the same stream.
int enqueue_one_step(cmf_lattice *L) {
  HIP_TRY(launch_lattice_step(L, L->parity, 0, partials_buf(L, 0), L->stream));
  HIP_TRY(launch_finalize(partials_buf(L, 0), L->nparts, L->level2, L->series, L->cap,
                          L->step_dev, 0, 1, L->mass0,
                          !(L->desc.flags & CMF_FLAG_NO_STATS), L->stream));
  L->parity ^= 1;
  return CMF_OK;
}

// Time n full steps (fused step + statistics finalize) as direct launches.
int time_full_steps(cmf_lattice *L, int n, double *ms_out) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  HIP_TRY(hipEventCreate(&e0));
  hipError_t e = hipEventCreate(&e1);
  if (e == hipSuccess) e = hipEventRecord(e0, L->stream);
  int rc = CMF_OK;
  for (int s = 0; s < n && e == hipSuccess && rc == CMF_OK; ++s) rc = enqueue_one_step(L);
  if (e == hipSuccess) e = hipEventRecord(e1, L->stream);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = 0.0f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (rc != CMF_OK) return rc;
  if (e != hipSuccess) return fail(CMF_EHIP, "timing failed: %s", hipGetErrorString(e));
  *ms_out = ms;
  return CMF_OK;
}

// Steps of a forked run starting from buffer `parity` (step j reads
// buf[parity ^ (j & 1)]) and the statistics reductions of their batches.
struct LatticeRun {
  cmf_lattice *L;
  int parity;
  hipError_t operator()(int j, hipStream_t s) const {
    return launch_lattice_step(L, parity ^ (j & 1), j, partials_buf(L, j % (2 * L->stat_batch)), s);
  }
};
struct LatticeFin {
  cmf_lattice *L;
  hipError_t operator()(int j0, int count, int bump, hipStream_t s) const {
    // j0 is a multiple of stat_batch: the batch's slots are consecutive
    return launch_finalize_batch(partials_buf(L, j0 % (2 * L->stat_batch)),
                                 (int64_t)kPartStride * L->partials_cap, count, L->nparts,
                                 L->level2, L->series, L->cap, L->step_dev, j0, bump, L->mass0,
                                 true, s);
  }
};

int capture_graph(cmf_lattice *L, int parity) {
  const bool stats = !(L->desc.flags & CMF_FLAG_NO_STATS);
  return capture_forked(L->stream, L->forked, stats, L->stat_batch, L->step_dev,
                        LatticeRun{L, parity}, LatticeFin{L}, &L->graph[parity]);
}

// n <= kGraphSteps direct steps in the forked form
int run_direct(cmf_lattice *L, int n) {
  const bool stats = !(L->desc.flags & CMF_FLAG_NO_STATS);
  int rc = run_forked(L->stream, L->forked, stats, L->stat_batch, L->step_dev,
                      LatticeRun{L, L->parity}, LatticeFin{L}, n);
  if (rc == CMF_OK) L->parity ^= (n & 1);
  return rc;
}

// A run of n steps of a fused lattice: launches of odd numbers of steps, at
// most kFusedSteps, as even as possible and as few as leave the state in the
// buffer that single steps would (each launch goes from one buffer to the
// other, so their number must be odd when n is).  The statistics of up to
// fused_slots steps are reduced at once, on the same stream: a reduction
// takes about as long as one launch, far less than the event waits of a
// second stream.
int run_fused(cmf_lattice *L, int n) {
  const bool stats = !(L->desc.flags & CMF_FLAG_NO_STATS);
  const int64_t pstride = (int64_t)kPartStride * L->partials_cap;
  const int slots = L->fused_slots, kmax = kFusedSteps < slots ? kFusedSteps : slots - 1;
  int m = (n + kmax - 1) / kmax;
  m += (m ^ n) & 1;
  const int pairs = (n - m) / 2;
  hipError_t e = hipSuccess;
  int done = 0, reduced = 0;
  for (int c = 0; c < m && e == hipSuccess; ++c) {
    const int k = 1 + 2 * (pairs / m + (c < pairs % m ? 1 : 0));
    auto reduce = [&]() {
      if (!stats || done == reduced) return hipSuccess;
      const hipError_t x = launch_finalize_batch(L->partials, pstride, done - reduced, L->nparts, L->level2, L->series,
                                   L->cap, L->step_dev, reduced, 0, L->mass0, true, L->stream);
      reduced = done;
      return x;
    };
    if (done + k - reduced > slots) e = reduce();
    if (e == hipSuccess)
      e = launch_step_fused(L->storage, L->general, L->fused, step_params(L), L->buf[L->parity],
                            L->buf[L->parity ^ 1], L->step_dev, done, k,
                            stats ? L->partials + (done - reduced) * pstride : nullptr, pstride,
                            L->stream);
    if (e == hipSuccess) {
      L->parity ^= 1;
      done += k;
      if (c == m - 1) e = reduce();
    }
  }
  if (e == hipSuccess) e = launch_bump_step(L->step_dev, n, L->stream);
  if (e != hipSuccess) return fail(CMF_EHIP, "step launch failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

// Copies of device arrays into the caller's pageable memory.  The runtime's
// own copy moves them through its staging buffers on one thread, 17 GB/s into
// memory that has been written before and 10 into fresh pages (a numpy array),
// against 56 GB/s of the link to pinned memory.  Large arrays therefore go
// through a ring of pinned chunks that kFetchThreads threads empty into the
// caller's array, whose page faults they share (57 MB into a new numpy array 5.8 ->
// 2.1 ms, 453 MB 45 -> 12).

// chunks 0 .. n - 1 in order: copies enqueued and waited for by this thread
// (the only one that calls the runtime), emptied by the others; chunk c uses
// slot c mod kFetchSlots once chunk c - kFetchSlots is out
hipError_t fetch_chunks(char *dst, const char *src, size_t bytes, FetchRing &ring) {
  const int64_t n = (int64_t)((bytes + kFetchChunk - 1) / kFetchChunk);
  std::mutex mu;
  std::condition_variable cv;
  int64_t landed = 0, taken = 0;
  bool stop = false;
  std::vector<char> out(n, 0);  // all guarded by mu
  auto size_of = [&](int64_t c) {
    const size_t at = (size_t)c * kFetchChunk;
    return bytes - at < kFetchChunk ? bytes - at : kFetchChunk;
  };
  auto work = [&]() {
    std::unique_lock<std::mutex> lk(mu);
    while (!stop && taken < n) {
      const int64_t c = taken++;
      cv.wait(lk, [&] { return landed > c || stop; });
      if (landed <= c) break;
      lk.unlock();
      memcpy(dst + (size_t)c * kFetchChunk, ring.pin + (size_t)(c % kFetchSlots) * kFetchChunk, size_of(c));
      lk.lock();
      out[c] = 1;
      cv.notify_all();
    }
  };
  std::vector<std::thread> threads;
  threads.reserve(kFetchThreads);
  try {
    for (int t = 0; t < kFetchThreads; ++t) threads.emplace_back(work);
  } catch (...) {
    // no thread or no memory for one: those that run are enough, if any do,
    // and must not be left joinable by an exception
  }
  if (threads.empty()) return hipErrorOutOfMemory;
  hipError_t e = hipSuccess;
  int64_t issued = 0;
  for (int64_t c = 0; c < n && e == hipSuccess; ++c) {
    for (; issued < n && issued < c + kFetchSlots && e == hipSuccess; ++issued) {
      if (issued >= kFetchSlots) {
        // the slot's last chunk is out, or waited for where chunk c needs it
        std::unique_lock<std::mutex> lk(mu);
        if (issued == c) cv.wait(lk, [&] { return out[issued - kFetchSlots] != 0; });
        if (!out[issued - kFetchSlots]) break;
      }
      const int slot = (int)(issued % kFetchSlots);
      e = hipMemcpyAsync(ring.pin + (size_t)slot * kFetchChunk, src + (size_t)issued * kFetchChunk,
                         size_of(issued), hipMemcpyDeviceToHost, nullptr);
      if (e == hipSuccess) e = hipEventRecord(ring.ready[slot], nullptr);
    }
    if (e == hipSuccess) e = hipEventSynchronize(ring.ready[c % kFetchSlots]);
    {
      std::lock_guard<std::mutex> lk(mu);
      if (e == hipSuccess)
        landed = c + 1;
      else
        stop = true;
    }
    cv.notify_all();
  }
  for (auto &t : threads) t.join();
  (void)hipStreamSynchronize(nullptr);  // no copy into the ring outlives it
  return e;
}

// `bytes` from device memory at src to dst, after the work already on s;
// returns when they are there (through the default stream, as hipMemcpy).
hipError_t fetch(FetchUser &user, void *dst, const void *src, size_t bytes, hipStream_t s) {
  const hipError_t w = hipStreamSynchronize(s);
  if (w != hipSuccess) return w;
  if (bytes >= 2 * kFetchChunk) {
    if (FetchRing *ring = user.take()) {
      hipError_t e = hipErrorOutOfMemory;
      try {
        e = fetch_chunks((char *)dst, (const char *)src, bytes, *ring);
      } catch (const std::bad_alloc &) {
      }
      user.give(ring);
      if (e == hipSuccess) return e;
      (void)hipGetLastError();
    }
  }
  return hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
}

// Rows of steps [first, step), at most cap of them, from a series ring on the
// device: the run up to the ring's end and the one from its start, or, of a
// small ring, all of it (a copy takes 6 us, a larger one hardly more).
hipError_t copy_series(const double *series, int cap, int64_t first, int64_t step,
                       std::vector<double> &rows) {
  rows.resize((size_t)(step - first) * kSeriesStride);
  if (step > first && first % cap + step - first > cap && cap <= 512) {
    std::vector<double> ring((size_t)cap * kSeriesStride);
    const hipError_t e = hipMemcpy(ring.data(), series, sizeof(double) * ring.size(), hipMemcpyDeviceToHost);
    for (int64_t s = first; s < step && e == hipSuccess; ++s)
      memcpy(rows.data() + (s - first) * kSeriesStride, ring.data() + (s % cap) * kSeriesStride,
             sizeof(double) * kSeriesStride);
    return e;
  }
  for (int64_t s = first; s < step;) {
    const int64_t at = s % cap, n = step - s < cap - at ? step - s : cap - at;
    const hipError_t e = hipMemcpy(rows.data() + (s - first) * kSeriesStride,
                                   series + at * kSeriesStride,
                                   sizeof(double) * kSeriesStride * n, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    s += n;
  }
  return hipSuccess;
}

void release(cmf_lattice *L) {
  if (!L) return;
  if (L->stream) (void)hipStreamSynchronize(L->stream);
  for (int k = 0; k < 2; ++k) {
    if (L->graph[k]) (void)hipGraphExecDestroy(L->graph[k]);
    if (L->buf[k] && L->own_bufs && !(k == 1 && L->buf[1] == L->buf[0])) (void)hipFree(L->buf[k]);
  }
  if (L->partials) (void)hipFree(L->partials);
  if (L->level2) (void)hipFree(L->level2);
  if (L->series) (void)hipFree(L->series);
  if (L->step_dev) (void)hipFree(L->step_dev);
  if (L->sk_has_plan) (void)hipfftDestroy(L->sk_plan);
  for (void *p : {(void *)L->sk_fields, L->sk_F, (void *)L->sk_acc, (void *)L->sk_out,
                  (void *)L->sk_perm, (void *)L->sk_off, (void *)L->vel_ws})
    if (p) (void)hipFree(p);
  forked_release(L->forked);
  if (L->own_stream && L->stream) (void)hipStreamDestroy(L->stream);
  delete L;
}

int validate(const cmf_desc *d) {
  if (!d) return fail(CMF_EINVAL, "desc is NULL");
  if (d->q != 9 && d->q != 19 && d->q != 27)
    return fail(CMF_EINVAL, "q must be 9, 19 or 27, got %d", d->q);
  if (d->nx < 1 || d->ny < 1 || d->nz < 1)
    return fail(CMF_EINVAL, "box edges must be >= 1 (%d, %d, %d)", d->nx, d->ny, d->nz);
  if (d->q == 9 && d->nz != 1) return fail(CMF_EINVAL, "D2Q9 needs nz = 1, got %d", d->nz);
  if (!sqrt_norms_consistent(d->q))
    return fail(CMF_EINVAL, "internal: the kernels' sqrt(b_v) table does not match the basis");
  const int64_t N = (int64_t)d->nx * d->ny * d->nz;
  if (N >= (int64_t)1 << 31) return fail(CMF_EINVAL, "N = %lld sites exceeds 2^31 - 1", (long long)N);
  if (d->nx >= (1 << 28)) return fail(CMF_EINVAL, "nx = %d is not below 2^28", d->nx);
  if (d->storage < kF64 || d->storage > kBF16) return fail(CMF_EINVAL, "unknown storage %d", d->storage);
  if (!(d->rho0 > 0.0) || !isfinite(d->rho0)) return fail(CMF_EINVAL, "rho0 must be > 0");
  if (!(d->tau >= 0.5) || !isfinite(d->tau)) return fail(CMF_EINVAL, "tau must be >= 0.5");
  if (!(d->kT >= 0.0) || !isfinite(d->kT)) return fail(CMF_EINVAL, "kT must be >= 0");
  if (d->lambda)
    for (int v = 0; v < d->q; ++v)
      if (!(d->lambda[v] >= 0.0 && d->lambda[v] <= 2.0))
        return fail(CMF_EINVAL, "lambda[%d] = %g outside [0, 2]", v, d->lambda[v]);
  if (d->series_capacity < 0) return fail(CMF_EINVAL, "series_capacity < 0");
  return CMF_OK;
}

}  // namespace

extern "C" {

const char *cmf_version(void) { return "cmflb 0.1 (gfx950)"; }

const char *cmf_last_error(void) { return g_last_error.c_str(); }

int cmf_device_count(void) {
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess) return 0;
  return n;
}

namespace {

// host checks of the fields of an equilibrium initialisation: positive
// finite densities, finite velocities
int check_init_fields(int64_t N, const double *rho, const double *u) {
  if (rho)
    for (int64_t s = 0; s < N; ++s)
      if (!(rho[s] > 0.0) || !isfinite(rho[s]))
        return fail(CMF_EINVAL, "rho[%lld] = %g is not a positive density", (long long)s, rho[s]);
  if (u)
    for (int64_t s = 0; s < 3 * N; ++s)
      if (!isfinite(u[s]))
        return fail(CMF_EINVAL, "u[%lld] = %g is not finite", (long long)s, u[s]);
  return CMF_OK;
}

// device copies of the optional rho (N) and u (3 N) fields; on failure
// nothing stays allocated
hipError_t upload_init_fields(int64_t N, const double *rho, const double *u, double **drho,
                              double **du) {
  *drho = *du = nullptr;
  hipError_t e = hipSuccess;
  if (rho) {
    e = hipMalloc((void **)drho, sizeof(double) * N);
    if (e == hipSuccess) e = hipMemcpy(*drho, rho, sizeof(double) * N, hipMemcpyHostToDevice);
  }
  if (e == hipSuccess && u) {
    e = hipMalloc((void **)du, sizeof(double) * 3 * N);
    if (e == hipSuccess) e = hipMemcpy(*du, u, sizeof(double) * 3 * N, hipMemcpyHostToDevice);
  }
  if (e != hipSuccess) {
    if (*drho) (void)hipFree(*drho);
    if (*du) (void)hipFree(*du);
    *drho = *du = nullptr;
  }
  return e;
}

// timing events, all or none
int create_events(std::vector<hipEvent_t> &ev) {
  for (auto &x : ev) {
    const hipError_t e = hipEventCreate(&x);
    if (e != hipSuccess) {
      for (auto &y : ev)
        if (y) (void)hipEventDestroy(y);
      return fail(CMF_EHIP, "hipEventCreate failed: %s", hipGetErrorString(e));
    }
  }
  return CMF_OK;
}

// bytes of one population buffer (q x N elements, rounded up to 256)
size_t buffer_bytes(const cmf_desc *d) {
  return ((size_t)d->q * d->nx * d->ny * d->nz * storage_bytes(d->storage) + 255) / 256 * 256;
}

// `p` must point into a device allocation of the current device with at
// least `bytes` bytes from p to the allocation's end (host-side queries
// only: a wrong pointer or a short buffer becomes CMF_EINVAL instead of a
// kernel access out of bounds).
int check_device_span(const void *p, size_t bytes, const char *what) {
  hipPointerAttribute_t attr;
  int dev = 0;
  if (hipPointerGetAttributes(&attr, p) != hipSuccess || attr.type != hipMemoryTypeDevice ||
      hipGetDevice(&dev) != hipSuccess || attr.device != dev) {
    (void)hipGetLastError();
    return fail(CMF_EINVAL, "%s is not device memory of the current device", what);
  }
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess) {
    (void)hipGetLastError();
    return fail(CMF_EINVAL, "%s: the allocation holding it is not known to HIP", what);
  }
  const uintptr_t b = reinterpret_cast<uintptr_t>(base), a = reinterpret_cast<uintptr_t>(p);
  if (a < b || a - b > size || size - (a - b) < bytes)
    return fail(CMF_EINVAL, "%s: %zu bytes from it to the end of its allocation, %zu needed",
                what, a < b || a - b > size ? (size_t)0 : size - (a - b), bytes);
  return CMF_OK;
}

// population buffers of a lattice: one with in-place streaming, else two
int buffer_count(const cmf_desc *d) { return (d->flags & CMF_FLAG_IN_PLACE) ? 1 : 2; }

// in-place streaming addresses each z plane (ny q nx values) with 32-bit
// byte offsets
int check_in_place(const cmf_desc *d) {
  if (!(d->flags & CMF_FLAG_IN_PLACE)) return CMF_OK;
  const int64_t plane = (int64_t)d->ny * d->q * d->nx * storage_bytes(d->storage);
  if (plane >= ((int64_t)1 << 32))
    return fail(CMF_EUNSUPPORTED, "in-place streaming needs each z plane below 4 GiB (%lld bytes)",
                (long long)plane);
  return CMF_OK;
}

int create_lattice(const cmf_desc *desc, void *hip_stream, void *ext, size_t ext_bytes,
                   cmf_lattice **out) {
  if (!out) return fail(CMF_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = validate(desc);
  if (rc != CMF_OK) return rc;
  rc = check_in_place(desc);
  if (rc != CMF_OK) return rc;
  if (ext) {
    const size_t need = buffer_count(desc) * buffer_bytes(desc);
    if (reinterpret_cast<uintptr_t>(ext) % 256 != 0)
      return fail(CMF_EINVAL, "external buffer is not 256-byte aligned");
    if (ext_bytes < need)
      return fail(CMF_EINVAL, "external buffer holds %zu bytes, the lattice needs %zu", ext_bytes, need);
    rc = check_device_span(ext, need, "external buffer");
    if (rc != CMF_OK) return rc;
  }
  cmf_lattice *L = new cmf_lattice();
  L->desc = *desc;
  L->desc.lambda = nullptr;
  L->q = desc->q;
  L->storage = desc->storage;
  L->N = (int64_t)desc->nx * desc->ny * desc->nz;
  L->cap = desc->series_capacity > 0 ? desc->series_capacity : 4096;
  const int q = L->q;

  // rates (the paper's pattern unless given) and the FP64 per-mode
  // constants
  ModeConstants mc;
  mode_constants(desc, mc);
  L->general = mc.general;
  L->nt_stores = ((int64_t)desc->nx * storage_bytes(desc->storage)) % kLineBytes == 0;
  L->in_place = (desc->flags & CMF_FLAG_IN_PLACE) != 0;
  double amp[27];
  float scale[27];
  for (int v = 0; v < q; ++v) {
    L->lambda[v] = mc.lambda[v];
    L->w[v] = mc.w[v];
    amp[v] = mc.amp[v];
    scale[v] = mc.scale[v];
  }
  L->mass0 = (double)L->N * desc->rho0;
  for (int v = 0; v < q; ++v) {
    L->amp[v] = amp[v];
    L->scale[v] = scale[v];
  }

  L->cp.nx = desc->nx;
  L->cp.ny = desc->ny;
  L->cp.nz = desc->nz;
  L->cp.pitch = 0;
  L->cp.layout = kLayoutPull;
  L->cp.rho0 = desc->rho0;
  for (int i = 0; i < q; ++i) {
    L->cp.w[i] = L->w[i];
    L->cp.scale[i] = scale[i];
    L->cp.iscale[i] = 1.0f / scale[i];
  }

  hipError_t e = hipGetDevice(&L->device);
  if (e != hipSuccess) {
    release(L);
    return fail(CMF_EHIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  }
  if (hip_stream) {
    L->stream = (hipStream_t)hip_stream;
  } else {
    e = hipStreamCreate(&L->stream);
    if (e != hipSuccess) {
      release(L);
      return fail(CMF_EHIP, "hipStreamCreate failed: %s", hipGetErrorString(e));
    }
    L->own_stream = true;
  }
  const size_t bytes = buffer_bytes(desc);
  if (ext) {
    L->own_bufs = false;
    L->buf[0] = ext;
    L->buf[1] = L->in_place ? ext : static_cast<char *>(ext) + bytes;
  } else {
    for (int k = 0; k < buffer_count(desc); ++k) {
      if (hipMalloc(&L->buf[k], bytes) != hipSuccess) {
        release(L);
        return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
      }
    }
    if (L->in_place) L->buf[1] = L->buf[0];
  }
  if (hipMalloc((void **)&L->series, sizeof(double) * kSeriesStride * L->cap) != hipSuccess ||
      hipMalloc((void **)&L->level2, sizeof(double) * kPartStride * kMaxLevel2 * kStatBatch) !=
          hipSuccess ||
      hipMalloc((void **)&L->step_dev, sizeof(int64_t)) != hipSuccess) {
    release(L);
    return fail(CMF_ENOMEM, "hipMalloc of statistics buffers failed");
  }
  // launch shape: a tuned one for this key if known, else the defaults
  {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, L->device) == hipSuccess && prop.multiProcessorCount > 0)
      L->cus = prop.multiProcessorCount;
    int block = default_block(*desc, L->cus);
    int grid = default_grid(L, block);
    lookup_tuned(L, &block, &grid);
    const int be = env_int("CMF_BLOCK", 0), ge = env_int("CMF_GRID", 0);
    if (be == 64 || be == 128 || be == 192 || be == 256) block = be;
    if (ge > 0) grid = ge;
    L->shape_set = be == block || ge > 0;
    rc = apply_launch(L, block, grid, L->amp, L->scale);
    if (rc != CMF_OK) {
      release(L);
      return rc;
    }
  }
  *out = L;
  rc = cmf_init_equilibrium(L, nullptr, nullptr);
  if (rc != CMF_OK) {
    release(L);
    *out = nullptr;
    return rc;
  }
  return CMF_OK;
}

}  // namespace

int cmf_create(const cmf_desc *desc, void *hip_stream, cmf_lattice **out) {
  return create_lattice(desc, hip_stream, nullptr, 0, out);
}

int cmf_create_external(const cmf_desc *desc, void *dev_ptr, size_t bytes, void *hip_stream,
                        cmf_lattice **out) {
  if (!dev_ptr) return fail(CMF_EINVAL, "dev_ptr is NULL");
  return create_lattice(desc, hip_stream, dev_ptr, bytes, out);
}

size_t cmf_external_bytes(const cmf_desc *desc) {
  if (validate(desc) != CMF_OK || check_in_place(desc) != CMF_OK) return 0;
  return buffer_count(desc) * buffer_bytes(desc);
}

int cmf_destroy(cmf_lattice *L) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  release(L);
  return CMF_OK;
}

int cmf_init_equilibrium(cmf_lattice *L, const double *rho, const double *u) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  int rc = check_init_fields(L->N, rho, u);
  if (rc != CMF_OK) return rc;
  HIP_TRY(hipStreamSynchronize(L->stream));
  double *drho = nullptr, *du = nullptr;
  hipError_t e = upload_init_fields(L->N, rho, u, &drho, &du);
  if (e == hipSuccess) {
    L->parity = 0;
    e = launch_init_eq(L->q, L->storage, conv(L), drho, du, L->buf[0], L->stream);
  }
  if (e == hipSuccess) e = launch_zero_i64(L->step_dev, 1, L->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
  if (drho) (void)hipFree(drho);
  if (du) (void)hipFree(du);
  if (e != hipSuccess) return fail(CMF_EHIP, "equilibrium initialisation failed: %s", hipGetErrorString(e));
  L->read_step = 0;
  return CMF_OK;
}

int cmf_set_populations(cmf_lattice *L, const double *f) {
  if (!L || !f) return fail(CMF_EINVAL, "NULL argument");
  HIP_TRY(hipStreamSynchronize(L->stream));
  double *df = nullptr;
  const size_t bytes = sizeof(double) * L->q * L->N;
  if (hipMalloc((void **)&df, bytes) != hipSuccess)
    return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  hipError_t e = hipMemcpy(df, f, bytes, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = launch_set_state(L->q, L->storage, conv(L), df, L->buf[L->parity], L->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
  (void)hipFree(df);
  if (e != hipSuccess) return fail(CMF_EHIP, "set_populations failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_get_populations(cmf_lattice *L, double *f) {
  if (!L || !f) return fail(CMF_EINVAL, "NULL argument");
  HIP_TRY(hipStreamSynchronize(L->stream));
  double *df = nullptr;
  const size_t bytes = sizeof(double) * L->q * L->N;
  if (hipMalloc((void **)&df, bytes) != hipSuccess)
    return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  hipError_t e = launch_get_state(L->q, L->storage, conv(L), L->buf[L->parity], df, L->stream);
  if (e == hipSuccess) e = fetch(L->fetches, f, df, bytes, L->stream);
  (void)hipFree(df);
  if (e != hipSuccess) return fail(CMF_EHIP, "get_populations failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_gather_sites(cmf_lattice *L, const int64_t *sites, int64_t n, double *out) {
  if (!L || (n > 0 && (!sites || !out))) return fail(CMF_EINVAL, "NULL argument");
  if (n < 0) return fail(CMF_EINVAL, "n < 0");
  if (n == 0) return CMF_OK;
  for (int64_t k = 0; k < n; ++k)
    if (sites[k] < 0 || sites[k] >= L->N)
      return fail(CMF_EINVAL, "site %lld outside [0, %lld)", (long long)sites[k], (long long)L->N);
  HIP_TRY(hipStreamSynchronize(L->stream));
  int64_t *ds = nullptr;
  double *dout = nullptr;
  if (hipMalloc((void **)&ds, sizeof(int64_t) * n) != hipSuccess ||
      hipMalloc((void **)&dout, sizeof(double) * L->q * n) != hipSuccess) {
    if (ds) (void)hipFree(ds);
    return fail(CMF_ENOMEM, "hipMalloc failed");
  }
  hipError_t e = hipMemcpy(ds, sites, sizeof(int64_t) * n, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = launch_gather(L->q, L->storage, conv(L), L->buf[L->parity], ds, n, dout, L->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
  if (e == hipSuccess) e = hipMemcpy(out, dout, sizeof(double) * L->q * n, hipMemcpyDeviceToHost);
  (void)hipFree(ds);
  (void)hipFree(dout);
  if (e != hipSuccess) return fail(CMF_EHIP, "gather_sites failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_step(cmf_lattice *L, int64_t nsteps) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (nsteps < 0) return fail(CMF_EINVAL, "nsteps < 0");
  const bool graphs = !(L->desc.flags & CMF_FLAG_NO_GRAPH) && !L->graphs_dropped;
  int64_t left = nsteps;
  while (L->fused && left > 2) {
    const int n = left < (1 << 20) ? (int)left : 1 << 20;
    int rc = run_fused(L, n);
    if (rc != CMF_OK) return rc;
    left -= n;
  }
  while (graphs && left >= kGraphSteps) {
    if (!L->graph[L->parity]) {
      int rc = capture_graph(L, L->parity);
      if (rc != CMF_OK) return rc;
    }
    HIP_TRY(hipGraphLaunch(L->graph[L->parity], L->stream));
    left -= kGraphSteps;  // an even number of steps: parity unchanged
  }
  while (left > 0) {
    const int n = left < kGraphSteps ? (int)left : kGraphSteps;
    int rc = run_direct(L, n);
    if (rc != CMF_OK) return rc;
    left -= n;
  }
  return CMF_OK;
}

int cmf_profile_steps(cmf_lattice *L, int64_t nsteps, double *kernel_ms) {
  if (!L || !kernel_ms) return fail(CMF_EINVAL, "NULL argument");
  if (nsteps < 0) return fail(CMF_EINVAL, "nsteps < 0");
  *kernel_ms = 0.0;
  if (nsteps == 0) return CMF_OK;
  std::vector<hipEvent_t> ev(2 * nsteps, nullptr);
  int rc = create_events(ev);
  if (rc != CMF_OK) return rc;
  // batches of stat_batch steps, each kernel between its own event pair and
  // the batch's statistics reduction after the batch, so that only event
  // markers separate consecutive step kernels
  const int K = L->stat_batch;
  const bool stats = !(L->desc.flags & CMF_FLAG_NO_STATS);
  for (int64_t s0 = 0; s0 < nsteps && rc == CMF_OK; s0 += K) {
    const int cnt = nsteps - s0 < K ? (int)(nsteps - s0) : K;
    hipError_t e = hipSuccess;
    for (int j = 0; j < cnt && e == hipSuccess; ++j) {
      e = hipEventRecord(ev[2 * (s0 + j)], L->stream);
      if (e == hipSuccess) e = launch_lattice_step(L, L->parity, j, partials_buf(L, j), L->stream);
      if (e == hipSuccess) e = hipEventRecord(ev[2 * (s0 + j) + 1], L->stream);
      if (e == hipSuccess) L->parity ^= 1;
    }
    if (e == hipSuccess && stats)
      e = launch_finalize_batch(partials_buf(L, 0), (int64_t)kPartStride * L->partials_cap, cnt,
                                L->nparts, L->level2, L->series, L->cap, L->step_dev, 0, 0,
                                L->mass0, true, L->stream);
    if (e == hipSuccess) e = launch_bump_step(L->step_dev, cnt, L->stream);
    if (e != hipSuccess) rc = fail(CMF_EHIP, "profiled step failed: %s", hipGetErrorString(e));
  }
  hipError_t e = hipStreamSynchronize(L->stream);
  if (rc == CMF_OK && e != hipSuccess) rc = fail(CMF_EHIP, "hipStreamSynchronize failed: %s", hipGetErrorString(e));
  double total = 0.0;
  for (int64_t s = 0; s < nsteps && rc == CMF_OK; ++s) {
    float ms = 0.0f;
    e = hipEventElapsedTime(&ms, ev[2 * s], ev[2 * s + 1]);
    if (e != hipSuccess) rc = fail(CMF_EHIP, "hipEventElapsedTime failed: %s", hipGetErrorString(e));
    total += ms;
  }
  for (auto &x : ev) (void)hipEventDestroy(x);
  *kernel_ms = total;
  return rc;
}

int cmf_sk_reset(cmf_lattice *L, int32_t nbins) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (nbins < 1 || nbins > kSkMaxBins)
    return fail(CMF_EINVAL, "nbins must be in [1, %d], got %d", kSkMaxBins, nbins);
  HIP_TRY(hipStreamSynchronize(L->stream));
  const int nx = L->desc.nx, ny = L->desc.ny, nz = L->desc.nz;
  const int64_t M = (int64_t)(nx / 2 + 1) * ny * nz;
  if (!L->sk_has_plan) {
    // all buffers and the plan, or none of them
    auto drop = [&]() {
      for (void **p : {(void **)&L->sk_fields, &L->sk_F, (void **)&L->sk_acc, (void **)&L->sk_perm}) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
      }
    };
    drop();
    if (hipMalloc((void **)&L->sk_fields, sizeof(float) * 4 * L->N) != hipSuccess ||
        hipMalloc(&L->sk_F, sizeof(float) * 2 * 4 * M) != hipSuccess ||
        hipMalloc((void **)&L->sk_acc, sizeof(double) * 4 * M) != hipSuccess ||
        hipMalloc((void **)&L->sk_perm, sizeof(int32_t) * M) != hipSuccess) {
      drop();
      return fail(CMF_ENOMEM, "structure-factor allocation failed");
    }
    // the four fields as one batch, a quarter of the launches; one field per
    // call for boxes that fill the chip by themselves (and whose transforms'
    // workspace would be four times as large), or where the batch is refused
    int dims3[3] = {nz, ny, nx};
    const int rank = nz > 1 ? 3 : 2;
    L->sk_batch = L->N <= kSkBatchSites ? 4 : 1;
    hipfftResult fr = HIPFFT_SUCCESS;
    if (L->sk_batch == 4)
      fr = hipfftPlanMany(&L->sk_plan, rank, dims3 + 3 - rank, nullptr, 1, (int)L->N, nullptr, 1,
                          (int)M, HIPFFT_R2C, 4);
    if (L->sk_batch == 1 || fr != HIPFFT_SUCCESS) {
      (void)hipGetLastError();
      L->sk_batch = 1;
      fr = nz > 1 ? hipfftPlan3d(&L->sk_plan, nz, ny, nx, HIPFFT_R2C)
                  : hipfftPlan2d(&L->sk_plan, ny, nx, HIPFFT_R2C);
    }
    if (fr != HIPFFT_SUCCESS) {
      drop();
      return fail(CMF_EHIP, "hipfft plan failed (%d)", (int)fr);
    }
    if (hipfftSetStream(L->sk_plan, L->stream) != HIPFFT_SUCCESS) {
      (void)hipfftDestroy(L->sk_plan);
      drop();
      return fail(CMF_EHIP, "hipfftSetStream failed");
    }
    L->sk_has_plan = true;
    L->sk_M = M;
  }
  if (L->sk_nbins != nbins) {
    L->sk_nbins = 0;  // no shells until the new ones are in place
    if (L->sk_off) (void)hipFree(L->sk_off);
    if (L->sk_out) (void)hipFree(L->sk_out);
    L->sk_off = nullptr;
    L->sk_out = nullptr;
    int32_t *counts = nullptr;
    if (hipMalloc((void **)&L->sk_off, sizeof(int64_t) * (nbins + 1)) != hipSuccess ||
        hipMalloc((void **)&L->sk_out, sizeof(double) * 6 * nbins * (1 + kSkParts)) != hipSuccess ||
        hipMalloc((void **)&counts, sizeof(int32_t) * kSkChunks * nbins) != hipSuccess)
      return fail(CMF_ENOMEM, "structure-factor allocation failed");
    hipError_t e = launch_sk_shells(nx, ny, nz, nbins, M, counts, L->sk_perm, L->sk_off, L->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
    (void)hipFree(counts);
    if (e != hipSuccess) return fail(CMF_EHIP, "shell sort failed: %s", hipGetErrorString(e));
    L->sk_nbins = nbins;
  }
  HIP_TRY(hipMemsetAsync(L->sk_acc, 0, sizeof(double) * 4 * M, L->stream));
  HIP_TRY(hipStreamSynchronize(L->stream));
  L->sk_samples = 0;
  return CMF_OK;
}

int cmf_sk_accumulate(cmf_lattice *L) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (!L->sk_nbins) return fail(CMF_EINVAL, "call cmf_sk_reset first");
  HIP_TRY(launch_macro_dev(L->q, L->storage, conv(L), L->buf[L->parity], L->sk_fields, L->stream));
  for (int f = 0; f < 4; f += L->sk_batch) {
    hipfftResult fr = hipfftExecR2C(L->sk_plan, (hipfftReal *)(L->sk_fields + f * L->N),
                                    (hipfftComplex *)L->sk_F + f * L->sk_M);
    if (fr != HIPFFT_SUCCESS) return fail(CMF_EHIP, "hipfftExecR2C failed (%d)", (int)fr);
  }
  HIP_TRY(launch_sk_accumulate(L->sk_F, L->sk_M, 1.0 / (double)L->N, L->sk_acc, L->stream));
  ++L->sk_samples;
  return CMF_OK;
}

int cmf_sk_shells(cmf_lattice *L, double *out, int64_t *nsamples) {
  if (!L || !out) return fail(CMF_EINVAL, "NULL argument");
  if (!L->sk_nbins) return fail(CMF_EINVAL, "call cmf_sk_reset first");
  const int nb = L->sk_nbins;
  HIP_TRY(launch_sk_segments(L->sk_acc, L->sk_M, L->desc.nx, L->desc.ny, L->desc.nz, nb,
                             L->sk_perm, L->sk_off, L->sk_out + 6 * nb, L->sk_out, L->stream));
  HIP_TRY(hipStreamSynchronize(L->stream));
  std::vector<double> raw(6 * nb);
  HIP_TRY(hipMemcpy(raw.data(), L->sk_out, sizeof(double) * 6 * nb, hipMemcpyDeviceToHost));
  const double ns = L->sk_samples > 0 ? (double)L->sk_samples : 1.0;
  for (int b = 0; b < nb; ++b) {
    const double w = raw[6 * b + 1];
    out[6 * b + 0] = w > 0 ? raw[6 * b] / w : 0.0;
    out[6 * b + 1] = w;
    for (int c = 2; c < 6; ++c) out[6 * b + c] = w > 0 ? raw[6 * b + c] / w / ns : 0.0;
  }
  if (nsamples) *nsamples = L->sk_samples;
  return CMF_OK;
}

int cmf_get_launch(cmf_lattice *L, cmf_launch *out) {
  if (!L || !out) return fail(CMF_EINVAL, "NULL argument");
  out->block = L->block;
  out->grid = L->grid;
  out->ms_per_step = 0.0;
  return CMF_OK;
}

int cmf_set_launch(cmf_lattice *L, int32_t block, int32_t grid) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (!(block == 64 || block == 128 || block == 192 || block == 256))
    return fail(CMF_EINVAL, "block must be 64, 128, 192 or 256, got %d", block);
  if (grid < 1) return fail(CMF_EINVAL, "grid must be >= 1, got %d", grid);
  HIP_TRY(hipStreamSynchronize(L->stream));
  const bool set0 = L->shape_set;
  L->shape_set = true;
  const int rc = apply_launch(L, block, grid, L->amp, L->scale);
  if (rc != CMF_OK) L->shape_set = set0;
  return rc;
}

int cmf_autotune(cmf_lattice *L, int32_t steps_per_trial, cmf_launch *trials, int32_t cap,
                 int32_t *n_out) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (steps_per_trial < 1) return fail(CMF_EINVAL, "steps_per_trial must be >= 1");
  if (n_out) *n_out = 0;
  HIP_TRY(hipStreamSynchronize(L->stream));
  // snapshot: current population buffer, step counter, series ring
  const size_t bytes = ((size_t)L->q * L->N * storage_bytes(L->storage) + 255) / 256 * 256;
  void *saved = nullptr;
  double *saved_series = nullptr;
  if (hipMalloc(&saved, bytes) != hipSuccess) return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  if (hipMalloc((void **)&saved_series, sizeof(double) * kSeriesStride * L->cap) != hipSuccess) {
    (void)hipFree(saved);
    return fail(CMF_ENOMEM, "hipMalloc of the statistics snapshot failed");
  }
  int64_t step0 = 0;
  const int parity0 = L->parity;
  const int block0 = L->block, grid0 = L->grid;
  hipError_t e = hipMemcpyAsync(saved, L->buf[parity0], bytes, hipMemcpyDeviceToDevice, L->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(saved_series, L->series, sizeof(double) * kSeriesStride * L->cap,
                       hipMemcpyDeviceToDevice, L->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(&step0, L->step_dev, sizeof(int64_t), hipMemcpyDeviceToHost, L->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
  if (e != hipSuccess) {
    (void)hipFree(saved);
    (void)hipFree(saved_series);
    return fail(CMF_EHIP, "autotune snapshot failed: %s", hipGetErrorString(e));
  }
  std::vector<int> blocks;
  for (int b = 64; b <= 256; b += 64)
    if (b == 64 || b - 64 < L->desc.nx || flat_plane_tiles(L->desc, b)) blocks.push_back(b);
  std::vector<cmf_launch> done;
  int rc = CMF_OK;
  const bool set0 = L->shape_set;
  L->shape_set = false;
  const bool one_tile = choose_tile_rows(L) > 0;
  for (int b : blocks) {
    std::vector<int> grids;
    if (!one_tile)
      for (int m : {1, 2, 4, 8, 16, 32}) grids.push_back(m * L->cus);
    grids.push_back(ntiles_for(L, b));
    int last = -1;
    for (int g : grids) {
      const int gg = g < ntiles_for(L, b) ? g : ntiles_for(L, b);
      if (gg == last || !launchable(gg, b)) continue;
      last = gg;
      rc = apply_launch(L, b, gg, L->amp, L->scale);
      if (rc != CMF_OK) break;
      double warm = 0.0, ms = 0.0;
      rc = time_full_steps(L, 1, &warm);
      if (rc == CMF_OK) rc = time_full_steps(L, steps_per_trial, &ms);
      if (rc != CMF_OK) break;
      done.push_back(cmf_launch{b, gg, ms / steps_per_trial});
    }
    if (rc != CMF_OK) break;
  }
  // restore the state exactly
  L->parity = parity0;
  e = hipMemcpyAsync(L->buf[parity0], saved, bytes, hipMemcpyDeviceToDevice, L->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(L->series, saved_series, sizeof(double) * kSeriesStride * L->cap,
                       hipMemcpyDeviceToDevice, L->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(L->step_dev, &step0, sizeof(int64_t), hipMemcpyHostToDevice, L->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(L->stream);
  (void)hipFree(saved);
  (void)hipFree(saved_series);
  if (rc == CMF_OK && e != hipSuccess) rc = fail(CMF_EHIP, "autotune restore failed: %s", hipGetErrorString(e));
  if (rc != CMF_OK) {
    L->shape_set = set0;
    (void)apply_launch(L, block0, grid0, L->amp, L->scale);
    return rc;
  }
  size_t best = 0;
  for (size_t k = 1; k < done.size(); ++k)
    if (done[k].ms_per_step < done[best].ms_per_step) best = k;
  rc = apply_launch(L, done[best].block, done[best].grid, L->amp, L->scale);
  if (rc != CMF_OK) return rc;
  remember_tuned(L, done[best].block, done[best].grid, done[best].ms_per_step);
  if (trials)
    for (size_t k = 0; k < done.size() && (int32_t)k < cap; ++k) trials[k] = done[k];
  if (n_out) *n_out = (int32_t)done.size();
  return CMF_OK;
}

int cmf_synchronize(cmf_lattice *L) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  HIP_TRY(hipStreamSynchronize(L->stream));
  return CMF_OK;
}

int cmf_get_step(cmf_lattice *L, int64_t *step) {
  if (!L || !step) return fail(CMF_EINVAL, "NULL argument");
  HIP_TRY(hipStreamSynchronize(L->stream));
  HIP_TRY(hipMemcpy(step, L->step_dev, sizeof(int64_t), hipMemcpyDeviceToHost));
  return CMF_OK;
}

int cmf_set_step(cmf_lattice *L, int64_t step) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (step < 0 || step >= kMaxStep)
    return fail(CMF_EINVAL, "step %lld outside [0, 2^56)", (long long)step);
  HIP_TRY(hipStreamSynchronize(L->stream));
  HIP_TRY(hipMemcpy(L->step_dev, &step, sizeof(int64_t), hipMemcpyHostToDevice));
  L->read_step = step;
  return CMF_OK;
}

int cmf_stats(cmf_lattice *L, cmf_moments *out, int64_t cap, int64_t *n_out) {
  if (!L || !n_out || (cap > 0 && !out)) return fail(CMF_EINVAL, "NULL argument");
  if (cap < 0) return fail(CMF_EINVAL, "cap < 0");
  *n_out = 0;
  int64_t step = 0;
  int rc = cmf_get_step(L, &step);
  if (rc != CMF_OK) return rc;
  if (L->desc.flags & CMF_FLAG_NO_STATS) {
    L->read_step = step;
    return CMF_OK;
  }
  int64_t first = L->read_step;
  if (step - first > L->cap) first = step - L->cap;
  if (step - first > cap) first = step - cap;
  std::vector<double> rows;
  HIP_TRY(copy_series(L->series, L->cap, first, step, rows));
  bool bad = false;
  for (int64_t s = first; s < step; ++s) {
    const double *r = rows.data() + (s - first) * kSeriesStride;
    cmf_moments &m = out[s - first];
    m.step = r[0];
    m.sum_rho = r[1];
    for (int a = 0; a < 3; ++a) {
      m.sum_j[a] = r[2 + a];
      m.sum_u[a] = r[5 + a];
      m.sum_u2[a] = r[8 + a];
    }
    m.nonfinite = r[11];
    if (m.nonfinite != 0.0) bad = true;
  }
  *n_out = step - first;
  L->read_step = step;
  if (bad) return fail(CMF_ENONFINITE, "non-finite density or velocity in a recorded step");
  return CMF_OK;
}

int cmf_sample_macro(cmf_lattice *L, void *rho_dev, void *u_dev) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  int rc = rho_dev ? check_device_span(rho_dev, sizeof(float) * L->N, "rho_dev") : CMF_OK;
  if (rc == CMF_OK && u_dev) rc = check_device_span(u_dev, sizeof(float) * 3 * L->N, "u_dev");
  if (rc != CMF_OK) return rc;
  HIP_TRY(launch_macro(L->q, L->storage, conv(L), L->buf[L->parity], (float *)rho_dev,
                       (float *)u_dev, L->stream));
  return CMF_OK;
}

int cmf_get_macro(cmf_lattice *L, double *rho, double *u) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (!rho && !u) return CMF_OK;
  HIP_TRY(hipStreamSynchronize(L->stream));
  double *d = nullptr;
  const size_t bytes = sizeof(double) * 4 * L->N;
  if (hipMalloc((void **)&d, bytes) != hipSuccess)
    return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  hipError_t e = launch_macro(L->q, L->storage, conv(L), L->buf[L->parity], d, d + L->N, L->stream);
  if (e == hipSuccess && rho) e = fetch(L->fetches, rho, d, sizeof(double) * L->N, L->stream);
  if (e == hipSuccess && u) e = fetch(L->fetches, u, d + L->N, sizeof(double) * 3 * L->N, L->stream);
  (void)hipFree(d);
  if (e != hipSuccess) return fail(CMF_EHIP, "get_macro failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_velocity_pdf(cmf_lattice *L, int32_t nbins, double xmax, double *moments,
                     int64_t *counts) {
  if (!L) return fail(CMF_EINVAL, "lattice is NULL");
  if (counts && (nbins < 1 || nbins > kVelMaxBins))
    return fail(CMF_EINVAL, "nbins = %d outside [1, %d]", nbins, kVelMaxBins);
  if (counts && !(xmax > 0.0 && isfinite(xmax))) return fail(CMF_EINVAL, "xmax must be > 0");
  if (!moments && !counts) return CMF_OK;
  // the workspace stays with the lattice (about 300 KB): the result, the
  // counts right after it, the block sums
  const size_t ncounts = counts ? 3 * ((size_t)nbins + 2) : 0;
  const size_t result = sizeof(VelState) + sizeof(int64_t) * 3 * (kVelMaxBins + 2);
  if (!L->vel_ws &&
      hipMalloc((void **)&L->vel_ws, result + sizeof(double) * kVelCols * kVelGrid) != hipSuccess)
    return fail(CMF_ENOMEM, "hipMalloc failed");
  VelState *st = reinterpret_cast<VelState *>(L->vel_ws);
  unsigned long long *dcounts = reinterpret_cast<unsigned long long *>(L->vel_ws + sizeof(VelState));
  double *partials = reinterpret_cast<double *>(L->vel_ws + result);
  // a lattice of two buffers of its own has room for the velocities in the
  // one that the next step overwrites
  const size_t need = sizeof(double) * (L->q == 9 ? 2 : 3) * (size_t)L->N;
  const bool room = L->own_bufs && !L->in_place && buffer_bytes(&L->desc) >= need;
  HIP_TRY(launch_vel_stats(L->q, L->storage, conv(L), L->buf[L->parity],
                           room ? static_cast<double *>(L->buf[L->parity ^ 1]) : nullptr,
                           counts ? nbins : 1, xmax, partials, st, counts ? dcounts : nullptr,
                           L->stream));
  std::vector<char> host(sizeof(VelState) + sizeof(int64_t) * ncounts);
  HIP_TRY(hipMemcpyAsync(host.data(), L->vel_ws, host.size(), hipMemcpyDeviceToHost, L->stream));
  HIP_TRY(hipStreamSynchronize(L->stream));
  if (moments) memcpy(moments, host.data() + offsetof(VelState, moments), sizeof st->moments);
  if (counts) memcpy(counts, host.data() + sizeof(VelState), sizeof(int64_t) * ncounts);
  return CMF_OK;
}

int cmf_noise_sample(int32_t q, uint64_t seed, uint32_t replica, int64_t step, int64_t site0,
                     int64_t n, int32_t fp64, double *out) {
  if (q != 9 && q != 19 && q != 27) return fail(CMF_EINVAL, "q must be 9, 19 or 27");
  if (step < 0 || step >= kMaxStep) return fail(CMF_EINVAL, "step outside [0, 2^56)");
  if (n < 0 || site0 < 0 || site0 + n > ((int64_t)1 << 32)) return fail(CMF_EINVAL, "bad site range");
  if (n == 0) return CMF_OK;
  if (!out) return fail(CMF_EINVAL, "out is NULL");
  double *d = nullptr;
  if (hipMalloc((void **)&d, sizeof(double) * q * n) != hipSuccess) return fail(CMF_ENOMEM, "hipMalloc failed");
  hipError_t e = launch_noise(q, fp64, (uint32_t)seed, (uint32_t)(seed >> 32), replica, (uint64_t)step,
                              site0, n, d,
                              nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(out, d, sizeof(double) * q * n, hipMemcpyDeviceToHost);
  (void)hipFree(d);
  if (e != hipSuccess) return fail(CMF_EHIP, "noise_sample failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_philox_words(const uint32_t *ctr, int64_t n, uint32_t key0, uint32_t key1, uint32_t *out) {
  if (n < 0) return fail(CMF_EINVAL, "n < 0");
  if (n == 0) return CMF_OK;
  if (!ctr || !out) return fail(CMF_EINVAL, "NULL argument");
  uint32_t *dc = nullptr, *dout = nullptr;
  if (hipMalloc((void **)&dc, 16 * n) != hipSuccess || hipMalloc((void **)&dout, 16 * n) != hipSuccess) {
    if (dc) (void)hipFree(dc);
    return fail(CMF_ENOMEM, "hipMalloc failed");
  }
  hipError_t e = hipMemcpy(dc, ctr, 16 * n, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = launch_philox(dc, n, key0, key1, dout, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(out, dout, 16 * n, hipMemcpyDeviceToHost);
  (void)hipFree(dc);
  (void)hipFree(dout);
  if (e != hipSuccess) return fail(CMF_EHIP, "philox_words failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_stream_copy(size_t bytes, int32_t reps, double *best_ms) {
  if (!best_ms || reps < 1 || bytes == 0) return fail(CMF_EINVAL, "bad arguments");
  const size_t n16 = (bytes + 15) / 16;
  void *a = nullptr, *b = nullptr;
  if (hipMalloc(&a, n16 * 16) != hipSuccess || hipMalloc(&b, n16 * 16) != hipSuccess) {
    if (a) (void)hipFree(a);
    return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", n16 * 16);
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipMemset(a, 0, n16 * 16);
  if (e == hipSuccess) e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e == hipSuccess) e = launch_stream_copy(a, b, n16, nullptr);  // warm-up
  double best = 1e30;
  for (int r = 0; r < reps && e == hipSuccess; ++r) {
    e = hipEventRecord(e0, nullptr);
    if (e == hipSuccess) e = launch_stream_copy(a, b, n16, nullptr);
    if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e == hipSuccess && ms < best) best = ms;
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(a);
  (void)hipFree(b);
  if (e != hipSuccess) return fail(CMF_EHIP, "stream copy failed: %s", hipGetErrorString(e));
  *best_ms = best;
  return CMF_OK;
}

}  // extern "C"

// ---- one step without allocation ------------------------------------------
// Device scratch of cmf_step_noalloc, one copy per GPU the library runs on
// (held until the process ends): the per-workgroup partial sums of the
// statistics (kNoAllocMaxGrid rows), the second-level rows of their
// reduction (kMaxLevel2 rows) and the step counter the kernels read.  In
// host code `scratch` only names the symbol; its device address comes from
// hipGetSymbolAddress, once per device (scratch_address).
namespace {
constexpr int kNoAllocMaxGrid = 65536;
constexpr size_t kScratchPartials = (size_t)kNoAllocMaxGrid * kPartStride;
constexpr size_t kScratchLevel2 = (size_t)kMaxLevel2 * kPartStride;
constexpr size_t kScratchDoubles = kScratchPartials + kScratchLevel2 + 1;
static __device__ __align__(256) double scratch[kScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first
// call on that device, with that device current).
int scratch_address(double **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(CMF_EHIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(CMF_EUNSUPPORTED, "device %d: at most %d devices are supported", dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(CMF_EHIP, "hipGetSymbolAddress of the scratch array failed: %s",
                  hipGetErrorString(e));
    g_scratch_dev[dev] = static_cast<double *>(ptr);
  }
  *out = g_scratch_dev[dev];
  return CMF_OK;
}
}  // namespace

extern "C" int cmf_step_noalloc(const cmf_desc *desc, const void *src, void *dst, int64_t step,
                                int32_t block, int32_t grid, double *stats_dev,
                                void *hip_stream) {
  int rc = validate(desc);
  if (rc != CMF_OK) return rc;
  if (desc->flags & CMF_FLAG_IN_PLACE)
    return fail(CMF_EUNSUPPORTED, "cmf_step_noalloc is a two-buffer pull step (no CMF_FLAG_IN_PLACE)");
  if (!src || !dst || src == dst) return fail(CMF_EINVAL, "src and dst must be two different buffers");
  if (reinterpret_cast<uintptr_t>(src) % 256 != 0 || reinterpret_cast<uintptr_t>(dst) % 256 != 0)
    return fail(CMF_EINVAL, "src and dst must be 256-byte aligned");
  if (step < 0 || step >= kMaxStep)
    return fail(CMF_EINVAL, "step %lld outside [0, 2^56)", (long long)step);
  if (!valid_launch(block, grid))
    return fail(CMF_EINVAL, "block must be 64, 128, 192 or 256 and grid >= 1, got (%d, %d)", block,
                grid);
  if (grid > kNoAllocMaxGrid)
    return fail(CMF_EINVAL,
                "grid %d exceeds %d: the scratch holds the partial sums of at most %d workgroups",
                grid, kNoAllocMaxGrid, kNoAllocMaxGrid);
  const size_t state_bytes =
      (size_t)desc->q * desc->nx * desc->ny * desc->nz * storage_bytes(desc->storage);
  rc = check_device_span(src, state_bytes, "src");
  if (rc == CMF_OK) rc = check_device_span(dst, state_bytes, "dst");
  if (rc == CMF_OK && stats_dev)
    rc = check_device_span(stats_dev, kSeriesStride * sizeof(double), "stats_dev");
  if (rc != CMF_OK) return rc;
  double *scr = nullptr;
  rc = scratch_address(&scr);
  if (rc != CMF_OK) return rc;
  ModeConstants mc;
  mode_constants(desc, mc);
  StepParams<double> pd;
  StepParams<float> pf;
  const bool f64 = desc->storage == kF64;
  if (f64)
    fill_params(*desc, mc.lambda, mc.amp, mc.scale, block, pd);
  else
    fill_params(*desc, mc.lambda, mc.amp, mc.scale, block, pf);
  const int ntiles = f64 ? pd.ntiles : pf.ntiles;
  const int g = grid < ntiles ? grid : ntiles;
  const bool nt = ((int64_t)desc->nx * storage_bytes(desc->storage)) % kLineBytes == 0;
  const double mass0 = (double)desc->nx * desc->ny * desc->nz * desc->rho0;
  int64_t *step_dev = reinterpret_cast<int64_t *>(scr + kScratchPartials + kScratchLevel2);
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e = launch_set_i64(step_dev, step, s);
  if (e == hipSuccess)
    e = launch_step(desc->q, desc->storage, mc.general, nt, kStreamPull,
                    f64 ? (const void *)&pd : (const void *)&pf,
                    src, dst, step_dev, 0, scr, g, block, s);
  if (e == hipSuccess && stats_dev)
    e = launch_finalize(scr, g, scr + kScratchPartials, stats_dev, 1, step_dev, 0, 0, mass0, true, s);
  if (e != hipSuccess) return fail(CMF_EHIP, "step launch failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

// ===========================================================================
// batched ensembles
// ===========================================================================
struct cmf_ensemble {
  struct Rep {
    cmf_desc desc;
    int64_t N = 0;
    int64_t offset = 0;  // elements
    int64_t pitch = 0;   // elements per population array: N rounded up to 64
    int tile0 = 0, ntiles = 0, spt = 1, tsites = 0;
    ConvParams cp;
  };
  int n = 0;
  int storage = 1;
  uint32_t flags = 0;
  bool general = false;
  bool own_stream = false;
  hipStream_t stream = nullptr;
  std::vector<Rep> reps;
  std::vector<ModeConstants> mcs;
  int spt9 = kEnsembleSpt9, spt3d = kEnsembleSpt27;  // sites per thread of a tile
  int tiles_cap = 0;  // tiles the tile map is allocated for
  size_t parts_cap = 0;  // partial rows allocated: 2 stat_batch per tile needed
  int stat_batch = 1;    // steps per statistics reduction
  void *arena[2] = {nullptr, nullptr};
  size_t arena_bytes = 0;
  int parity = 0;
  void *d_reps = nullptr;
  int32_t *d_tile_rep = nullptr;
  int ntiles = 0;
  int64_t total_sites = 0;
  double *partials = nullptr;
  double *series = nullptr;
  double *d_mass0 = nullptr;
  int cap = 4096;
  int64_t *step_dev = nullptr;
  std::vector<int64_t> read_step;
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  bool graphs_dropped = false;  // a new tile shape dropped captured graphs
  ForkedRun forked;
  FetchUser fetches;
};

namespace {

// multiplier and shifts of the exact division by d >= 1 that
// udiv_invariant applies (Granlund and Montgomery, PLDI 1994, Fig. 4.1):
// l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1, s1 = min(l, 1),
// s2 = max(l - 1, 0)
void invariant_divisor(uint32_t d, uint32_t *m, uint32_t *sh) {
  int l = 0;
  while ((1ull << l) < d) ++l;
  *m = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
  *sh = (uint32_t)(l < 1 ? l : 1) | ((uint32_t)(l > 1 ? l - 1 : 0) << 8);
}

template <typename R>
void fill_replica(const cmf_desc &d, const ModeConstants &mc, const cmf_ensemble::Rep &rp,
                  ReplicaParams<R> &p) {
  memset(&p, 0, sizeof p);
  p.q = d.q;
  p.nx = d.nx;
  p.ny = d.ny;
  p.nz = d.nz;
  p.nsites = (int32_t)rp.N;
  p.tile0 = rp.tile0;
  p.ntiles = rp.ntiles;
  p.spt = rp.spt;
  p.tsites = rp.tsites;
  p.pitch = (int32_t)rp.pitch;
  invariant_divisor((uint32_t)d.nx, &p.div_nx, &p.sh_nx);
  invariant_divisor((uint32_t)d.ny, &p.div_ny, &p.sh_ny);
  p.noise = d.kT > 0.0 ? 1 : 0;
  p.offset = rp.offset;
  p.key0 = (uint32_t)d.seed;
  p.key1 = (uint32_t)(d.seed >> 32);
  p.replica = d.replica;
  p.rho0 = (R)d.rho0;
  for (int v = 0; v < d.q; ++v) {
    p.amp[v] = (R)mc.amp[v];
    p.oml[v] = (R)(1.0 - mc.lambda[v]);
    p.lam[v] = (R)mc.lambda[v];
  }
  p.amp1 = (R)sqrt(d.kT / kCs2);
  class_scales(d.q, d.storage, mc.scale, p.scale, p.iscale);
}

void ens_release(cmf_ensemble *E) {
  if (!E) return;
  if (E->stream) (void)hipStreamSynchronize(E->stream);
  for (int k = 0; k < 2; ++k) {
    if (E->graph[k]) (void)hipGraphExecDestroy(E->graph[k]);
    if (E->arena[k]) (void)hipFree(E->arena[k]);
  }
  if (E->d_reps) (void)hipFree(E->d_reps);
  if (E->d_tile_rep) (void)hipFree(E->d_tile_rep);
  if (E->partials) (void)hipFree(E->partials);
  if (E->series) (void)hipFree(E->series);
  if (E->d_mass0) (void)hipFree(E->d_mass0);
  if (E->step_dev) (void)hipFree(E->step_dev);
  forked_release(E->forked);
  if (E->own_stream && E->stream) (void)hipStreamDestroy(E->stream);
  delete E;
}

double *ens_partials_buf(const cmf_ensemble *E, int b) {
  return E->partials + (size_t)b * kPartStride * E->ntiles;
}

// One direct step (as enqueue_one_step of a lattice).
int ens_enqueue_step(cmf_ensemble *E) {
  HIP_TRY(launch_ensemble_step(E->storage, E->general, E->d_reps, E->d_tile_rep, E->ntiles,
                               E->arena[E->parity], E->arena[1 - E->parity], E->step_dev, 0,
                               ens_partials_buf(E, 0), E->stream));
  HIP_TRY(launch_ensemble_finalize(E->storage, E->d_reps, E->n, ens_partials_buf(E, 0), 0, 1,
                                   E->series, E->cap, E->step_dev, 0, 1, E->d_mass0,
                                   !(E->flags & CMF_FLAG_NO_STATS), E->stream));
  E->parity ^= 1;
  return CMF_OK;
}

struct EnsembleRun {
  cmf_ensemble *E;
  int parity;
  hipError_t operator()(int j, hipStream_t s) const {
    const int b = parity ^ (j & 1);
    return launch_ensemble_step(E->storage, E->general, E->d_reps, E->d_tile_rep,
                                E->ntiles, E->arena[b], E->arena[b ^ 1], E->step_dev, j,
                                ens_partials_buf(E, j % (2 * E->stat_batch)), s);
  }
};
struct EnsembleFin {
  cmf_ensemble *E;
  hipError_t operator()(int j0, int count, int bump, hipStream_t s) const {
    // j0 is a multiple of stat_batch: the batch's slots are consecutive
    return launch_ensemble_finalize(E->storage, E->d_reps, E->n,
                                    ens_partials_buf(E, j0 % (2 * E->stat_batch)),
                                    (int64_t)kPartStride * E->ntiles, count, E->series, E->cap,
                                    E->step_dev, j0, bump, E->d_mass0, true, s);
  }
};

int ens_capture(cmf_ensemble *E, int parity) {
  const bool stats = !(E->flags & CMF_FLAG_NO_STATS);
  return capture_forked(E->stream, E->forked, stats, E->stat_batch, E->step_dev,
                        EnsembleRun{E, parity}, EnsembleFin{E}, &E->graph[parity]);
}

int ens_run_direct(cmf_ensemble *E, int n) {
  const bool stats = !(E->flags & CMF_FLAG_NO_STATS);
  int rc = run_forked(E->stream, E->forked, stats, E->stat_batch, E->step_dev,
                      EnsembleRun{E, E->parity}, EnsembleFin{E}, n);
  if (rc == CMF_OK) E->parity ^= (n & 1);
  return rc;
}

int ens_check_index(cmf_ensemble *E, int32_t index) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (index < 0 || index >= E->n) return fail(CMF_EINVAL, "replica index %d outside [0, %d)", index, E->n);
  return CMF_OK;
}

void *ens_replica_buffer(cmf_ensemble *E, int index) {
  return (char *)E->arena[E->parity] + E->reps[index].offset * storage_bytes(E->storage);
}

// Tile the replicas, 3-D replicas first, then D2Q9, each in creation order:
// a tile of a replica is spt x kEnsembleBlock consecutive sites, spt = spt9
// (D2Q9) or spt3d (D3Q19, D3Q27), the last tile of a replica ragged.  Uploads the tile map and the replica
// records, grows the tile map and the partial-sum buffers when needed and
// drops captured graphs.  The stream must be idle.
int ens_build_tiles(cmf_ensemble *E, int spt9, int spt3d) {
  std::vector<int32_t> tile_rep;
  std::vector<int> tile0(E->n), ntl(E->n), spt(E->n), tsites(E->n);
  for (int pass = 0; pass < 2; ++pass)
    for (int r = 0; r < E->n; ++r) {
      const int q = E->reps[r].desc.q;
      if ((pass == 0) != (q != 9)) continue;
      tile0[r] = (int)tile_rep.size();
      spt[r] = q == 9 ? spt9 : spt3d;
      tsites[r] = spt[r] * kEnsembleBlock;
      const int64_t n = (E->reps[r].N + tsites[r] - 1) / tsites[r];
      if ((int64_t)tile_rep.size() + n >= ((int64_t)1 << 31))
        return fail(CMF_EINVAL, "ensemble has too many tiles");
      ntl[r] = (int)n;
      tile_rep.insert(tile_rep.end(), ntl[r], r);
    }
  const int nt = (int)tile_rep.size();
  // statistics of K steps per reduction, as a lattice, while the partial sums
  // stay within kEnsRingBytes (64 replicas of 64 x 48: 478 -> 365 us
  // per 32 graph-replayed steps, 754 -> 313 per 31 direct ones; the
  // 0.95 ms steps of the 320-replica set hide one reduction per step)
  int K = kStatBatch;
  while (K > 1 && 2 * (size_t)K * sizeof(double) * kPartStride * nt > kEnsRingBytes) K /= 2;
  const size_t rows = 2 * (size_t)K * nt;
  if (nt > E->tiles_cap || rows > E->parts_cap) {
    // allocate first, so that a failure leaves the current tiling usable
    int32_t *map = nullptr;
    double *parts = nullptr;
    if (hipMalloc((void **)&map, sizeof(int32_t) * nt) != hipSuccess ||
        hipMalloc((void **)&parts, sizeof(double) * kPartStride * rows) != hipSuccess) {
      if (map) (void)hipFree(map);
      return fail(CMF_ENOMEM, "allocation of the tile map (%d tiles) failed", nt);
    }
    if (E->d_tile_rep) (void)hipFree(E->d_tile_rep);
    if (E->partials) (void)hipFree(E->partials);
    E->d_tile_rep = map;
    E->partials = parts;
    E->tiles_cap = nt;
    E->parts_cap = rows;
  }
  E->stat_batch = K;
  for (int r = 0; r < E->n; ++r) {
    E->reps[r].tile0 = tile0[r];
    E->reps[r].ntiles = ntl[r];
    E->reps[r].spt = spt[r];
    E->reps[r].tsites = tsites[r];
  }
  E->ntiles = nt;
  E->spt9 = spt9;
  E->spt3d = spt3d;
  hipError_t e = hipMemcpy(E->d_tile_rep, tile_rep.data(), sizeof(int32_t) * nt, hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    if (E->storage == kF64) {
      std::vector<ReplicaParams<double>> h(E->n);
      for (int r = 0; r < E->n; ++r) fill_replica(E->reps[r].desc, E->mcs[r], E->reps[r], h[r]);
      e = hipMemcpy(E->d_reps, h.data(), sizeof(ReplicaParams<double>) * E->n, hipMemcpyHostToDevice);
    } else {
      std::vector<ReplicaParams<float>> h(E->n);
      for (int r = 0; r < E->n; ++r) fill_replica(E->reps[r].desc, E->mcs[r], E->reps[r], h[r]);
      e = hipMemcpy(E->d_reps, h.data(), sizeof(ReplicaParams<float>) * E->n, hipMemcpyHostToDevice);
    }
  }
  drop_graphs(E);
  if (e != hipSuccess) return fail(CMF_EHIP, "tile map upload failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

}  // namespace

extern "C" {

int cmf_ensemble_create(const cmf_desc *descs, int32_t n, void *hip_stream, cmf_ensemble **out) {
  if (!out) return fail(CMF_EINVAL, "out is NULL");
  *out = nullptr;
  if (!descs || n < 1) return fail(CMF_EINVAL, "need at least one descriptor");
  for (int r = 0; r < n; ++r) {
    int rc = validate(&descs[r]);
    if (rc != CMF_OK) return fail(rc, "replica %d: %s", r, g_last_error.c_str());
    if (descs[r].storage != descs[0].storage) return fail(CMF_EINVAL, "replica %d: storage differs from replica 0", r);
    if (descs[r].flags != descs[0].flags) return fail(CMF_EINVAL, "replica %d: flags differ from replica 0", r);
    if (descs[r].flags & CMF_FLAG_IN_PLACE)
      return fail(CMF_EUNSUPPORTED, "replica %d: in-place streaming is for single lattices", r);
    // ensemble tiles address a replica's buffer (q arrays of N rounded up
    // to 64) with 32-bit byte offsets
    const int64_t n_pad = ((int64_t)descs[r].nx * descs[r].ny * descs[r].nz + 63) / 64 * 64;
    const int64_t bytes = (int64_t)descs[r].q * n_pad * storage_bytes(descs[r].storage);
    if (bytes >= ((int64_t)1 << 32))
      return fail(CMF_EINVAL, "replica %d: %lld population bytes; an ensemble member holds below 4 GiB",
                  r, (long long)bytes);
  }
  cmf_ensemble *E = new cmf_ensemble();
  E->n = n;
  E->storage = descs[0].storage;
  E->flags = descs[0].flags;
  E->cap = descs[0].series_capacity > 0 ? descs[0].series_capacity : 4096;
  E->reps.resize(n);
  E->read_step.assign(n, 0);
  E->mcs.resize(n);
  std::vector<ModeConstants> &mcs = E->mcs;
  int64_t offset = 0;
  for (int r = 0; r < n; ++r) {
    cmf_ensemble::Rep &rp = E->reps[r];
    rp.desc = descs[r];
    rp.desc.lambda = nullptr;
    rp.N = (int64_t)descs[r].nx * descs[r].ny * descs[r].nz;
    rp.offset = offset;
    rp.pitch = (rp.N + 63) / 64 * 64;
    offset += (int64_t)descs[r].q * rp.pitch;
    mode_constants(&descs[r], mcs[r]);
    if (mcs[r].general) E->general = true;
    rp.cp.nx = descs[r].nx;
    rp.cp.ny = descs[r].ny;
    rp.cp.nz = descs[r].nz;
    rp.cp.pitch = rp.pitch;
    rp.cp.layout = kLayoutPull;
    rp.cp.rho0 = descs[r].rho0;
    for (int i = 0; i < descs[r].q; ++i) {
      rp.cp.w[i] = mcs[r].w[i];
      rp.cp.scale[i] = mcs[r].scale[i];
      rp.cp.iscale[i] = 1.0f / mcs[r].scale[i];
    }
    E->total_sites += rp.N;
  }
  // sites per thread of the tiles (cmf_ensemble_set_tiles / _autotune;
  // CMF_ENSEMBLE_SPT9 / CMF_ENSEMBLE_SPT27, the latter for both 3-D
  // lattices, override the defaults, 1..16)
  const int spt9 = env_int("CMF_ENSEMBLE_SPT9", kEnsembleSpt9, 1, 16);
  const int spt27 = env_int("CMF_ENSEMBLE_SPT27", kEnsembleSpt27, 1, 16);
  E->arena_bytes = ((size_t)offset * storage_bytes(E->storage) + 255) / 256 * 256;
  hipError_t e = hip_stream ? hipSuccess : hipStreamCreate(&E->stream);
  if (hip_stream) E->stream = (hipStream_t)hip_stream; else E->own_stream = true;
  if (e != hipSuccess) {
    ens_release(E);
    return fail(CMF_EHIP, "hipStreamCreate failed: %s", hipGetErrorString(e));
  }
  const size_t rec = E->storage == kF64 ? sizeof(ReplicaParams<double>) : sizeof(ReplicaParams<float>);
  bool ok = hipMalloc(&E->arena[0], E->arena_bytes) == hipSuccess &&
            hipMalloc(&E->arena[1], E->arena_bytes) == hipSuccess &&
            hipMalloc(&E->d_reps, rec * n) == hipSuccess &&
            hipMalloc((void **)&E->series, sizeof(double) * kSeriesStride * E->cap * n) == hipSuccess &&
            hipMalloc((void **)&E->d_mass0, sizeof(double) * n) == hipSuccess &&
            hipMalloc((void **)&E->step_dev, sizeof(int64_t)) == hipSuccess;
  if (!ok) {
    ens_release(E);
    return fail(CMF_ENOMEM, "ensemble allocation (%zu bytes per arena) failed", E->arena_bytes);
  }
  {
    const int rc = ens_build_tiles(E, spt9, spt27);
    if (rc != CMF_OK) {
      const std::string msg = g_last_error;
      ens_release(E);
      return fail(rc, "%s", msg.c_str());
    }
  }
  std::vector<double> mass0(n);
  for (int r = 0; r < n; ++r) mass0[r] = (double)E->reps[r].N * descs[r].rho0;
  e = hipMemcpy(E->d_mass0, mass0.data(), sizeof(double) * n, hipMemcpyHostToDevice);
  // at rest every deviation is exactly zero
  if (e == hipSuccess) e = hipMemsetAsync(E->arena[0], 0, E->arena_bytes, E->stream);
  if (e == hipSuccess) e = launch_zero_i64(E->step_dev, 1, E->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  if (e != hipSuccess) {
    ens_release(E);
    return fail(CMF_EHIP, "ensemble initialisation failed: %s", hipGetErrorString(e));
  }
  *out = E;
  return CMF_OK;
}

int cmf_ensemble_destroy(cmf_ensemble *E) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  ens_release(E);
  return CMF_OK;
}

int cmf_ensemble_info(cmf_ensemble *E, int32_t *n_replicas, int64_t *total_sites, int64_t *n_tiles) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (n_replicas) *n_replicas = E->n;
  if (total_sites) *total_sites = E->total_sites;
  if (n_tiles) *n_tiles = E->ntiles;
  return CMF_OK;
}

int cmf_ensemble_get_tiles(cmf_ensemble *E, cmf_ensemble_tiles *out) {
  if (!E || !out) return fail(CMF_EINVAL, "NULL argument");
  out->spt9 = E->spt9;
  out->spt3d = E->spt3d;
  out->ms_per_step = 0.0;
  return CMF_OK;
}

int cmf_ensemble_set_tiles(cmf_ensemble *E, int32_t spt9, int32_t spt3d) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (spt9 < 1 || spt9 > 16 || spt3d < 1 || spt3d > 16)
    return fail(CMF_EINVAL, "sites per thread must be in [1, 16], got %d and %d", spt9, spt3d);
  HIP_TRY(hipStreamSynchronize(E->stream));
  return ens_build_tiles(E, spt9, spt3d);
}

int cmf_ensemble_autotune(cmf_ensemble *E, int32_t steps_per_trial, cmf_ensemble_tiles *trials,
                          int32_t cap, int32_t *n_out) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (steps_per_trial < 1) return fail(CMF_EINVAL, "steps_per_trial must be >= 1");
  if (n_out) *n_out = 0;
  HIP_TRY(hipStreamSynchronize(E->stream));
  bool has2d = false, has3d = false;
  for (const auto &rp : E->reps) (rp.desc.q == 9 ? has2d : has3d) = true;
  std::vector<int> c9 = has2d ? std::vector<int>{1, 2, 3, 4, 6, 8} : std::vector<int>{E->spt9};
  std::vector<int> c3 = has3d ? std::vector<int>{1, 2, 3, 4, 6, 8} : std::vector<int>{E->spt3d};
  // snapshot: current arena, step counter, statistics rings
  const size_t series_bytes = sizeof(double) * kSeriesStride * E->cap * E->n;
  void *saved = nullptr, *saved_series = nullptr;
  if (hipMalloc(&saved, E->arena_bytes) != hipSuccess) return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", E->arena_bytes);
  if (hipMalloc(&saved_series, series_bytes) != hipSuccess) {
    (void)hipFree(saved);
    return fail(CMF_ENOMEM, "hipMalloc of the statistics snapshot failed");
  }
  const int parity0 = E->parity, spt9_0 = E->spt9, spt3d_0 = E->spt3d;
  int64_t step0 = 0;
  hipError_t e = hipMemcpyAsync(saved, E->arena[parity0], E->arena_bytes, hipMemcpyDeviceToDevice, E->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(saved_series, E->series, series_bytes, hipMemcpyDeviceToDevice, E->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(&step0, E->step_dev, sizeof(int64_t), hipMemcpyDeviceToHost, E->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  if (e != hipSuccess) {
    (void)hipFree(saved);
    (void)hipFree(saved_series);
    return fail(CMF_EHIP, "ensemble autotune snapshot failed: %s", hipGetErrorString(e));
  }
  std::vector<cmf_ensemble_tiles> done;
  int rc = CMF_OK;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = fail(CMF_EHIP, "hipEventCreate failed");
  for (int a : c9) {
    for (int b : c3) {
      if (rc != CMF_OK) break;
      rc = ens_build_tiles(E, a, b);
      if (rc != CMF_OK) break;
      rc = ens_enqueue_step(E);  // untimed
      hipError_t x = hipSuccess;
      if (rc == CMF_OK) x = hipEventRecord(e0, E->stream);
      for (int k = 0; k < steps_per_trial && rc == CMF_OK && x == hipSuccess; ++k) rc = ens_enqueue_step(E);
      if (rc == CMF_OK && x == hipSuccess) x = hipEventRecord(e1, E->stream);
      if (rc == CMF_OK && x == hipSuccess) x = hipEventSynchronize(e1);
      float ms = 0.0f;
      if (rc == CMF_OK && x == hipSuccess) x = hipEventElapsedTime(&ms, e0, e1);
      if (rc == CMF_OK && x != hipSuccess) rc = fail(CMF_EHIP, "ensemble autotune timing failed: %s", hipGetErrorString(x));
      if (rc == CMF_OK) done.push_back(cmf_ensemble_tiles{a, b, (double)ms / steps_per_trial});
    }
    if (rc != CMF_OK) break;
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  // restore the state exactly
  (void)hipStreamSynchronize(E->stream);
  E->parity = parity0;
  e = hipMemcpyAsync(E->arena[parity0], saved, E->arena_bytes, hipMemcpyDeviceToDevice, E->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(E->series, saved_series, series_bytes, hipMemcpyDeviceToDevice, E->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(E->step_dev, &step0, sizeof(int64_t), hipMemcpyHostToDevice, E->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  (void)hipFree(saved);
  (void)hipFree(saved_series);
  if (rc == CMF_OK && e != hipSuccess) rc = fail(CMF_EHIP, "ensemble autotune restore failed: %s", hipGetErrorString(e));
  if (rc != CMF_OK || done.empty()) {
    const std::string msg = rc != CMF_OK ? g_last_error : std::string("no trial ran");
    (void)ens_build_tiles(E, spt9_0, spt3d_0);
    return fail(rc != CMF_OK ? rc : CMF_EHIP, "%s", msg.c_str());
  }
  size_t best = 0;
  for (size_t k = 1; k < done.size(); ++k)
    if (done[k].ms_per_step < done[best].ms_per_step) best = k;
  rc = ens_build_tiles(E, done[best].spt9, done[best].spt3d);
  if (rc != CMF_OK) return rc;
  if (trials)
    for (size_t k = 0; k < done.size() && (int32_t)k < cap; ++k) trials[k] = done[k];
  if (n_out) *n_out = (int32_t)done.size();
  return CMF_OK;
}

int cmf_ensemble_init_equilibrium(cmf_ensemble *E, int32_t index, const double *rho, const double *u) {
  int rc = ens_check_index(E, index);
  if (rc != CMF_OK) return rc;
  cmf_ensemble::Rep &rp = E->reps[index];
  rc = check_init_fields(rp.N, rho, u);
  if (rc != CMF_OK) return rc;
  HIP_TRY(hipStreamSynchronize(E->stream));
  double *drho = nullptr, *du = nullptr;
  hipError_t e = upload_init_fields(rp.N, rho, u, &drho, &du);
  if (e == hipSuccess)
    e = launch_init_eq(rp.desc.q, E->storage, rp.cp, drho, du, ens_replica_buffer(E, index), E->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  if (drho) (void)hipFree(drho);
  if (du) (void)hipFree(du);
  if (e != hipSuccess) return fail(CMF_EHIP, "ensemble init failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_ensemble_set_populations(cmf_ensemble *E, int32_t index, const double *f) {
  int rc = ens_check_index(E, index);
  if (rc != CMF_OK) return rc;
  if (!f) return fail(CMF_EINVAL, "f is NULL");
  cmf_ensemble::Rep &rp = E->reps[index];
  HIP_TRY(hipStreamSynchronize(E->stream));
  const size_t bytes = sizeof(double) * rp.desc.q * rp.N;
  double *df = nullptr;
  if (hipMalloc((void **)&df, bytes) != hipSuccess) return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  hipError_t e = hipMemcpy(df, f, bytes, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = launch_set_state(rp.desc.q, E->storage, rp.cp, df, ens_replica_buffer(E, index), E->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  (void)hipFree(df);
  if (e != hipSuccess) return fail(CMF_EHIP, "ensemble set_populations failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_ensemble_get_populations(cmf_ensemble *E, int32_t index, double *f) {
  int rc = ens_check_index(E, index);
  if (rc != CMF_OK) return rc;
  if (!f) return fail(CMF_EINVAL, "f is NULL");
  cmf_ensemble::Rep &rp = E->reps[index];
  HIP_TRY(hipStreamSynchronize(E->stream));
  const size_t bytes = sizeof(double) * rp.desc.q * rp.N;
  double *df = nullptr;
  if (hipMalloc((void **)&df, bytes) != hipSuccess) return fail(CMF_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  hipError_t e = launch_get_state(rp.desc.q, E->storage, rp.cp, ens_replica_buffer(E, index), df, E->stream);
  if (e == hipSuccess) e = fetch(E->fetches, f, df, bytes, E->stream);
  (void)hipFree(df);
  if (e != hipSuccess) return fail(CMF_EHIP, "ensemble get_populations failed: %s", hipGetErrorString(e));
  return CMF_OK;
}

int cmf_ensemble_step(cmf_ensemble *E, int64_t nsteps) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (nsteps < 0) return fail(CMF_EINVAL, "nsteps < 0");
  const bool graphs = !(E->flags & CMF_FLAG_NO_GRAPH) && !E->graphs_dropped;
  int64_t left = nsteps;
  while (graphs && left >= kGraphSteps) {
    if (!E->graph[E->parity]) {
      int rc = ens_capture(E, E->parity);
      if (rc != CMF_OK) return rc;
    }
    HIP_TRY(hipGraphLaunch(E->graph[E->parity], E->stream));
    left -= kGraphSteps;
  }
  while (left > 0) {
    const int n = left < kGraphSteps ? (int)left : kGraphSteps;
    int rc = ens_run_direct(E, n);
    if (rc != CMF_OK) return rc;
    left -= n;
  }
  return CMF_OK;
}

int cmf_ensemble_profile_steps(cmf_ensemble *E, int64_t nsteps, double *kernel_ms) {
  if (!E || !kernel_ms) return fail(CMF_EINVAL, "NULL argument");
  if (nsteps < 0) return fail(CMF_EINVAL, "nsteps < 0");
  *kernel_ms = 0.0;
  std::vector<hipEvent_t> ev(2 * nsteps, nullptr);
  const int rc = create_events(ev);
  if (rc != CMF_OK) return rc;
  hipError_t e = hipSuccess;
  for (int64_t s = 0; s < nsteps && e == hipSuccess; ++s) {
    e = hipEventRecord(ev[2 * s], E->stream);
    if (e == hipSuccess)
      e = launch_ensemble_step(E->storage, E->general, E->d_reps, E->d_tile_rep, E->ntiles,
                               E->arena[E->parity], E->arena[1 - E->parity], E->step_dev, 0,
                               ens_partials_buf(E, 0), E->stream);
    if (e == hipSuccess) e = hipEventRecord(ev[2 * s + 1], E->stream);
    if (e == hipSuccess)
      e = launch_ensemble_finalize(E->storage, E->d_reps, E->n, ens_partials_buf(E, 0), 0, 1,
                                   E->series, E->cap, E->step_dev, 0, 1, E->d_mass0,
                                   !(E->flags & CMF_FLAG_NO_STATS), E->stream);
    E->parity ^= 1;
  }
  if (e == hipSuccess) e = hipStreamSynchronize(E->stream);
  double total = 0.0;
  for (int64_t s = 0; s < nsteps && e == hipSuccess; ++s) {
    float ms = 0.0f;
    e = hipEventElapsedTime(&ms, ev[2 * s], ev[2 * s + 1]);
    total += ms;
  }
  for (auto &x : ev) (void)hipEventDestroy(x);
  if (e != hipSuccess) return fail(CMF_EHIP, "ensemble profiling failed: %s", hipGetErrorString(e));
  *kernel_ms = total;
  return CMF_OK;
}

int cmf_ensemble_synchronize(cmf_ensemble *E) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  HIP_TRY(hipStreamSynchronize(E->stream));
  return CMF_OK;
}

int cmf_ensemble_get_step(cmf_ensemble *E, int64_t *step) {
  if (!E || !step) return fail(CMF_EINVAL, "NULL argument");
  HIP_TRY(hipStreamSynchronize(E->stream));
  HIP_TRY(hipMemcpy(step, E->step_dev, sizeof(int64_t), hipMemcpyDeviceToHost));
  return CMF_OK;
}

int cmf_ensemble_set_step(cmf_ensemble *E, int64_t step) {
  if (!E) return fail(CMF_EINVAL, "ensemble is NULL");
  if (step < 0 || step >= kMaxStep)
    return fail(CMF_EINVAL, "step %lld outside [0, 2^56)", (long long)step);
  HIP_TRY(hipStreamSynchronize(E->stream));
  HIP_TRY(hipMemcpy(E->step_dev, &step, sizeof(int64_t), hipMemcpyHostToDevice));
  for (auto &r : E->read_step) r = step;
  return CMF_OK;
}

int cmf_ensemble_stats(cmf_ensemble *E, int32_t index, cmf_moments *out, int64_t cap, int64_t *n_out) {
  int rc = ens_check_index(E, index);
  if (rc != CMF_OK) return rc;
  if (!n_out || (cap > 0 && !out)) return fail(CMF_EINVAL, "NULL argument");
  if (cap < 0) return fail(CMF_EINVAL, "cap < 0");
  *n_out = 0;
  int64_t step = 0;
  rc = cmf_ensemble_get_step(E, &step);
  if (rc != CMF_OK) return rc;
  if (E->flags & CMF_FLAG_NO_STATS) {
    E->read_step[index] = step;
    return CMF_OK;
  }
  int64_t first = E->read_step[index];
  if (step - first > E->cap) first = step - E->cap;
  if (step - first > cap) first = step - cap;
  std::vector<double> rows;
  HIP_TRY(copy_series(E->series + (size_t)index * E->cap * kSeriesStride, E->cap, first, step, rows));
  bool bad = false;
  for (int64_t s = first; s < step; ++s) {
    const double *r = rows.data() + (s - first) * kSeriesStride;
    cmf_moments &m = out[s - first];
    m.step = r[0];
    m.sum_rho = r[1];
    for (int a = 0; a < 3; ++a) {
      m.sum_j[a] = r[2 + a];
      m.sum_u[a] = r[5 + a];
      m.sum_u2[a] = r[8 + a];
    }
    m.nonfinite = r[11];
    if (m.nonfinite != 0.0) bad = true;
  }
  *n_out = step - first;
  E->read_step[index] = step;
  if (bad) return fail(CMF_ENONFINITE, "non-finite density or velocity in a recorded step");
  return CMF_OK;
}

}  // extern "C"
