// cmflb_kernels.hip -- gfx950 kernels of libcmflb besides the fused steps
// (cmflb_step.h, cmflb_ensemble.hip): the statistics reductions, the state
// conversion and diagnostic kernels and their launchers.
#include "cmflb_step.h"
#include "cmflb_sums.h"

namespace cmf {

// ---------------------------------------------------------------------------
// statistics finalize: fixed-order FP64 sums of the block partials (in two
// levels when there are many blocks) into the series row of the current
// step, then advance the step counter
// ---------------------------------------------------------------------------
// first level: block (r, y) sums partial rows [r chunk, (r + 1) chunk) of
// step y of a batch (its rows from partials + y pstride) into level-2 row
// y gridDim.x + r
__global__ __launch_bounds__(256) void k_reduce_partials(
    const double *__restrict__ partials, int nparts, int chunk, int64_t pstride,
    double *__restrict__ level2) {
  const int lo = blockIdx.x * chunk;
  const int hi = lo + chunk < nparts ? lo + chunk : nparts;
  block_sum_rows(partials + blockIdx.y * pstride, lo, hi,
                 level2 + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kPartStride);
}

// The statistics row of step *step_ptr + step_off + y for block y of a
// batch (its nrows rows from rows + y rstride); *step_ptr advances by `bump`
// (0 inside a run of steps, which advances it once at its end; a batch of
// more than one step passes 0).
__global__ __launch_bounds__(256) void k_finalize(
    const double *__restrict__ rows, int nrows, int64_t rstride, double *__restrict__ series,
    int cap, int64_t *__restrict__ step_ptr, int step_off, int bump, double mass0,
    int stats) {
  __shared__ double tot[kNAcc];
  const int64_t base = *step_ptr;
  const int64_t step = base + step_off + blockIdx.x;
  // with a ring shorter than the batch, a later step of the same batch
  // takes the same row: only the latest of them writes it, as if the steps
  // had been reduced one after the other
  if (stats && blockIdx.x + (int64_t)cap >= gridDim.x) {
    block_sum_rows(rows + blockIdx.x * rstride, 0, nrows, tot);
    __syncthreads();
    if (threadIdx.x == 0) {
      double *row = series + (step % cap) * kSeriesStride;
      row[0] = (double)step;
      row[1] = mass0 + tot[0];
#pragma unroll
      for (int k = 1; k < kNAcc; ++k) row[1 + k] = tot[k];
    }
  }
  if (threadIdx.x == 0 && bump) *step_ptr = base + bump;
}

// ---------------------------------------------------------------------------
// state conversion kernels (FP64 arithmetic)
// ---------------------------------------------------------------------------
// Where the buffer holds the pre-collision populations of one site, for the
// buffer's layout (cp.layout, see Layout) and order (row-interleaved, or one
// array per population when cp.pitch > 0): the columns x - c_x and the first
// elements of the row blocks (y - c_y, z - c_z) that it pulls from, index
// c + 1, all of them the site's own in the natural layout.  Sites are below
// 2^31, so the site index takes two 32-bit divisions, once per site.  With
// 64-bit divisions per population the arithmetic, not the bytes, bounded
// every kernel that reads a state (D3Q27 128^3 FP32: velocity PDFs 1118 ->
// 318 us, one structure-factor sample 459 -> 200 us).
template <class L>
struct SiteAddr {
  uint32_t xs[3];
  int64_t rows[3][3];
  int64_t unit;  // elements from one population of a row block to the next
  bool swapped;
  __device__ __forceinline__ SiteAddr(const ConvParams &cp, uint32_t s) {
    const uint32_t nx = (uint32_t)cp.nx, ny = (uint32_t)cp.ny;
    const uint32_t row = s / nx;
    const int x = (int)(s - row * nx);
    const int z = L::D == 3 ? (int)(row / ny) : 0;
    const int y = (int)(row - (uint32_t)z * ny);
    swapped = cp.layout == kLayoutSwapped;
    const int d = cp.layout == kLayoutNatural ? 0 : 1;
    const int64_t block = cp.pitch > 0 ? (int64_t)cp.nx : (int64_t)cp.nx * L::Q;
    unit = cp.pitch > 0 ? cp.pitch : (int64_t)cp.nx;
#pragma unroll
    for (int a = 0; a < 3; ++a) xs[a] = (uint32_t)wrap_sub(x, d * (a - 1), cp.nx);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const int zz = L::D == 3 ? wrap_sub(z, d * (b - 1), cp.nz) : 0;
#pragma unroll
      for (int a = 0; a < 3; ++a)
        rows[a][b] = ((int64_t)wrap_sub(y, d * (a - 1), cp.ny) + (int64_t)cp.ny * zz) * block;
    }
  }
  // element offset of population i
  __device__ __forceinline__ int64_t operator()(const ConvParams &cp, int i) const {
    const int own = cp.pitch > 0 ? i : pop_slot<L>(i);
    const int opp = cp.pitch > 0 ? opposite<L>(i) : pop_slot<L>(opposite<L>(i));
    return rows[L::cy[i] + 1][L::cz[i] + 1] + (swapped ? opp : own) * unit + xs[L::cx[i] + 1];
  }
};

// d_eq = f_eq(rho, u) - w rho0 = T(u)^-1 (rho e_0 - rho0 G(u)), evaluated at
// site s and written to the buffer slot that the next pull reads from.
template <class L, typename S>
__global__ __launch_bounds__(256) void k_init_eq(const ConvParams cp,
                                                 const double *__restrict__ rho,
                                                 const double *__restrict__ u,
                                                 S *__restrict__ buf) {
  using ST = Store<S, double>;
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  const SiteAddr<L> at(cp, (uint32_t)s);
  const double r = rho ? rho[s] : cp.rho0;
  const double ux = u ? u[s] : 0.0, uy = u ? u[N + s] : 0.0,
               uz = u ? u[2 * N + s] : 0.0;
  double t[L::NT];
#pragma unroll
  for (int k = 0; k < L::NT; ++k) t[k] = 0.0;
  t[0] = r;
  if constexpr (L::Q == 19) {
    double dd[19];
    d3q19::shift_inverse(t, ux, uy, uz);
    t[0] = r - cp.rho0;
    d3q19::populations(t, dd);
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
      ST::store(buf + at(cp, i), dd[i],
                cp.iscale[i]);
  } else {
    add_rest_moments<L::D, double>(t, -cp.rho0, ux, uy, uz);
    const Axis<double> ax(ux), ay(uy), az(uz);
    tensor_inv<L::D, double>(t, ax, ay, az);
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
      ST::store(buf + at(cp, i),
                t[pop_pos<L>(i)], cp.iscale[i]);
  }
}

template <class L, typename S>
__global__ __launch_bounds__(256) void k_set_state(const ConvParams cp,
                                                   const double *__restrict__ f,
                                                   S *__restrict__ buf) {
  using ST = Store<S, double>;
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  const SiteAddr<L> at(cp, (uint32_t)s);
#pragma unroll
  for (int i = 0; i < L::Q; ++i)
    ST::store(buf + at(cp, i),
              f[(int64_t)i * N + s] - cp.w[i] * cp.rho0, cp.iscale[i]);
}

template <class L, typename S>
__global__ __launch_bounds__(256) void k_get_state(const ConvParams cp,
                                                   const S *__restrict__ buf,
                                                   double *__restrict__ f) {
  using ST = Store<S, double>;
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  const SiteAddr<L> at(cp, (uint32_t)s);
#pragma unroll
  for (int i = 0; i < L::Q; ++i)
    f[(int64_t)i * N + s] =
        cp.w[i] * cp.rho0 +
        ST::load(buf + at(cp, i),
                 cp.scale[i]);
}

template <class L, typename S>
__global__ __launch_bounds__(256) void k_gather(const ConvParams cp,
                                                const S *__restrict__ buf,
                                                const int64_t *__restrict__ sites,
                                                int64_t n,
                                                double *__restrict__ out) {
  using ST = Store<S, double>;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const SiteAddr<L> at(cp, (uint32_t)sites[k]);
#pragma unroll
  for (int i = 0; i < L::Q; ++i)
    out[k * L::Q + i] =
        cp.w[i] * cp.rho0 +
        ST::load(buf + at(cp, i),
                 cp.scale[i]);
}

// drho and rho u of the pre-collision state at site s, FP64
template <class L, typename S>
__device__ __forceinline__ void site_moments(const ConvParams &cp, const S *__restrict__ buf,
                                             uint32_t s, double &drho, double *j) {
  using ST = Store<S, double>;
  const SiteAddr<L> at(cp, s);
  drho = j[0] = j[1] = j[2] = 0.0;
#pragma unroll
  for (int i = 0; i < L::Q; ++i) {
    const double d = ST::load(buf + at(cp, i), cp.scale[i]);
    drho += d;
    j[0] += L::cx[i] * d;
    j[1] += L::cy[i] * d;
    j[2] += L::cz[i] * d;
  }
}

template <class L, typename S, typename T>
__global__ __launch_bounds__(256) void k_macro(const ConvParams cp,
                                               const S *__restrict__ buf,
                                               T *__restrict__ rho_out,
                                               T *__restrict__ u_out) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  double drho, j[3];
  site_moments<L, S>(cp, buf, (uint32_t)s, drho, j);
  const double rho = cp.rho0 + drho;
  if (rho_out) rho_out[s] = (T)rho;
  if (u_out) {
    u_out[s] = (T)(j[0] / rho);
    u_out[N + s] = (T)(j[1] / rho);
    u_out[2 * N + s] = (T)(j[2] / rho);
  }
}

template <class L, typename R>
__global__ __launch_bounds__(256) void k_noise(uint32_t key0, uint32_t key1,
                                               uint32_t replica, uint64_t step,
                                               int64_t site0, int64_t n,
                                               double *__restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  R eta[L::NNOISE];
  site_normals<L, R>((uint32_t)(site0 + k), step, replica, key0, key1, eta);
  for (int v = 0; v < L::Q; ++v)
    out[k * L::Q + v] =
        v < L::FIRST_NOISY ? 0.0 : (double)eta[v - L::FIRST_NOISY];
}

__global__ __launch_bounds__(256) void k_philox(const uint32_t *__restrict__ ctr,
                                                int64_t n, uint32_t key0,
                                                uint32_t key1,
                                                uint32_t *__restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const U4 w = philox4x32_10(ctr[4 * k], ctr[4 * k + 1], ctr[4 * k + 2],
                             ctr[4 * k + 3], key0, key1);
  out[4 * k] = w.x;
  out[4 * k + 1] = w.y;
  out[4 * k + 2] = w.z;
  out[4 * k + 3] = w.w;
}

// plain streaming copy of n16 16-byte elements (the HBM calibration kernel)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void cmf_stream_copy_kernel(
    const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n16; k += stride)
    __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

__global__ void k_zero_i64(int64_t *p, int64_t n) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = 0;
}

__global__ void k_set_i64(int64_t *p, int64_t v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// ---------------------------------------------------------------------------
// structure factor (amortized diagnostic): fields, |FFT|^2 accumulation and
// deterministic shell binning
// ---------------------------------------------------------------------------
// drho = rho - rho0, u_x, u_y, u_z of the pre-collision state as 4 FP32
// planes of N values (FP64 arithmetic, rounded once).
template <class L, typename S>
__global__ __launch_bounds__(256) void k_macro_dev(const ConvParams cp,
                                                   const S *__restrict__ buf,
                                                   float *__restrict__ out) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  double drho, j[3];
  site_moments<L, S>(cp, buf, (uint32_t)s, drho, j);
  const double rho = cp.rho0 + drho;
  out[s] = (float)drho;
  out[N + s] = (float)(j[0] / rho);
  out[2 * N + s] = (float)(j[1] / rho);
  out[3 * N + s] = (float)(j[2] / rho);
}

// acc[f][m] += |F_f(m)|^2 / N for the 4 transformed fields (M modes each)
__global__ __launch_bounds__(256) void k_sk_accumulate(
    const float2 *__restrict__ F, int64_t M, double inv_n,
    double *__restrict__ acc) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= 4 * M) return;
  const float2 c = F[m];
  acc[m] += ((double)c.x * c.x + (double)c.y * c.y) * inv_n;
}

// shell of half-spectrum mode m (nxh = nx/2 + 1 modes along x), with the
// Hermitian weight of the modes the real transform does not store
struct ShellGeom {
  int nx, ny, nz, nxh, nbins;
  double kmax;
};

__device__ __forceinline__ int shell_of(const ShellGeom &g, int64_t m,
                                        double *weight, double *kmag) {
  // modes are fewer than sites, below 2^31
  const uint32_t um = (uint32_t)m, r = um / (uint32_t)g.nxh;
  const int kx = (int)(um - r * (uint32_t)g.nxh);
  const int kz0 = (int)(r / (uint32_t)g.ny), ky0 = (int)(r - (uint32_t)kz0 * (uint32_t)g.ny);
  const int ky = ky0 <= g.ny / 2 ? ky0 : ky0 - g.ny;
  const int kz = kz0 <= g.nz / 2 ? kz0 : kz0 - g.nz;
  const double two_pi = 6.283185307179586;
  const double ax = two_pi * kx / g.nx, ay = two_pi * ky / g.ny,
               az = two_pi * kz / g.nz;
  const double k = sqrt(ax * ax + ay * ay + az * az);
  *kmag = k;
  const bool self = kx == 0 || (g.nx % 2 == 0 && kx == g.nx / 2);
  *weight = self ? 1.0 : 2.0;
  if (kx == 0 && ky == 0 && kz == 0) return -1;  // k = 0 excluded
  int b = (int)(k / g.kmax * g.nbins);
  return b < g.nbins ? b : g.nbins - 1;
}

// The modes of every shell, in ascending order (k = 0 belongs to none): a
// counting sort in chunks of `chunk` modes, one wave each.  First the counts
// of every chunk,
__global__ __launch_bounds__(64) void k_sk_count(const ShellGeom g, int64_t M, int64_t chunk,
                                                 int32_t *__restrict__ counts) {
  extern __shared__ int32_t cnt[];
  for (int b = threadIdx.x; b < g.nbins; b += 64) cnt[b] = 0;
  __syncthreads();
  const int64_t lo = blockIdx.x * chunk, hi = lo + chunk < M ? lo + chunk : M;
  for (int64_t m = lo + threadIdx.x; m < hi; m += 64) {
    double w, k;
    const int b = shell_of(g, m, &w, &k);
    if (b >= 0) atomicAdd(&cnt[b], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < g.nbins; b += 64) counts[(int64_t)blockIdx.x * g.nbins + b] = cnt[b];
}

// then the start of every shell (off, nbins + 1 entries) and, in place of the
// counts, of every chunk's part of it (one workgroup of 1024 >= nbins threads),
__global__ __launch_bounds__(1024) void k_sk_starts(int32_t *__restrict__ counts, int nchunks,
                                                    int nbins, int64_t *__restrict__ off) {
  __shared__ int64_t sum[1024];
  const int b = threadIdx.x;
  int64_t total = 0;
  if (b < nbins)
    for (int c = 0; c < nchunks; ++c) total += counts[(int64_t)c * nbins + b];
  sum[b] = total;
  __syncthreads();
  for (int h = 1; h < 1024; h *= 2) {
    const int64_t below = b >= h ? sum[b - h] : 0;
    __syncthreads();
    sum[b] += below;
    __syncthreads();
  }
  if (b >= nbins) return;
  off[b + 1] = sum[b];
  if (b == 0) off[0] = 0;
  int64_t at = sum[b] - total;  // modes are fewer than 2^31
  for (int c = 0; c < nchunks; ++c) {
    const int32_t n = counts[(int64_t)c * nbins + b];
    counts[(int64_t)c * nbins + b] = (int32_t)at;
    at += n;
  }
}

// then the modes: 64 at a time, each after the lanes below it with its shell
__global__ __launch_bounds__(64) void k_sk_scatter(const ShellGeom g, int64_t M, int64_t chunk,
                                                   const int32_t *__restrict__ starts,
                                                   int32_t *__restrict__ perm) {
  extern __shared__ int32_t cnt[];
  for (int b = threadIdx.x; b < g.nbins; b += 64) cnt[b] = starts[(int64_t)blockIdx.x * g.nbins + b];
  __syncthreads();
  const int64_t lo = blockIdx.x * chunk, hi = lo + chunk < M ? lo + chunk : M;
  const int lane = threadIdx.x;
  for (int64_t m0 = lo; m0 < hi; m0 += 64) {
    const int64_t m = m0 + lane;
    double w, k;
    const int b = m < hi ? shell_of(g, m, &w, &k) : -1;
    uint64_t left = __ballot(b >= 0);
    while (left) {  // one shell per turn, that of the lowest lane left
      const int shell = __shfl(b, __ffsll((unsigned long long)left) - 1);
      const uint64_t same = __ballot(b == shell);
      const int base = cnt[shell];
      if (b == shell) perm[base + __popcll(same & (((uint64_t)1 << lane) - 1))] = (int32_t)m;
      if (lane == 0) cnt[shell] = base + __popcll(same);
      __syncthreads();
      left &= ~same;
    }
  }
}

// Shell sums in a fixed order: workgroup (b, p) sums part p of the modes of
// shell b (listed contiguously in `perm`, shell b in [off[b], off[b + 1])),
// out[b kSkParts + p] = (sum w k, sum w, sum w S_rho, sum w S_ux, sum w S_uy,
// sum w S_uz); k_sk_total adds the parts.  One workgroup per shell left the
// chip to the few that hold most modes (48 shells, whole call: D3Q27 128^3 216
// -> 64 us, 256^3 1880 -> 178).
constexpr int kSkCols = 6;
__global__ __launch_bounds__(256) void k_sk_segments(const double *__restrict__ acc,
                                                     int64_t M, const ShellGeom g,
                                                     const int32_t *__restrict__ perm,
                                                     const int64_t *__restrict__ off,
                                                     double *__restrict__ out) {
  const int b = blockIdx.x;
  const int64_t lo = off[b], n = off[b + 1] - lo;
  const int64_t j1 = lo + n * (blockIdx.y + 1) / kSkParts;
  double s[kSkCols] = {0, 0, 0, 0, 0, 0};
  for (int64_t j = lo + n * blockIdx.y / kSkParts + threadIdx.x; j < j1; j += blockDim.x) {
    const int64_t m = perm[j];
    double w, k;
    shell_of(g, m, &w, &k);
    s[0] += w * k;
    s[1] += w;
#pragma unroll
    for (int f = 0; f < 4; ++f) s[2 + f] += w * acc[f * M + m];
  }
  __shared__ double sh[256][kSkCols];
#pragma unroll
  for (int c = 0; c < kSkCols; ++c) sh[threadIdx.x][c] = s[c];
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h)
#pragma unroll
      for (int c = 0; c < kSkCols; ++c) sh[threadIdx.x][c] += sh[threadIdx.x + h][c];
    __syncthreads();
  }
  if (threadIdx.x < kSkCols)
    out[((int64_t)b * kSkParts + blockIdx.y) * kSkCols + threadIdx.x] = sh[0][threadIdx.x];
}

__global__ __launch_bounds__(256) void k_sk_total(const double *__restrict__ parts, int n,
                                                  double *__restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double *p = parts + (int64_t)(i / kSkCols) * kSkParts * kSkCols + i % kSkCols;
  double s = p[0];
  for (int j = 1; j < kSkParts; ++j) s += p[j * kSkCols];
  out[i] = s;
}

// ---------------------------------------------------------------------------
// velocity statistics of the pre-collision state (Test 7, Fig. 8): moments
// about the mean and normalised histograms, FP64 per site
// ---------------------------------------------------------------------------
// Three passes, each needing the result of the one before (VelState, on the
// device, so that the host waits once): the means, the central moments, the
// histogram.  The first reads the populations, which bound it, and leaves the
// velocities in `keep` when the caller has room for them (dims N doubles, a
// quarter of the bytes of a D3Q27 FP32 state); the others read those, or the
// populations again.  D3Q27 FP32 with 40 bins: 128^3 318 us with three passes
// over the populations and the host between them, 128 now (45 + 11 + 29 us in
// the passes; reading the state once takes 38); 256^3 711 us (433 + 89 + 29).
template <class L, typename S>
struct PopVelocity {
  ConvParams cp;
  const S *buf;
  __device__ __forceinline__ void operator()(int64_t s, double *u) const {
    double drho, j[3];
    site_moments<L, S>(cp, buf, (uint32_t)s, drho, j);
    const double rho = cp.rho0 + drho;
    u[0] = j[0] / rho;
    u[1] = j[1] / rho;
    u[2] = j[2] / rho;
  }
};

template <int DIMS>
struct KeptVelocity {
  const double *u;
  int64_t n;
  __device__ __forceinline__ void operator()(int64_t s, double *v) const {
    v[2] = 0.0;
#pragma unroll
    for (int a = 0; a < DIMS; ++a) v[a] = u[a * n + s];
  }
};

// fixed-order sum of COLS values per thread over the workgroup into out
template <int COLS>
__device__ __forceinline__ void block_sum_cols(const double *acc, double *out) {
  __shared__ double sh[256][COLS];
#pragma unroll
  for (int k = 0; k < COLS; ++k) sh[threadIdx.x][k] = acc[k];
  __syncthreads();
  for (int h = 128; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h)
#pragma unroll
      for (int k = 0; k < COLS; ++k) sh[threadIdx.x][k] += sh[threadIdx.x + h][k];
    __syncthreads();
  }
  if (threadIdx.x < COLS) out[threadIdx.x] = sh[0][threadIdx.x];
}

// per-block sums of u_a, each block over a fixed set of sites in a fixed order
template <class SRC>
__global__ __launch_bounds__(256) void k_vel_sums(const SRC src, int64_t N, int dims,
                                                  double *__restrict__ keep,
                                                  double *__restrict__ partials) {
  double acc[3] = {0.0, 0.0, 0.0};
  for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256) {
    double u[3];
    src(s, u);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      acc[a] += u[a];
      if (keep && a < dims) keep[a * N + s] = u[a];
    }
  }
  block_sum_cols<3>(acc, partials + (int64_t)blockIdx.x * kVelCols);
}

// per-block sums of (u_a - c_a)^p, p = 1..4, a = x, y, z (column 4 a + p - 1)
template <class SRC>
__global__ __launch_bounds__(256) void k_vel_moments(const SRC src, int64_t N,
                                                     const VelState *__restrict__ st,
                                                     double *__restrict__ partials) {
  double acc[kVelCols], c[3];
#pragma unroll
  for (int k = 0; k < kVelCols; ++k) acc[k] = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) c[a] = st->centre[a];
  for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256) {
    double u[3];
    src(s, u);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double v = u[a] - c[a], v2 = v * v;
      acc[4 * a] += v;
      acc[4 * a + 1] += v2;
      acc[4 * a + 2] += v2 * v;
      acc[4 * a + 3] += v2 * v2;
    }
  }
  block_sum_cols<kVelCols>(acc, partials + (int64_t)blockIdx.x * kVelCols);
}

// One workgroup: fixed-order sum of the COLS columns of the block rows, then
// the means (COLS = 3; the counts are cleared for the histogram) or the
// central moments about them.
template <int COLS>
__global__ __launch_bounds__(256) void k_vel_final(const double *__restrict__ partials, int nparts,
                                                   double n, VelState *__restrict__ st,
                                                   unsigned long long *__restrict__ counts,
                                                   int ncounts) {
  __shared__ double h[COLS];
  double acc[COLS];
#pragma unroll
  for (int k = 0; k < COLS; ++k) acc[k] = 0.0;
  for (int b = threadIdx.x; b < nparts; b += 256)
#pragma unroll
    for (int k = 0; k < COLS; ++k) acc[k] += partials[(int64_t)b * kVelCols + k];
  block_sum_cols<COLS>(acc, h);
  for (int k = threadIdx.x; k < ncounts; k += 256) counts[k] = 0ull;
  __syncthreads();
  if (threadIdx.x >= 3) return;
  const int a = threadIdx.x;
  if constexpr (COLS == 3) {
    st->centre[a] = h[a] / n;
  } else {
    // central moments about the FP64 mean; the residual first moment
    // d = sum (u - mean) / N corrects them to the exact mean
    const double d = h[4 * a] / n, s2 = h[4 * a + 1] / n, s3 = h[4 * a + 2] / n,
                 s4 = h[4 * a + 3] / n;
    const double var = s2 - d * d;
    const double m3 = s3 - 3.0 * d * s2 + 2.0 * d * d * d;
    const double m4 = s4 - 4.0 * d * s3 + 6.0 * d * d * s2 - 3.0 * d * d * d * d;
    const double mean = st->centre[a] + d;
    st->centre[a] = mean;
    st->inv_sigma[a] = var > 0.0 ? 1.0 / sqrt(var) : 0.0;
    st->moments[4 * a] = mean;
    st->moments[4 * a + 1] = var;
    st->moments[4 * a + 2] = var > 0.0 ? m3 / (var * sqrt(var)) : 0.0;
    st->moments[4 * a + 3] = var > 0.0 ? m4 / (var * var) : 0.0;
  }
}

// histogram of x = (u_a - centre_a) / sigma_a: bin 0 counts x < -xmax (and
// non-finite x), bins 1..nbins split [-xmax, xmax) evenly, bin nbins + 1
// counts x >= xmax; LDS counters per block, in `copies` sets that
// neighbouring lanes use in turn (most sites of a Gaussian fall into a few
// bins), integer totals (order-free)
template <class SRC>
__global__ __launch_bounds__(256) void k_vel_hist(const SRC src, int64_t N,
                                                  const VelState *__restrict__ st, int dims,
                                                  int nbins, double xmax, int copies,
                                                  unsigned long long *__restrict__ counts) {
  extern __shared__ uint32_t hist[];
  const int nb2 = nbins + 2;
  for (int k = threadIdx.x; k < copies * 3 * nb2; k += 256) hist[k] = 0u;
  __syncthreads();
  uint32_t *own = hist + (threadIdx.x % copies) * 3 * nb2;
  double c[3], inv[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c[a] = st->centre[a];
    inv[a] = st->inv_sigma[a];
  }
  const double width = 2.0 * xmax / nbins;
  for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < N; s += (int64_t)gridDim.x * 256) {
    double u[3];
    src(s, u);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (a >= dims) continue;
      const double x = (u[a] - c[a]) * inv[a];
      int b;
      if (!(x >= -xmax)) {
        b = 0;
      } else if (x >= xmax) {
        b = nbins + 1;
      } else {
        b = 1 + (int)floor((x + xmax) / width);
        b = b > nbins ? nbins : b;
      }
      atomicAdd(&own[a * nb2 + b], 1u);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < 3 * nb2; k += 256) {
    unsigned long long t = 0;
    for (int j = 0; j < copies; ++j) t += hist[j * 3 * nb2 + k];
    if (t) atomicAdd(&counts[k], t);
  }
}

__global__ void k_bump_step(int64_t *step_ptr, int64_t by) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *step_ptr = *step_ptr + by;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_step(int q, int storage, bool general, bool nt, int mode,
                       const void *params, const void *src, void *dst,
                       const int64_t *step_ptr, int step_off, double *partials,
                       int grid, int block, hipStream_t stream) {
  if (mode == kStreamPull)
    return launch_step_pull(q, storage, general, nt, params, src, dst, step_ptr, step_off,
                            partials, grid, block, stream);
  if (mode == kStreamAAEven || mode == kStreamAAOdd)
    return launch_step_in_place(q, storage, general, nt, mode == kStreamAAOdd, params, dst,
                                step_ptr, step_off, partials, grid, block, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_finalize(const double *partials, int nparts, double *level2,
                           double *series, int cap, int64_t *step_ptr, int step_off,
                           int bump, double mass0, bool stats, hipStream_t stream) {
  return launch_finalize_batch(partials, 0, 1, nparts, level2, series, cap, step_ptr, step_off,
                               bump, mass0, stats, stream);
}

hipError_t launch_finalize_batch(const double *partials, int64_t pstride, int count, int nparts,
                                 double *level2, double *series, int cap, int64_t *step_ptr,
                                 int step_off, int bump, double mass0, bool stats,
                                 hipStream_t stream) {
  if (count < 1 || (count > 1 && bump != 0)) return hipErrorInvalidValue;
  const double *rows = partials;
  int nrows = nparts;
  int64_t rstride = pstride;
  if (stats && nparts > kSingleLevelRows) {
    int nb = (nparts + kLevel2Threshold - 1) / kLevel2Threshold;
    if (nb > kMaxLevel2) nb = kMaxLevel2;
    const int chunk = (nparts + nb - 1) / nb;
    nb = (nparts + chunk - 1) / chunk;
    hipLaunchKernelGGL(k_reduce_partials, dim3(nb, count), dim3(256), 0, stream, partials,
                       nparts, chunk, pstride, level2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    rows = level2;
    nrows = nb;
    rstride = (int64_t)nb * kPartStride;
  }
  hipLaunchKernelGGL(k_finalize, dim3(count), dim3(256), 0, stream, rows, nrows, rstride,
                     series, cap, step_ptr, step_off, bump, mass0, stats ? 1 : 0);
  return hipGetLastError();
}

template <class T>
struct Tag {
  using type = T;
};

// call f(Tag<Lattice>, Tag<StorageType>) for a runtime (q, storage)
template <class F>
hipError_t with_lattice_storage(int q, int storage, F &&f) {
  auto by_storage = [&](auto lt) -> hipError_t {
    switch (storage) {
      case kF64: return f(lt, Tag<double>{});
      case kF32: return f(lt, Tag<float>{});
      case kF16: return f(lt, Tag<__half>{});
      case kBF16: return f(lt, Tag<__hip_bfloat16>{});
    }
    return hipErrorInvalidValue;
  };
  if (q == 9) return by_storage(Tag<D2Q9>{});
  if (q == 19) return by_storage(Tag<D3Q19>{});
  if (q == 27) return by_storage(Tag<D3Q27>{});
  return hipErrorInvalidValue;
}

hipError_t launch_init_eq(int q, int storage, const ConvParams &cp,
                          const double *rho, const double *u, void *buf,
                          hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_init_eq<L, S>), dim3(blocks_for(N, 256)), dim3(256),
                       0, stream, cp, rho, u, static_cast<S *>(buf));
    return hipGetLastError();
  });
}

hipError_t launch_set_state(int q, int storage, const ConvParams &cp,
                            const double *f, void *buf, hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_set_state<L, S>), dim3(blocks_for(N, 256)),
                       dim3(256), 0, stream, cp, f, static_cast<S *>(buf));
    return hipGetLastError();
  });
}

hipError_t launch_get_state(int q, int storage, const ConvParams &cp,
                            const void *buf, double *f, hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_get_state<L, S>), dim3(blocks_for(N, 256)),
                       dim3(256), 0, stream, cp, static_cast<const S *>(buf), f);
    return hipGetLastError();
  });
}

hipError_t launch_gather(int q, int storage, const ConvParams &cp,
                         const void *buf, const int64_t *sites, int64_t n,
                         double *out, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_gather<L, S>), dim3(blocks_for(n, 256)), dim3(256), 0,
                       stream, cp, static_cast<const S *>(buf), sites, n, out);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t macro_t(int q, int storage, const ConvParams &cp, const void *buf, T *rho,
                   T *u, hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_macro<L, S, T>), dim3(blocks_for(N, 256)), dim3(256), 0,
                       stream, cp, static_cast<const S *>(buf), rho, u);
    return hipGetLastError();
  });
}

hipError_t launch_macro(int q, int storage, const ConvParams &cp,
                        const void *buf, float *rho, float *u,
                        hipStream_t stream) {
  return macro_t<float>(q, storage, cp, buf, rho, u, stream);
}

hipError_t launch_macro(int q, int storage, const ConvParams &cp,
                        const void *buf, double *rho, double *u,
                        hipStream_t stream) {
  return macro_t<double>(q, storage, cp, buf, rho, u, stream);
}

hipError_t launch_noise(int q, int fp64, uint32_t key0, uint32_t key1,
                        uint32_t replica, uint64_t step, int64_t site0,
                        int64_t n, double *out, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const unsigned g = blocks_for(n, 256);
  if (q == 9) {
    if (fp64)
      hipLaunchKernelGGL((k_noise<D2Q9, double>), dim3(g), dim3(256), 0, stream,
                         key0, key1, replica, step, site0, n, out);
    else
      hipLaunchKernelGGL((k_noise<D2Q9, float>), dim3(g), dim3(256), 0, stream,
                         key0, key1, replica, step, site0, n, out);
  } else if (q == 19) {
    if (fp64)
      hipLaunchKernelGGL((k_noise<D3Q19, double>), dim3(g), dim3(256), 0,
                         stream, key0, key1, replica, step, site0, n, out);
    else
      hipLaunchKernelGGL((k_noise<D3Q19, float>), dim3(g), dim3(256), 0, stream,
                         key0, key1, replica, step, site0, n, out);
  } else if (q == 27) {
    if (fp64)
      hipLaunchKernelGGL((k_noise<D3Q27, double>), dim3(g), dim3(256), 0,
                         stream, key0, key1, replica, step, site0, n, out);
    else
      hipLaunchKernelGGL((k_noise<D3Q27, float>), dim3(g), dim3(256), 0, stream,
                         key0, key1, replica, step, site0, n, out);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, int64_t n, uint32_t key0,
                         uint32_t key1, uint32_t *out, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_philox, dim3(blocks_for(n, 256)), dim3(256), 0, stream,
                     ctr, n, key0, key1, out);
  return hipGetLastError();
}

hipError_t launch_stream_copy(const void *src, void *dst, size_t n16,
                              hipStream_t stream) {
  if (n16 == 0) return hipSuccess;
  // one 16-byte element per thread (a grid-stride loop only beyond 2^30
  // workgroups): the fastest plain copy measured on gfx950
  size_t blocks = (n16 + 255) / 256;
  if (blocks > ((size_t)1 << 30)) blocks = (size_t)1 << 30;
  hipLaunchKernelGGL(cmf_stream_copy_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     stream, static_cast<const u32x4 *>(src),
                     static_cast<u32x4 *>(dst), n16);
  return hipGetLastError();
}

hipError_t launch_bump_step(int64_t *step_ptr, int64_t by, hipStream_t stream) {
  hipLaunchKernelGGL(k_bump_step, dim3(1), dim3(64), 0, stream, step_ptr, by);
  return hipGetLastError();
}

hipError_t launch_macro_dev(int q, int storage, const ConvParams &cp,
                            const void *buf, float *out, hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    hipLaunchKernelGGL((k_macro_dev<L, S>), dim3(blocks_for(N, 256)), dim3(256), 0,
                       stream, cp, static_cast<const S *>(buf), out);
    return hipGetLastError();
  });
}

hipError_t launch_sk_accumulate(const void *F, int64_t M, double inv_n,
                                double *acc, hipStream_t stream) {
  hipLaunchKernelGGL(k_sk_accumulate, dim3(blocks_for(4 * M, 256)), dim3(256), 0,
                     stream, static_cast<const float2 *>(F), M, inv_n, acc);
  return hipGetLastError();
}

ShellGeom shell_geom(int nx, int ny, int nz, int nbins) {
  ShellGeom g;
  g.nx = nx;
  g.ny = ny;
  g.nz = nz;
  g.nxh = nx / 2 + 1;
  g.nbins = nbins;
  const double pi = 3.141592653589793;
  g.kmax = pi * sqrt((nx > 1 ? 1.0 : 0.0) + (ny > 1 ? 1.0 : 0.0) + (nz > 1 ? 1.0 : 0.0)) *
           (1.0 + 1e-12);
  return g;
}

hipError_t launch_sk_shells(int nx, int ny, int nz, int nbins, int64_t M, int32_t *counts,
                            int32_t *perm, int64_t *off, hipStream_t stream) {
  const ShellGeom g = shell_geom(nx, ny, nz, nbins);
  int64_t chunk = ((M + kSkChunks - 1) / kSkChunks + 63) / 64 * 64;
  if (chunk < 512) chunk = 512;
  const int nchunks = (int)((M + chunk - 1) / chunk);
  const size_t lds = sizeof(int32_t) * nbins;
  hipLaunchKernelGGL(k_sk_count, dim3(nchunks), dim3(64), lds, stream, g, M, chunk, counts);
  hipLaunchKernelGGL(k_sk_starts, dim3(1), dim3(1024), 0, stream, counts, nchunks, nbins, off);
  hipLaunchKernelGGL(k_sk_scatter, dim3(nchunks), dim3(64), lds, stream, g, M, chunk, counts, perm);
  return hipGetLastError();
}

hipError_t launch_sk_segments(const double *acc, int64_t M, int nx, int ny, int nz,
                              int nbins, const int32_t *perm, const int64_t *off, double *parts,
                              double *out, hipStream_t stream) {
  hipLaunchKernelGGL(k_sk_segments, dim3(nbins, kSkParts), dim3(256), 0, stream, acc, M,
                     shell_geom(nx, ny, nz, nbins), perm, off, parts);
  hipLaunchKernelGGL(k_sk_total, dim3(blocks_for(kSkCols * nbins, 256)), dim3(256), 0, stream,
                     parts, kSkCols * nbins, out);
  return hipGetLastError();
}

hipError_t launch_vel_stats(int q, int storage, const ConvParams &cp, const void *buf,
                            double *keep, int nbins, double xmax, double *partials, VelState *st,
                            unsigned long long *counts, hipStream_t stream) {
  const int64_t N = (int64_t)cp.nx * cp.ny * cp.nz;
  const int dims = q == 9 ? 2 : 3, ncounts = counts ? 3 * (nbins + 2) : 0;
  const int grid = (int)(blocks_for(N, 256) < (unsigned)kVelGrid ? blocks_for(N, 256) : kVelGrid);
  // fewer workgroups for the histogram, each of which adds its counts to the
  // totals; as many copies of its counters as 32 KB hold
  const int hgrid = grid < kVelHistGrid ? grid : kVelHistGrid;
  int copies = 1;
  while (copies < 8 && 2 * copies * 3 * (nbins + 2) * (int)sizeof(uint32_t) <= 32768) copies *= 2;
  const size_t lds = sizeof(uint32_t) * copies * 3 * (size_t)(nbins + 2);
  auto rest = [&](auto src) {
    using SRC = decltype(src);
    hipLaunchKernelGGL((k_vel_moments<SRC>), dim3(grid), dim3(256), 0, stream, src, N, st, partials);
    hipLaunchKernelGGL((k_vel_final<kVelCols>), dim3(1), dim3(256), 0, stream, partials, grid,
                       (double)N, st, nullptr, 0);
    if (counts)
      hipLaunchKernelGGL((k_vel_hist<SRC>), dim3(hgrid), dim3(256), lds, stream, src, N, st, dims,
                         nbins, xmax, copies, counts);
    return hipGetLastError();
  };
  return with_lattice_storage(q, storage, [&](auto lt, auto stt) {
    using L = typename decltype(lt)::type;
    using S = typename decltype(stt)::type;
    const PopVelocity<L, S> src{cp, static_cast<const S *>(buf)};
    hipLaunchKernelGGL((k_vel_sums<PopVelocity<L, S>>), dim3(grid), dim3(256), 0, stream, src, N,
                       dims, keep, partials);
    hipLaunchKernelGGL((k_vel_final<3>), dim3(1), dim3(256), 0, stream, partials, grid, (double)N,
                       st, counts, ncounts);
    if (keep) return rest(KeptVelocity<L::D>{keep, N});
    return rest(src);
  });
}

hipError_t launch_set_i64(int64_t *p, int64_t v, hipStream_t stream) {
  hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(64), 0, stream, p, v);
  return hipGetLastError();
}

hipError_t launch_zero_i64(int64_t *p, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_i64, dim3(blocks_for(n, 256)), dim3(256), 0, stream,
                     p, n);
  return hipGetLastError();
}

}  // namespace cmf
