// cmflb_step_fused.hip -- several D2Q9 steps per launch for small boxes.
//
// A step of a box of up to a few hundred thousand sites takes a few
// microseconds whatever its size: the launch, one pass of loads and stores
// through caches that the eight XCDs do not share, and one wavefront's
// collision in a row.  This kernel takes `nsteps` steps per launch: a
// workgroup owns a tile, pulls the populations of its tile and the nsteps - 1
// sites around it from HBM, and steps that region, one site narrower on each
// side per step, from LDS to LDS; the last step writes the tile's own sites.
// The sites around the tile are computed by its neighbours too; the same
// arithmetic on the same values gives the same bits, so tiles need no
// exchange and the populations equal those of single steps.
//
// Why seven steps in tiles of 16 x (4 to 16): a launch and its one pass
// through HBM take about 4.5 us, a step in LDS 0.8-2 us (one to three
// wavefronts' collisions in a row on each SIMD, the noise above all), and the
// region grows with the steps; 64^2 FP32 took 5.4 / 3.0 / 2.65 / 2.57 / 2.75 us
// per step with 1 / 3 / 5 / 7 / 9 steps per launch.  The sums of a step's
// statistics run in the next step's time on the wave that has no sites (in the
// sites' waves, ahead of their work, they took 0.8 us per step).  FP32 with
// statistics: 64^2 5.96 -> 1.70, 200^2 6.36 -> 2.59, 400 x 300 8.50 -> 4.85 us
// per step; the floor of 200^2 is 0.5 us (2.9 MB per step, or 342
// instructions per site).
#include "cmflb_step.h"

namespace cmf {

namespace {

// the distinct statistics columns of D2Q9: sum_jz is an exact zero and
// sum_uz2 equals sum_uz (zeros, or NaN where rho is not finite)
constexpr int kCols2 = 9;
constexpr int kColOf[kNAcc] = {0, 1, 2, -1, 3, 4, 5, 6, 7, 5, 8};

// LDS of a workgroup with tiles of kCell x TY sites: two buffers of the Q
// populations of a region of RX x RY sites, then two of the statistics
// columns of the tile, kCellPitch values per cell.  The sizes are
// compile-time constants, so a site's 2 Q accesses share three addresses.
template <typename S, typename R, int TY>
struct FusedLds {
  static constexpr int RX = kCell + 2 * (kFusedSteps - 1), RY = TY + 2 * (kFusedSteps - 1);
  typename Store<S, R>::bits_t pop[2][D2Q9::Q][RX * RY];
  alignas(16) R stat[2][kCols2][TY * kCellPitch];
};

template <typename S, typename R, bool GENERAL, int TY>
__global__ __launch_bounds__(1024) void k_step_fused(
    const S *__restrict__ src, S *__restrict__ dst, const StepParams<R> p,
    const int64_t *__restrict__ step_ptr, int step_off, int nsteps, double *__restrict__ partials,
    int64_t pstride) {
  using L = D2Q9;
  using ST = Store<S, R>;
  using Lds = FusedLds<S, R, TY>;
  constexpr int Q = L::Q, RX = Lds::RX;
  constexpr uint32_t B = sizeof(S);
  extern __shared__ double fused_lds[];
  Lds &lds = *reinterpret_cast<Lds *>(fused_lds);
  const uint64_t step0 = (uint64_t)(*step_ptr + step_off);
  const int nx = p.nx, ny = p.ny;
  const int x0 = (blockIdx.x % p.ncx) * kCell, y0 = (blockIdx.x / p.ncx) * TY;
  const int w = nx - x0 < kCell ? nx - x0 : kCell;
  const int hgt = ny - y0 < TY ? ny - y0 : TY;
  const uint32_t bytes = (uint32_t)Q * (uint32_t)nx * (uint32_t)ny * B;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(src, bytes);
  const __amdgpu_buffer_rsrc_t rd = make_rsrc(dst, bytes);
  const uint32_t rowb = (uint32_t)nx * B;
  if (partials && w < kCell)  // sites missing from the cells of a row's end
    for (int i = threadIdx.x; i < 2 * kCols2 * TY * kCellPitch; i += blockDim.x)
      (&lds.stat[0][0][0])[i] = R(0);
  __syncthreads();

  // sums of step j's cells, from the values its sites left in LDS, by the
  // last threads: the sites of a step go to the first ones
  auto reduce = [&](int j) {
    double *out = partials + (int64_t)j * pstride + ((int64_t)y0 * p.ncx + x0 / kCell) * kPartStride;
    for (int i = (int)(blockDim.x - 1 - threadIdx.x); i < kNAcc * hgt; i += blockDim.x) {
      const int r = i / kNAcc, k = i - r * kNAcc;
      const int col = k < 3 ? k : k == 9 ? 5 : k == 10 ? 8 : k - 1;
      const double s = k == 3 ? 0.0 : cell_sum(&lds.stat[j & 1][col][r * kCellPitch]);
      out[(int64_t)r * p.ncx * kPartStride + k] = s;
    }
  };

  // step j: the first from HBM, the last to HBM, the others from LDS to LDS
  // (`first` and `last` a constant's type where each kind has its own code)
  auto step = [&](auto first, auto last, int j) {
    constexpr bool LAST = std::is_same<decltype(last), std::true_type>::value;
    constexpr bool INNER = std::is_same<decltype(last), std::false_type>::value;
    if (partials && !first) reduce(j - 1);
    const int h = LAST ? 0 : nsteps - 1 - j;  // sites computed beyond the tile
    const int rw = w + 2 * h, area = rw * (hgt + 2 * h);
    // i / rw by a multiplication, exact for i < 4096 and rw <= 256 (i (m rw
    // - 2^20) <= i rw < 2^20 with m = 2^20 / rw + 1)
    const uint32_t m = (1u << 20) / (uint32_t)rw + 1u;
    for (int i = threadIdx.x; i < area; i += blockDim.x) {
      const int ry = (int)(((uint32_t)i * m) >> 20), rx = i - ry * rw;
      int gx = x0 - h + rx, gy = y0 - h + ry;
      gx = gx < 0 ? gx + nx : gx >= nx ? gx - nx : gx;
      gy = gy < 0 ? gy + ny : gy >= ny ? gy - ny : gy;
      const int lidx = (ry + j) * RX + rx + j;  // in the first step's region
      // (FP64 draws when it collides: 64^2 without noise 1.51 against 1.58 us)
      Pulled<L, S, R, sizeof(S) == 4> f{p.scale};
      if (first) {
        const uint32_t xs[3] = {(uint32_t)wrap_sub(gx, -1, nx) * B, (uint32_t)gx * B,
                                (uint32_t)wrap_sub(gx, 1, nx) * B};
        const uint32_t ys[3] = {(uint32_t)wrap_sub(gy, -1, ny) * Q * rowb, (uint32_t)gy * Q * rowb,
                                (uint32_t)wrap_sub(gy, 1, ny) * Q * rowb};
#pragma unroll
        for (int q = 0; q < Q; ++q)
          f.keep(q, buf_load<S, false>(rs, ys[L::cy[q] + 1] + xs[L::cx[q] + 1],
                                       (uint32_t)pop_slot<L>(q) * rowb));
      } else {
        const auto *from = &lds.pop[(j & 1) ^ 1][0][lidx];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          f.keep(q, from[q * RX * Lds::RY - L::cy[q] * RX - L::cx[q]]);
      }
      const auto normals = f.normals(p, (uint32_t)(gx + nx * gy), step0 + j);
      R *d = f.d;
      SiteStats<R> st;
      collide_site<L, R, GENERAL, sizeof(S) == 2>(d, p, normals, st);
      if (INNER || h > 0) {
        auto *to = &lds.pop[j & 1][0][lidx];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          to[q * RX * Lds::RY] = ST::to_bits(d[q], p.iscale[weight_class<L>(q)]);
      } else {
#pragma unroll
        for (int q = 0; q < Q; ++q)
          buf_store<S, false>(ST::to_bits(d[q], p.iscale[weight_class<L>(q)]), rd,
                              (uint32_t)gy * Q * rowb + (uint32_t)gx * B,
                              (uint32_t)pop_slot<L>(q) * rowb);
      }
      const int ix = rx - h, iy = ry - h;
      if (partials && ix >= 0 && ix < w && iy >= 0 && iy < hgt) {
        R *v = &lds.stat[j & 1][0][iy * kCellPitch + ix];
#pragma unroll
        for (int k = 0; k < kNAcc; ++k)
          if (kColOf[k] >= 0 && k != 9) v[kColOf[k] * TY * kCellPitch] = st.v[k];
      }
    }
    __syncthreads();
  };
  // The first and last step in code of their own take 7-10 % less time (us per
  // step, 64^2 FP32 1.87 -> 1.71, 200^2 2.77 -> 2.59, 250 x 255 FP16 3.41 -> 3.14);
  // FP64 then spills scalar registers (64^2 1.49 -> 1.57) and keeps one loop.
  if (sizeof(R) == 8 || nsteps == 1) {
    for (int j = 0; j < nsteps; ++j) step(j == 0, j, j);
  } else {
    step(std::true_type{}, std::false_type{}, 0);
    for (int j = 1; j < nsteps - 1; ++j) step(std::false_type{}, std::false_type{}, j);
    step(std::false_type{}, std::true_type{}, nsteps - 1);
  }
  if (partials) reduce(nsteps - 1);
}

template <typename S, typename R, bool GENERAL, int TY>
hipError_t fused(const void *params, const void *src, void *dst, const int64_t *step_ptr,
                 int step_off, int nsteps, double *partials, int64_t pstride, hipStream_t stream) {
  const StepParams<R> &p = *static_cast<const StepParams<R> *>(params);
  using Lds = FusedLds<S, R, TY>;
  static_assert(Lds::RX * Lds::RY < 4096 && Lds::RX <= 256 && sizeof(Lds) <= 160 * 1024, "region");
  // the sites of the first (largest) step in one pass, and a wave for the sums
  const int h = 2 * (nsteps - 1);
  int threads = ((kCell + h) * (TY + h) + 63) / 64 * 64 + 64;
  if (threads > 1024) threads = 1024;
  hipLaunchKernelGGL((k_step_fused<S, R, GENERAL, TY>), dim3(p.ncx * ((p.ny + TY - 1) / TY)),
                     dim3(threads), sizeof(Lds), stream, static_cast<const S *>(src),
                     static_cast<S *>(dst), p, step_ptr, step_off, nsteps, partials, pstride);
  return hipGetLastError();
}

template <typename S, typename R, bool GENERAL>
hipError_t by_tile(int ty, const void *params, const void *src, void *dst, const int64_t *step_ptr,
                   int off, int nsteps, double *partials, int64_t pstride, hipStream_t stream) {
  switch (ty) {
    case 4:
      return fused<S, R, GENERAL, 4>(params, src, dst, step_ptr, off, nsteps, partials, pstride, stream);
    case 8:
      return fused<S, R, GENERAL, 8>(params, src, dst, step_ptr, off, nsteps, partials, pstride, stream);
    case 12:
      return fused<S, R, GENERAL, 12>(params, src, dst, step_ptr, off, nsteps, partials, pstride, stream);
    case 16:
      return fused<S, R, GENERAL, 16>(params, src, dst, step_ptr, off, nsteps, partials, pstride, stream);
  }
  return hipErrorInvalidValue;
}

template <typename S, typename R>
hipError_t by_rates(bool general, int ty, const void *params, const void *src, void *dst,
                    const int64_t *step_ptr, int off, int nsteps, double *partials,
                    int64_t pstride, hipStream_t stream) {
  return general ? by_tile<S, R, true>(ty, params, src, dst, step_ptr, off, nsteps, partials, pstride, stream)
                 : by_tile<S, R, false>(ty, params, src, dst, step_ptr, off, nsteps, partials, pstride, stream);
}

}  // namespace

hipError_t launch_step_fused(int storage, bool general, int ty, const void *params,
                             const void *src, void *dst, const int64_t *step_ptr, int step_off,
                             int nsteps, double *partials, int64_t pstride, hipStream_t stream) {
  if (nsteps < 1 || nsteps > kFusedSteps || nsteps % 2 == 0 || src == dst) return hipErrorInvalidValue;
  switch (storage) {
    case kF64:
      return by_rates<double, double>(general, ty, params, src, dst, step_ptr, step_off, nsteps, partials, pstride, stream);
    case kF32:
      return by_rates<float, float>(general, ty, params, src, dst, step_ptr, step_off, nsteps, partials, pstride, stream);
    case kF16:
      return by_rates<__half, float>(general, ty, params, src, dst, step_ptr, step_off, nsteps, partials, pstride, stream);
    case kBF16:
      return by_rates<__hip_bfloat16, float>(general, ty, params, src, dst, step_ptr, step_off, nsteps, partials, pstride, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace cmf
