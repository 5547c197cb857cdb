// Spatially varying PSF (gfx950): reconstruction of an image's PSF at a position from its
// eigen-images and the fit of a Gaussian mixture to it (Section 2.2.2, Table 1: E principal
// images on a side x side grid centred on a source, loadings varying smoothly over the
// image; Section 2.2.3: the PSF approximated by a mixture of bivariate normals).
//
// k_psf_fit: one workgroup of 256 threads per fit, all arithmetic in FP64.  The PSF image
// (at most 63 x 63 knots) is formed once in LDS; each expectation-maximisation iteration
// evaluates the K component densities at every knot, accumulates per component the weighted
// sums of 1, dx, dy, dx^2, dx dy, dy^2 over the responsibilities, reduces them across the
// workgroup in a fixed order (wavefront butterflies, then the four wavefronts in order) and
// forms the next mixture.  Deterministic: no atomics.
//
// Bound by FP64 VALU issue (one operation per lane every 4 cycles), so the split and the
// algebra spare operations: a thread owns one knot column (256 / side row strips of it), so
// that dx, the exponent's column terms and the moments in dx are formed once per iteration
// instead of once per knot (three running sums per component, not six); K is a template
// parameter; the covariance's inverse and normaliser are formed once per component and
// iteration; the exponential is exp2_fp64.  4000 fits of K = 3 on 51 x 51 knots, 30
// iterations: 3.54 ms before (one column-free loop for every K, divisions and library exponentials
// per knot), 1.30 ms after, about 32 operations per component and knot.
#include <hip/hip_runtime.h>
#include <math.h>

#include <cstring>

#include "device.h"
#include "pixmath.h"
#include "plan.h"

namespace celmi {

constexpr int kPsfThreads = 256;
constexpr int kPsfWaves = kPsfThreads / kWave;
constexpr int kPsfMaxSide = CEL_PSF_MAX_SIDE;
constexpr int kPsfSums = 6 * kMaxPsf;

struct PsfFitArgs {
  int32_t n_images, n_eigen, side;
  const double* eigen;      // [n_images][n_eigen][side][side]
  const double* coef;       // [n_images][n_eigen][6]
  const double* size;       // [n_images][2]: W, H
  const int32_t* fit_img;   // [n]
  const double* fit_xy;     // [n][2]
  int32_t n_iter;
  double* out;              // [n][kMaxPsf][6]
  int32_t* err;
};

// Sum each of the L per-thread values over the workgroup in a fixed order: the first
// wavefront's lanes l < L return the sum of value l (the other threads' result is not used).
template <int L>
__device__ __forceinline__ double block_sum(const double (&v)[L], double (*red)[kPsfSums]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double s = wave_sums<L>(v, lane);
  const int slot = wave_sums_slot<L>(lane);
  if (slot >= 0) red[wv][slot] = s;
  __syncthreads();
  double t = 0.0;
  if ((int)threadIdx.x < L)
#pragma unroll
    for (int w = 0; w < kPsfWaves; ++w) t += red[w][threadIdx.x];
  return t;
}

// 1 / x: the hardware's approximation with two Newton steps (not a finite number where 1 / x
// is not).
__device__ __forceinline__ double reciprocal(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

template <int K>
__global__ __launch_bounds__(kPsfThreads) void k_psf_fit(PsfFitArgs a) {
  extern __shared__ double wts[];   // side * side
  __shared__ double red[kPsfWaves][kPsfSums];
  __shared__ double mean[2];
  // a component's density: mean, covariance yy, -2 xy and xx, and, each in two parts, the
  // exponent's factor -log2(e) / (2 det) and weight / (2 pi sqrt(det)): a knot's rounding
  // averages out over the knots, a component's would shift the whole fit
  enum { kMx, kMy, kYY, kXY, kXX, kH, kHLo, kW, kWLo, kCf };
  __shared__ double cf[K][kCf];
  const int f = blockIdx.x;
  const int tid = threadIdx.x;
  const int n = a.fit_img[f];
  double* out = a.out + (int64_t)f * kMaxPsf * 6;
  if (n < 0 || n >= a.n_images) {   // a bad image index: this fit's rows are NaN
    if (tid < kMaxPsf * 6) out[tid] = NAN;
    if (tid == 0 && a.err) atomicOr(a.err, CEL_DEVERR_BAD_INDEX);
    return;
  }
  const int side = a.side, npx = side * side, E = a.n_eigen;
  const double c = 0.5 * (side - 1);
  // this thread's knots: column j, rows row0, row0 + strips, ... (threads past the last whole
  // strip have none); in row-major order its knot index advances by strips * side
  const int strips = kPsfThreads / side, row0 = tid / side, j = tid - row0 * side;
  const int pend = row0 < strips ? npx : 0, pstep = strips * side;
  const double dx = j - c;
  // loadings at the fit position: quadratic in u = x / W, v = y / H
  const double u = a.fit_xy[2 * f] / a.size[2 * n], v = a.fit_xy[2 * f + 1] / a.size[2 * n + 1];
  const double mono[6] = {1.0, u, v, u * u, u * v, v * v};
  double load[kMaxPsf];
#pragma unroll
  for (int e = 0; e < kMaxPsf; ++e) {
    double s = 0.0;
    if (e < E)
#pragma unroll
      for (int t = 0; t < 6; ++t) s += a.coef[((int64_t)n * E + e) * 6 + t] * mono[t];
    load[e] = s;
  }
  // the PSF image, negative values clipped; its mass and centroid
  const double* eig = a.eigen + (int64_t)n * E * npx;
  double m3[3] = {0.0, 0.0, 0.0};
  double dy = row0 - c;
  for (int p = tid; p < pend; p += pstep, dy += strips) {
    double s = 0.0;
    for (int e = 0; e < E; ++e) s += load[e] * eig[(int64_t)e * npx + p];
    s = s > 0.0 ? s : 0.0;
    wts[p] = s;
    m3[0] += s;
    m3[2] = fma(s, dy, m3[2]);
  }
  m3[1] = m3[0] * dx;
  double sum = block_sum<3>(m3, red);
  const double M = __shfl(sum, 0, 64);   // (first wavefront; as everything derived from sums)
  const double mx = __shfl(sum, 1, 64) / M, my = __shfl(sum, 2, 64) / M;
  if (tid == 0) {
    mean[0] = mx;
    mean[1] = my;
  }
  __syncthreads();
  // central second moments (a second pass, about the centroid)
  {
    const double ex = dx - mean[0], ym = mean[1];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    dy = row0 - c;
    for (int p = tid; p < pend; p += pstep, dy += strips) {
      const double s = wts[p], ey = dy - ym, sy = s * ey;
      s0 += s;
      s1 += sy;
      s2 = fma(sy, ey, s2);
    }
    const double m2[3] = {ex * ex * s0, ex * s1, s2};
    sum = block_sum<3>(m2, red);
  }
  // the mixture: component k in lane k of the first wavefront
  double mix[6];
  {   // the start: every component at the centroid, covariance scaled by 2^(k - (K-1)/2)
    const double fac = exp2((double)tid - 0.5 * (K - 1));
    mix[0] = 1.0 / K;
    mix[1] = mx;
    mix[2] = my;
#pragma unroll
    for (int q = 0; q < 3; ++q) mix[3 + q] = fac * __shfl(sum, q, 64) / M;
  }
  for (int it = 0; it < a.n_iter; ++it) {
    if (tid < K) {
      const double det = mix[3] * mix[5] - mix[4] * mix[4];
      // -log2(e) / 2 and 2 pi as sums of two doubles
      constexpr double kL = -0.5 * kLog2e, kLLo = -0.5 * 2.0355273740931033e-17;
      constexpr double kP = 2.0 * M_PI, kPLo = 2.4492935982947064e-16;
      const double h = kL / det;
      const double r = sqrt(det), r_lo = fma(-r, r, det) / (2.0 * r);
      const double n = kP * r, n_lo = fma(kP, r, -n) + kP * r_lo + kPLo * r;
      const double w = mix[0] / n;
      cf[tid][kMx] = mix[1];
      cf[tid][kMy] = mix[2];
      cf[tid][kYY] = mix[5];
      cf[tid][kXY] = -2.0 * mix[4];
      cf[tid][kXX] = mix[3];
      cf[tid][kH] = h;
      cf[tid][kHLo] = (fma(-h, det, kL) + kLLo) / det;
      cf[tid][kW] = w;
      cf[tid][kWLo] = (fma(-w, n, mix[0]) - w * n_lo) / n;
    }
    __syncthreads();   // cf is written; red is free again
    double e0[K], e1[K], e2[K], h[K], h_lo[K], wn[K], wn_lo[K], ym[K], s0[K], s1[K], s2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double ex = dx - cf[k][kMx];
      ym[k] = cf[k][kMy];
      e0[k] = cf[k][kYY] * ex * ex;
      e1[k] = cf[k][kXY] * ex;
      e2[k] = cf[k][kXX];
      h[k] = cf[k][kH];
      h_lo[k] = cf[k][kHLo];
      wn[k] = cf[k][kW];
      wn_lo[k] = cf[k][kWLo];
      s0[k] = s1[k] = s2[k] = 0.0;
    }
    dy = row0 - c;
    for (int p = tid; p < pend; p += pstep, dy += strips) {
      double comp[K], tot = 0.0;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double ey = dy - ym[k];
        const double e = exp2_fp64(fma(ey, fma(e2[k], ey, e1[k]), e0[k]), h[k], h_lo[k]);
        comp[k] = fma(wn[k], e, wn_lo[k] * e);
        tot += comp[k];
      }
      if (!(tot > 0.0)) continue;
      // the responsibilities comp / tot (at most 1) times the knot's weight, by one quotient
      // weight / tot unless that (or 1 / tot) leaves the range
      double t = wts[p] * reciprocal(tot);
      if (!(t <= 1e300)) {
        t = reciprocal(tot * 0x1p600);
#pragma unroll
        for (int k = 0; k < K; ++k) comp[k] = comp[k] * 0x1p600 * t;
        t = wts[p];
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double r = comp[k] * t, ry = r * dy;
        s0[k] += r;
        s1[k] += ry;
        s2[k] = fma(ry, dy, s2[k]);
      }
    }
    double acc[6 * K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double sx = s0[k] * dx;
      acc[6 * k + 0] = s0[k];
      acc[6 * k + 1] = sx;
      acc[6 * k + 2] = s1[k];
      acc[6 * k + 3] = sx * dx;
      acc[6 * k + 4] = s1[k] * dx;
      acc[6 * k + 5] = s2[k];
    }
    sum = block_sum<6 * K>(acc, red);
    if (tid < 64) {
      double sm[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) sm[q] = __shfl(sum, (6 * tid + q) & 63, 64);
      const double nk = sm[0];
      if (tid < K && nk > 1e-12 * M) {   // a component with no weight keeps its parameters
        const double ax = sm[1] / nk, ay = sm[2] / nk;
        mix[0] = nk / M;
        mix[1] = ax;
        mix[2] = ay;
        mix[3] = sm[3] / nk - ax * ax;
        mix[4] = sm[4] / nk - ax * ay;
        mix[5] = sm[5] / nk - ay * ay;
      }
    }
  }
  // weights normalised to one; rows beyond K zero
  if (tid < 64) {
    double wsum = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) wsum += __shfl(mix[0], k, 64);
    if (tid < kMaxPsf) {
#pragma unroll
      for (int q = 0; q < 6; ++q) out[6 * tid + q] = tid >= K ? 0.0 : q == 0 ? mix[0] / wsum : mix[q];
    }
  }
}

}  // namespace celmi

using namespace celmi;

extern "C" cel_status cel_psf_fit(cel_ctx* ctx, const cel_psf_model* model, int32_t n_fits, const int32_t* fit_img,
                                  const double* fit_xy, int32_t n_comp, int32_t n_iter, double* out, void* stream) {
  if (!ctx || !model || n_fits < 0 || n_comp < 1 || n_iter < 0 || n_iter > 100000) return CEL_EINVAL;
  if (n_comp > kMaxPsf || model->n_eigen > CEL_MAX_EIGEN || model->side > kPsfMaxSide) return CEL_EUNSUPPORTED;
  if (model->n_images < 0 || model->n_eigen < 1 || model->side < 3 || model->side % 2 == 0) return CEL_EINVAL;
  if (n_fits == 0) return CEL_OK;
  if (!fit_img || !fit_xy || !out || !model->eigen || !model->coef || !model->size || model->n_images < 1)
    return CEL_EINVAL;
  if (hipSetDevice(ctx->device) != hipSuccess) return CEL_EHIP;
  PsfFitArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n_images = model->n_images;
  a.n_eigen = model->n_eigen;
  a.side = model->side;
  a.eigen = model->eigen;
  a.coef = model->coef;
  a.size = model->size;
  a.fit_img = fit_img;
  a.fit_xy = fit_xy;
  a.n_iter = n_iter;
  a.out = out;
  a.err = ctx->d_err;
  const size_t lds = sizeof(double) * (size_t)a.side * a.side;
  void (*const kernels[kMaxPsf])(PsfFitArgs) = {k_psf_fit<1>, k_psf_fit<2>, k_psf_fit<3>, k_psf_fit<4>};
  hipLaunchKernelGGL(kernels[n_comp - 1], dim3(n_fits), dim3(kPsfThreads), lds, (hipStream_t)stream, a);
  return hipGetLastError() == hipSuccess ? CEL_OK : CEL_EHIP;
}
