// Device helpers shared by the celmi kernels (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "device.h"

namespace celmi {

// ----------------------------------------------------------------------------------------
// precision helpers

// 2^x in FP64: x = n + f with n the nearest integer, 2^f = 1 + f g(f) with g the polynomial
// of degree 10 interpolating (2^f - 1) / f at the Chebyshev nodes of [-1/2, 1/2] (relative
// error 2.0e-17 with the coefficients as doubles; 0.8 ulp with the evaluation's rounding),
// scaled by 2^n (n saturates as an integer: overflow to infinity, underflow to 0).  0 at
// -infinity; infinity or NaN at +infinity; NaN stays NaN.  About 18 operations against the
// library's 26.
//
// The conversion is the instruction's own, which saturates and takes NaN to 0; the language's
// is undefined beyond the integers, where exponents of narrow components do lie.
__device__ __forceinline__ int saturated_int(double n) {
  int i;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(n));
  return i;
}
__device__ __forceinline__ double exp2_reduced(double f, double n) {
  double r = 4.4549605981865186e-10;
  r = fma(f, r, 7.072585949269223e-09);
  r = fma(f, r, 1.0178062445845774e-07);
  r = fma(f, r, 1.321544258792169e-06);
  r = fma(f, r, 1.525273382983612e-05);
  r = fma(f, r, 1.540353044173605e-04);
  r = fma(f, r, 1.3333558146416936e-03);
  r = fma(f, r, 9.618129107606888e-03);
  r = fma(f, r, 5.55041086648216e-02);
  r = fma(f, r, 2.4022650695910097e-01);
  r = fma(f, r, 6.931471805599453e-01);
  return __builtin_amdgcn_ldexp(fma(f, r, 1.0), saturated_int(n));
}
__device__ __forceinline__ double exp2_fp64(double x) {
  const double n = rint(x), r = exp2_reduced(x - n, n);
  return x < -1100.0 ? 0.0 : r;
}
// 2^(q h) for a factor h = hi + lo: no rounding of the product or of h
__device__ __forceinline__ double exp2_fp64(double q, double hi, double lo) {
  const double n = rint(q * hi), r = exp2_reduced(fma(q, lo, fma(q, hi, -n)), n);
  return q * hi < -1100.0 ? 0.0 : r;
}

template <typename T> __device__ __forceinline__ T fexp2(T x);
template <> __device__ __forceinline__ float fexp2<float>(float x) { return __builtin_amdgcn_exp2f(x); }
template <> __device__ __forceinline__ double fexp2<double>(double x) { return exp2_fp64(x); }

constexpr double kLn2 = 0.69314718055994530942;

// x log(E/x) for a count x > 0 and a rate E > 0: the part of the centred Poisson term that
// cancels against E - x, so the quotient must be accurate to the last bit or two.  float:
// the quotient from the hardware reciprocal with one residual correction (within an ulp of
// E/x for normal operands), the logarithm from the hardware log2 (operands here are
// normal: x >= 1, E at least the patch's smallest sky value); double: library division
// and logarithm.
template <typename T> __device__ __forceinline__ T x_log_ratio(T x, T E);
template <> __device__ __forceinline__ float x_log_ratio<float>(float x, float E) {
  const float r = __builtin_amdgcn_rcpf(x);
  float q = E * r;
  q = fmaf(fmaf(-x, q, E), r, q);
  return x * (__builtin_amdgcn_logf(q) * (float)kLn2);
}
template <> __device__ __forceinline__ double x_log_ratio<double>(double x, double E) { return x * log(E / x); }

// 1/E for the adjoint coefficients (float: hardware reciprocal, within 1 ulp)
template <typename T> __device__ __forceinline__ T frcp(T E);
template <> __device__ __forceinline__ float frcp<float>(float E) { return __builtin_amdgcn_rcpf(E); }
template <> __device__ __forceinline__ double frcp<double>(double E) { return 1.0 / E; }

constexpr double kLog2e = 1.4426950408889634074;
constexpr double kLog2TwoPi = 2.6514961294723187980;   // log2(2 pi)
constexpr double kNegHuge = -1.0e30;
// Block -> position in a cost-sorted work list, XCD-aware.  Workgroups are dispatched to
// the 8 XCDs in turn (block b on XCD b mod 8), each XCD with its own L2.  Consecutive
// positions of the list (the chunks of one patch, sorted next to each other) are handed to
// one XCD in groups of kXcdGroup, so they share its L2 (tables, neighbour maps); the list
// order across groups, and so the large-first balance, is kept.  A tail that does not fill
// whole groups maps to itself.
constexpr int kXcds = 8;
constexpr int kXcdGroup = 4;
__device__ __forceinline__ int xcd_position(int b, int n) {
  constexpr int span = kXcds * kXcdGroup;
  const int full = (n / span) * span;
  if (b >= full) return b;
  const int xcd = b % kXcds, slot = b / kXcds;
  return ((slot / kXcdGroup) * kXcds + xcd) * kXcdGroup + slot % kXcdGroup;
}

// Component cut (reading of the kernels' truncation): a mixture component is skipped over a
// wavefront's pixel box when its contribution to the expected count there, flux times
// density, stays below 2^-kRelCut of the patch's smallest sky value -- far below the
// resolution of the rate in the kernel's precision (2^-24 in float32, 2^-53 in float64).
template <typename T>
constexpr double rel_cut_log2() {
  return sizeof(T) == 8 ? 60.0 : 30.0;
}

// Value of one mixture component at offset (dx, dy) from its centre, given the monomials
// xx = dx^2, xy = 2 dx dy, yy = dy^2 and its record q = (q0, q1, q2, log2 weight):
// 2^(q0 xx + q1 xy + q2 yy + lw) -- the form for values alone (neighbour maps, Hessian);
// the pixel kernel, which needs u = P d for the derivatives anyway, forms the exponent
// from u (the same value up to rounding).
template <typename T>
__device__ __forceinline__ T comp_value(const T* __restrict__ q, T xx, T xy, T yy) {
  return fexp2<T>(fma(q[0], xx, fma(q[1], xy, fma(q[2], yy, q[3]))));
}


// squared radius beyond which 2^(lw - log2(e)/2 d^T C^{-1} d) < 2^cut (-1: never above it;
// +inf when the component is not finite, so that NaN parameters reach the rate)
__device__ __forceinline__ double cut_radius2(double lw, double cxx, double cxy, double cyy, double cut) {
  const double room = lw - cut;
  const double lmax = 0.5 * (cxx + cyy) + sqrt(0.25 * (cxx - cyy) * (cxx - cyy) + cxy * cxy);
  if (isnan(room) || !isfinite(lmax)) return INFINITY;
  if (!(room > 0)) return -1.0;
  return room * lmax * (2.0 / kLog2e);
}

// log2 threshold on a component's density for a source of expected flux L on a patch whose
// sky is at least sky_min; -inf (keep everything) when either is not a positive finite
// number, so that non-finite parameters still propagate to the objective
template <typename T>
__device__ __forceinline__ double density_cut_log2(double L, double sky_min, double log2_L, double log2_sky_min) {
  const double c = log2_sky_min - log2_L - rel_cut_log2<T>();
  return (L > 0 && sky_min > 0 && isfinite(c)) ? c : -INFINITY;
}

// log l_b = log r + W[b] . c,  c_k = ln(l_{k+1} / l_k), reference band r = index 2
static __device__ __constant__ double c_W[5][4] = {
    {-1, -1, 0, 0}, {0, -1, 0, 0}, {0, 0, 0, 0}, {0, 0, 1, 0}, {0, 0, 1, 1}};

__device__ __forceinline__ double sigmoid(double x) { return 1.0 / (1.0 + exp(-x)); }



// Squared distance from (mx, my) to the wavefront's pixel box [bx0, bx1] x [by0, by1].
// The component cut compares a wavefront-uniform squared distance d2 (>= +0, possibly +inf)
// with a stored squared cut radius that is never -0 or NaN (the tables are written so).  For
// such values the order of IEEE floats is the signed order of their bit patterns, so the
// float path takes each test as an integer compare of scalar registers instead of one vector
// compare per component; the double path compares the values.
__device__ __forceinline__ int cut_key(float x) { return __float_as_int(x); }
__device__ __forceinline__ double cut_key(double x) { return x; }
__device__ __forceinline__ int uniform_cut_key(float d2) { return __builtin_amdgcn_readfirstlane(__float_as_int(d2)); }
__device__ __forceinline__ double uniform_cut_key(double d2) { return d2; }

template <typename T>
__device__ __forceinline__ T box_dist2(T mx, T my, const T* box) {
  const T ddx = fmax(fmax(box[0] - mx, mx - box[1]), (T)0);
  const T ddy = fmax(fmax(box[2] - my, my - box[3]), (T)0);
  return fma(ddx, ddx, ddy * ddy);
}

// Pixel box (patch-local columns x0..x1, rows y0..y1) of the run [base, end) of a
// row-major patch of width w.
template <typename T>
__device__ __forceinline__ void run_box(int base, int end, int w, T* box) {
  const int last = end - 1;
  const int r0 = base / w, r1 = last / w;
  box[0] = (T)(r0 == r1 ? base - r0 * w : 0);
  box[1] = (T)(r0 == r1 ? last - r1 * w : w - 1);
  box[2] = (T)r0;
  box[3] = (T)r1;
}

template <typename T>
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Wavefront sums of M values per lane together.  At each lane offset O = 32, 16, ... a lane
// keeps half of its values (the first half when bit O of its index is clear, else the second)
// and adds the partner lane's copies of those, so the values per lane halve at every step
// (M/2 + M/4 + ... exchanges instead of 6 M); once one value is left a plain butterfly
// finishes.  Every sum takes the same additions, in the same pairing and operand order, as
// wave_sum's butterfly, so the results are bitwise those of M wave_sum calls.  U is the
// type the lanes hold (float values are exchanged as floats and widened before the first
// addition, which is exact).  Lane l returns the sum of value wave_sums_slot<M>(l) (-1: none;
// each value has exactly one such lane).
template <int M, int O = 32, typename U>
__device__ __forceinline__ double wave_sums(const U* v, int lane) {
  if constexpr (M == 1) {
    double x = (double)v[0];
#pragma unroll
    for (int off = O; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
  } else {
    static_assert(O >= 1, "more values than lanes");
    constexpr int A = (M + 1) / 2, B = M - A;
    const bool hi = (lane & O) != 0;
    double w[A];
#pragma unroll
    for (int i = 0; i < A; ++i) {
      const U f = v[i], s = i < B ? v[A + i] : (U)0;
      const U send = hi ? f : s;
      w[i] = (double)(hi ? s : f) + (double)__shfl_xor(send, O, 64);
    }
    return wave_sums<A, O / 2, double>(w, lane);
  }
}

// flags[i] for a wavefront-uniform i, known to be uniform (bytes come by vector loads, and a
// pointer formed from one would make every load through it a vector load too)
__device__ __forceinline__ int uniform_byte(const uint8_t* flags, int i) {
  return __builtin_amdgcn_readfirstlane((int)flags[i]);
}

// the lane that wave_sums leaves holding the sum of value q (the lowest such lane)
template <int M, int O = 32>
__host__ __device__ constexpr int wave_sums_lane(int q) {
  if constexpr (M == 1) {
    return 0;
  } else {
    constexpr int A = (M + 1) / 2;
    return q < A ? wave_sums_lane<A, O / 2>(q) : O + wave_sums_lane<A, O / 2>(q - A);
  }
}

// a double held by lane l, read by every lane (l wavefront-uniform)
__device__ __forceinline__ double read_lane(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

template <int M, int O = 32>
__device__ __forceinline__ int wave_sums_slot(int lane) {
  if constexpr (M == 1) {
    return (O == 0 || (lane & (2 * O - 1)) == 0) ? 0 : -1;
  } else {
    constexpr int A = (M + 1) / 2, B = M - A;
    const int r = wave_sums_slot<A, O / 2>(lane);
    if (r < 0) return -1;
    if (lane & O) return r < B ? A + r : -1;
    return r;
  }
}

// LDS written by lanes of one wavefront, read by other lanes of it
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// The value `v` of the lane whose index differs in bit OFF (1, 2 or 4), by data-parallel moves
// instead of an LDS permute.  The move for 4 reverses a group of 8 lanes: it is an exchange for
// values that the lanes of each quad already share.
template <int OFF>
__device__ __forceinline__ double dpp_xor(double v) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4, "");
  constexpr int ctrl = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : 0x141;
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// sum and maximum over each group of 8 lanes, the same bits in every lane of a group
__device__ __forceinline__ double sum8(double v) {
  v += dpp_xor<1>(v);
  v += dpp_xor<2>(v);
  return v + dpp_xor<4>(v);
}
__device__ __forceinline__ double max8(double v) {
  v = fmax(v, dpp_xor<1>(v));
  v = fmax(v, dpp_xor<2>(v));
  return fmax(v, dpp_xor<4>(v));
}

// Transcendental functions of a source's parameters, one argument per lane and broadcast, so
// that each function's code runs once per wavefront (all 64 lanes active) instead of once per
// value.
struct SourceExps {
  double rv[2], cv[2][4];        // flux and colour variances exp(th[5 + i]), exp(th[15 + 4 i + k])
  double rad;                    // exp(th[24])
  double a, prof, axis;          // sigmoid(th[2]), sigmoid(th[25]), sigmoid(th[26])
};

__device__ __forceinline__ SourceExps source_exps(const double* th, int lane) {
  double x = 0.0;
#pragma unroll
  for (int l = 0; l < 14; ++l) {
    const double v = l < 2 ? th[5 + l] : l < 10 ? th[13 + l] : l == 10 ? th[24] : l == 11 ? -th[2]
                     : l == 12 ? -th[25] : -th[26];
    x = lane == l ? v : x;
  }
  double e = exp(x);
  if (lane >= 11) e = 1.0 / (1.0 + e);
  SourceExps r;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    r.rv[i] = read_lane(e, i);
#pragma unroll
    for (int k = 0; k < 4; ++k) r.cv[i][k] = read_lane(e, 2 + 4 * i + k);
  }
  r.rad = read_lane(e, 10);
  r.a = read_lane(e, 11);
  r.prof = read_lane(e, 12);
  r.axis = read_lane(e, 13);
  return r;
}

// Colour bounds of both types (Section 4.2.3 at their optimal weights): the values
// -log sum_j w_j exp(-D_j) and their gradients with respect to the colour means (gm) and
// log colour variances (gv), summed over the prior components j with weights xi_j,
// computed by a whole wavefront (all 64 lanes active): lane 8 i + j
// takes prior component j of type i (lanes 16..63 repeat lanes 0..15), the maximum,
// normaliser and gradient sums are combined by fixed butterflies within each group of 8
// lanes, and every lane receives both types' results.
__device__ inline void colour_bound_wave(const DPrior& pr, const double* th, const SourceExps& ex, int lane, double* kc,
                                         double (*gm)[4], double (*gv)[4]) {
  static_assert(CEL_N_COLOUR_COMPONENTS == 8, "one lane per prior colour component, groups of 8");
  const int i = (lane >> 3) & 1, j = lane & 7;
  double cm[4], cv[4], lcv[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {   // selects, not a lane-dependent index into th
    cm[k] = i ? th[11 + k] : th[7 + k];
    lcv[k] = i ? th[19 + k] : th[15 + k];
    cv[k] = i ? ex.cv[1][k] : ex.cv[0][k];
  }
  const double sum_lcv = lcv[0] + lcv[1] + lcv[2] + lcv[3];
  double tr = 0, maha = 0, row[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    tr += pr.c_prec[i][j][k][k] * cv[k];
    double r = 0;
#pragma unroll
    for (int l = 0; l < 4; ++l) r += pr.c_prec[i][j][k][l] * (cm[l] - pr.c_mean[i][j][l]);
    row[k] = r;
    maha += (cm[k] - pr.c_mean[i][j][k]) * r;
  }
  const double e = pr.c_logw[i][j] - 0.5 * (tr + maha - 4.0 + pr.c_logdet[i][j] - sum_lcv);
  const double mx = max8(e);
  const double w = exp(e - mx);
  const double z = sum8(w);
  const double xi = w / z;
  double part[9];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    part[k] = sum8(xi * row[k]);
    part[4 + k] = sum8(xi * 0.5 * (pr.c_prec[i][j][k][k] * cv[k] - 1.0));
  }
  part[8] = -(mx + log(z));
  // lanes 0..7 hold type 0, lanes 8..15 type 1
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    gm[0][k] = read_lane(part[k], 0);
    gm[1][k] = read_lane(part[k], 8);
    gv[0][k] = read_lane(part[4 + k], 0);
    gv[1][k] = read_lane(part[4 + k], 8);
  }
  kc[0] = read_lane(part[8], 0);
  kc[1] = read_lane(part[8], 8);
}

// KL(q(z_s) || p(z_s)) and its gradient in the unconstrained coordinates (equations eq:kl,
// kleq; Supplement A with the readings: flux KL is the normal KL of log r with variances;
// colour KL is the bound of Section 4.2.3 at its optimal weights; point-mass terms are
// minus the log prior density; direction and angle terms are constants and dropped), by a
// whole wavefront (all lanes active; every lane gets the value and applies the gradient to
// its own g).  Subtracts gs times the gradient from g.  Its time is the latency of its
// transcendental functions (14 exponentials, six log1p, four logarithms when each lane took
// them all), so they are taken across lanes: the finalisation of 3 sources without a gradient,
// little else than the KL, 9.1 -> 6.4 us.
__device__ inline double kl_source_wave(const DPrior& pr, const double* th, const SourceExps& ex, double* g, double gs,
                                        int lane) {
  double kc[2], gm[2][4], gv[2][4];
  colour_bound_wave(pr, th, ex, lane, kc, gm, gv);
  // lanes 0-2: softplus(x) = max(x, 0) + log1p(exp(-|x|)) of the type, profile and axis logits
  // (the second term serves x and -x); lanes 3-5: logs of the flux and radius prior variances
  const double lx = lane == 0 ? th[2] : lane == 1 ? th[25] : th[26];
  const double sp = log1p(exp(-fabs(lx)));
  const double lg = log(lane == 3 ? pr.r[0][1] : lane == 4 ? pr.r[1][1] : 2.0 * M_PI * pr.radius[1]);
  const double l1p[3] = {read_lane(sp, 0), read_lane(sp, 1), read_lane(sp, 2)};
  const double log_R2[2] = {read_lane(lg, 3), read_lane(lg, 4)}, log_E2 = read_lane(lg, 5);
  auto softplus = [](double x, double l) { return fmax(x, 0.0) + l; };
  const double eta = th[2];
  const double a = ex.a;
  const double log_a = -softplus(-eta, l1p[0]), log_1ma = -softplus(eta, l1p[0]);
  double kl = a * (log_a - pr.log_a) + (1.0 - a) * (log_1ma - pr.log_1ma);
  double dk_da = eta - pr.logit_a;          // d KL_a / d a
  const double q[2] = {1.0 - a, a};
  double part[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double rm = th[3 + i], lrv = th[5 + i], rv = ex.rv[i];
    const double R1 = pr.r[i][0], R2 = pr.r[i][1];
    const double kr = 0.5 * (log_R2[i] - lrv) + (rv + (rm - R1) * (rm - R1)) / (2.0 * R2) - 0.5;
    g[3 + i] -= gs * q[i] * (rm - R1) / R2;
    g[5 + i] -= gs * q[i] * (-0.5 + rv / (2.0 * R2));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      g[7 + 4 * i + k] -= gs * q[i] * gm[i][k];
      g[15 + 4 * i + k] -= gs * q[i] * gv[i][k];
    }
    part[i] = kr + kc[i];
    kl += q[i] * part[i];
  }
  dk_da += part[1] - part[0];
  g[2] -= gs * (dk_da * a * (1.0 - a));
  // radius: point mass vs log-normal
  const double lr = th[24], E1 = pr.radius[0], E2 = pr.radius[1];
  kl += lr + 0.5 * log_E2 + (lr - E1) * (lr - E1) / (2.0 * E2);
  g[24] -= gs * (1.0 + (lr - E1) / E2);
  // profile and axis: point mass vs Beta
  {
    const double e = th[25], p = ex.prof, lp = -softplus(-e, l1p[1]), lq = -softplus(e, l1p[1]);
    kl += -(pr.profile[0] - 1.0) * lp - (pr.profile[1] - 1.0) * lq + pr.lbeta_profile;
    g[25] -= gs * (-(pr.profile[0] - 1.0) * (1.0 - p) + (pr.profile[1] - 1.0) * p);
  }
  {
    const double e = th[26], p = ex.axis, lp = -softplus(-e, l1p[2]), lq = -softplus(e, l1p[2]);
    kl += -(pr.axis[0] - 1.0) * lp - (pr.axis[1] - 1.0) * lq + pr.lbeta_axis;
    g[26] -= gs * (-(pr.axis[0] - 1.0) * (1.0 - p) + (pr.axis[1] - 1.0) * p);
  }
  return kl;
}

}  // namespace celmi
