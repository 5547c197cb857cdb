// Trust-region Newton block step and block coordinate ascent (Sections 4.3-4.4).
//
// One Newton iteration on a set of pairwise non-overlapping sources (a colour class):
//   1. component tables of the stepped sources at the current iterate (in a sweep an accepted
//      trial's tables are kept for it)
//   2. the objective, gradient and exact Hessian: k_hess per work item, k_hess_finalize per
//      source.  On request instead the Hessian's pixel part by central differences of the
//      pixel gradient (variants 1..54 at theta +/- h e_k, k_fd_hessian), its KL part
//      analytically, since the tight colour-prior mixture makes the KL's higher derivatives
//      far too large for differencing
//   3. k_trsolve, kTrWaves wavefronts per source: convergence tests and the trust-region
//      subproblem in FP64, its multiplier by L D L^T factorisations of B + lambda I for
//      several lambda at a time; where none gives the step (the hard case) the
//      eigen-decomposition of B = -H by one-sided Jacobi and the secular equation; the
//      trial point
//   4. the objective at the trial points (last variant)
//   5. k_accept: ratio of actual to predicted gain, acceptance and radius update
// Trust-region constants (the paper prints none): accept if rho > eta (0.1); radius
// shrinks to |p|/4 if rho < 1/4 and doubles (to at most radius_max) if rho > 3/4 with the
// step on the boundary; converged if |g|_inf <= gtol max(1, |L_s|/n_pix), the predicted
// gain <= ftol max(1, |L_s|), or radius < radius_min.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "device.h"
#include "kernels.h"
#include "launch_rules.h"
#include "pixmath.h"
#include "plan.h"
#include "trbracket.h"

namespace celmi {

constexpr int kN = kParamN;   // 27
static_assert(((kN + 1) / 2) % 2 == 0, "the Jacobi half-columns hold an even number of rows");
constexpr int kLd = kN + 1;   // padded LDS row



// Hessian of KL_s in the unconstrained coordinates (the same KL as the objective: the type
// KL, the normal KL of log r, the colour bound F = -log sum_j w_j exp(-D_j), and minus the
// log prior densities of the radius, profile and axis point masses), times sc, added into
// B (27 rows of stride LD).  KL = KL_a(eta) + KL_radius + KL_profile + KL_axis
// + (1 - a) K_0 + a K_1; grad F = sum_j xi_j dD_j and
// hess F = sum_j xi_j (d2D_j - dD_j dD_j^T) + grad F grad F^T in the 8 colour variables.
// Computed by a whole wavefront (all 64 lanes active, B in LDS): lane
// 8 i + j takes prior colour component j of type i -- its weight xi_j, dD_j and d2D_j --
// and the sums over j of xi_j (d2D_j - dD_j dD_j^T) and xi_j dD_j are formed through LDS
// in fixed order (work: 16 x 44 and 2 x 44 doubles); lanes then add the two 8 x 8 colour
// blocks and lane 0 the remaining terms.
constexpr int kKlw = 44;   // 36 upper-triangle entries of the 8 x 8 block + 8 gradient entries
template <int LD>
__device__ void kl_hessian_wave(const DPrior& pr, const double* th, double (*B)[LD], double sc, int lane,
                                double (*work)[kKlw], double (*sums)[kKlw]) {
  static_assert(CEL_N_COLOUR_COMPONENTS == 8, "one lane per prior colour component, groups of 8");
  const int i = (lane >> 3) & 1, j = lane & 7;
  double cm[4], cv[4], lcv = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {   // selects, not a lane-dependent index into th
    cm[k] = i ? th[11 + k] : th[7 + k];
    const double l = i ? th[19 + k] : th[15 + k];
    cv[k] = exp(l);
    lcv += l;
  }
  double tr = 0, maha = 0, dD[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    tr += pr.c_prec[i][j][k][k] * cv[k];
    double r = 0;
#pragma unroll
    for (int l = 0; l < 4; ++l) r += pr.c_prec[i][j][k][l] * (cm[l] - pr.c_mean[i][j][l]);
    dD[k] = r;
    dD[4 + k] = 0.5 * (pr.c_prec[i][j][k][k] * cv[k] - 1.0);
    maha += (cm[k] - pr.c_mean[i][j][k]) * r;
  }
  const double e = pr.c_logw[i][j] - 0.5 * (tr + maha - 4.0 + pr.c_logdet[i][j] - lcv);
  double mx = e;
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  const double ex = exp(e - mx);
  double z = ex;
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) z += __shfl_xor(z, off, 64);
  const double xi = ex / z;
  const double kc = -(mx + log(z));   // the colour bound of type i
  if (lane < 16) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int w = u; w < 8; ++w) {
        double d2 = 0.0;
        if (u < 4 && w < 4) d2 = pr.c_prec[i][j][u][w];
        else if (u == w) d2 = 0.5 * pr.c_prec[i][j][u - 4][u - 4] * cv[u - 4];
        work[lane][n++] = xi * (d2 - dD[u] * dD[w]);
      }
#pragma unroll
    for (int u = 0; u < 8; ++u) work[lane][36 + u] = xi * dD[u];
  }
  wave_lds_sync();
  for (int e2 = lane; e2 < 2 * kKlw; e2 += 64) {
    const int ii = e2 / kKlw, q = e2 % kKlw;
    double acc = 0;
    for (int jj = 0; jj < 8; ++jj) acc += work[8 * ii + jj][q];
    sums[ii][q] = acc;
  }
  wave_lds_sync();
  const double eta = th[2], a = sigmoid(eta), aa = a * (1.0 - a);
  // colour blocks: entry (u, w) of type ii, lanes 0..63 twice
  for (int e2 = lane; e2 < 2 * 64; e2 += 64) {
    const int ii = e2 / 64, u = (e2 % 64) / 8, w = e2 % 8;
    const int lo = u < w ? u : w, hi = u < w ? w : u;
    const int n = lo * 8 - lo * (lo - 1) / 2 + (hi - lo);
    const double q = ii == 0 ? 1.0 - a : a;
    const double hf = sums[ii][n] + sums[ii][36 + u] * sums[ii][36 + w];
    const int iu = u < 4 ? 7 + 4 * ii + u : 15 + 4 * ii + (u - 4);
    const int iw = w < 4 ? 7 + 4 * ii + w : 15 + 4 * ii + (w - 4);
    B[iu][iw] += sc * (q * hf);
  }
  const double kc1 = __shfl(kc, 8, 64);
  if (lane == 0) {
    double K[2];
    const double kcs[2] = {kc, kc1};
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
      const double rm = th[3 + ii], lrv = th[5 + ii], rv = exp(lrv);
      const double R1 = pr.r[ii][0], R2 = pr.r[ii][1];
      const double q = ii == 0 ? 1.0 - a : a;
      const double sg = ii == 0 ? -aa : aa;   // d^2 KL / d eta d theta_k = sg dK_i/dtheta_k
      K[ii] = 0.5 * (log(R2) - lrv) + (rv + (rm - R1) * (rm - R1)) / (2.0 * R2) - 0.5 + kcs[ii];
      const double dm = (rm - R1) / R2, dv = -0.5 + rv / (2.0 * R2);
      B[3 + ii][3 + ii] += sc * (q / R2);
      B[5 + ii][5 + ii] += sc * (q * rv / (2.0 * R2));
      B[2][3 + ii] += sc * (sg * dm);
      B[3 + ii][2] += sc * (sg * dm);
      B[2][5 + ii] += sc * (sg * dv);
      B[5 + ii][2] += sc * (sg * dv);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int iu = u < 4 ? 7 + 4 * ii + u : 15 + 4 * ii + (u - 4);
        B[2][iu] += sc * (sg * sums[ii][36 + u]);
        B[iu][2] += sc * (sg * sums[ii][36 + u]);
      }
    }
    // type weight: dKL/deta = a(1-a) [eta - logit A + K1 - K0]
    const double t = eta - pr.logit_a + K[1] - K[0];
    B[2][2] += sc * (aa * (1.0 - 2.0 * a) * t + aa);
    // point masses
    B[24][24] += sc * (1.0 / pr.radius[1]);
    {
      const double p = sigmoid(th[25]);
      B[25][25] += sc * ((pr.profile[0] + pr.profile[1] - 2.0) * p * (1.0 - p));
    }
    {
      const double p = sigmoid(th[26]);
      B[26][26] += sc * ((pr.axis[0] + pr.axis[1] - 2.0) * p * (1.0 - p));
    }
  }
  wave_lds_sync();
}

// ----------------------------------------------------------------------------------------
// Analytic Hessian of the pixel part of L_s (Section 4.3 uses a dense Newton Hessian).
//
// Per patch the pixel sum depends on theta_s through 11 primitives
//   y = (a, L0, L1, e0, e1, mu_x, mu_y, S_xx, S_xy, S_yy, pi)
// (type probability, flux moments L_i = E[l | a=i] and e_i = expm1(Var log l | a=i), the
// pixel-frame centre and galaxy covariance, the de Vaucouleurs weight), with
//   E_s = w0 L0 f0 + w1 L1 f1,  V_s = w0 L0^2 e0 f0^2 + w1 L1^2 e1 f1^2 + w0 w1 d^2,
//   d = L0 f0 - L1 f1,  w0 = 1 - a, w1 = a.
// For T(E, V) = -E + x (log E - V / (2 E^2)):  T_E = c_E, T_V = c_V,
//   T_EE = -x/E^2 - 3 x V / E^4, T_EV = x / E^3, T_VV = 0, so per pixel
//   d2T/du dv = T_EE E_u E_v + T_EV (E_u V_v + E_v V_u) + c_E E_uv + c_V V_uv.
// f0, f1 and their first and second derivatives in (mu, S, pi) are sums of normal densities
// times Hermite polynomials (gal_hess).  The kernel sums G_u and the 66 entries Q_uv
// per work item; k_hess_finalize maps them to theta_s by the chain rule.

constexpr int kPrim = 11;
constexpr int kHQ = 66;
constexpr int kHSlots = 80;   // T, T_own, G[11], Q[66], pad

__host__ __device__ constexpr int qidx(int u, int v) { return u * kPrim - u * (u - 1) / 2 + (v - u); }
__host__ __device__ constexpr int zidx(int i, int j) { return i * 6 - i * (i - 1) / 2 + (j - i); }

template <typename T>
struct PixH {
  T f0, f1;
  T g0[6];   // mu_x, mu_y, S_xx, S_xy, S_yy, pi
  T g1[2];
  T h0[21];  // upper triangle (zidx)
  T h1[3];   // xx, xy, yy
};

// A galaxy component's record: with c the exponent's scale and P' = c^2 P,
//   (c P_xx, c P_xy, c P_yy, log2 weight), (P'_xx, P'_xy, P'_yy, tau / 2), 2 P', 3 P'.
constexpr int kHRec = 16;

// One galaxy component of one profile.  All derivatives of N = weight * normal(p; m, C) in
// (m, S) are spatial ones, for the normal obeys the heat equation dN/dC = d2N/dm dm / 2 and
// dC = tau dS: with the Hermite polynomials H of u = P d,
//   dN/dm_a = N u_a, d2N/dm_a dm_b = N H_ab, dN/dS_ab = (tau/2) N H_ab (twice that for the
//   off-diagonal), d2N/dm_c dS_ab = (tau/2) N H_abc, d2N/dS_ab dS_cd = (tau/2)^2 N H_abcd,
//   H_ab = u_a u_b - P_ab, H_abc = u_c H_ab - P_ac u_b - P_bc u_a,
//   H_abcd = u_d H_abc - P_ad H_bc - P_bd H_ac - P_cd H_ab.
// They depend on the index counts alone: 3 + 4 + 5 values serve the 3 + 6 + 6 second
// derivatives, by recurrence, with u' = c u (order-n sums carry c^n, divided back per pixel).
// gs: sums of (tau/2) N H'_ab; h2, h3, h4: profile-weighted sums of N H', (tau/2) N H',
// (tau/2)^2 N H'.
template <typename T>
__device__ __forceinline__ void gal_hess(const T* q, T wP, T dx, T dy, T& f, T* gm, T* gs, T* h2, T* h3, T* h4) {
#pragma clang fp contract(off)
  const T ux = fma(q[0], dx, q[1] * dy);
  const T uy = fma(q[1], dx, q[2] * dy);
  const T N = fexp2<T>(fma(dx, ux, fma(dy, uy, q[3])));
  const T *P = q + 4, *P2 = q + 8, *P3 = q + 11;
  const T xx = fma(ux, ux, -P[0]), xy = fma(ux, uy, -P[1]), yy = fma(uy, uy, -P[2]);
  const T xxx = ux * (xx - P2[0]), xxy = fma(uy, xx, -P2[1] * ux);
  const T xyy = fma(ux, yy, -P2[1] * uy), yyy = uy * (yy - P2[2]);
  const T xxxx = fma(ux, xxx, -P3[0] * xx), xxxy = fma(uy, xxx, -P3[1] * xx);
  const T xxyy = fma(uy, xxy, fma(-P2[1], xy, -P[2] * xx));
  const T xyyy = fma(ux, yyy, -P3[1] * yy), yyyy = fma(uy, yyy, -P3[2] * yy);
  f += N;
  gm[0] = fma(N, ux, gm[0]);
  gm[1] = fma(N, uy, gm[1]);
  const T Nt = N * q[7], Nw = N * wP, Nwt = Nw * q[7], Nwtt = Nwt * q[7];
  gs[0] = fma(Nt, xx, gs[0]);
  gs[1] = fma(Nt, xy, gs[1]);
  gs[2] = fma(Nt, yy, gs[2]);
  h2[0] = fma(Nw, xx, h2[0]);
  h2[1] = fma(Nw, xy, h2[1]);
  h2[2] = fma(Nw, yy, h2[2]);
  h3[0] = fma(Nwt, xxx, h3[0]);
  h3[1] = fma(Nwt, xxy, h3[1]);
  h3[2] = fma(Nwt, xyy, h3[2]);
  h3[3] = fma(Nwt, yyy, h3[3]);
  h4[0] = fma(Nwtt, xxxx, h4[0]);
  h4[1] = fma(Nwtt, xxxy, h4[1]);
  h4[2] = fma(Nwtt, xxyy, h4[2]);
  h4[3] = fma(Nwtt, xyyy, h4[3]);
  h4[4] = fma(Nwtt, yyyy, h4[4]);
}

template <typename T, int NEXP, int NDEV>
__device__ __forceinline__ void eval_own_hess(const Table<T>* __restrict__ tb,
                                              const T (*__restrict__ rec)[2 * kMaxProf][kHRec], int K, T px, T py,
                                              const T* box, PixH<T>& o) {
#pragma clang fp contract(off)
  T fe = 0, fd = 0, gme[2] = {0, 0}, gmd[2] = {0, 0}, gse[3] = {0, 0, 0}, gsd[3] = {0, 0, 0};
  T h2[3] = {0, 0, 0}, h3[4] = {0, 0, 0, 0}, h4[5] = {0, 0, 0, 0, 0};
  T f1 = 0, g1x = 0, g1y = 0, h1[3] = {0, 0, 0};
  const T pi = tb->hdr[7], omp = (T)1 - pi;
  for (int k = 0; k < K; ++k) {
    const T mx = tb->star[k][0], my = tb->star[k][1];
    const T dx = px - mx, dy = py - my;
    const T xx = dx * dx, xy = (T)2 * dx * dy, yy = dy * dy;
    const auto d2k = uniform_cut_key(box_dist2<T>(mx, my, box));
    // the cut radii of this PSF component, read before any is used (one wait for all)
    T rc[NEXP + NDEV];
#pragma unroll
    for (int j = 0; j < NEXP + NDEV; ++j) rc[j] = tb->rc2[k][j < NEXP ? j : kMaxProf + (j - NEXP)];
    if (!(d2k > cut_key(tb->rc2s[k]))) {
      const T Pxx = tb->star[k][2], Pxy = tb->star[k][3], Pyy = tb->star[k][4];
      const T ux = fma(Pxx, dx, Pxy * dy), uy = fma(Pxy, dx, Pyy * dy);
      const T N = comp_value<T>(tb->sq[k], xx, xy, yy);
      f1 += N;
      g1x = fma(N, ux, g1x);
      g1y = fma(N, uy, g1y);
      h1[0] = fma(N, fma(ux, ux, -Pxx), h1[0]);
      h1[1] = fma(N, fma(ux, uy, -Pxy), h1[1]);
      h1[2] = fma(N, fma(uy, uy, -Pyy), h1[2]);
    }
#pragma unroll
    for (int j = 0; j < NEXP; ++j)
      if (!(d2k > cut_key(rc[j]))) gal_hess<T>(rec[k][j], omp, dx, dy, fe, gme, gse, h2, h3, h4);
#pragma unroll
    for (int j = 0; j < NDEV; ++j)
      if (!(d2k > cut_key(rc[NEXP + j]))) gal_hess<T>(rec[k][kMaxProf + j], pi, dx, dy, fd, gmd, gsd, h2, h3, h4);
  }
  // the orders' scales divided back; the off-diagonal S derivatives count twice
  constexpr double c1 = 1.0 / kExpScale;
  constexpr T s1 = (T)c1, s2 = (T)(c1 * c1), s3 = (T)(c1 * c1 * c1), s4 = (T)(c1 * c1 * c1 * c1);
  o.f1 = f1;
  o.g1[0] = g1x;
  o.g1[1] = g1y;
  o.h1[0] = h1[0];
  o.h1[1] = h1[1];
  o.h1[2] = h1[2];
  o.f0 = fma(pi, fd, omp * fe);
  constexpr T m2[3] = {s2, (T)2 * s2, s2};
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    o.g0[e] = s1 * fma(pi, gmd[e], omp * gme[e]);
    o.h0[zidx(e, 5)] = s1 * (gmd[e] - gme[e]);
  }
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    o.g0[2 + e] = m2[e] * fma(pi, gsd[e], omp * gse[e]);
    o.h0[zidx(2 + e, 5)] = m2[e] * (gsd[e] - gse[e]);
  }
  o.g0[5] = fd - fe;
  o.h0[zidx(0, 0)] = s2 * h2[0];
  o.h0[zidx(0, 1)] = s2 * h2[1];
  o.h0[zidx(1, 1)] = s2 * h2[2];
  o.h0[zidx(0, 2)] = s3 * h3[0];
  o.h0[zidx(0, 3)] = (T)2 * s3 * h3[1];
  o.h0[zidx(0, 4)] = s3 * h3[2];
  o.h0[zidx(1, 2)] = s3 * h3[1];
  o.h0[zidx(1, 3)] = (T)2 * s3 * h3[2];
  o.h0[zidx(1, 4)] = s3 * h3[3];
  o.h0[zidx(2, 2)] = s4 * h4[0];
  o.h0[zidx(2, 3)] = (T)2 * s4 * h4[1];
  o.h0[zidx(2, 4)] = s4 * h4[2];
  o.h0[zidx(3, 3)] = (T)4 * s4 * h4[2];
  o.h0[zidx(3, 4)] = (T)2 * s4 * h4[3];
  o.h0[zidx(4, 4)] = s4 * h4[4];
  o.h0[zidx(5, 5)] = 0;
}

struct HessArgs {
  const DTask* tasks;
  const int32_t* order;
  const DPatch* patches;
  const int32_t* nbr_idx;
  const void* tables;          // variant-0 tables
  const void* xs;
  const void* maps;
  double* hslots;              // [n_tasks][kHSlots]
  const uint8_t* active;
  const int32_t* img_npsf;
  const uint8_t* cur;          // per source: the variant holding its tables (null = 0)
  int64_t variant_stride;
};

// The float form is held to three wavefronts per SIMD (153 VGPRs, nothing spilled; at the two
// wavefronts that 194 VGPRs allowed the kernel stalled on latency).  The double form keeps its
// natural allocation.
// Bound by VALU issue, about 53 slots per galaxy component and pixel (84 when each second
// derivative had its own formula and per-component constants came by scalar loads from the
// table; the records are now formed once per item in LDS): Hessians of 200 sources (3.7e6
// active pixels) 397 -> 250 us per call, a Newton step of 339 sources 964 -> 622 us.
//
// W = 1: one wavefront per work item.  W > 1: that many per item, a pass of 64 pixels each,
// for launches whose items leave the chip idle; as in the pixel kernel they add to the item's
// per-lane sums in turn, in the order of one wavefront, and the products are written out
// fused, so that an item's sums do not depend on the launch's size.  They add to the 79 sums
// where they are, in LDS: carried through the loop over the turns in registers they took 187
// VGPRs (two wavefronts per SIMD) where 126 do (four); 1395 items 71 -> 53 us, 425 items 29 -> 27.
template <typename T, int NEXP, int NDEV, int W>
__global__ __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? (W > 1 ? 4 : 3) : 1))) void k_hess(HessArgs a) {
#pragma clang fp contract(off)
  const int pos = xcd_position((int)blockIdx.x, (int)gridDim.x);
  const int t = a.order ? a.order[pos] : pos;
  const DTask task = a.tasks[t];
  const DPatch P = a.patches[task.patch];
  if (a.active && !a.active[P.src]) return;
  const Table<T>* __restrict__ tb = reinterpret_cast<const Table<T>*>(a.tables) +
                                    (a.cur ? uniform_byte(a.cur, P.src) * a.variant_stride : 0) + task.patch;
  const int K = a.img_npsf[P.img];
  const int lane = threadIdx.x & 63, wave = W > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  // the galaxy components' records, one component per lane
  __shared__ __align__(16) T rec[kMaxPsf][2 * kMaxProf][kHRec];
  static_assert(kMaxPsf * 2 * kMaxProf <= 64, "one component per lane");
  // (W > 1) the item's per-lane sums
  __shared__ T chain[W > 1 ? kPrim + kHQ : 1][64];
  __shared__ double chain_t[W > 1 ? 2 : 1][64];
  if constexpr (W > 1) {
    for (int u = wave; u < kPrim + kHQ; u += W) chain[u][lane] = 0;
    if (wave < 2) chain_t[wave][lane] = 0;
  }
  if (threadIdx.x < K * 2 * kMaxProf) {
    const T* q = &tb->gq[0][0][0] + lane * 8;
    T* r = &rec[0][0][0] + lane * kHRec;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = q[e];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      r[8 + e] = (T)2 * q[4 + e];
      r[11 + e] = (T)3 * q[4 + e];
    }
  }
  __syncthreads();
  const T L0 = tb->hdr[0], L1 = tb->hdr[1], w0 = tb->hdr[2], w1 = tb->hdr[3];
  const T e0 = tb->hdr[8], e1 = tb->hdr[9];
  const T w01 = w0 * w1, aa = w1, oma2 = fma((T)-2, aa, (T)1);
  double tsum = 0, town = 0;
  T G[kPrim], Q[kHQ];
#pragma unroll
  for (int u = 0; u < kPrim; ++u) G[u] = 0;
#pragma unroll
  for (int u = 0; u < kHQ; ++u) Q[u] = 0;
  // what the pixels are added to
  auto Gs = [&](int u) -> T& { return W > 1 ? chain[W > 1 ? u : 0][lane] : G[u]; };
  auto Qs = [&](int u) -> T& { return W > 1 ? chain[W > 1 ? kPrim + u : 0][lane] : Q[u]; };
  // this lane's patch-local pixel coordinates, advanced by 64 W pixels per pass with a carry
  constexpr int step = 64 * W;
  const int step_rows = step / P.w, step_cols = step - step_rows * P.w;
  int row = (task.pix_begin + (int)threadIdx.x) / P.w;
  int col = task.pix_begin + (int)threadIdx.x - row * P.w;
  for (int pass = task.pix_begin; pass < task.pix_end; pass += step) {
    const int base = pass + wave * 64;
    const bool any = W == 1 || base < task.pix_end;
    int idx = base + lane;
    const bool valid = idx < task.pix_end;
    if (!valid) idx = task.pix_begin;
    T xv, sky;
    if constexpr (sizeof(T) == 8) {
      const double2 xs = reinterpret_cast<const double2*>(a.xs)[P.off + idx];
      xv = xs.x; sky = xs.y;
    } else {
      const float2 xs = reinterpret_cast<const float2*>(a.xs)[P.off + idx];
      xv = xs.x; sky = xs.y;
    }
    int ibox[4];
    run_box<int>(base, max(min(base + 64, task.pix_end), base + 1), P.w, ibox);
    const T box[4] = {(T)ibox[0], (T)ibox[1], (T)ibox[2], (T)ibox[3]};
    PixH<T> o;
    if (W == 1) __builtin_assume(K >= 1);   // images have 1..kMaxPsf PSF components (checked at prepare)
    eval_own_hess<T, NEXP, NDEV>(tb, rec, any ? K : 0, (T)col, (T)row, box, o);
    T Eb = sky, Vb = 0;
    bool own = true;
    for (int nb = P.nbr_begin; nb < (any ? P.nbr_end : P.nbr_begin); ++nb) {
      const DPatch Qp = a.patches[a.nbr_idx[nb]];
      const int ox = P.x0 - Qp.x0, oy = P.y0 - Qp.y0;
      // a neighbour whose rectangle misses this pass's pixel box is skipped as a whole
      if (ibox[0] + ox >= Qp.w || ibox[1] + ox < 0 || ibox[2] + oy >= Qp.h || ibox[3] + oy < 0) continue;
      const int cx = col + ox, cy = row + oy;
      if (valid && (unsigned)cx < (unsigned)Qp.w && (unsigned)cy < (unsigned)Qp.h) {
        const int64_t at = Qp.off + (cy * Qp.w + cx);
        if constexpr (sizeof(T) == 8) {
          const double2 ev = reinterpret_cast<const double2*>(a.maps)[at];
          Eb += ev.x; Vb += ev.y;
        } else {
          const float2 ev = reinterpret_cast<const float2*>(a.maps)[at];
          Eb += ev.x; Vb += ev.y;
        }
        if (Qp.src < P.src) own = false;
      }
    }
    auto add_pixels = [&] {
      const T f0 = o.f0, f1 = o.f1;
      const T a0 = L0 * f0, a1 = L1 * f1, d = a0 - a1;
      const T Es = fma(w0, a0, w1 * a1);
      const T k0 = w0 * L0 * L0 * e0, k1 = w1 * L1 * L1 * e1;
      const T Vs = fma(k0 * f0, f0, fma(k1 * f1, f1, w01 * d * d));
      const T E = Eb + Es, V = Vb + Vs, x = xv;
      const T invE = frcp<T>(E);
      const T xr = x * invE * invE;
      T Tm = fma((T)-0.5 * xr, V, (x > (T)0 ? x_log_ratio<T>(x, E) : (T)0) - (E - x));
      T cE = fma(xr * invE, V, (x - E) * invE);
      T cV = (T)-0.5 * xr;
      T TEE = -fma((T)3 * xr * V * invE, invE, xr);
      T TEV = xr * invE;
      if (!valid) Tm = cE = cV = TEE = TEV = 0;
      double &t_sum = W > 1 ? chain_t[0][lane] : tsum, &t_own = W > 1 ? chain_t[W > 1][lane] : town;
      t_sum += (double)Tm;
      t_own += own ? (double)Tm : 0.0;
      // The z-derivatives of E_s and V_s are the vectors g0 and g1 (g1 and h1 vanish outside the
      // centre coordinates z < 2) with weights fixed per pixel, and so is everything built of
      // them:
      //   E_z = al0 g0 + al1 g1,  V_z = be0 g0 + be1 g1,  d_z = L0 g0 - L1 g1,
      //   al_i = w_i L_i,  be0 = 2 (k0 f0 + w01 d L0),  be1 = 2 (k1 f1 - w01 d L1).
      // T_EE E_u E_v + T_EV (E_u V_v + V_u E_v) = E_u a_v + c_u E_v with a = T_EE E + T_EV V,
      // c = T_EV V; a_z = A0 g0 + A1 g1, c_z = C0 g0 + C1 g1.
      const T cV2 = (T)2 * cV;
      const T ea0 = e0 * a0, ea1 = e1 * a1, w01d = w01 * d;
      const T al0 = w0 * L0, al1 = w1 * L1;
      const T be0 = (T)2 * fma(k0, f0, w01d * L0), be1 = (T)2 * fma(k1, f1, -(w01d * L1));
      const T A0 = fma(TEE, al0, TEV * be0), A1 = fma(TEE, al1, TEV * be1), C0 = TEV * be0, C1 = TEV * be1;
      // the (z, z) block: with E_zz = w0 L0 h0 + w1 L1 h1 and
      //   V_zz = 2 (k0 (g0 g0^T + f0 h0) + k1 (g1 g1^T + f1 h1) + w01 (d_z d_z^T + d (L0 h0 - L1 h1))),
      // c_E E_zz + c_V V_zz = rho0 h0 + rho1 h1 + 2 c_V (k0 g0 g0^T + k1 g1 g1^T + w01 d_z d_z^T),
      // rho_i = c_E al_i + c_V be_i; altogether
      //   rho0 h0 + rho1 h1 + s00 g0 g0^T + s01 (g0 g1^T + g1 g0^T) + s11 g1 g1^T
      const T rho0 = fma(cE, al0, cV * be0), rho1 = fma(cE, al1, cV * be1);
      const T s00 = fma(cV2, fma(w01 * L0, L0, k0), al0 * (A0 + C0));
      const T s11 = fma(cV2, fma(w01 * L1, L1, k1), al1 * (A1 + C1));
      const T s01 = fma(-cV2, w01 * L0 * L1, fma(C0, al1, al0 * A1));
      T Pz[6], Rz[2];
#pragma unroll
      for (int i = 0; i < 6; ++i) Pz[i] = s00 * o.g0[i];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        Pz[i] = fma(s01, o.g1[i], Pz[i]);
        Rz[i] = fma(s01, o.g0[i], s11 * o.g1[i]);
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) {
#pragma unroll
        for (int j = i; j < 6; ++j) {
          T q = Qs(qidx(5 + i, 5 + j));
          q = fma(rho0, o.h0[zidx(i, j)], q);
          q = fma(Pz[i], o.g0[j], q);
          if (i < 2 && j < 2) {
            q = fma(rho1, o.h1[i + j], q);
            q = fma(Rz[i], o.g1[j], q);
          }
          Qs(qidx(5 + i, 5 + j)) = q;
        }
      }
      // the amplitude coordinates u < 5 (E_u vanishes in the two variances u = 3, 4)
      const T Eu[3] = {-d, w0 * f0, w1 * f1};
      const T Vu[5] = {fma(oma2 * d, d, fma(ea1, a1, -(ea0 * a0))), (T)2 * fma(w0 * ea0, f0, w01d * f0),
                       (T)2 * fma(w1 * ea1, f1, -(w01d * f1)), w0 * a0 * a0, w1 * a1 * a1};
      T av[5], cu[5];
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        Gs(u) = fma(cV, Vu[u], Gs(u));
        cu[u] = TEV * Vu[u];
        av[u] = cu[u];
        if (u < 3) {
          Gs(u) = fma(cE, Eu[u], Gs(u));
          av[u] = fma(TEE, Eu[u], cu[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 5; ++u) {
#pragma unroll
        for (int v = u; v < 5; ++v) {
          T q = Qs(qidx(u, v));
          if (v < 3) q = fma(cu[u], Eu[v], q);
          if (u < 3) q = fma(Eu[u], av[v], q);
          Qs(qidx(u, v)) = q;
        }
      }
      // second derivatives of E_s and V_s
      auto add = [&](int u, int v, T x, T y) { Qs(qidx(u, v)) = fma(x, y, Qs(qidx(u, v))); };
      const T f00 = f0 * f0, f11 = f1 * f1;
      add(0, 0, cV2, -(d * d));
      add(0, 1, cE, -f0);
      add(0, 1, cV2, fma(oma2 * d, f0, -(ea0 * f0)));
      add(0, 2, cE, f1);
      add(0, 2, cV2, fma(-(oma2 * d), f1, ea1 * f1));
      add(0, 3, cV, -(a0 * a0));
      add(0, 4, cV, a1 * a1);
      add(1, 1, cV2, fma(w0, e0, w01) * f00);
      add(1, 2, cV2, -(w01 * f0 * f1));
      add(1, 3, cV2, w0 * a0 * f0);
      add(2, 2, cV2, fma(w1, e1, w01) * f11);
      add(2, 4, cV2, w1 * a1 * f1);
      // the (amplitude, z) pairs: E_u a_z + c_u E_z and the second derivatives
      //   c_E (-d_z) + c_V (-2 L0^2 e0 f0 g0 + 2 L1^2 e1 f1 g1 + 2 (1 - 2a) d d_z)      (u = 0)
      //   c_E w0 g0 + c_V (4 w0 L0 e0 f0 g0 + 2 w01 (f0 d_z + d g0))                    (u = 1)
      //   c_E w1 g1 + c_V (4 w1 L1 e1 f1 g1 - 2 w01 (f1 d_z + d g1))                    (u = 2)
      //   c_V 2 w0 L0^2 f0 g0 (u = 3),  c_V 2 w1 L1^2 f1 g1 (u = 4)
      // as t0 g0 + t1 g1
      const T c0 = fma(cV2 * oma2, d, -cE), c1 = cV2 * w01 * f0, c2 = -(cV2 * w01 * f1);
      T t0[5], t1[5];
#pragma unroll
      for (int u = 0; u < 5; ++u) {
        t0[u] = cu[u] * al0;
        t1[u] = cu[u] * al1;
        if (u < 3) {
          t0[u] = fma(Eu[u], A0, t0[u]);
          t1[u] = fma(Eu[u], A1, t1[u]);
        }
      }
      t0[0] += fma(c0, L0, -(cV2 * L0 * ea0));
      t1[0] += fma(-c0, L1, cV2 * L1 * ea1);
      t0[1] += fma(c1, L0, fma(cE, w0, cV2 * fma((T)2 * w0, ea0, w01d)));
      t1[1] = fma(-c1, L1, t1[1]);
      t0[2] = fma(c2, L0, t0[2]);
      t1[2] += fma(-c2, L1, fma(cE, w1, cV2 * fma((T)2 * w1, ea1, -w01d)));
      t0[3] = fma(cV2, al0 * a0, t0[3]);
      t1[4] = fma(cV2, al1 * a1, t1[4]);
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        Gs(5 + j) = fma(rho0, o.g0[j], Gs(5 + j));
        if (j < 2) Gs(5 + j) = fma(rho1, o.g1[j], Gs(5 + j));
#pragma unroll
        for (int u = 0; u < 5; ++u) {
          T q = fma(t0[u], o.g0[j], Qs(qidx(u, 5 + j)));
          if (j < 2) q = fma(t1[u], o.g1[j], q);
          Qs(qidx(u, 5 + j)) = q;
        }
      }
    };
    if constexpr (W == 1) {
      add_pixels();
    } else {
      // the wavefronts' turns; every wavefront meets at the barrier after each
      for (int turn = 0; turn < W; ++turn) {
        if (turn == wave) add_pixels();
        __syncthreads();
      }
    }
    col += step_cols;
    row += step_rows;
    if (col >= P.w) {
      col -= P.w;
      row += 1;
    }
  }
  if constexpr (W > 1) {   // one wavefront stores the item's sums
    if (wave != W - 1) return;
#pragma unroll
    for (int u = 0; u < kPrim; ++u) G[u] = chain[u][lane];
#pragma unroll
    for (int u = 0; u < kHQ; ++u) Q[u] = chain[kPrim + u][lane];
    tsum = chain_t[0][lane];
    town = chain_t[1][lane];
  }
  // the slot row's 79 wavefront sums, formed together in two groups (the first 64 of the 77
  // first- and second-order sums, exchanged in the pixel precision at the first step; then
  // the two objective sums with the last 13); the lane holding a sum stores it
  double* out = a.hslots + (int64_t)t * kHSlots;
  constexpr int kGQ = kPrim + kHQ, kA = 64, kB = 2 + kGQ - kA;
  {
    T v[kA];
#pragma unroll
    for (int i = 0; i < kA; ++i) v[i] = i < kPrim ? G[i] : Q[i - kPrim];
    const double sv = wave_sums<kA, 32, T>(v, lane);
    const int sl = wave_sums_slot<kA>(lane);
    if (sl >= 0) out[2 + sl] = sv;
  }
  {
    double v[kB];
    v[0] = tsum;
    v[1] = town;
#pragma unroll
    for (int i = 2; i < kB; ++i) v[i] = (double)Q[kA + i - 2 - kPrim];
    const double sv = wave_sums<kB>(v, lane);
    const int sl = wave_sums_slot<kB>(lane);
    if (sl >= 0) out[sl < 2 ? sl : kA + sl] = sv;
  }
}

// Sigma_s(angle, log r, logit axis) and its first and second derivatives in those three
// coordinates (Section 2.1.2): out d1[t][e], d2[t][t'][e] with e = (xx, xy, yy).
__device__ void sigma_derivs(double ang, double lr, double eta, double d1[3][3], double d2[3][3][3]) {
  const double c = cos(ang), s = sin(ang), r2 = exp(2.0 * lr), rho = sigmoid(eta);
  const double rp = rho * (1.0 - rho), rpp = rp * (1.0 - 2.0 * rho);
  const double sig[3] = {r2 * (c * c + rho * rho * s * s), r2 * (rho * rho - 1.0) * c * s,
                         r2 * (s * s + rho * rho * c * c)};
  const double dt[3] = {2.0 * r2 * c * s * (rho * rho - 1.0), r2 * (rho * rho - 1.0) * (c * c - s * s),
                        -2.0 * r2 * c * s * (rho * rho - 1.0)};
  const double dtt[3] = {2.0 * r2 * (rho * rho - 1.0) * (c * c - s * s), -4.0 * r2 * (rho * rho - 1.0) * c * s,
                         -2.0 * r2 * (rho * rho - 1.0) * (c * c - s * s)};
  const double dr[3] = {2.0 * rho * r2 * s * s, 2.0 * rho * r2 * c * s, 2.0 * rho * r2 * c * c};
  const double drr[3] = {2.0 * r2 * s * s, 2.0 * r2 * c * s, 2.0 * r2 * c * c};
  const double dtr[3] = {4.0 * rho * r2 * c * s, 2.0 * rho * r2 * (c * c - s * s), -4.0 * rho * r2 * c * s};
  for (int e = 0; e < 3; ++e) {
    d1[0][e] = dt[e];
    d1[1][e] = 2.0 * sig[e];
    d1[2][e] = dr[e] * rp;
    d2[0][0][e] = dtt[e];
    d2[1][1][e] = 4.0 * sig[e];
    d2[2][2][e] = drr[e] * rp * rp + dr[e] * rpp;
    d2[0][1][e] = d2[1][0][e] = 2.0 * dt[e];
    d2[1][2][e] = d2[2][1][e] = 2.0 * dr[e] * rp;
    d2[0][2][e] = d2[2][0][e] = dtr[e] * rp;
  }
}

// S = A M A^T for a symmetric M given as (xx, xy, yy)
__device__ __forceinline__ void conj_A(const double A[2][2], const double* m, double* out) {
  const double t00 = A[0][0] * m[0] + A[0][1] * m[1], t01 = A[0][0] * m[1] + A[0][1] * m[2];
  const double t10 = A[1][0] * m[0] + A[1][1] * m[1], t11 = A[1][0] * m[1] + A[1][1] * m[2];
  out[0] = t00 * A[0][0] + t01 * A[0][1];
  out[1] = t00 * A[1][0] + t01 * A[1][1];
  out[2] = t10 * A[1][0] + t11 * A[1][1];
}

struct HessFinArgs {
  const int32_t* job_src;
  int32_t n_jobs;
  const uint8_t* active;
  const double* theta;
  const double* hslots;
  const int32_t* patch_ptr;
  const DPatch* patches;
  const double* pix_const;
  const cel_image* images;
  const DPrior* prior;
  double* local;               // [S]
  double* grad;                // [S][32]
  double* hess;                // [S][27][27]
  int32_t* err;                // device condition word (non-finite Hessian entries)
};

// Sparsity of J = dr/dtheta (r: the 11 primitive coordinates, theta: the 27 parameters):
// column k has jcount(k) nonzero rows jrow(k, e) -- the centre rows for the position, the
// flux rows m_i / v_i for the flux and colour parameters, the three S rows for the angle,
// radius and axis, and one row each for the type and profile logits.
__device__ __forceinline__ int jcount(int k) { return k < 2 ? 2 : (k == 23 || k == 24 || k == 26) ? 3 : 1; }
__device__ __forceinline__ int jrow(int k, int e) {
  if (k < 2) return 5 + e;
  if (k == 2) return 0;
  if (k < 5) return 1 + 2 * (k - 3);
  if (k < 7) return 2 + 2 * (k - 5);
  if (k < 15) return 1 + 2 * ((k - 7) / 4);
  if (k < 23) return 2 + 2 * ((k - 15) / 4);
  if (k == 25) return 10;
  return 7 + e;
}

// k_hess_finalize: a source's Hessian, gradient and local objective from its work items' sums,
// one workgroup per source.  Its time is the latency of dependent FP64 chains, so the
// independent parts run on wavefronts of their own: kHParts of them take a contiguous share
// of the patches each, one the KL value and gradient, one the KL Hessian; the parts are
// added in LDS in a fixed order.  Per patch H += J^T (Qr J) is formed in two products over
// the at most three nonzero rows of J's columns, upper triangle only (six entries per lane in
// registers).  3 sources of 5 patches: 46 us as two kernels (four part wavefronts, then the
// parts' sum with the KL terms), 13 us here; 200 sources 57 / 14.7; 339 of 10 patches 61 / 36.
constexpr int kHParts = 8;
constexpr int kHWaves = kHParts + 2;
constexpr int kHTri = kN * (kN + 1) / 2;      // 378
constexpr int kHPer = (kHTri + 63) / 64;      // per lane
constexpr int kHU = 2 + kPrim + kHQ;

// entry e of the upper triangle of a kN x kN matrix, row by row
__device__ __forceinline__ void tri_entry(int e, int& i, int& k) {
  const float b = 2 * kN + 1;
  i = (int)((b - sqrtf(b * b - 8.0f * (float)e)) * 0.5f);
  i = min(max(i, 0), kN - 1);
  if (i * (2 * kN + 1 - i) / 2 > e) --i;
  else if ((i + 1) * (2 * kN - i) / 2 <= e) ++i;
  k = e - i * (2 * kN + 1 - i) / 2 + i;
}

struct HessPartLds {
  // (once its patches are done: the part's Hessian, gradient and local objective)
  double sm[kHU], Lf[2], ev[2];   // a patch's sums and flux moments
  double Qr[kPrim][kPrim], Gr[kPrim], QJ[kPrim][kN];
  // column k of dr/dtheta: rows jr[k][e] with values jv[k][e] (zero past jcount(k)); dg the
  // diagonal and sblk the S-block second-derivative terms
  double jv[kN][3], dg[kN], sblk[3][3];
  int jr[kN][3];
  double th[kN], sd1[3][3], sd2[3][3][3];
  double rv[2], cvv[2][4];
};
static_assert(sizeof(HessPartLds) >= (kHTri + kN + 1) * sizeof(double), "a part's sums fit over its work arrays");

__global__ __launch_bounds__(64 * kHWaves) void k_hess_finalize(HessFinArgs a) {
  const int s = a.job_src ? a.job_src[blockIdx.x] : (int)blockIdx.x;
  if (a.active && !a.active[s]) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __shared__ HessPartLds part_lds[kHParts];
  auto part = [&](int q) { return reinterpret_cast<double*>(&part_lds[q]); };
  __shared__ double Hk[kN][kLd], klg[kN + 1];        // minus the KL's Hessian and gradient; its value
  const double* theta = a.theta + (int64_t)s * kThetaN;
  if (w == kHParts) {
    double thr[kThetaN], gk[kThetaN];
#pragma unroll
    for (int k = 0; k < kThetaN; ++k) {
      thr[k] = theta[k];
      gk[k] = 0.0;
    }
    // (every lane: gk = -grad KL)
    const double kv = kl_source_wave(*a.prior, thr, source_exps(thr, lane), gk, 1.0, lane);
    if (lane == 0) {
      klg[kN] = kv;
#pragma unroll
      for (int k = 0; k < kN; ++k) klg[k] = gk[k];
    }
  } else if (w == kHParts + 1) {
    __shared__ double klw[16][kKlw], kls[2][kKlw];
    double thr[kThetaN];
#pragma unroll
    for (int k = 0; k < kThetaN; ++k) thr[k] = theta[k];
    for (int idx = lane; idx < kN * kN; idx += 64) Hk[idx / kN][idx % kN] = 0.0;
    wave_lds_sync();
    kl_hessian_wave<kLd>(*a.prior, thr, Hk, -1.0, lane, klw, kls);
  } else {
    HessPartLds& m = part_lds[w];
    if (lane < kN) m.th[lane] = theta[lane];
    wave_lds_sync();
    if (lane == 0) sigma_derivs(m.th[23], m.th[24], m.th[26], m.sd1, m.sd2);
    if (lane < kN) {
#pragma unroll
      for (int e = 0; e < 3; ++e) m.jr[lane][e] = e < jcount(lane) ? jrow(lane, e) : jrow(lane, 0);
    }
    // flux and colour variances, one per lane
    if (lane >= 1 && lane < 11) {
      const int l = lane - 1;
      const double e = exp(l < 2 ? m.th[5 + l] : m.th[15 + (l - 2)]);
      if (l < 2) m.rv[l] = e;
      else m.cvv[(l - 2) / 4][(l - 2) % 4] = e;
    }
    wave_lds_sync();
    // this lane's Hessian entries (ti, tk) = entry lane + 64 m accumulate in registers
    double hacc[kHPer], gsum = 0.0, local = 0.0;
    int ti[kHPer], tk[kHPer];
#pragma unroll
    for (int q = 0; q < kHPer; ++q) {
      hacc[q] = 0.0;
      tri_entry(min(lane + 64 * q, kHTri - 1), ti[q], tk[q]);
    }
    const double aa = sigmoid(m.th[2]), pi = sigmoid(m.th[25]);
    // this part's patches: a contiguous share of the source's
    const int q0 = a.patch_ptr[s], nq = a.patch_ptr[s + 1] - q0, per = (nq + kHParts - 1) / kHParts;
    const int p0 = q0 + min(nq, w * per), p1 = q0 + min(nq, (w + 1) * per);
    for (int p = p0; p < p1; ++p) {
      {
        const cel_image& im = a.images[a.patches[p].img];
        // the work items' sums, four items' loads at a time
        const int t1 = a.patches[p].task_end;
        double s0 = 0.0, s1 = 0.0;
        for (int t = a.patches[p].task_begin; t < t1; t += 4) {
          double x[4], y[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double* row = a.hslots + (int64_t)min(t + u, t1 - 1) * kHSlots;
            x[u] = row[lane];
            y[u] = row[min(64 + lane, kHU - 1)];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            s0 += t + u < t1 ? x[u] : 0.0;
            s1 += t + u < t1 ? y[u] : 0.0;
          }
        }
        m.sm[lane] = s0;
        if (64 + lane < kHU) m.sm[64 + lane] = s1;
        // flux moments of the patch's band: L_i = iota exp(m_i + v_i / 2) and e_i = exp(v_i),
        // lane 2 w + i
        if (lane < 4) {
          const int i = lane & 1, which = (lane >> 1) & 1;
          double mean = m.th[3 + i], var = m.rv[i];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double W = c_W[im.band][c];
            mean += W * m.th[7 + 4 * i + c];
            var += W * W * m.cvv[i][c];
          }
          const double ex = exp(which == 0 ? mean + 0.5 * var : var);
          if (which == 0) m.Lf[i] = im.iota * ex;
          else m.ev[i] = ex;
        }
        wave_lds_sync();
        const double *sm = m.sm, *Lf = m.Lf, *ev = m.ev;
        local += sm[0] + a.pix_const[2 * p];
        // stage 1: y = (a, L0, L1, e0, e1, z) -> r = (a, m0, v0, m1, v1, z).  Each r is reached
        // from at most two y: a <- a; m_i <- L_i (dL/dm = L); v_i <- L_i (L/2) and e_i (e^v);
        // z <- z.  Qr = Jy^T Qy Jy + sum_u g_u d2y_u/dr2, Gr = Jy^T g.  Written without
        // branches: the second source of an r that has one is given weight 0.
        auto ysrc = [&](int r, int* u, double* j) {
          const bool flux = r >= 1 && r <= 4;
          const int i = (r - 1) >> 1;
          const bool var = flux && ((r & 1) == 0);
          const double L = i ? Lf[1] : Lf[0], e = i ? ev[1] : ev[0];
          u[0] = flux ? 1 + i : r;
          j[0] = flux ? (var ? 0.5 * L : L) : 1.0;
          u[1] = var ? 3 + i : u[0];
          j[1] = var ? e : 0.0;
        };
        for (int idx = lane; idx < kPrim * kPrim; idx += 64) {
          const int r = idx / kPrim, r2 = idx % kPrim;
          int ua[2], ub[2];
          double ja[2], jb[2];
          ysrc(r, ua, ja);
          ysrc(r2, ub, jb);
          double v = 0;
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
              const int u = ua[x], z = ub[y];
              v += ja[x] * sm[2 + kPrim + (u <= z ? qidx(u, z) : qidx(z, u))] * jb[y];
            }
          // second derivatives of y in r: L_i: mm = L, mv = L/2, vv = L/4; e_i: vv = e^v
          if (r >= 1 && r <= 4 && r2 >= 1 && r2 <= 4 && ((r - 1) >> 1) == ((r2 - 1) >> 1)) {
            const int i = (r - 1) >> 1;
            const double gL = sm[3 + i], ge = sm[5 + i];
            const double L = i ? Lf[1] : Lf[0], e = i ? ev[1] : ev[0];
            const int nv = ((r & 1) == 0) + ((r2 & 1) == 0);   // how many of r, r2 are v_i
            v += gL * L * (nv == 0 ? 1.0 : nv == 1 ? 0.5 : 0.25) + (nv == 2 ? ge * e : 0.0);
          }
          m.Qr[r][r2] = v;
        }
        if (lane < kPrim) {
          int ua[2];
          double ja[2];
          ysrc(lane, ua, ja);
          m.Gr[lane] = ja[0] * sm[2 + ua[0]] + ja[1] * sm[2 + ua[1]];
        }
        wave_lds_sync();   // Gr is read below
        // stage 2: the nonzero values of column k of J = dr/dtheta (zero-padded to 3), all
        // candidates formed and one selected
        if (lane < kN) {
          const int k = lane;
          const double A00 = im.A[0][0], A01 = im.A[0][1], A10 = im.A[1][0], A11 = im.A[1][1];
          const int c = (k - 7) & 3, tv = (k - 15) >> 2;
          const double W = c_W[im.band][c];
          const int t = k == 23 ? 0 : k == 24 ? 1 : 2;
          double sv[3];
          conj_A(im.A, m.sd1[t], sv);
          const bool sk = k == 23 || k == 24 || k == 26;
          double v0 = 0.0;
          v0 = k == 0 ? A00 : k == 1 ? A01 : v0;
          v0 = k == 2 ? aa * (1.0 - aa) : v0;
          v0 = (k == 3 || k == 4) ? 1.0 : v0;
          v0 = (k == 5 || k == 6) ? m.rv[k == 6] : v0;
          v0 = (k >= 7 && k < 15) ? W : v0;
          v0 = (k >= 15 && k < 23) ? W * W * m.cvv[tv & 1][c] : v0;
          v0 = k == 25 ? pi * (1.0 - pi) : v0;
          v0 = sk ? sv[0] : v0;
          m.jv[k][0] = v0;
          m.jv[k][1] = k == 0 ? A10 : k == 1 ? A11 : sk ? sv[1] : 0.0;
          m.jv[k][2] = sk ? sv[2] : 0.0;
          // the diagonal second-derivative terms sum_r Gr[r] d2r/dtheta_k^2 (outside the S block)
          double dgk = 0.0;
          dgk = k == 2 ? m.Gr[0] * aa * (1.0 - aa) * (1.0 - 2.0 * aa) : dgk;
          dgk = (k == 5 || k == 6) ? m.Gr[2 + 2 * (k - 5)] * m.rv[k == 6] : dgk;
          dgk = (k >= 15 && k < 23) ? m.Gr[2 + 2 * (tv & 1)] * W * W * m.cvv[tv & 1][c] : dgk;
          dgk = k == 25 ? m.Gr[10] * pi * (1.0 - pi) * (1.0 - 2.0 * pi) : dgk;
          m.dg[k] = dgk;
        }
        // S block (angle, radius, axis): sum_r Gr[r] d2S_r/dt dt'
        if (lane >= 32 && lane < 41) {
          const int si = (lane - 32) / 3, sk = (lane - 32) % 3;
          double sv[3];
          conj_A(im.A, m.sd2[si][sk], sv);
          m.sblk[si][sk] = m.Gr[7] * sv[0] + m.Gr[8] * sv[1] + m.Gr[9] * sv[2];
        }
        wave_lds_sync();
        // QJ = Qr J, then H += J^T QJ + the second-derivative terms (columns zero-padded; the
        // rows of column k are jr[k][e])
        for (int idx = lane; idx < kPrim * kN; idx += 64) {
          const int r = idx / kN, k = idx % kN;
          double v = 0;
#pragma unroll
          for (int y = 0; y < 3; ++y) v += m.Qr[r][m.jr[k][y]] * m.jv[k][y];
          m.QJ[r][k] = v;
        }
        if (lane < kN)
          gsum += m.jv[lane][0] * m.Gr[m.jr[lane][0]] + m.jv[lane][1] * m.Gr[m.jr[lane][1]] +
                  m.jv[lane][2] * m.Gr[m.jr[lane][2]];
        wave_lds_sync();
#pragma unroll
        for (int q6 = 0; q6 < kHPer; ++q6) {
          const int i = ti[q6], k = tk[q6];
          double v = 0;
#pragma unroll
          for (int x = 0; x < 3; ++x) v += m.jv[i][x] * m.QJ[m.jr[i][x]][k];
          if (i == k) v += m.dg[i];
          const int si = i == 23 ? 0 : i == 24 ? 1 : i == 26 ? 2 : -1;
          const int sk = k == 23 ? 0 : k == 24 ? 1 : k == 26 ? 2 : -1;
          if (si >= 0 && sk >= 0) v += m.sblk[si][sk];
          hacc[q6] += v;
        }
        wave_lds_sync();
      }
    }
#pragma unroll
    for (int q = 0; q < kHPer; ++q)
      if (lane + 64 * q < kHTri) part(w)[lane + 64 * q] = hacc[q];
    if (lane < kN) part(w)[kHTri + lane] = gsum;
    if (lane == 0) part(w)[kHTri + kN] = local;   // (every lane holds the same sum)
  }
  __syncthreads();
  bool fin = true;
  for (int e = threadIdx.x; e < kHTri + kN + 1; e += 64 * kHWaves) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kHParts; ++q) v += part(q)[e];
    if (e < kHTri) {
      int i, k;
      tri_entry(e, i, k);
      v += Hk[i][k];
      fin = fin && isfinite(v);
      a.hess[(int64_t)s * kN * kN + i * kN + k] = v;
      a.hess[(int64_t)s * kN * kN + k * kN + i] = v;
    } else if (e < kHTri + kN) {
      a.grad[(int64_t)s * kThetaN + e - kHTri] = v + klg[e - kHTri];
    } else {
      a.local[s] = v - klg[kN];
    }
  }
  if (threadIdx.x >= kN && threadIdx.x < kThetaN) a.grad[(int64_t)s * kThetaN + threadIdx.x] = 0.0;
  if (a.err && !fin) atomicOr(a.err, CEL_DEVERR_NONFINITE_HESSIAN);
}

struct TrArgs {
  const int32_t* job_src;     // sources of this launch
  int32_t n_jobs;
  const uint8_t* active;
  const double* v_grad;       // gradient at the iterate [S][32]
  const double* v_local;      // L_s at the iterate [S]
  const double* hess;         // Hessian of L_s [S][27][27]
  const double* theta;
  const double* radius;
  const double* npix;         // active pixels per source
  double gtol, ftol, radius_min;
  double* theta_trial;        // out [S][32]
  uint8_t* trial_active;      // out: 1 = trial point to evaluate
  double* pred;               // out: predicted gain
  double* pnorm;              // out: |p|
  int32_t* status;            // out: CONVERGED / NONFINITE for sources not tried
  int32_t* err;               // device condition word
};

// Hessian of L_s from central differences of the pixel gradient (variants 1..54 hold the
// gradients at theta_s +/- h e_k), symmetrised, minus the analytic KL Hessian (the tight
// colour-prior mixture makes the KL's higher derivatives too large for differencing).
struct FdHessArgs {
  const int32_t* job_src;
  int32_t n_jobs, S;
  const uint8_t* active;
  const double* v_grad;       // [variants][S][32]
  double fd_step;
  const double* theta;
  const DPrior* prior;
  double* hess;               // out [S][27][27]
};

__global__ __launch_bounds__(64) void k_fd_hessian(FdHessArgs a) {
  const int s = a.job_src ? a.job_src[blockIdx.x] : (int)blockIdx.x;
  if (a.active && !a.active[s]) return;
  const int lane = threadIdx.x;
  __shared__ double H[kN][kLd];
  __shared__ double th[kN];
  const int64_t vs = (int64_t)a.S * kThetaN;
  const double h2 = 2.0 * a.fd_step;
  for (int idx = lane; idx < kN * kN; idx += 64) {
    const int i = idx / kN, k = idx % kN;
    const double hik = (a.v_grad[(int64_t)(1 + k) * vs + (int64_t)s * kThetaN + i] -
                        a.v_grad[(int64_t)(1 + kN + k) * vs + (int64_t)s * kThetaN + i]) / h2;
    const double hki = (a.v_grad[(int64_t)(1 + i) * vs + (int64_t)s * kThetaN + k] -
                        a.v_grad[(int64_t)(1 + kN + i) * vs + (int64_t)s * kThetaN + k]) / h2;
    H[i][k] = 0.5 * (hik + hki);
  }
  if (lane < kN) th[lane] = a.theta[(int64_t)s * kThetaN + lane];
  __syncthreads();
  __shared__ double klw[16][kKlw], kls[2][kKlw];
  kl_hessian_wave<kLd>(*a.prior, th, H, -1.0, lane, klw, kls);
  for (int idx = lane; idx < kN * kN; idx += 64) a.hess[(int64_t)s * kN * kN + idx] = H[idx / kN][idx % kN];
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// (B + D) p = g by an unpivoted L D L^T factorisation of one wavefront, D = lam I with a further
// 1 at decoupled coordinates (`pivot`: this lane's entry): lane c < 27 holds column c in
// registers, a step broadcasts the pivot column by lane reads, and p is p_c in lane c.  Returns
// false (uniformly) when a pivot is not positive: B + D is not positive definite.  Otherwise
// sums: |p|^2, p . w with w = (B + D)^-1 p, and g . p, in every lane, and w itself, like p,
// where |p| is within 1e-7 of the radius.
// Unlike an eigen-decomposition, whose errors are relative to |B|, the factorisation keeps
// the small entries of a badly scaled B (a type logit far from 0) to relative precision.
__device__ __forceinline__ bool ldl_solve(const double (*B)[kLd], double pivot, double g_c, double radius, int lane,
                                          double& p, double& w, double* sums) {
  // The lane's index, made to look new at every step (`x`: a value formed there): comparisons
  // with it are then made where they are used, where 27 masks held in scalar registers would
  // leave the lane reads one register pair, and a wait each.
  auto lane_at = [&](double x) {
    int l = lane;
    asm("" : "+v"(l) : "v"(__double2loint(x)));
    return l;
  };
  const int cc = lane < kN ? lane : 0;
  double A[kN], z = g_c, iown = 0.0;
#pragma unroll
  for (int r = 0; r < kN; ++r) A[r] = B[r][cc] + (r == lane ? pivot : 0.0);
  auto reciprocal = [](double d) {
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    return fma(fma(-d, y, 1.0), y, y);
  };
  double d = read_lane(A[0], 0), inv = reciprocal(d), dmin = d;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const int ln = lane_at(inv);
    const double l = ln > j ? A[j] * inv : 0.0;   // L[c][j] (lanes past 26 repeat column 0's rows)
    iown = ln == j ? inv : iown;
    const double zj = read_lane(z, j);
    if (j + 1 < kN) {   // the next pivot first: its reciprocal is the chain's latency
      A[j + 1] = fma(-read_lane(A[j + 1], j), l, A[j + 1]);
      d = read_lane(A[j + 1], j + 1);
      dmin = fmin(dmin, d);
      inv = reciprocal(d);
    }
    constexpr int kRun = 8;   // lane reads issued together, ahead of the products that wait for them
#pragma unroll
    for (int r0 = j + 2; r0 < kN; r0 += kRun) {
      double v[kRun];
#pragma unroll
      for (int u = 0; u < kRun; ++u)
        if (r0 + u < kN) v[u] = read_lane(A[r0 + u], j);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kRun; ++u)
        if (r0 + u < kN) A[r0 + u] = fma(-v[u], l, A[r0 + u]);
    }
    z = fma(-zj, l, z);
  }
  if (!(dmin > 1e-290)) return false;
  // column c below the diagonal now holds D_c L[r][c], row j of the columns right of it
  // D_j L[c][j]
  p = z * iown;
#pragma unroll
  for (int k = kN - 1; k > 0; --k) {
    const double l = lane_at(p) < k ? A[k] * iown : 0.0;   // L[k][c]
    p = fma(-read_lane(p, k), l, p);
  }
  double q = p;
#pragma unroll
  for (int j = 0; j < kN - 1; ++j) {
    const double l = lane_at(q) > j ? A[j] * read_lane(iown, j) : 0.0;
    q = fma(-read_lane(q, j), l, q);
  }
  const bool own = lane < kN;
  const double v[3] = {own ? p * p : 0.0, own ? q * q * iown : 0.0, own ? z * z * iown : 0.0};
  const double sv = wave_sums<3>(v, lane);
#pragma unroll
  for (int i = 0; i < 3; ++i) sums[i] = read_lane(sv, wave_sums_lane<3>(i));
  w = 0.0;
  if (fabs(sqrt(sums[0]) - radius) <= 1e-7 * radius) {
    w = q * iown;
#pragma unroll
    for (int k = kN - 1; k > 0; --k) {
      const double l = lane_at(w) < k ? A[k] * iown : 0.0;
      w = fma(-read_lane(w, k), l, w);
    }
  }
  return true;
}

// The trust-region subproblem: max g . p - p^T B p / 2 with |p| <= radius, one workgroup of
// kTrWaves wavefronts per source.  Its cost is the latency of a dependent FP64 chain, so the
// wavefronts factorise B + lam I at different multipliers at once (trbracket.h chooses them).
// What this cannot certify -- no root (the hard case), or a step that lies along directions of
// almost no gradient, where the hard case's rule decides -- goes to the eigen-decomposition
// below.  A point with |p| within 1e-7 of the radius is moved onto the boundary along dp/dlam.
// Coordinates that are zero throughout B and g (a type weight of exactly 0 or 1 leaves the other
// type's so) are out of the factorisations, by a unit pivot: B is singular by them alone, and
// without them lam = 0 tells at once whether the step is inside the region, to be completed
// among them by the eigen-decomposition, or on its boundary.
// One factorisation and its solves take 6-7 us (2200 issue slots, a third of them lane
// reads); three to five rounds for most sources.  The eigen-decomposition alone, one
// wavefront: 113 us for 3 sources, 131 us for 339; this: 33 us and 70 us.  Where both are
// needed the rounds come on top: one for a decoupled interior step, four for another singular
// one, at most twelve (78 us) for most others.
//
// Eigen-decomposition (first wavefront): one-sided (Hestenes) Jacobi on
// W = B + c I, c = 1.001 |B|_F (positive definite, so its singular vectors are B's
// eigenvectors and its singular values the shifted eigenvalues).  Lane k holds column k of
// W in registers; in round r of a sweep the lanes pair up by the round-robin (circle)
// schedule -- columns (r + m, r - m) mod 27 for m = 1..13, column r with the zero column 27
// -- exchange columns with one shuffle per entry, and orthogonalise each pair by the
// rotation that diagonalises its 2x2 Gram block.  Sweeps stop when a whole sweep finds
// every pair orthogonal to 1e-15; then lambda_k = |w_k| - c and v_k = w_k / |w_k|.
__global__ __launch_bounds__(64 * kTrWaves) void k_trsolve(TrArgs a) {
  const int s = a.job_src ? a.job_src[blockIdx.x] : (int)blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (a.active && !a.active[s]) {
    if (tid == 0) a.trial_active[s] = 0;
    return;
  }
  __shared__ double B[kN][kLd];
  __shared__ double V[kN][kLd];
  __shared__ double g[kN], lam[kN], y[kN], gt[kN];
  __shared__ int outcome;   // 0 continue, 1 non-finite, 2 converged
  const double L = a.v_local[s];
  const double radius = a.radius[s];
  // B = -H (the Hessian of L_s, pixel and KL parts), symmetrised
  for (int idx = tid; idx < kN * kN; idx += 64 * kTrWaves) {
    const int i = idx / kN, k = idx % kN;
    B[i][k] = -0.5 * (a.hess[(int64_t)s * kN * kN + i * kN + k] + a.hess[(int64_t)s * kN * kN + k * kN + i]);
  }
  if (tid < kN) g[tid] = a.v_grad[(int64_t)s * kThetaN + tid];
  __syncthreads();
  // finiteness and the gradient test (wave reductions: every lane holds the same result)
  double bad = 0.0, gm = 0.0, fro = 0.0;
  for (int idx = lane; idx < kN * kN; idx += 64) {
    const double b = B[idx / kN][idx % kN];
    if (!isfinite(b)) bad = 1.0;
    fro += b * b;
  }
  if (lane < kN) {
    if (!isfinite(g[lane])) bad = 1.0;
    gm = fabs(g[lane]);
  }
  bad = wave_max(bad);
  const double gmax = wave_max(gm);
  fro = wave_sum<double>(fro);
  if (bad != 0.0 || !isfinite(L) || !isfinite(radius)) {
    if (tid == 0) {
      a.status[s] = CEL_ST_NONFINITE;
      a.trial_active[s] = 0;
      if (a.err) atomicOr(a.err, CEL_DEVERR_NONFINITE_STEP);
    }
    return;
  }
  if (gmax <= a.gtol * fmax(1.0, fabs(L) / fmax(a.npix[s], 1.0)) || radius < a.radius_min) {
    if (tid == 0) {
      a.status[s] = CEL_ST_CONVERGED;
      a.trial_active[s] = 0;
    }
    return;
  }
  {
    __shared__ double res[2][kTrWaves][3];   // a wavefront's |p| (-1: not positive definite), Newton point, multiplier
    const double g_c = lane < kN ? g[lane] : 0.0;
    const double gnorm = sqrt(wave_sum<double>(g_c * g_c));
    // Gershgorin's discs and the diagonal bound B's least eigenvalue
    double low = 0.0, dia = 0.0;
    bool dec = false;   // this lane's coordinate is zero throughout
    if (lane < kN) {
      double off = 0.0;
      for (int r = 0; r < kN; ++r) off += r == lane ? 0.0 : fabs(B[r][lane]);
      low = fmax(off - B[lane][lane], 0.0);
      dia = fmax(-B[lane][lane], 0.0);
      dec = off == 0.0 && B[lane][lane] == 0.0 && g_c == 0.0;
    }
    TrBracket br;
    br.start(wave_max(dia), wave_max(low), gnorm, radius, __any(dec));
    double lam = br.first(wave);
    int winner = TrBracket::kMore;
    for (int round = 0; round < kTrRounds && winner == TrBracket::kMore; ++round) {
      double p, w, sums[3], np = -1.0, newton = 0.0;
      if (ldl_solve(B, lam + (dec ? 1.0 : 0.0), g_c, radius, lane, p, w, sums)) {
        np = sqrt(sums[0]);
        newton = lam + (sums[0] / sums[1]) * (np - radius) / radius;
      }
      double(*rs)[3] = res[round & 1];
      if (lane == 0) {
        rs[wave][0] = np;
        rs[wave][1] = newton;
        rs[wave][2] = lam;
      }
      __syncthreads();
      // every thread draws the same conclusions from the wavefronts' results
      winner = br.take(round, rs);
      if (winner == wave) {
        // the step, its predicted gain g.p - p^T B p / 2 (B p = g - lam p) and norm
        const bool edge = lam > 0.0 || np > radius;
        const bool ok = !edge || sums[0] / sums[1] > 1e-6 * gnorm / radius;
        // onto the boundary along dp/dlam = -w, which leaves an error of the second order in
        // |p| / radius - 1 (and takes up the rounding of |p| near the pole)
        const double t = edge ? 0.5 * (radius * radius - sums[0]) / sums[1] : 0.0;
        p = fma(t, w, p);
        if (edge) np = radius;
        const double pr = 0.5 * (sums[2] - t * t * sums[1] + lam * np * np);
        const bool go = pr > a.ftol * fmax(1.0, fabs(L));
        if (lane == 0) {
          outcome = ok ? (go ? 0 : 2) : 3;
          if (ok) {
            a.pred[s] = pr;
            a.pnorm[s] = np;
            if (!go) a.status[s] = CEL_ST_CONVERGED;
            a.trial_active[s] = go ? 1 : 0;
          }
        }
        if (ok && go && lane < kThetaN)
          a.theta_trial[(int64_t)s * kThetaN + lane] = a.theta[(int64_t)s * kThetaN + lane] + (lane < kN ? p : 0.0);
      }
      lam = br.next(wave);
    }
    __syncthreads();
    if (winner >= 0 && outcome != 3) return;
  }
  if (wave != 0) return;
  const double cs = sqrt(fro) * 1.001 + 1e-300;
  // Lane 32 h + c holds rows 14 h .. 14 h + 13 of column c (c < 27; column 27 is the idle
  // partner of the odd-size round-robin), so a round exchanges and rotates 14 entries per
  // lane; sums over a column add the two halves (lanes c and c + 32).
  constexpr int kH = (kN + 1) / 2;
  const int half = lane >> 5, col = lane & 31;
  auto hsum = [&](double v) { return v + __shfl_xor(v, 32, 64); };
  double w[kH];
#pragma unroll
  for (int i = 0; i < kH; ++i) {
    const int row = half * kH + i;
    w[i] = (col < kN && row < kN) ? B[row][col] + (row == col ? cs : 0.0) : 0.0;
  }
  for (int sweep = 0; sweep < 40; ++sweep) {
    double rotated = 0.0;
    // squared column norm, exact at the start of a sweep and carried through its rotations
    // (|c w + cp pw|^2 = c^2 al + cp^2 be + 2 c cp ga)
    double al;
    {
      double a0 = 0.0, a1 = 0.0;
#pragma unroll
      for (int i = 0; i < kH; i += 2) {
        a0 = fma(w[i], w[i], a0);
        a1 = fma(w[i + 1], w[i + 1], a1);
      }
      al = hsum(a0 + a1);
    }
    for (int r = 0; r < kN; ++r) {
      const int pc = col > kN ? col : col == kN ? r : col == r ? kN : ((2 * r - col) % kN + kN) % kN;
      const int pt = half * 32 + pc;
      double pw[kH];
      const double be = __shfl(al, pt, 64);
#pragma unroll
      for (int i = 0; i < kH; ++i) pw[i] = __shfl(w[i], pt, 64);
      double g0 = 0.0, g1 = 0.0;   // two chains for the dot product
#pragma unroll
      for (int i = 0; i < kH; i += 2) {
        g0 = fma(w[i], pw[i], g0);
        g1 = fma(w[i + 1], pw[i + 1], g1);
      }
      const double ga = hsum(g0 + g1);
      const bool lowside = col < pc;
      const double alo = lowside ? al : be, ahi = lowside ? be : al;
      double c = 1.0, sn = 0.0;
      // the pair is rotated unless orthogonal to 1e-15 of its norms' product
      // (|ga| > 1e-15 sqrt(alo ahi), compared squared)
      if (ga * ga > 1e-30 * (alo * ahi)) {
        // t = tan of the rotation angle, the root of smaller magnitude of t^2 + 2 zeta t - 1 = 0
        // with zeta = (ahi - alo) / (2 ga), written without zeta: with d = ahi - alo,
        // t = sign(d) 2 ga / (|d| + sqrt(d^2 + 4 ga^2)) (d = 0: t = sign(ga), both roots of
        // size 1 annihilate the pair); c = 1 / sqrt(1 + t^2), |t| <= 1
        const double d = ahi - alo;
        const double r = sqrt(fma(d, d, 4.0 * ga * ga));
        const double t = (d >= 0.0 ? 2.0 * ga : -2.0 * ga) / (fabs(d) + r);
        c = rsqrt(fma(t, t, 1.0));
        sn = c * t;
        rotated = 1.0;
      }
      const double cp = lowside ? -sn : sn;
#pragma unroll
      for (int i = 0; i < kH; ++i) w[i] = fma(c, w[i], cp * pw[i]);
      al = c * c * al + cp * cp * be + 2.0 * c * cp * ga;
    }
    if (wave_max(rotated) == 0.0) break;
  }
  {
    double nn = 0.0;
#pragma unroll
    for (int i = 0; i < kH; ++i) nn = fma(w[i], w[i], nn);
    const double sig = sqrt(hsum(nn)), inv = 1.0 / sig;
    double acc = 0.0;   // gt = V^T g
#pragma unroll
    for (int i = 0; i < kH; ++i) {
      const int row = half * kH + i;
      if (col < kN && row < kN) {
        const double v = w[i] * inv;
        V[row][col] = v;
        acc = fma(v, g[row], acc);
      }
    }
    acc = hsum(acc);
    if (col < kN && half == 0) {
      lam[col] = sig - cs;
      gt[col] = acc;
    }
  }
  wave_lds_sync();
  bool go = false;
  {
  // the trust-region subproblem in the eigenbasis; scalar logic runs identically on every
  // lane, sums over the 27 eigenvalues are wave reductions
  const bool own = lane < kN;
  const double lam_l = own ? lam[lane] : 0.0, gt_l = own ? gt[lane] : 0.0;
  const double gnorm = sqrt(wave_sum<double>(own ? g[lane] * g[lane] : 0.0));
  double lmin = lam[0];
  int imin = 0;
  for (int i = 1; i < kN; ++i)
    if (lam[i] < lmin) {
      lmin = lam[i];
      imin = i;
    }
  const bool low_l = own && fabs(lam_l - lmin) <= 1e-12 * fmax(1.0, fabs(lmin));
  // shifted eigenvalues d_i = lam_i + lo >= 0 (exact zero at the lowest): the multiplier is
  // lo + mu, and |p|^2 = sum gt_i^2 / (d_i + mu)^2 keeps its precision near the pole
  const double lo = fmax(0.0, -lmin);
  const double dl = own ? lam_l + lo : 0.0;
  auto norm_mu = [&](double m) {
    const double v = own ? gt_l / (dl + m) : 0.0;
    return sqrt(wave_sum<double>(v * v));
  };
  double mu = -1.0;   // chosen shifted multiplier (< 0: not yet found)
  bool hard = false;
  if (lmin > 0 && norm_mu(0.0) <= radius) mu = 0.0;
  double tau_hard = 0.0;
  if (mu < 0) {
    const double notorth = wave_max((low_l && fabs(gt_l) > 1e-12 * fmax(gnorm, 1e-300)) ? 1.0 : 0.0);
    if (notorth == 0.0) {
      const double v = (own && !low_l) ? gt_l / dl : 0.0;
      const double nr = wave_sum<double>(v * v);
      if (sqrt(nr) <= radius) {
        hard = true;
        mu = 0.0;
        tau_hard = sqrt(fmax(radius * radius - nr, 0.0));
      }
    }
  }
  if (mu < 0) {
    // boundary multiplier: |p| = radius for mu in (0, inf).  Safeguarded Newton on
    // 1/radius - 1/|p|, convex and decreasing in mu (Nocedal & Wright, Algorithm 4.3, in
    // the eigenbasis: |q|^2 = sum gt_i^2 / (d_i + mu)^3), inside a bracket [aa, bb] with
    // |p(aa)| > radius >= |p(bb)|, bisecting when a step leaves it; 4-13 steps to
    // |p| = radius (1 + O(eps)).
    double hi = gnorm / radius + 1.0;
    while (norm_mu(hi) > radius) hi *= 2.0;
    double aa = 0.0, bb = hi;
    const double glow = wave_max(low_l ? fabs(gt_l) : 0.0);
    double mc = lmin > 0 ? 0.0 : 0.5 * glow / radius;   // left of the root
    if (!(mc >= aa && mc < bb) || (lmin <= 0 && !(mc > 0.0))) mc = 0.5 * (aa + bb);
    for (int it = 0; it < 200 && mu < 0; ++it) {
      const double v = own ? 1.0 / (dl + mc) : 0.0;
      const double pv = gt_l * v;
      const double s1 = wave_sum<double>(pv * pv), s2 = wave_sum<double>(pv * pv * v);
      const double np = sqrt(s1);
      if (np > radius) aa = mc;
      else bb = mc;
      double nx = mc + (s1 / s2) * (np - radius) / radius;
      if (!(nx > aa && nx < bb)) nx = 0.5 * (aa + bb);
      if (fabs(np - radius) <= 4.0 * DBL_EPSILON * radius || nx == mc) mu = mc;   // converged
      else if (bb - aa <= 4.0 * DBL_EPSILON * bb) mu = bb;                        // bracket closed
      mc = nx;
    }
    if (mu < 0) mu = bb;
  }
  // step in the eigenbasis (hard case: completed along the lowest eigenvector, oriented so
  // that its largest-magnitude entry is positive), predicted gain and norm
  double yl = 0.0;
  if (own) yl = (hard && low_l) ? 0.0 : gt_l / (dl + mu);
  if (hard && lane == imin) {
    int am = 0;
    for (int i = 1; i < kN; ++i)
      if (fabs(V[i][imin]) > fabs(V[am][imin])) am = i;
    yl = V[am][imin] < 0 ? -tau_hard : tau_hard;
  }
  const double gp = wave_sum<double>(gt_l * yl), pBp = wave_sum<double>(lam_l * yl * yl), nn = wave_sum<double>(yl * yl);
  if (own) y[lane] = yl;
  const double pr = gp - 0.5 * pBp;
  go = pr > a.ftol * fmax(1.0, fabs(L));
  if (lane == 0) {
    a.pred[s] = pr;
    a.pnorm[s] = sqrt(nn);
    if (!go) a.status[s] = CEL_ST_CONVERGED;
    a.trial_active[s] = go ? 1 : 0;
    outcome = go ? 0 : 2;
  }
  }
  wave_lds_sync();
  if (outcome) return;
  if (tid < kThetaN) {
    double v = a.theta[(int64_t)s * kThetaN + tid];
    if (tid < kN) {
      double step = 0;
      for (int i = 0; i < kN; ++i) step += V[tid][i] * y[i];
      v += step;
    }
    a.theta_trial[(int64_t)s * kThetaN + tid] = v;
  }
}

struct AcceptArgs {
  const int32_t* job_src;     // stepped sources (null: source = job); with `skipped` all sources are jobs
  int32_t n_jobs;
  int32_t skipped;            // 1: sources not flagged in active get the skipped status
  uint8_t* active;            // stepped sources (cleared on convergence when clear_done)
  int32_t clear_done;
  const uint8_t* trial_active;
  const double* local0;       // L_s at the iterate
  const double* local_trial;  // L_s at the trial point
  const double* pred;
  const double* pnorm;
  double* theta;
  const double* theta_trial;
  double* radius;
  int32_t* status;
  double* out_local;          // may be null
  double eta, radius_max;
  uint8_t* cur;               // an accepted source's tables are its trial's (may be null)
};

// 32 lanes per source, one of its parameters each (one thread per source copied them one
// after another: 7 us a launch, whatever the number of sources); the skipped sources' status
// in the same launch.
__global__ __launch_bounds__(256) void k_accept(AcceptArgs a) {
  const int jj = blockIdx.x * 8 + (int)(threadIdx.x >> 5), k = threadIdx.x & 31;
  static_assert(kThetaN == 32, "one lane per parameter");
  if (jj >= a.n_jobs) return;
  const int s = a.job_src ? a.job_src[jj] : jj;
  if (!a.active[s]) {
    if (a.skipped && k == 0) {
      a.status[s] = CEL_ST_SKIPPED;
      if (a.out_local) a.out_local[s] = __longlong_as_double(0x7ff8000000000000LL);
    }
    return;
  }
  const double L = a.local0[s], Lt = a.local_trial[s], pn = a.pnorm[s], pred = a.pred[s], radius = a.radius[s];
  const double trial = a.theta_trial[(int64_t)s * kThetaN + k];
  double Lout = L;
  if (a.trial_active[s]) {
    double r = radius;
    int st = CEL_ST_REJECTED;
    if (!isfinite(Lt)) {
      r = 0.25 * pn;
    } else {
      const double rho = (Lt - L) / pred;
      if (rho < 0.25) r = 0.25 * pn;
      else if (rho > 0.75 && pn >= 0.99 * r) r = fmin(2.0 * r, a.radius_max);
      if (rho > a.eta) {
        st = CEL_ST_ACCEPTED;
        a.theta[(int64_t)s * kThetaN + k] = trial;
        Lout = Lt;
      }
    }
    if (k == 0) {
      a.radius[s] = r;
      a.status[s] = st;
      if (a.cur && st == CEL_ST_ACCEPTED) a.cur[s] ^= 1;
    }
  } else if (a.clear_done && k == 0) {
    a.active[s] = 0;   // converged or non-finite: done for this colour class
  }
  if (a.out_local && k == 0) a.out_local[s] = Lout;
}

__global__ __launch_bounds__(256) void k_skipped(const uint8_t* __restrict__ mask, int S, int32_t* status,
                                                 double* out_local) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S || mask[s]) return;
  status[s] = CEL_ST_SKIPPED;
  if (out_local) out_local[s] = __longlong_as_double(0x7ff8000000000000LL);
}

// fills: radius <- r0 for all sources; active <- (colour == c) for one class, its tables in
// variant 0
__global__ __launch_bounds__(256) void k_fill_radius(double* radius, int S, double r0) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s < S) radius[s] = r0;
}
__global__ __launch_bounds__(256) void k_set_active(uint8_t* active, uint8_t* cur, const int32_t* __restrict__ colour,
                                                    int S, int c) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S) return;
  active[s] = colour[s] == c ? 1 : 0;
  cur[s] = 0;
}
__global__ __launch_bounds__(256) void k_count_active(const uint8_t* __restrict__ active, const int32_t* __restrict__ list,
                                                      int n, int32_t* out) {
  __shared__ int sh[256];
  int c = 0;
  for (int i = threadIdx.x; i < n; i += 256) c += active[list[i]];
  sh[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

template <typename T>
static hipError_t launch_hess_t(cel_plan* p, const int32_t* order, int n_items, const uint8_t* active,
                                const uint8_t* cur, hipStream_t sm) {
  if (n_items <= 0) return hipSuccess;
  HessArgs ha;
  std::memset(&ha, 0, sizeof(ha));
  ha.tasks = p->d_tasks;
  ha.order = order;
  ha.patches = p->d_patches;
  ha.nbr_idx = p->d_nbr;
  ha.tables = sizeof(T) == 8 ? (const void*)p->tables_d : (const void*)p->tables_f;
  ha.xs = sizeof(T) == 8 ? (const void*)p->d_xs64 : (const void*)p->d_xs;
  ha.maps = sizeof(T) == 8 ? (const void*)p->d_maps64 : (const void*)p->d_maps;
  ha.hslots = p->d_hslots;
  ha.active = active;
  ha.img_npsf = p->d_npsf;
  ha.cur = cur;
  ha.variant_stride = p->P;
  const bool std_prof = p->nexp == 6 && p->ndev == 8;
  if constexpr (sizeof(T) == 4) {
    const int waves = hessian_waves(item_groups(p, 1), n_items);
    if (waves == 8) {
      if (std_prof) hipLaunchKernelGGL((k_hess<T, 6, 8, 8>), dim3(n_items), dim3(64 * 8), 0, sm, ha);
      else hipLaunchKernelGGL((k_hess<T, 8, 8, 8>), dim3(n_items), dim3(64 * 8), 0, sm, ha);
      return hipGetLastError();
    }
    if (waves == 4) {
      if (std_prof) hipLaunchKernelGGL((k_hess<T, 6, 8, 4>), dim3(n_items), dim3(64 * 4), 0, sm, ha);
      else hipLaunchKernelGGL((k_hess<T, 8, 8, 4>), dim3(n_items), dim3(64 * 4), 0, sm, ha);
      return hipGetLastError();
    }
  }
  if (std_prof) hipLaunchKernelGGL((k_hess<T, 6, 8, 1>), dim3(n_items), dim3(64), 0, sm, ha);
  else hipLaunchKernelGGL((k_hess<T, 8, 8, 1>), dim3(n_items), dim3(64), 0, sm, ha);
  return hipGetLastError();
}

// Analytic per-source Hessians (pixel and KL parts) of the sources flagged in `active` among
// `srcs` (device list, n_src entries; null = 0..S-1), with their gradients and local objectives.
// The base tables and maps must be current.
static hipError_t enqueue_hessian(cel_plan* p, const double* theta, const int32_t* order, int n_items,
                                  const int32_t* srcs, int n_src, const uint8_t* active, double* local,
                                  double* grad, double* hess, hipStream_t sm,
                                  const uint8_t* cur = nullptr) {
  const bool fp64 = p->opt.pixel_fp64 || p->opt.hessian_fp64;
  hipError_t e = fp64 ? launch_hess_t<double>(p, order, n_items, active, cur, sm)
                      : launch_hess_t<float>(p, order, n_items, active, cur, sm);
  if (e != hipSuccess || n_src <= 0) return e;
  HessFinArgs fa;
  std::memset(&fa, 0, sizeof(fa));
  fa.job_src = srcs;
  fa.n_jobs = n_src;
  fa.active = active;
  fa.theta = theta;
  fa.hslots = p->d_hslots;
  fa.patch_ptr = p->d_patch_ptr;
  fa.patches = p->d_patches;
  fa.pix_const = p->d_pixconst;
  fa.images = p->d_images;
  fa.prior = p->d_prior;
  fa.local = local;
  fa.grad = grad;
  fa.hess = hess;
  fa.err = p->d_err;
  hipLaunchKernelGGL(k_hess_finalize, dim3(n_src), dim3(64 * kHWaves), 0, sm, fa);
  return hipGetLastError();
}

// What of the iterate's tables and neighbour moment maps a Newton iteration finds made: nothing
// (the difference Hessian, whose gradient pass makes them); all of them, in variant 0; or, in a
// sweep, the maps (none of the class's neighbours has moved since they were made: once per class)
// and each stepped source's tables in the variant that d_cur names -- the trial's tables go to its
// other variant, and an accepted trial's are the next iterate's, which spares an iteration the
// rebuild (8 us of a small class's 110).
enum class Made { kNothing, kSweep, kAll };

// One Newton iteration of colour class `cls` on the sources flagged in `active`; with
// mark_skipped (all flagged sources are the class's) the others get the skipped status.
static hipError_t enqueue_newton_class(cel_plan* p, double* theta, double* radius, uint8_t* active, int cls,
                                       int32_t* status, double* out_local, bool clear_done, hipStream_t sm,
                                       Made made = Made::kNothing, bool mark_skipped = false) {
  const bool fp64 = p->opt.pixel_fp64 || p->opt.hessian_fp64;
  const int nsrc = (int)p->class_src[cls].size();
  if (nsrc == 0) return hipSuccess;
  hipError_t e;
  uint8_t* cur = made == Made::kSweep ? p->d_cur : nullptr;
  if (!p->opt.hessian_fd) {   // the exact Hessians with the gradients
    e = enqueue_hessian(p, theta, p->d_class_tasks[cls], (int)p->class_tasks[cls].size(), p->d_class_src[cls], nsrc,
                        active, p->v_local, p->v_grad, p->d_hess, sm, cur);
  } else {
    // gradients at the iterate and at the 54 central-difference points, then the Hessians
    e = eval_any(p, theta, nullptr, 0, 2 * kParamN + 1, true, cls, active, sm, true, fp64);
    if (e == hipSuccess) {
      FdHessArgs fa;
      std::memset(&fa, 0, sizeof(fa));
      fa.job_src = p->d_class_src[cls];
      fa.n_jobs = nsrc;
      fa.S = p->S;
      fa.active = active;
      fa.v_grad = p->v_grad;
      fa.fd_step = p->opt.fd_step;
      fa.theta = theta;
      fa.prior = p->d_prior;
      fa.hess = p->d_hess;
      hipLaunchKernelGGL(k_fd_hessian, dim3(nsrc), dim3(64), 0, sm, fa);
      e = hipGetLastError();
    }
  }
  if (e != hipSuccess) return e;
  TrArgs ta;
  std::memset(&ta, 0, sizeof(ta));
  ta.job_src = p->d_class_src[cls];
  ta.n_jobs = nsrc;
  ta.active = active;
  ta.v_grad = p->v_grad;
  ta.v_local = p->v_local;
  ta.hess = p->d_hess;
  ta.theta = theta;
  ta.radius = radius;
  ta.npix = p->d_npix;
  ta.gtol = p->opt.gtol;
  ta.ftol = p->opt.ftol;
  ta.radius_min = p->opt.radius_min;
  ta.theta_trial = p->d_theta_trial;
  ta.trial_active = p->d_trial_active;
  ta.pred = p->d_pred;
  ta.pnorm = p->d_step_norm;
  ta.status = status;
  ta.err = p->d_err;
  hipLaunchKernelGGL(k_trsolve, dim3(nsrc), dim3(64 * kTrWaves), 0, sm, ta);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // objective at the trial points, by the objective's own pixel form, so that an accepted source's
  // L_s is the number that an evaluation at the new iterate gives (exponents from the pixel's
  // monomials instead: 12860 items 76 -> 67 us, but other last bits)
  e = eval_any(p, theta, p->d_theta_trial, p->trial_variant, 1, false, cls, p->d_trial_active, sm, false, fp64, nullptr,
               nullptr, cur);
  if (e != hipSuccess) return e;
  AcceptArgs aa;
  std::memset(&aa, 0, sizeof(aa));
  aa.job_src = mark_skipped ? nullptr : p->d_class_src[cls];
  aa.n_jobs = mark_skipped ? p->S : nsrc;
  aa.skipped = mark_skipped ? 1 : 0;
  aa.active = active;
  aa.clear_done = clear_done ? 1 : 0;
  aa.trial_active = p->d_trial_active;
  aa.local0 = p->v_local;
  aa.local_trial = p->v_local + (int64_t)p->trial_variant * p->S;
  aa.pred = p->d_pred;
  aa.pnorm = p->d_step_norm;
  aa.theta = theta;
  aa.theta_trial = p->d_theta_trial;
  aa.radius = radius;
  aa.status = status;
  aa.out_local = out_local;
  aa.eta = p->opt.eta;
  aa.radius_max = p->opt.radius_max;
  aa.cur = cur;
  hipLaunchKernelGGL(k_accept, dim3((aa.n_jobs + 7) / 8), dim3(256), 0, sm, aa);
  return hipGetLastError();
}

}  // namespace celmi

using namespace celmi;

static cel_status newton_scratch(cel_plan* p) {
  const bool fp64 = p->opt.pixel_fp64 || p->opt.hessian_fp64;
  // analytic Hessian: variants 0 (iterate) and 1 (trial); differences: 0, 1..54, 55 (trial)
  p->fd_mode = p->opt.hessian_fd ? 1 : 0;
  p->trial_variant = p->opt.hessian_fd ? kVariants - 1 : 1;
  cel_status st = ensure_variants(p, p->trial_variant + 1, fp64);
  if (st) return st;
  return ensure_newton(p);
}

extern "C" cel_status cel_newton_step(cel_ctx* ctx, const cel_plan* cplan, double* theta, double* radius,
                                      const uint8_t* mask, int32_t* step_status, double* elbo_local, void* stream) {
  if (!ctx || !cplan) return CEL_EINVAL;
  cel_plan* p = const_cast<cel_plan*>(cplan);
  if (p->S > 0 && (!theta || !radius || !step_status)) return CEL_EINVAL;
  if (hipSetDevice(p->device) != hipSuccess) return CEL_EHIP;
  hipStream_t sm = (hipStream_t)stream;
  // the stepped sources must be pairwise non-overlapping
  std::vector<uint8_t> m(p->S, 1);
  if (mask)
    for (int s = 0; s < p->S; ++s) m[s] = mask[s] ? 1 : 0;
  for (int s = 0; s < p->S; ++s)
    if (m[s])
      for (int t : p->adj[s])
        if (m[t]) return CEL_EINVAL;
  cel_status st = newton_scratch(p);
  if (st) return st;
  if (p->S == 0) return CEL_OK;
  // The stepped sources never overlap one another, so none is a neighbour of another: the
  // tables and neighbour maps made once at the iterate serve all of them, and the sources
  // of several colour classes are stepped as one batch (the step class).
  std::vector<int> used;
  for (int c = 0; c < p->n_colours; ++c) {
    bool any = false;
    for (int s : p->class_src[c]) any = any || m[s];
    if (any) used.push_back(c);
  }
  int cls = used.empty() ? -1 : used[0];
  const bool union_class = used.size() > 1 && !p->opt.hessian_fd;
  if (union_class) cls = p->n_colours;
  hipError_t e = stage_selection(p, m, union_class, sm);
  const bool maps_once = !p->opt.hessian_fd;
  if (maps_once && e == hipSuccess && cls >= 0)
    e = prep_base(p, theta, sm, p->opt.pixel_fp64 || p->opt.hessian_fp64, p->d_mask);
  const bool one = maps_once && cls >= 0;   // one batch holds every stepped source
  if (one) {
    if (e == hipSuccess)
      e = enqueue_newton_class(p, theta, radius, p->d_mask, cls, step_status, elbo_local, false, sm, Made::kAll, true);
  } else {
    for (int c : used) {
      if (e != hipSuccess) break;
      e = enqueue_newton_class(p, theta, radius, p->d_mask, c, step_status, elbo_local, false, sm);
    }
  }
  if (e == hipSuccess && !one) {
    hipLaunchKernelGGL(k_skipped, dim3((p->S + 255) / 256), dim3(256), 0, sm, p->d_mask, p->S, step_status,
                       elbo_local);
    e = hipGetLastError();
  }
  return e == hipSuccess ? CEL_OK : CEL_EHIP;
}

extern "C" cel_status cel_sweep(cel_ctx* ctx, const cel_plan* cplan, double* theta, double* radius, int32_t* status,
                                const cel_sweep_opts* opts, cel_sweep_report* report, void* stream) {
  if (!ctx || !cplan) return CEL_EINVAL;
  cel_plan* p = const_cast<cel_plan*>(cplan);
  if (p->S > 0 && (!theta || !radius || !status)) return CEL_EINVAL;
  cel_sweep_opts o;
  std::memset(&o, 0, sizeof(o));
  o.n_sweeps = 3;
  o.max_newton_iters = 50;
  o.use_graph = 1;
  if (opts) {
    if (opts->n_sweeps < 0 || opts->max_newton_iters < 0 || opts->max_classes < 0 || opts->start_colour < 0 ||
        (opts->start_colour > 0 && opts->start_colour >= cplan->n_colours))
      return CEL_EINVAL;
    o = *opts;
  }
  if (hipSetDevice(p->device) != hipSuccess) return CEL_EHIP;
  hipStream_t sm = (hipStream_t)stream;
  cel_status st = newton_scratch(p);
  if (st) return st;
  // graphs cannot be captured on the null stream: run on the plan's own stream after the
  // caller's prior work, and synchronise before returning (the call is synchronous anyway)
  if (o.use_graph && sm == nullptr) {
    if (hipStreamSynchronize(sm) != hipSuccess) return CEL_EHIP;
    sm = p->own_stream;
  }
  const auto t0 = std::chrono::steady_clock::now();
  int64_t steps = 0;
  hipError_t e = hipSuccess;
  const int S = p->S;
  if (S > 0 && o.start_colour == 0) {   // a fresh pass: every status starts as skipped
    hipLaunchKernelGGL(k_set_active, dim3((S + 255) / 256), dim3(256), 0, sm, p->d_mask, p->d_cur, p->d_colour, S, -1);
    e = hipGetLastError();
    if (e == hipSuccess)
      hipLaunchKernelGGL(k_skipped, dim3((S + 255) / 256), dim3(256), 0, sm, p->d_mask, S, status, nullptr);
  }
  // one captured graph per colour class: a full Newton iteration of the class
  if (o.use_graph && p->graphs.size() != (size_t)p->n_colours) {
    for (auto& g : p->graphs) (void)hipGraphExecDestroy(g.exec);
    p->graphs.assign(p->n_colours, {});
  }
  const int check_every = 4;
  int classes = 0, sweeps_done = 0, next_colour = 0;
  bool stopped = false;
  for (int sw = 0; sw < o.n_sweeps && e == hipSuccess && S > 0 && !stopped; ++sw) {
    const int c0 = sw == 0 ? o.start_colour : 0;
    if (c0 == 0) {   // trust radii restart at each pass
      hipLaunchKernelGGL(k_fill_radius, dim3((S + 255) / 256), dim3(256), 0, sm, radius, S, p->opt.radius0);
      if ((e = hipGetLastError()) != hipSuccess) break;
    }
    for (int c = c0; c < p->n_colours && e == hipSuccess; ++c) {
      if (o.max_classes > 0 && classes == o.max_classes) {
        stopped = true;
        next_colour = c;
        break;
      }
      ++classes;
      const int nsrc = (int)p->class_src[c].size();
      hipLaunchKernelGGL(k_set_active, dim3((S + 255) / 256), dim3(256), 0, sm, p->d_mask, p->d_cur, p->d_colour, S, c);
      if ((e = hipGetLastError()) != hipSuccess) break;
      // the neighbours of this class keep their parameters during its iterations: their
      // moment maps are made once here (analytic Hessian path)
      const bool maps_once = !p->opt.hessian_fd;
      if (maps_once &&
          (e = prep_base(p, theta, sm, p->opt.pixel_fp64 || p->opt.hessian_fp64, p->d_mask)) != hipSuccess)
        break;
      hipGraphExec_t exec = nullptr;
      if (o.use_graph) {
        auto& G = p->graphs[c];
        if (!G.exec || G.theta != theta || G.radius != radius || G.status != status || G.stream != sm) {
          if (G.exec) (void)hipGraphExecDestroy(G.exec);
          G.exec = nullptr;
          hipGraph_t graph;
          e = hipStreamBeginCapture(sm, hipStreamCaptureModeThreadLocal);
          if (e != hipSuccess) break;
          hipError_t e2 = enqueue_newton_class(p, theta, radius, p->d_mask, c, status, nullptr, true, sm,
                                                maps_once ? Made::kSweep : Made::kNothing);
          e = hipStreamEndCapture(sm, &graph);
          if (e2 != hipSuccess) e = e2;
          if (e != hipSuccess) break;
          e = hipGraphInstantiate(&G.exec, graph, nullptr, nullptr, 0);
          (void)hipGraphDestroy(graph);
          if (e != hipSuccess) break;
          G.theta = theta;
          G.radius = radius;
          G.status = status;
          G.stream = sm;
        }
        exec = G.exec;
      }
      for (int it = 0; it < o.max_newton_iters && e == hipSuccess; ++it) {
        if (exec) e = hipGraphLaunch(exec, sm);
        else e = enqueue_newton_class(p, theta, radius, p->d_mask, c, status, nullptr, true, sm,
                                                maps_once ? Made::kSweep : Made::kNothing);
        ++steps;
        if (e != hipSuccess) break;
        if ((it + 1) % check_every == 0 || it + 1 == o.max_newton_iters) {
          hipLaunchKernelGGL(k_count_active, dim3(1), dim3(256), 0, sm, p->d_mask, p->d_class_src[c], nsrc,
                             p->d_counter);
          e = hipMemcpyAsync(p->h_counter, p->d_counter, sizeof(int32_t), hipMemcpyDeviceToHost, sm);
          if (e == hipSuccess) e = hipStreamSynchronize(sm);
          if (e != hipSuccess) break;
          if (*p->h_counter == 0) break;
        }
      }
    }
    if (!stopped && e == hipSuccess) ++sweeps_done;
  }
  if (e == hipSuccess && S > 0) e = launch_total_after_eval(p, theta, sm);
  double tot = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(p->h_total, p->d_total, sizeof(double), hipMemcpyDeviceToHost, sm);
  if (e == hipSuccess) e = hipStreamSynchronize(sm);
  if (e == hipSuccess) tot = S > 0 ? *p->h_total : 0.0;
  if (report) {
    report->elbo_total = tot;
    report->n_colours = p->n_colours;
    report->n_newton_steps = steps;
    report->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    report->sweeps_done = sweeps_done;
    report->next_colour = next_colour;
  }
  return e == hipSuccess ? CEL_OK : CEL_EHIP;
}

extern "C" cel_status cel_elbo_hessian(cel_ctx* ctx, const cel_plan* cplan, const double* theta, const uint8_t* mask,
                                       double* hess, double* grad, double* elbo_local, void* stream) {
  if (!ctx || !cplan) return CEL_EINVAL;
  cel_plan* p = const_cast<cel_plan*>(cplan);
  if (p->S > 0 && (!theta || !hess)) return CEL_EINVAL;
  if (hipSetDevice(p->device) != hipSuccess) return CEL_EHIP;
  hipStream_t sm = (hipStream_t)stream;
  cel_status st = newton_scratch(p);
  if (st) return st;
  if (p->S == 0) return CEL_OK;
  const bool fp64 = p->opt.pixel_fp64 || p->opt.hessian_fp64;
  if (hipEventSynchronize(p->mask_copied) != hipSuccess) return CEL_EHIP;
  for (int s = 0; s < p->S; ++s) p->h_mask[s] = mask ? (mask[s] ? 1 : 0) : 1;
  hipError_t e = hipMemcpyAsync(p->d_mask, p->h_mask, p->S, hipMemcpyHostToDevice, sm);
  if (e == hipSuccess) e = hipEventRecord(p->mask_copied, sm);
  if (e == hipSuccess) e = prep_base(p, theta, sm, fp64);
  if (e == hipSuccess)
    e = enqueue_hessian(p, theta, p->d_order, (int)p->n_tasks, nullptr, p->S, p->d_mask,
                        elbo_local ? elbo_local : p->v_local, grad ? grad : p->v_grad, hess, sm);
  return e == hipSuccess ? CEL_OK : CEL_EHIP;
}
