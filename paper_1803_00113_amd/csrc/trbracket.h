// The search for the trust-region multiplier: max g . p - p^T B p / 2 with |p| <= radius by
// trial multipliers lam, kTrWaves at a time, of which only |p(lam)| and its slope are known
// (p = (B + lam I)^-1 g; nothing where B + lam I is not positive definite).
//
// lam = 0 is the solution if B is positive definite and |p| <= radius; else |p(lam)| = radius,
// and with psi(lam) = 1/|p(lam)| increasing, concave and nearly linear right of the pole, the
// Newton points of psi = 1/radius lie left of the root (Nocedal & Wright, Algorithm 4.3) and
// the secant through a point on either side right of it: together they bracket it ever more
// tightly.  The next multipliers are both of them, the cubic lam(psi) through the two points'
// values and slopes, and a point in the bracket's larger part.
//
// Plain arithmetic without a device function, so that it runs on the host as well.
#pragma once
#include <float.h>
#include <math.h>

#ifdef __HIPCC__
#define CEL_HD __host__ __device__ __forceinline__
#else
#define CEL_HD inline
#endif

namespace celmi {

constexpr int kTrWaves = 4;   // multipliers per round
// The search is given up after kTrBlind rounds that have found nothing positive definite left of
// the root, and after kTrRounds in any case.  With almost no gradient along the least eigenvalue's
// direction it halves its way to the pole for 10 to 40 rounds, when the eigen-decomposition (17
// rounds' time) is the cheaper.  Of 16000 steps of survey and field workloads 0.04 % found that
// point after more than 8 rounds, the last in the 10th; nine in ten ended within 5 rounds, all
// within 12.
constexpr int kTrBlind = 12, kTrRounds = 16;

struct TrBracket {
  enum { kMore = -1, kNone = -2 };
  double radius, scale;   // scale = |g| / radius
  bool zero, decoupled;
  // lo: not right of the root, hi: not left of it; near and far: the best Newton and secant
  // points; the closest points of each side with known norms (0: none) and their Newton points
  double lo, hi, near, far, ll, nl, tl, nr, tr;
  double mid;             // the cubic's multiplier

  // below: the diagonal bounds the least eigenvalue from above by -below; disc: Gershgorin's
  // discs bound it from below by -disc (both >= 0).  dec: coordinates of B and g that are zero
  // throughout were left out of the norms (a unit pivot put in their place).
  CEL_HD void start(double below, double disc, double gnorm, double r, bool dec) {
    radius = r;
    scale = gnorm / r;
    decoupled = dec;
    lo = below;
    hi = 1.001 * (scale + disc);   // |p(lam)| <= |g| / (lam + least eigenvalue)
    near = lo;
    far = hi;
    ll = nl = tl = nr = tr = mid = 0.0;
    zero = lo == 0.0;
  }

  // the first multipliers: 0 (unless the diagonal rules it out) and fractions of |g| / radius
  CEL_HD double first(int w) const { return w == 0 && zero ? 0.0 : lo + ldexp(scale, 2 * w - 2 * kTrWaves + 2); }

  // A round's results: |p| (-1: not positive definite), the Newton point and the multiplier.
  // Returns the index of the multiplier that solves the problem (to 1e-7 of the radius), kMore,
  // or kNone where a step along the least eigenvalue's direction is what is left.
  CEL_HD int take(int round, const double (*rs)[3]) {
    // the Newton step; with decoupled coordinates B is singular, and the step is completed in them
    if (round == 0 && zero && rs[0][0] >= 0.0 && rs[0][0] <= radius) return decoupled ? kNone : 0;
    double best = INFINITY;
    int ibest = -1;
    for (int w = 0; w < kTrWaves; ++w) {
      const double nw = rs[w][0], lw = rs[w][2];
      if (nw >= 0.0 && nw <= radius) {
        if (lw <= hi) {
          hi = lw;
          nr = nw;
          tr = rs[w][1];
        }
      } else {
        lo = fmax(lo, lw);
        if (nw >= 0.0 && lw >= ll) {
          ll = lw;
          nl = nw;
          tl = rs[w][1];
        }
      }
      if (nw >= 0.0) {
        near = fmax(near, rs[w][1]);
        if (fabs(nw - radius) < best) {
          best = fabs(nw - radius);
          ibest = w;
        }
      }
    }
    // close enough to the boundary for a first-order correction
    if (ibest >= 0 && best <= 1e-7 * radius) return ibest;
    // Nothing positive definite is known left of the root and the bracket is small: from hi to
    // a root in it, directions of curvature above 4 (hi - lo) would grow by a quarter at most.
    // With |p(hi)| <= radius / 2 the rest, more than half of |p|^2, would lie along directions
    // of less curvature than that, which is not a step to take from here (a curvature below
    // 1e-6 |g| / radius); and a bracket below 2^-46 |g| / radius moves no other step by 1e-7.
    if (nl == 0.0 && nr > 0.0 && hi - lo <= (nr <= 0.5 * radius ? 0x1p-23 : 0x1p-46) * scale) return kNone;
    if (nl == 0.0 && round >= kTrBlind - 1) return kNone;
    near = fmax(near, lo);
    far = fmin(far, hi);
    if (nl > 0.0 && nr > 0.0) {
      // psi = 1 / radius at t between the points
      const double pl = 1.0 / nl, pr = 1.0 / nr, t = (1.0 / radius - pl) / (pr - pl), u = 1.0 - t;
      far = fmin(far, ll + t * (hi - ll));
      // slopes dlam/dt by the Newton points, (tl - ll) / t and (hi - tr) / u
      mid = u * u * ((1.0 + 2.0 * t) * ll + (tl - ll)) + t * t * ((3.0 - 2.0 * t) * hi - (hi - tr));
    }
    if (!(far - near > 4.0 * DBL_EPSILON * far)) {
      if (!(hi - lo > 4.0 * DBL_EPSILON * hi)) return kNone;   // bracket closed
      near = lo, far = hi;   // (crossed by rounding: back to what is certain)
    }
    return kMore;
  }

  // the next round's multipliers
  CEL_HD double next(int w) const {
    if (nl > 0.0 && nr > 0.0 && near > lo) {
      const double third = (far - near) / 3.0, half = near + 1.5 * third;
      const double m = mid > near && mid < far ? mid : half;
      return w == 0 ? near : w == 1 ? far : w == 2 ? m : m < half ? far - third : near + third;
    }
    if (nr > 0.0)   // nothing positive definite left of the root yet
      return near + (far - near) * ldexp(1.0, -2 * w - 1);
    return fmin(fmax(near, 1e-9 * far) * ldexp(1.0, 2 * w + 1), far);   // nothing right of it
  }
};

}  // namespace celmi
