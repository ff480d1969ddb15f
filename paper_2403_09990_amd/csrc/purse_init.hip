// Step I of the paper ("The CLOSURE Algorithm"): candidate start poses, each
// kept when it lies in S.  One trial per lane, or per quad of lanes for the
// perspective-3-point trials of a small launch; instance j runs M_j trials (its
// sample count in the batch).
//
// - 3D-3D (random sample averaging with a minimal solver): three distinct
//   correspondences, a random point inside each of their balls, Arun's
//   method on the three pairs.
// - 2D-3D: three distinct correspondences, a random point inside each of
//   their ellipses, and the perspective-3-point problem for the three
//   bearing rays: with s2 = u s1 and s3 = v s1 along the rays, the law of
//   cosines for the three pairs gives u = N(v) / D(v) and a quartic in v;
//   its real roots (found by bracketing between the roots of its
//   derivatives and bisection, in float64) give the camera points, and Arun's
//   method the pose.  Roots are taken in increasing v; the first solution
//   in S is kept.
// - pose regression (eq. PURSEregression): a random convex combination of
//   the hypotheses, R = proj_SO3(sum w_i R_i), t = sum w_i t_i, with weights
//   uniform on the simplex.
//
// Random numbers: Philox4x64-10; pose regression key (seed, 3), counter
// (trial, i, 0, 0), word 0 for the weight of hypothesis i; the keypoint
// sets key (seed, 4), counter (trial, k, 0, 0): k = 0 picks the
// correspondences, k = 1..3 the point in the k-th constraint.
#include "purse_fit.hpp"
#include "purse_launch.hpp"
#include "purse_traj.hpp"

namespace purse {

namespace {

constexpr int kInitBlock = 256;
constexpr int kInitQuadTrials = 384;  // trials per compute unit up to which a quad runs each

__device__ __forceinline__ void philox_u3(uint64_t seed, uint64_t key1, uint64_t c0, uint64_t c1, double u[3]) {
  uint64_t c[4] = {c0, c1, 0ull, 0ull};
  philox4x64_10(c, seed, key1);
  for (int q = 0; q < 3; ++q) u[q] = (double)(c[q] >> 40) * 0x1p-24;
}

// True unless the three points are collinear (to float64 resolution).
__device__ __forceinline__ bool has_area(const double P[3][3]) {
  double e1[3], e2[3];
  for (int r = 0; r < 3; ++r) {
    e1[r] = P[1][r] - P[0][r];
    e2[r] = P[2][r] - P[0][r];
  }
  const double c0 = e1[1] * e2[2] - e1[2] * e2[1], c1 = e1[2] * e2[0] - e1[0] * e2[2],
               c2 = e1[0] * e2[1] - e1[1] * e2[0];
  const double n1 = e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2];
  const double n2 = e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2];
  return c0 * c0 + c1 * c1 + c2 * c2 > 1e-24 * n1 * n2;
}

// Arun's method on three pairs P_k -> X_k (float64): R = proj_SO3(sum
// (X_k - Xbar)(P_k - Pbar)^T), t = Xbar - R Pbar.  False if degenerate.
__device__ bool arun3(const double P[3][3], const double X[3][3], double R[9], double t[3]) {
  double pb[3] = {0, 0, 0}, xb[3] = {0, 0, 0};
  for (int k = 0; k < 3; ++k)
    for (int r = 0; r < 3; ++r) {
      pb[r] += P[k][r] / 3.0;
      xb[r] += X[k][r] / 3.0;
    }
  double H[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = 0; k < 3; ++k)
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) H[3 * r + c] += (X[k][r] - xb[r]) * (P[k][c] - pb[c]);
  // Three pairs give a rank-two H whose determinant is zero up to rounding,
  // so polar_so3's flag for "det < 0 with close smaller singular values"
  // says nothing here: the polar factor u1 v1^T + u2 v2^T + (u1 x u2)(v1 x
  // v2)^T is well defined whenever both triangles have area.
  polar_so3<double>(H, R, 12);
  for (int r = 0; r < 3; ++r) t[r] = xb[r] - (R[3 * r] * pb[0] + R[3 * r + 1] * pb[1] + R[3 * r + 2] * pb[2]);
  // collinear points (a rank-one H) leave the rotation about their line open
  return has_area(P) && has_area(X);
}

// Three distinct indices of n, in the order drawn.
__device__ __forceinline__ void pick_three(const double u[3], int n, int idx[3]) {
  int taken[3];
  for (int q = 0; q < 3; ++q) {
    int x = (int)floor(u[q] * (double)(n - q));
    // skip the indices already taken, smallest first
    int s0 = q > 0 ? taken[0] : INT32_MAX, s1 = q > 1 ? taken[1] : INT32_MAX;
    if (s1 < s0) {
      const int tmp = s0;
      s0 = s1;
      s1 = tmp;
    }
    if (x >= s0) ++x;
    if (x >= s1) ++x;
    taken[q] = x;
    idx[q] = x;
  }
}

__device__ __forceinline__ double polyval(const double *c, int deg, double x) {
  double v = c[0];
  for (int k = 1; k <= deg; ++k) v = v * x + c[k];
  return v;
}

// Real roots of a polynomial of degree <= 4 (highest coefficient first),
// ascending: the roots of its derivative bracket the monotone pieces, each
// bisected to float64 resolution (every degree handled the same way).
__device__ int real_roots4(const double *c4, double roots[4]) {
  double c[5][5];  // c[d]: the (4 - d)-th derivative's coefficients, degree d
  for (int k = 0; k <= 4; ++k) c[4][k] = c4[k];
  for (int d = 4; d > 1; --d)
    for (int k = 0; k < d; ++k) c[d - 1][k] = c[d][k] * (double)(d - k);
  // bound on every root (Cauchy) of the quartic
  double lead = c[4][0];
  if (lead == 0.0) return 0;
  double B = 0.0;
  for (int k = 1; k <= 4; ++k) B = fmax(B, fabs(c[4][k] / lead));
  B += 1.0;
  double r[4];
  int nr = 0;
  // degree 1
  if (c[1][0] != 0.0) {
    r[0] = -c[1][1] / c[1][0];
    nr = 1;
  }
  for (int d = 2; d <= 4; ++d) {
    double pts[6];
    int np = 0;
    pts[np++] = -B;
    for (int k = 0; k < nr; ++k)
      if (r[k] > -B && r[k] < B) pts[np++] = r[k];
    pts[np++] = B;
    int nn = 0;
    double rn[4];
    for (int k = 0; k + 1 < np; ++k) {
      double lo = pts[k], hi = pts[k + 1];
      double flo = polyval(c[d], d, lo), fhi = polyval(c[d], d, hi);
      if (flo == 0.0) {
        if (nn == 0 || rn[nn - 1] != lo) rn[nn++] = lo;
        continue;
      }
      if ((flo < 0.0) == (fhi < 0.0)) continue;
      for (int it = 0; it < 100; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        const double fm = polyval(c[d], d, mid);
        if ((fm < 0.0) == (flo < 0.0)) {
          lo = mid;
          flo = fm;
        } else {
          hi = mid;
        }
      }
      if (nn < 4) rn[nn++] = 0.5 * (lo + hi);
    }
    nr = nn;
    for (int k = 0; k < nn; ++k) r[k] = rn[k];
  }
  for (int k = 0; k < nr; ++k) roots[k] = r[k];
  return nr;
}

// Lane L of the quad hands its value to the quad.
template <int L>
__device__ __forceinline__ int quad_bcast(int x) {
  return __builtin_amdgcn_mov_dpp(x, L * 0x55, 0xF, 0xF, false);
}
template <int L>
__device__ __forceinline__ double quad_bcast(double x) {
  return __hiloint2double(quad_bcast<L>(__double2hiint(x)), quad_bcast<L>(__double2loint(x)));
}
// the same by a runtime lane, uniform over the quad
__device__ __forceinline__ double quad_pick(double x, int l) {
  const double a = quad_bcast<0>(x), b = quad_bcast<1>(x), c = quad_bcast<2>(x), d = quad_bcast<3>(x);
  return l == 0 ? a : (l == 1 ? b : (l == 2 ? c : d));
}

// real_roots4 by the four lanes of a quad, which all hold the quartic: lane q
// bisects the q-th monotone piece (degree d has at most d), the same steps on
// the same bracket, and the roots found are gathered in order.
__device__ __forceinline__ int real_roots4_quad(const double *c4, double roots[4], int q) {
  double c[5][5];
#pragma unroll
  for (int k = 0; k <= 4; ++k) c[4][k] = c4[k];
#pragma unroll
  for (int d = 4; d > 1; --d)
#pragma unroll
    for (int k = 0; k < d; ++k) c[d - 1][k] = c[d][k] * (double)(d - k);
  const double lead = c[4][0];
  if (lead == 0.0) return 0;
  double B = 0.0;
#pragma unroll
  for (int k = 1; k <= 4; ++k) B = fmax(B, fabs(c[4][k] / lead));
  B += 1.0;
  double r[4] = {0.0, 0.0, 0.0, 0.0};
  int nr = 0;
  if (c[1][0] != 0.0) {
    r[0] = -c[1][1] / c[1][0];
    nr = 1;
  }
#pragma unroll
  for (int d = 2; d <= 4; ++d) {
    // this lane's piece: the ends -B, the roots inside (-B, B), B
    double lo = -B, hi = B;
    int at = 0;  // interior points so far
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k < nr && r[k] > -B && r[k] < B) {
        if (at == q) hi = r[k];
        if (at + 1 == q) lo = r[k];
        ++at;
      }
    }
    const bool piece = q <= at;
    double flo = polyval(c[d], d, lo), fhi = polyval(c[d], d, hi);
    const bool zero = flo == 0.0;
    int found = 0;  // 1: a root in the piece, 2: at its lower end
    double root = 0.0;
    if (piece && zero) {
      found = 2;
      root = lo;
    } else if (piece && (flo < 0.0) != (fhi < 0.0)) {
      const bool neg = flo < 0.0;
      for (int it = 0; it < 100; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        const double fm = polyval(c[d], d, mid);
        if ((fm < 0.0) == neg)
          lo = mid;
        else
          hi = mid;
      }
      found = 1;
      root = 0.5 * (lo + hi);
    }
    const int fs[4] = {quad_bcast<0>(found), quad_bcast<1>(found), quad_bcast<2>(found), quad_bcast<3>(found)};
    const double rs[4] = {quad_bcast<0>(root), quad_bcast<1>(root), quad_bcast<2>(root), quad_bcast<3>(root)};
    int nn = 0;
    double last = 0.0, rn[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool take = fs[k] == 1 || (fs[k] == 2 && (nn == 0 || last != rs[k]));
#pragma unroll
      for (int w = 0; w < 4; ++w) rn[w] = take && w == nn ? rs[k] : rn[w];
      last = take ? rs[k] : last;
      nn += take ? 1 : 0;
    }
    nr = nn;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = rn[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) roots[k] = r[k];
  return nr;
}

// Polynomial helpers (highest degree first, fixed storage of 5).
__device__ __forceinline__ void pmul(const double *a, int da, const double *b, int db, double *out) {
  for (int k = 0; k <= da + db; ++k) out[k] = 0.0;
  for (int i = 0; i <= da; ++i)
    for (int jj = 0; jj <= db; ++jj) out[i + jj] += a[i] * b[jj];
}

// R_i of a pose-regression hypothesis from its stored quaternion (w, x, y,
// z), normalised, in float64.
__device__ void hyp_rotation(const float *q4, double R[9]) {
  const double q0 = q4[0], q1 = q4[1], q2 = q4[2], q3 = q4[3];
  const double s = 1.0 / sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
  const double w = q0 * s, x = q1 * s, y = q2 * s, z = q3 * s;
  R[0] = 1.0 - 2.0 * (y * y + z * z);
  R[1] = 2.0 * (x * y - w * z);
  R[2] = 2.0 * (x * z + w * y);
  R[3] = 2.0 * (x * y + w * z);
  R[4] = 1.0 - 2.0 * (x * x + z * z);
  R[5] = 2.0 * (y * z - w * x);
  R[6] = 2.0 * (x * z - w * y);
  R[7] = 2.0 * (y * z + w * x);
  R[8] = 1.0 - 2.0 * (x * x + y * y);
}

struct InitKp {
  const float *a, *c, *L, *beta;
};

// in_purse of (R, t) against every constraint of the instance (float64, the
// sampler's test with tolerance tau and depth > z_min).
__device__ bool in_s_keypoints(int kind, int n, const InitKp &kp, const float K[4], const double R[9],
                               const double t[3], double tau, double z_min) {
  for (int i = 0; i < n; ++i) {
    double P[3];
    for (int r = 0; r < 3; ++r)
      P[r] = R[3 * r] * kp.a[3 * i] + R[3 * r + 1] * kp.a[3 * i + 1] + R[3 * r + 2] * kp.a[3 * i + 2] + t[r];
    double rr;
    if (kind == PURSE_KIND_2D3D) {
      if (!(P[2] > z_min)) return false;
      const double e0 = K[0] * P[0] / P[2] + K[2] - kp.c[3 * i];
      const double e1 = K[1] * P[1] / P[2] + K[3] - kp.c[3 * i + 1];
      const float *l = kp.L + 4 * i;
      rr = sqrt(fmax(0.0, e0 * (l[0] * e0 + l[1] * e1) + e1 * (l[2] * e0 + l[3] * e1)));
    } else {
      const double e0 = P[0] - kp.c[3 * i], e1 = P[1] - kp.c[3 * i + 1], e2 = P[2] - kp.c[3 * i + 2];
      rr = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
    }
    if (!(rr <= (double)kp.beta[i] + tau)) return false;
  }
  return true;
}

}  // namespace

// The bearing of a random point inside the ellipse of keypoint i.
__device__ __forceinline__ void bearing_in_ellipse(const InitKp &kp, int i, const double u[3], const float K[4],
                                                   double f[3]) {
  double sp, cp;
  sincospi(2.0 * u[1], &sp, &cp);
  const double rad = sqrt(u[2]) * (double)kp.beta[i];
  const float *l = kp.L + 4 * i;
  // U^T U = Lambda, U = [[w0, w1], [0, w2]]; e = U^-1 y
  const double w0 = sqrt((double)l[0]), w1 = (double)l[1] / w0;
  const double w2 = sqrt(fmax(0.0, (double)l[3] - w1 * w1));
  const double y0 = rad * cp, y1 = rad * sp;
  const double e1 = y1 / w2, e0 = (y0 - w1 * e1) / w0;
  const double px = (double)kp.c[3 * i] + e0, py = (double)kp.c[3 * i + 1] + e1;
  double d[3] = {(px - K[2]) / K[0], (py - K[3]) / K[1], 1.0};
  const double nd = 1.0 / sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  for (int r = 0; r < 3; ++r) f[r] = d[r] * nd;
}

// The perspective-3-point equations of points Pm on the bearings f: the
// quartic in v, and u = N(v) / D(v), s1 = bb / sqrt(q(v)).
struct P3P {
  double q[3], N[3], D[2], bb, quart[5];
};

__device__ __forceinline__ void p3p_equations(const double Pm[3][3], const double f[3][3], P3P &e) {
  double dd[3];
  for (int r = 0; r < 3; ++r) dd[r] = Pm[1][r] - Pm[2][r];
  const double a = sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
  for (int r = 0; r < 3; ++r) dd[r] = Pm[0][r] - Pm[2][r];
  const double bb = sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
  for (int r = 0; r < 3; ++r) dd[r] = Pm[0][r] - Pm[1][r];
  const double c = sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
  const double ca = f[1][0] * f[2][0] + f[1][1] * f[2][1] + f[1][2] * f[2][2];
  const double cb = f[0][0] * f[2][0] + f[0][1] * f[2][1] + f[0][2] * f[2][2];
  const double cg = f[0][0] * f[1][0] + f[0][1] * f[1][1] + f[0][2] * f[1][2];
  const double Kc = (a * a - c * c) / (bb * bb);
  // q = v^2 - 2 cb v + 1; N = K q + 1 - v^2; D = -2 ca v + 2 cg
  const double q[3] = {1.0, -2.0 * cb, 1.0};
  const double N[3] = {Kc - 1.0, -2.0 * cb * Kc, Kc + 1.0};
  const double D[2] = {-2.0 * ca, 2.0 * cg};
  double DD[3], NN[5], ND[4], qDD[5];
  pmul(D, 1, D, 1, DD);
  pmul(N, 2, N, 2, NN);
  pmul(N, 2, D, 1, ND);
  pmul(q, 2, DD, 2, qDD);
  const double k2 = (c * c) / (bb * bb);
  for (int k = 0; k <= 4; ++k) {
    double v = NN[k] - k2 * qDD[k];
    if (k >= 1) v += -2.0 * cg * ND[k - 1];
    if (k >= 2) v += DD[k - 2];
    e.quart[k] = v;
  }
  for (int k = 0; k < 3; ++k) {
    e.q[k] = q[k];
    e.N[k] = N[k];
  }
  e.D[0] = D[0];
  e.D[1] = D[1];
  e.bb = bb;
}

// The pose of root v; false if it gives none.
__device__ __forceinline__ bool p3p_pose(const double Pm[3][3], const double f[3][3], const P3P &e, double v,
                                         double R[9], double t[3]) {
  if (!(v > 0.0)) return false;
  const double Dv = e.D[0] * v + e.D[1];
  if (fabs(Dv) < 1e-14) return false;
  const double uu = polyval(e.N, 2, v) / Dv;
  const double qv = polyval(e.q, 2, v);
  if (!(uu > 0.0) || !(qv > 0.0)) return false;
  const double s1 = e.bb / sqrt(qv);
  double X[3][3];
  for (int r = 0; r < 3; ++r) {
    X[0][r] = s1 * f[0][r];
    X[1][r] = uu * s1 * f[1][r];
    X[2][r] = v * s1 * f[2][r];
  }
  return arun3(Pm, X, R, t);
}

// One perspective-3-point trial by a quad of lanes: lane q draws and places
// the q-th point (1..3), bisects the q-th piece of each derivative, and
// solves and tests the q-th root's pose; the first lane whose pose is in S has
// the trial's.  The same arithmetic as the single lane's, whose chain of
// float64 steps (three points, up to nine bisections, up to four poses) is what
// a launch of few trials waits for (1500 trials of 10 keypoints: 0.082 -> 0.034
// ms).  Lanes of a quad enter together.
__device__ __forceinline__ bool p3p_quad(const InitKp &kp, int n, const float K[4], uint64_t seed, uint64_t s, int q,
                                         double tau, double z_min, double R[9], double t[3]) {
  double u[3];
  philox_u3(seed, 4ull, s, 0ull, u);
  int idx[3];
  pick_three(u, n, idx);
  double Pm[3][3];
  for (int k = 0; k < 3; ++k)
    for (int r = 0; r < 3; ++r) Pm[k][r] = kp.a[3 * idx[k] + r];
  double mine[3];
  {
    // (lane 0 repeats lane 1's)
    const int k = max(q, 1) - 1, i = k == 0 ? idx[0] : (k == 1 ? idx[1] : idx[2]);
    philox_u3(seed, 4ull, s, (uint64_t)(k + 1), u);
    bearing_in_ellipse(kp, i, u, K, mine);
  }
  double f[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    f[0][r] = quad_bcast<1>(mine[r]);
    f[1][r] = quad_bcast<2>(mine[r]);
    f[2][r] = quad_bcast<3>(mine[r]);
  }
  P3P e;
  p3p_equations(Pm, f, e);
  double roots[4];
  const int nr = real_roots4_quad(e.quart, roots, q);
  const double v = q == 0 ? roots[0] : (q == 1 ? roots[1] : (q == 2 ? roots[2] : roots[3]));
  const bool mine_ok = q < nr && p3p_pose(Pm, f, e, v, R, t) &&
                       in_s_keypoints(PURSE_KIND_2D3D, n, kp, K, R, t, tau, z_min);
  const int okay = mine_ok ? 1 : 0;
  const int first = quad_bcast<0>(okay) ? 0 : (quad_bcast<1>(okay) ? 1 : (quad_bcast<2>(okay) ? 2 : (quad_bcast<3>(okay) ? 3 : -1)));
  if (first < 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = k % 4 == 0 ? 1.0 : 0.0;
#pragma unroll
    for (int r = 0; r < 3; ++r) t[r] = 0.0;
    return false;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = quad_pick(R[k], first);
#pragma unroll
  for (int r = 0; r < 3; ++r) t[r] = quad_pick(t[r], first);
  return true;
}

// LANES = 4: a quad of lanes per trial of a 2D-3D instance (instances of other
// kinds use the first quarter of the grid).
template <int LANES>
__global__ void __launch_bounds__(kInitBlock) k_init(DevBatch b, DevParams p, float *poses, uint8_t *mask) {
  const int j = blockIdx.y;
  int64_t off, M;
  sample_range(b.sample_off, j, b.total_samples, b.max_samples, off, M);
  const int kind = b.kind[j];
  // lanes of a trial, and this lane's place among them
  const int per = LANES > 1 && kind == PURSE_KIND_2D3D ? LANES : 1, q4 = threadIdx.x % per;
  const int64_t s = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / per;
  if (s >= M) return;  // (the lanes of a quad together)
  const int n = b.n_kp[j];
  const int64_t ko = b.kp_off[j];
  const uint64_t seed = b.seed[j];
  float *out = poses + 12 * (off + s);
  double R[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, t[3] = {0, 0, 0};
  bool ok = false;
  const bool valid = n >= (kind == PURSE_KIND_REG ? 1 : 3) && n <= PURSE_MAX_KP && ko >= 0 &&
                     b.kp_off[j + 1] - ko == n && b.kp_off[j + 1] <= b.total_kp;
  const InitKp kp{b.model_pts + 3 * ko, b.centres + 3 * ko, b.shapes + 4 * ko, b.bounds + ko};
  if (valid && kind == PURSE_KIND_REG) {
    // convex combination of the hypotheses
    double M9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, wsum = 0.0;
    double tt[3] = {0, 0, 0};
    for (int i = 0; i < n; ++i) {
      double u[3];
      philox_u3(seed, 3ull, (uint64_t)s, (uint64_t)i, u);
      const double w = -log1p(-u[0]);
      double Ri[9];
      hyp_rotation(kp.L + 4 * i, Ri);
      for (int k = 0; k < 9; ++k) M9[k] += w * Ri[k];
      for (int r = 0; r < 3; ++r) tt[r] += w * kp.c[3 * i + r];
      wsum += w;
    }
    for (int k = 0; k < 9; ++k) M9[k] /= wsum;
    for (int r = 0; r < 3; ++r) t[r] = tt[r] / wsum;
    polar_so3<double>(M9, R, 12);
    ok = true;
    const double tau = p.tau3;
    for (int i = 0; i < n && ok; ++i) {
      double Ri[9];
      hyp_rotation(kp.L + 4 * i, Ri);
      double f = 0.0;
      for (int k = 0; k < 9; ++k) f += (R[k] - Ri[k]) * (R[k] - Ri[k]);
      double e2 = 0.0;
      for (int r = 0; r < 3; ++r) e2 += (t[r] - kp.c[3 * i + r]) * (t[r] - kp.c[3 * i + r]);
      ok = sqrt(f) <= (double)kp.a[3 * i] + tau && sqrt(e2) <= (double)kp.beta[i] + tau;
    }
  } else if (valid && (kind == PURSE_KIND_3D3D || kind == PURSE_KIND_2D3D)) {
    double u[3];
    philox_u3(seed, 4ull, (uint64_t)s, 0ull, u);
    int idx[3];
    pick_three(u, n, idx);
    double Pm[3][3];
    for (int k = 0; k < 3; ++k)
      for (int r = 0; r < 3; ++r) Pm[k][r] = kp.a[3 * idx[k] + r];
    const bool is2d = kind == PURSE_KIND_2D3D;
    float K[4] = {0, 0, 0, 0};
    if (is2d)
      for (int q = 0; q < 4; ++q) K[q] = b.intrinsics[4 * j + q];
    const double tau = is2d ? p.tau2 : p.tau3;
    if (!is2d) {
      double X[3][3];
      for (int k = 0; k < 3; ++k) {
        philox_u3(seed, 4ull, (uint64_t)s, (uint64_t)(k + 1), u);
        const double z = 1.0 - 2.0 * u[0];
        const double rho = sqrt(fmax(0.0, 1.0 - z * z));
        double sp, cp;
        sincospi(2.0 * u[1], &sp, &cp);
        const double rad = cbrt(u[2]) * (double)kp.beta[idx[k]];
        const double d[3] = {rho * cp, rho * sp, z};
        for (int r = 0; r < 3; ++r) X[k][r] = (double)kp.c[3 * idx[k] + r] + rad * d[r];
      }
      ok = arun3(Pm, X, R, t) && in_s_keypoints(kind, n, kp, K, R, t, tau, (double)p.z_min);
    } else {
      if constexpr (LANES > 1) {
        ok = p3p_quad(kp, n, K, seed, (uint64_t)s, q4, tau, (double)p.z_min, R, t);
      } else {
        double f[3][3];
        for (int k = 0; k < 3; ++k) {
          philox_u3(seed, 4ull, (uint64_t)s, (uint64_t)(k + 1), u);
          bearing_in_ellipse(kp, idx[k], u, K, f[k]);
        }
        P3P e;
        p3p_equations(Pm, f, e);
        double roots[4];
        const int nr = real_roots4(e.quart, roots);
        for (int k = 0; k < nr && !ok; ++k) {
          double Rk[9], tk[3];
          if (p3p_pose(Pm, f, e, roots[k], Rk, tk) && in_s_keypoints(kind, n, kp, K, Rk, tk, tau, (double)p.z_min)) {
            for (int q2 = 0; q2 < 9; ++q2) R[q2] = Rk[q2];
            for (int r = 0; r < 3; ++r) t[r] = tk[r];
            ok = true;
          }
        }
      }
    }
  }
  if (q4 != 0) return;
  float4 *o4 = reinterpret_cast<float4 *>(out);
  o4[0] = make_float4((float)R[0], (float)R[1], (float)R[2], (float)R[3]);
  o4[1] = make_float4((float)R[4], (float)R[5], (float)R[6], (float)R[7]);
  o4[2] = make_float4((float)R[8], (float)t[0], (float)t[1], (float)t[2]);
  mask[off + s] = ok ? PURSE_MASK_FEASIBLE : 0;
}

void launch_init(const DevBatch &b, const DevParams &p, float *poses, uint8_t *mask, hipStream_t stream) {
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    n_cu = 256;
  // Quads, in workgroups of one wavefront that spread over the compute units,
  // while the trials leave the chip idle: 65536 trials take 0.071 ms by quads
  // and 0.095 by lanes, 131072 0.128 and 0.125, 262144 0.243 and 0.229
  if (b.max_samples * (int64_t)b.n_inst <= (int64_t)n_cu * kInitQuadTrials) {
    const dim3 grid((unsigned)((b.max_samples * 4 + 63) / 64), (unsigned)b.n_inst);
    hipLaunchKernelGGL(k_init<4>, grid, dim3(64), 0, stream, b, p, poses, mask);
    return;
  }
  const dim3 grid((unsigned)((b.max_samples + kInitBlock - 1) / kInitBlock), (unsigned)b.n_inst);
  hipLaunchKernelGGL(k_init<1>, grid, dim3(kInitBlock), 0, stream, b, p, poses, mask);
}

}  // namespace purse
