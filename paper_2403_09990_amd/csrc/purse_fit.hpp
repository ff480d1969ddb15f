// Centre-fit building blocks shared by the prologue and the backward: DLT
// and weak-perspective starts, whitening of Lambda, the Gauss-Newton fit of
// the 2D-3D maximum-likelihood pose, Arun's fit for 3D-3D.
#pragma once

#include "purse_near.hpp"

namespace purse {

__device__ inline bool finite_f(float x) { return isfinite(x); }


// Whitening factor U = [[u00, u01], [0, u11]] with U^T U = Lambda.
template <typename T>
__device__ __forceinline__ void whiten_factor(const float *Lam, T w[3]) {
  T l00 = Lam[0], l01 = Lam[1], l11 = Lam[3];
  w[0] = sqrt((double)l00);
  w[1] = l01 / w[0];
  w[2] = sqrt((double)(l11 - w[1] * w[1]));
}

// Gauss-Newton centre fit of the 2D-3D maximum-likelihood pose (eq. MLE with
// rho = ||.||^2_Lambda): targets are the ellipse centres, each step about the
// pivot R Zbar + t of the current pose, iterated until the step is below
// kCentreTol (rotation) and kCentreTol (1 + |t|_inf) (translation), at most
// `steps` times.  T is double, or a dual number when the backward
// differentiates the fit; obs(i, z, w) gives keypoint i's image point and
// whitening factor.
constexpr double kCentreTol = 1e-13;

template <typename T, typename OBS>
__device__ bool gn_centre_2d(const float *Z, const OBS &obs, int n, const float K[4], int steps, double z_min,
                             T R[9], T t[3]) {
  double zb[3] = {0, 0, 0};
  for (int i = 0; i < n; ++i)
    for (int r = 0; r < 3; ++r) zb[r] += Z[3 * i + r];
  for (int r = 0; r < 3; ++r) zb[r] /= n;
  const double Kd[4] = {K[0], K[1], K[2], K[3]};
  for (int st = 0; st < steps; ++st) {
    T o[3];
    for (int r = 0; r < 3; ++r) o[r] = R[3 * r] * zb[0] + R[3 * r + 1] * zb[1] + R[3 * r + 2] * zb[2] + t[r];
    T A[21], g[6];
    for (int k = 0; k < 21; ++k) A[k] = T(0.0);
    for (int k = 0; k < 6; ++k) g[k] = T(0.0);
    for (int i = 0; i < n; ++i) {
      T P[3];
      for (int r = 0; r < 3; ++r)
        P[r] = R[3 * r] * (double)Z[3 * i] + R[3 * r + 1] * (double)Z[3 * i + 1] + R[3 * r + 2] * (double)Z[3 * i + 2] + t[r];
      if (!(value_of(P[2]) > z_min)) return false;
      T iz = T(1.0) / P[2];
      T u = Kd[0] * (P[0] * iz) + Kd[2], v = Kd[1] * (P[1] * iz) + Kd[3];
      T z[2], w[3];
      obs(i, z, w);
      T r0 = z[0] - u, r1 = z[1] - v;
      T rt0 = w[0] * r0 + w[1] * r1, rt1 = w[2] * r1;
      T pt[3] = {P[0] - o[0], P[1] - o[1], P[2] - o[2]};
      gn_accumulate<T>(P, pt, iz, T(Kd[0]), T(Kd[1]), w, rt0, rt1, A, g);
    }
    T d[6];
    if (!chol6_solve<T>(A, g, d)) return false;
    apply_update<T>(d, o, R, t);
    // converged: the step is at the float64 rounding level of the pose
    double dw = 0.0, dv = 0.0, tm = 0.0;
    for (int k = 0; k < 3; ++k) {
      dw = fmax(dw, fabs(value_of(d[k])));
      dv = fmax(dv, fabs(value_of(d[3 + k])));
      tm = fmax(tm, fabs(value_of(t[k])));
    }
    if (dw <= kCentreTol && dv <= kCentreTol * (1.0 + tm)) break;
  }
  for (int i = 0; i < n; ++i) {
    double pz = value_of(R[6]) * Z[3 * i] + value_of(R[7]) * Z[3 * i + 1] + value_of(R[8]) * Z[3 * i + 2] + value_of(t[2]);
    if (!(pz > z_min)) return false;
  }
  return true;
}

// gn_centre_2d<double> on a whole wavefront, for up to 64 keypoints: lane i
// takes keypoint i, the normal equations are summed over the wavefront in a
// fixed order (every lane ends with the same sums) and every lane then takes
// the same step, so the control flow stays wave-uniform.  The fit ends where the
// steps reach the rounding of the pose, whatever the rounding on the way.
template <typename OBS>
__device__ bool gn_centre_2d_wave(const float *Z, const OBS &obs, int n, const float K[4], int steps, double z_min,
                                  double R[9], double t[3]) {
  const int lane = threadIdx.x & 63;
  const double Kd[4] = {K[0], K[1], K[2], K[3]};
  const bool mine = lane < n;
  const int i = mine ? lane : 0;
  const double Zi[3] = {Z[3 * i], Z[3 * i + 1], Z[3 * i + 2]};
  double zi[2], wi[3];
  obs(i, zi, wi);
  double zb[3] = {mine ? Zi[0] : 0.0, mine ? Zi[1] : 0.0, mine ? Zi[2] : 0.0};
  wave_sums<3>(zb, n);
  for (int r = 0; r < 3; ++r) zb[r] /= n;
  for (int st = 0; st < steps; ++st) {
    double o[3];
    for (int r = 0; r < 3; ++r) o[r] = R[3 * r] * zb[0] + R[3 * r + 1] * zb[1] + R[3 * r + 2] * zb[2] + t[r];
    double A[27], *g = A + 21;
#pragma unroll
    for (int k = 0; k < 27; ++k) A[k] = 0.0;
    double P[3];
    for (int r = 0; r < 3; ++r) P[r] = R[3 * r] * Zi[0] + R[3 * r + 1] * Zi[1] + R[3 * r + 2] * Zi[2] + t[r];
    if (__ballot(mine && !(P[2] > z_min)) != 0ull) return false;
    if (mine) {
      const double iz = near_rcp(P[2]);
      const double u = Kd[0] * (P[0] * iz) + Kd[2], v = Kd[1] * (P[1] * iz) + Kd[3];
      const double r0 = zi[0] - u, r1 = zi[1] - v;
      const double rt0 = wi[0] * r0 + wi[1] * r1, rt1 = wi[2] * r1;
      const double pt[3] = {P[0] - o[0], P[1] - o[1], P[2] - o[2]};
      gn_accumulate<double>(P, pt, iz, Kd[0], Kd[1], wi, rt0, rt1, A, g);
    }
    wave_sums<27>(A, n);
    double L[21], dinv[6], d[6];
    if (!near_solve(A, g, L, dinv, d)) return false;
    near_update(d, o, R, t);
    double dw = 0.0, dv = 0.0, tm = 0.0;
    for (int k = 0; k < 3; ++k) {
      dw = fmax(dw, fabs(d[k]));
      dv = fmax(dv, fabs(d[3 + k]));
      tm = fmax(tm, fabs(t[k]));
    }
    if (dw <= kCentreTol && dv <= kCentreTol * (1.0 + tm)) break;
  }
  const double pz = R[6] * Zi[0] + R[7] * Zi[1] + R[8] * Zi[2] + t[2];
  return __ballot(mine && !(pz > z_min)) == 0ull;
}

// The starts of the fit on a whole wavefront, for the prologue and for the
// backward's re-run of a fit alike; the results are uniform.  The sums of the
// normal equations sit one per lane, the factorisation and the solves of the
// inverse iteration one row per lane, and the polar factor comes from Newton's
// iteration.  (Serial in one lane, the DLT start took 45 to 70 us, half of the
// prologue of a 2D-3D instance: 65536 samples of 16 keypoints 0.544 -> 0.491 ms.)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Direct linear transform in normalised image coordinates, model points
// centred and scaled for conditioning; the null vector of the 2N x 12 system
// comes from inverse iteration on its normal matrix.  Returns (R, t) with the
// sign fixed by det(P[:, :3]) > 0 and t = P[:, 3] / (mean singular value).
// buf: 64 x 7 doubles of LDS of the wavefront's own.
__device__ inline bool dlt_2d_wave(const float *Z, const float *z, int n, const float K[4], double (*buf)[7],
                                   double R[9], double t[3]) {
  const int lane = threadIdx.x & 63;
  const bool mine = lane < n;
  const int i = mine ? lane : 0;
  double Zi[3] = {Z[3 * i], Z[3 * i + 1], Z[3 * i + 2]};
  double zb[3] = {mine ? Zi[0] : 0.0, mine ? Zi[1] : 0.0, mine ? Zi[2] : 0.0};
  wave_sums<3>(zb, n);
  double ss[1] = {0.0};
  for (int r = 0; r < 3; ++r) {
    zb[r] /= n;
    Zi[r] -= zb[r];
    ss[0] += mine ? Zi[r] * Zi[r] : 0.0;
  }
  wave_sums<1>(ss, n);
  const double sc = sqrt(ss[0] / n);
  if (!(sc > 0)) return false;
  const double isc = 1.0 / sc;
  if (mine) {
    const double xn = ((double)z[3 * i] - K[2]) / K[0], yn = ((double)z[3 * i + 1] - K[3]) / K[1];
    for (int r = 0; r < 3; ++r) buf[lane][r] = Zi[r] * isc;
    buf[lane][3] = 1.0;
    buf[lane][4] = xn;
    buf[lane][5] = yn;
    buf[lane][6] = xn * xn + yn * yn;
  }
  wave_lds_fence();
  // lane 4 e + w: sum_i h_a h_b q_w, (a, b) the e-th pair (packed lower), q = 1,
  // xn, yn, xn^2 + yn^2
  const int e = lane >> 2, w = lane & 3;
  const int a = e >= 6 ? 3 : (e >= 3 ? 2 : (e >= 1 ? 1 : 0)), b = min(e - a * (a + 1) / 2, 3);
  double sum = 0.0;
  for (int k = 0; k < n; ++k) sum = fma(buf[k][a] * buf[k][b], buf[k][3 + w], sum);
  wave_lds_fence();
  double *S = &buf[0][0];
  if (lane < 40) S[lane] = sum;
  wave_lds_fence();
  // row r of the 12 x 12 normal matrix on lane r: blocks h h^T by 1 on the first
  // two diagonal blocks, -xn, -yn in the last row, xn^2 + yn^2 in the corner
  const int row = min(lane, 11), rp = row >> 2, ra = row & 3;
  double A[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    const int cp = c >> 2, ca = c & 3, hi = max(ra, ca), lo = min(ra, ca);
    const double *q = S + 4 * (hi * (hi + 1) / 2 + lo);
    double v = 0.0;
    if (rp == cp) v = rp == 2 ? q[3] : q[0];
    if (rp == 2 && cp < 2) v = -q[1 + cp];
    if (cp == 2 && rp < 2) v = -q[1 + rp];
    A[c] = v;
  }
  double tr = 0.0;
  for (int k = 0; k < 4; ++k) {
    const double *q = S + 4 * (k * (k + 1) / 2 + k);
    tr += 2.0 * q[0] + q[3];
  }
#pragma unroll
  for (int c = 0; c < 12; ++c) A[c] += lane == c ? 1e-13 * tr : 0.0;
  // Cholesky, right-looking; Lr: this lane's row below the diagonal, Lc: its
  // column below the diagonal, di: the reciprocal diagonal (uniform)
  double Lr[12], Lc[12], di[12];
#pragma unroll
  for (int j = 0; j < 12; ++j) Lr[j] = Lc[j] = 0.0;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    const double d = lane_value(A[j], j);
    ok = ok && d > 0.0;
    di[j] = near_rsq(d);
    const double l = A[j] * di[j];
    Lr[j] = lane > j && lane < 12 ? l : 0.0;
#pragma unroll
    for (int c = j + 1; c < 12; ++c) {
      const double lc = lane_value(l, c);
      Lc[c] = lane == j ? lc : Lc[c];
      A[c] = fma(-l, lc, A[c]);
    }
  }
  if (!ok) return false;
  double v = lane < 12 ? 1.0 + 0.01 * lane : 0.0;
  for (int it = 0; it < 80; ++it) {
    const double u = v;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double x = lane_value(v, k) * di[k];
      v = lane == k ? x : fma(-Lr[k], x, v);
    }
#pragma unroll
    for (int k = 11; k >= 0; --k) {
      const double x = lane_value(v, k) * di[k];
      v = lane == k ? x : fma(-Lc[k], x, v);
    }
    double nn[1] = {v * v};
    wave_sums<1>(nn, 16);
    v *= near_rsq(nn[0]);
    if (it >= 2 && __ballot(fabs(v - u) > 1e-14) == 0ull) break;
  }
  // undo the model normalisation: P = P' [[I/sc, -zb/sc], [0, 1]]
  double M[9], p3[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    double acc = lane_value(v, 4 * r + 3);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double q = lane_value(v, 4 * r + c) * isc;
      M[3 * r + c] = q;
      acc -= q * zb[c];
    }
    p3[r] = acc;
  }
  const double det = M[0] * (M[4] * M[8] - M[5] * M[7]) - M[1] * (M[3] * M[8] - M[5] * M[6]) +
                     M[2] * (M[3] * M[7] - M[4] * M[6]);
  if (det < 0) {
    for (int k = 0; k < 9; ++k) M[k] = -M[k];
    for (int r = 0; r < 3; ++r) p3[r] = -p3[r];
  }
  near_polar(M, R);
  // the mean singular value, tr(R^T M) / 3 (det M >= 0)
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) s += R[k] * M[k];
  s *= 1.0 / 3.0;
  if (!(s > 0)) return false;
  for (int r = 0; r < 3; ++r) t[r] = p3[r] / s;
  return true;
}

// Weak-perspective initialisation: least squares x_n = A Z + b (a scaled
// orthographic camera) by the 4x4 normal equations; s = mean row norm of A,
// R = proj_SO3 [A0/s; A1/s; A0 x A1 / s^2], t = (b / s, 1 / s).
__device__ inline bool affine_2d_wave(const float *Z, const float *z, int n, const float K[4], double R[9],
                                      double t[3]) {
  const int lane = threadIdx.x & 63;
  const bool mine = lane < n;
  const int i = mine ? lane : 0;
  double x[4] = {0, 0, 0, 0}, xn = 0.0, yn = 0.0;
  if (mine) {
    for (int r = 0; r < 3; ++r) x[r] = Z[3 * i + r];
    x[3] = 1.0;
    xn = ((double)z[3 * i] - K[2]) / K[0];
    yn = ((double)z[3 * i + 1] - K[3]) / K[1];
  }
  double G[18], *r0 = G + 10, *r1 = G + 14;  // (G packed lower)
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int b = 0; b <= a; ++b) G[tri(a, b)] = x[a] * x[b];
    r0[a] = x[a] * xn;
    r1[a] = x[a] * yn;
  }
  wave_sums<18>(G, n);
  // Cholesky of G (4x4) and two solves
  double L[10], di[4];
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double d = G[tri(j, j)];
#pragma unroll
    for (int k = 0; k < j; ++k) d -= L[tri(j, k)] * L[tri(j, k)];
    ok = ok && d > 0;
    di[j] = near_rsq(d);
#pragma unroll
    for (int c = j + 1; c < 4; ++c) {
      double v = G[tri(c, j)];
#pragma unroll
      for (int k = 0; k < j; ++k) v -= L[tri(c, k)] * L[tri(j, k)];
      L[tri(c, j)] = v * di[j];
    }
  }
  if (!ok) return false;
  double *rhs[2] = {r0, r1};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double *y = rhs[c];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double v = y[k];
#pragma unroll
      for (int q = 0; q < k; ++q) v -= L[tri(k, q)] * y[q];
      y[k] = v * di[k];
    }
#pragma unroll
    for (int k = 3; k >= 0; --k) {
      double v = y[k];
#pragma unroll
      for (int q = k + 1; q < 4; ++q) v -= L[tri(q, k)] * y[q];
      y[k] = v * di[k];
    }
  }
  const double s = 0.5 * (sqrt(r0[0] * r0[0] + r0[1] * r0[1] + r0[2] * r0[2]) +
                          sqrt(r1[0] * r1[0] + r1[1] * r1[1] + r1[2] * r1[2]));
  if (!(s > 0)) return false;
  double c3[3];
  cross3(r0, r1, c3);
  const double is = 1.0 / s;
  double M[9];
  for (int r = 0; r < 3; ++r) {
    M[r] = r0[r] * is;
    M[3 + r] = r1[r] * is;
    M[6 + r] = c3[r] * (is * is);
  }
  near_polar(M, R);
  t[0] = r0[3] * is;
  t[1] = r1[3] * is;
  t[2] = is;
  return true;
}

// Observations of the plain fit: float inputs, the whitening factors of Lambda
// computed once in float64 (3 doubles per keypoint, in LDS).
struct ObsCached {
  const float *z;
  const double *w;
  __device__ void operator()(int i, double zz[2], double ww[3]) const {
    zz[0] = z[3 * i];
    zz[1] = z[3 * i + 1];
    ww[0] = w[3 * i];
    ww[1] = w[3 * i + 1];
    ww[2] = w[3 * i + 2];
  }
};

// Weighted cost sum ||z_i - Pi(R Z_i + t)||^2_Lambda_i of a 2D-3D pose, on a
// whole wavefront: keypoint i on lane i.
template <typename OBS>
__device__ inline double cost_2d_wave(const float *Z, const OBS &obs, int n, const float K[4], const double R[9],
                                      const double t[3]) {
  const int lane = threadIdx.x & 63, i = lane < n ? lane : 0;
  const double m[3] = {Z[3 * i], Z[3 * i + 1], Z[3 * i + 2]};
  double P[3], zz[2], w[3];
  matvec3(R, m, P);
  for (int r = 0; r < 3; ++r) P[r] += t[r];
  const double iz = 1.0 / P[2];
  const double u = (double)K[0] * (P[0] * iz) + K[2], v = (double)K[1] * (P[1] * iz) + K[3];
  obs(i, zz, w);
  const double r0 = zz[0] - u, r1 = zz[1] - v;
  const double a = w[0] * r0 + w[1] * r1, b = w[2] * r1;
  double c[1] = {lane < n ? a * a + b * b : 0.0};
  wave_sums<1>(c, n);
  return c[0];
}

// Arun's method in float64: R = proj_SO3(sum (b_i - bbar)(a_i - abar)^T).
__device__ inline void kabsch_centre(const float *a, const float *b, int n, double R[9], double t[3]) {
  double ab[3] = {0, 0, 0}, bb[3] = {0, 0, 0};
  for (int i = 0; i < n; ++i)
    for (int r = 0; r < 3; ++r) {
      ab[r] += a[3 * i + r];
      bb[r] += b[3 * i + r];
    }
  for (int r = 0; r < 3; ++r) {
    ab[r] /= n;
    bb[r] /= n;
  }
  double H[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = 0; i < n; ++i)
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) H[3 * r + c] += ((double)b[3 * i + r] - bb[r]) * ((double)a[3 * i + c] - ab[c]);
  polar_so3<double>(H, R, 12);
  double ra[3];
  matvec3(R, ab, ra);
  for (int r = 0; r < 3; ++r) t[r] = bb[r] - ra[r];
}

}  // namespace purse
