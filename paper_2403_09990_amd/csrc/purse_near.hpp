// Float64 building blocks of the kernels that run few wavefronts (the
// prologue's fits, the backward's sweeps), where the length of the instruction
// chain is the time: sums over lanes by row permutations, reciprocals and roots
// by Newton steps, Exp by its series, the Gauss-Newton step.
#pragma once

#include "purse_device.hpp"

namespace purse {

// (bound_ctrl lets the compiler fold a float's move into its add)
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

template <int G, typename T>
__device__ __forceinline__ T group_sum(T x) {
  static_assert(G == 2 || G == 4 || G == 8 || G == 16, "lane groups within a row of 16");
  x += dpp_of<0xB1>(x);                // quad_perm [1,0,3,2]
  if (G >= 4) x += dpp_of<0x4E>(x);    // [2,3,0,1]
  if (G >= 8) x += dpp_of<0x141>(x);   // half mirror
  if (G >= 16) x += dpp_of<0x140>(x);  // row mirror
  return x;
}

// The sums of N values over a group of 16, a step of nine values at a time: a
// lone wavefront otherwise waits in each value's chain of four dependent steps
// (one instance of 12 keypoints, 100 iterations: 1.36 -> 1.23 ms; by the
// float64 4x4x4 matrix instruction against ones, 1.62).
template <int CTRL, int N, typename T>
__device__ __forceinline__ void group_step(T *x) {
  T y[N];
#pragma unroll
  for (int k = 0; k < N; ++k) y[k] = dpp_of<CTRL>(x[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) x[k] += y[k];
  __builtin_amdgcn_sched_barrier(0);
}
template <int N, typename T>
__device__ __forceinline__ void group_sums(T *x) {
  constexpr int M = N < 9 ? N : 9;
  group_step<0xB1, M>(x);
  group_step<0x4E, M>(x);
  group_step<0x141, M>(x);
  group_step<0x140, M>(x);
  if constexpr (N > M) group_sums<N - M>(x + M);
}

// Lane `lane`'s value, uniform.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// The sums of N values over the wavefront, uniform in every lane; n: lanes
// 0..n - 1 hold values, the others zeros (one row of 16 needs no more).
template <int N>
__device__ __forceinline__ void wave_sums(double *x, int n) {
  group_sums<N>(x);
  if (n <= 16) {
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = lane_value(x[k], 0);
  } else {
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = (lane_value(x[k], 0) + lane_value(x[k], 16)) + (lane_value(x[k], 32) + lane_value(x[k], 48));
  }
}

// (1 - cos x) / x^2 and (x - sin x) / x^3 from z = x^2: their Taylor series for
// |x| <= 1/2 (truncation below 1e-17), else by half angles.
__device__ __forceinline__ void exp_coeffs_bd(double z, double &B, double &Dc, double &A) {
  if (z <= 0.25) {
    B = 0.5 + z * (-1.0 / 24 + z * (1.0 / 720 + z * (-1.0 / 40320 + z * (1.0 / 3628800 + z * (-1.0 / 479001600 +
        z * (1.0 / 87178291200.0))))));
    Dc = 1.0 / 6 + z * (-1.0 / 120 + z * (1.0 / 5040 + z * (-1.0 / 362880 + z * (1.0 / 39916800 +
         z * (-1.0 / 6227020800.0 + z * (1.0 / 1307674368000.0))))));
    A = 1.0 - z * Dc;
  } else {
    const double x = sqrt(z);
    double s, c, sh, ch;
    sincos(x, &s, &c);
    sincos(0.5 * x, &sh, &ch);
    A = s / x;
    B = 2.0 * sh * sh / z;
    Dc = (1.0 - A) / z;
  }
}

// Reciprocal and reciprocal square root for chains of float64 steps: in float64
// the hardware approximation (2^-26 or better) and two Newton steps, a few units
// in the last place and a third of the instructions of the correctly rounded
// forms (arguments are depths, squared radii and pivots, far from the ends of
// the range).
__device__ __forceinline__ float near_rcp(float x) { return drcp(x); }
__device__ __forceinline__ float near_rsq(float x) { return drsqrt(x); }
__device__ __forceinline__ double near_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double near_rsq(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * fma(-x * r, r, 1.0), r, r);
  return fma(0.5 * fma(-x * r, r, 1.0), r, r);
}

// Exp of so(3) in float64: the Taylor series of its coefficients for angles up
// to 1/2 (no square root or trigonometric call), else the general form.
__device__ __forceinline__ void near_exp_so3(const double w[3], double E[9]) {
  const double z = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  if (z <= 0.25) {
    double B, Dc, A;
    exp_coeffs_bd(z, B, Dc, A);
    const double C = 1.0 - z * B;
    const double b0 = B * w[0], b1 = B * w[1], a0 = A * w[0], a1 = A * w[1], a2 = A * w[2];
    E[0] = C + b0 * w[0];
    E[4] = C + b1 * w[1];
    E[8] = C + B * w[2] * w[2];
    E[1] = b0 * w[1] - a2;
    E[3] = b0 * w[1] + a2;
    E[2] = b0 * w[2] + a1;
    E[6] = b0 * w[2] - a1;
    E[5] = b1 * w[2] - a0;
    E[7] = b1 * w[2] + a0;
  } else {
    exp_so3<double>(w, E);
  }
}

// The Gauss-Newton solve A d = g in float64: the factor's off-diagonal entries L
// and reciprocal diagonal dinv; false when a pivot is not positive.
__device__ __forceinline__ bool near_solve(const double A[21], const double g[6], double L[21], double dinv[6],
                                           double d[6]) {
  bool ok = true;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double v = A[tri(j, j)];
#pragma unroll
    for (int k = 0; k < j; ++k) v -= L[tri(j, k)] * L[tri(j, k)];
    ok = ok && v > 0.0;
    dinv[j] = near_rsq(v);
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      double x = A[tri(i, j)];
#pragma unroll
      for (int k = 0; k < j; ++k) x -= L[tri(i, k)] * L[tri(j, k)];
      L[tri(i, j)] = x * dinv[j];
    }
  }
  if (!ok) return false;
  chol6_subst<double>(L, dinv, g, d);  // (it reads no diagonal entry of L)
  return true;
}

// The left update about o by the step d.
__device__ __forceinline__ void near_update(const double d[6], const double o[3], double R[9], double t[3]) {
  double E[9], Rn[9], arm[3], e[3];
  near_exp_so3(d, E);
  matmul3(E, R, Rn);
#pragma unroll
  for (int r = 0; r < 3; ++r) arm[r] = t[r] - o[r];
  matvec3(E, arm, e);
#pragma unroll
  for (int r = 0; r < 3; ++r) t[r] = e[r] + o[r] + d[3 + r];
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = Rn[k];
}

// R = proj_SO3(M) in float64 for det M > 0 by Newton's iteration for the
// orthogonal polar factor, X <- (X + X^-T) / 2 from M scaled to unit mean square
// singular value: four to eight steps, each squaring the distance.  Jacobi
// (three quarters of the DLT start's chain) where det M is not clearly positive
// or the steps do not settle.
__device__ __forceinline__ void near_polar(const double M[9], double R[9]) {
  double f2 = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) f2 += M[k] * M[k];
  const double sc = near_rsq(f2 * (1.0 / 3.0));
  double X[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) X[k] = M[k] * sc;
  bool settled = false;
  for (int it = 0; it < 24; ++it) {
    double C[9];
    cross3(X + 3, X + 6, C);
    cross3(X + 6, X, C + 3);
    cross3(X, X + 3, C + 6);
    const double det = X[0] * C[0] + X[1] * C[1] + X[2] * C[2];
    if (!(det > 1e-6)) break;
    const double h = 0.5 * near_rcp(det);
    double move = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double y = fma(h, C[k], 0.5 * X[k]);
      move = fmax(move, fabs(y - X[k]));
      X[k] = y;
    }
    if (move < 1e-9) {  // (the next step would move by its square)
      settled = true;
      break;
    }
  }
  if (settled) {
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = X[k];
  } else {
    polar_so3<double>(M, R, 12);
  }
}

}  // namespace purse
