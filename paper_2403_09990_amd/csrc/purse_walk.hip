// The paper's Step II: the strategic random walk, sampling the rotation
// boundary and the translation boundary separately (Section "The CLOSURE
// Algorithm", Step II; Alg. "d S_R parallel sampler" and, in the appendix
// "Boundary Sampler Algorithms", Alg. "d S_t parallel sampler").
//
// One wavefront per walk.  Per iteration the lanes draw the N_P
// perturbations (up to four per lane) into LDS and rank them by the distance
// to the boundary min_i (beta_i - ||g_i||_Lambda_i) (eq. partial-s-dist) with
// N_P* rounds of a wavefront maximum (ties to the lower perturbation index),
// then test the N_P* x N_T candidates with in_purse, 64 at a time in the order
// of preference m N_P* + k (largest step scale, then highest rank), until a
// round holds a feasible one: its first lane hands its pose to the others.
// The walk's pose is wave-uniform; the keypoints of the walk's instance sit
// in LDS.
//
// Bounded by vector instructions at two wavefronts per SIMD (1000 walks of
// both modes): the ten Philox rounds of each draw (four 32-bit multiply-adds
// per 64-bit product), and the keypoint loop of the distances.  A
// perturbation is drawn once (the candidates and the move drew theirs again),
// set membership compares squares, and the roots and reciprocals of the
// distances are the exact short forms.  2000 walks of 10 iterations, 10
// keypoints: 0.345 -> 0.165 ms; 800 of 8, 3D-3D: 0.245 -> 0.104 ms.
#include "purse_fit.hpp"
#include "purse_launch.hpp"
#include "purse_traj.hpp"

namespace purse {

namespace {

constexpr int kWalkWaves = 4;  // walks per workgroup
constexpr int kWalkBlock = 64 * kWalkWaves;

struct WalkKp {
  float m[3];   // model point a_i / Z_i
  float c[3];   // b_i, or (z_i.x, z_i.y, 0); pose regression: t_i
  float w[3];   // 2D-3D: whitening factor of Lambda_i (upper triangle); pose regression:
                // (beta_i^R, radius_limit(beta_i^R + tau), 0)
  float beta;   // beta_i (pose regression: beta_i^t)
  float lim;    // radius_limit(beta_i + tau)
  float Ri[9];  // pose regression: the hypothesis' rotation R_i
};

// LDS written by other lanes of the wavefront is read after this.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Range of the arguments for which the short forms of the square root and the
// reciprocal are exact, gathered over the keypoints of a pose.
struct ShortRange {
  float lo = 1.f, hi = 1.f;
  __device__ __forceinline__ void see(float x) {
    lo = fminf(lo, x);
    hi = fmaxf(hi, x);
  }
  __device__ __forceinline__ bool exact() const { return lo >= kShortMin && hi <= kShortMax; }
};

// Squared r_i of keypoint k at (R, t) (r2; pose regression: of the translation,
// and f of the rotation ||R - R_i||_F); z is the depth (1 where there is none).
// SHORT: the reciprocal's short form, its argument noted in rg.
template <int KIND, bool SHORT>
__device__ __forceinline__ void walk_r2(const WalkKp &k, const float K[4], const float R[9], const float t[3],
                                        ShortRange &rg, float &z, float &r2, float &f) {
  z = 1.f;
  if (KIND == PURSE_KIND_REG) {
    f = 0.f;
#pragma unroll
    for (int q = 0; q < 9; ++q) f = fmaf(R[q] - k.Ri[q], R[q] - k.Ri[q], f);
    const float e0 = t[0] - k.c[0], e1 = t[1] - k.c[1], e2 = t[2] - k.c[2];
    r2 = fmaf(e0, e0, fmaf(e1, e1, e2 * e2));
    return;
  }
  float P[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) P[r] = fmaf(R[3 * r], k.m[0], fmaf(R[3 * r + 1], k.m[1], fmaf(R[3 * r + 2], k.m[2], t[r])));
  if (KIND == PURSE_KIND_2D3D) {
    z = P[2];
    if (SHORT) rg.see(fabsf(z));
    const float iz = SHORT ? short_rcp(z) : 1.f / z;
    const float e0 = fmaf(K[0], P[0] * iz, K[2]) - k.c[0];
    const float e1 = fmaf(K[1], P[1] * iz, K[3]) - k.c[1];
    const float et0 = fmaf(k.w[0], e0, k.w[1] * e1), et1 = k.w[2] * e1;
    r2 = fmaf(et0, et0, et1 * et1);
    return;
  }
  const float e0 = P[0] - k.c[0], e1 = P[1] - k.c[1], e2 = P[2] - k.c[2];
  r2 = fmaf(e0, e0, fmaf(e1, e1, e2 * e2));
}

// The boundary distance min_i (beta_i - r_i).
template <int KIND, bool SHORT>
__device__ __forceinline__ float walk_distance_of(const WalkKp *kp, int n, const float K[4], const float R[9],
                                                  const float t[3], ShortRange &rg) {
  float d = INFINITY;
#pragma unroll 2
  for (int i = 0; i < n; ++i) {
    const WalkKp k = kp[i];
    float z, r2, f;
    walk_r2<KIND, SHORT>(k, K, R, t, rg, z, r2, f);
    if (SHORT) rg.see(r2);
    if (KIND == PURSE_KIND_REG) {
      if (SHORT) rg.see(f);
      d = fminf(d, k.w[0] - (SHORT ? short_sqrt(f) : sqrtf(f)));
    }
    d = fminf(d, k.beta - (SHORT ? short_sqrt(r2) : sqrtf(r2)));
  }
  return d;
}

// By the short forms, without a branch per keypoint; with the functions
// themselves where an argument was out of their range (a pose on a keypoint).
template <int KIND>
__device__ __forceinline__ float walk_distance(const WalkKp *kp, int n, const float K[4], const float R[9],
                                               const float t[3]) {
  ShortRange rg;
  float d = walk_distance_of<KIND, true>(kp, n, K, R, t, rg);
  if (__builtin_expect(!rg.exact(), 0)) d = walk_distance_of<KIND, false>(kp, n, K, R, t, rg);
  return d;
}

// Whether the pose is in S (r_i <= beta_i + tau, depth > z_min); ends when no
// lane of the wavefront is.
template <int KIND>
__device__ __forceinline__ bool walk_inside(const WalkKp *kp, int n, const float K[4], const float R[9],
                                            const float t[3], float z_min) {
  bool ok = true;
  for (int i = 0; i < n; i += 2) {
    // (an odd count tests its last keypoint twice)
    const WalkKp k0 = kp[i], k1 = kp[min(i + 1, n - 1)];
    float z0, z1, r0, r1, f0 = 0.f, f1 = 0.f;
    ShortRange rg;
    walk_r2<KIND, true>(k0, K, R, t, rg, z0, r0, f0);
    walk_r2<KIND, true>(k1, K, R, t, rg, z1, r1, f1);
    if (KIND == PURSE_KIND_2D3D) {
      if (__builtin_expect(!rg.exact(), 0)) {
        walk_r2<KIND, false>(k0, K, R, t, rg, z0, r0, f0);
        walk_r2<KIND, false>(k1, K, R, t, rg, z1, r1, f1);
      }
      ok = ok & (z0 > z_min) & (z1 > z_min);
    }
    ok = ok & (r0 <= k0.lim) & (r1 <= k1.lim);
    if (KIND == PURSE_KIND_REG) ok = ok & (f0 <= k0.w[1]) & (f1 <= k1.w[1]);
    if (__ballot(ok) == 0ull) return false;
  }
  return ok;
}

// Three 24-bit uniforms of (walk, iteration, perturbation) under key
// (seed, 1 + mode): a direction and a magnitude fraction.
__device__ __forceinline__ void walk_draw(uint64_t seed, int mode, uint64_t walk, uint32_t it, uint32_t j,
                                          float dir[3], float &frac) {
  uint64_t c[4] = {walk, (uint64_t)it, (uint64_t)j, 0ull};
  philox4x64_10(c, seed, 1ull + (uint64_t)mode);
  const float u1 = (float)(c[0] >> 40) * 0x1p-24f;
  const float u2 = (float)(c[1] >> 40) * 0x1p-24f;
  frac = (float)(c[2] >> 40) * 0x1p-24f;
  const float z = 1.f - 2.f * u1;
  const float rho = exact_sqrt(fmaxf(0.f, 1.f - z * z));
  float sp, cp;
  sincospif(2.f * u2, &sp, &cp);
  dir[0] = rho * cp;
  dir[1] = rho * sp;
  dir[2] = z;
}

__device__ __forceinline__ void left_rotate(const float w[3], const float R[9], float out[9]) {
  float E[9];
  exp_so3(w, E);
  matmul3(E, R, out);
}

// Maximum over the wavefront (no NaN), in every lane: butterflies within rows
// of 16 lanes, then across the rows.
template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
  const int y = __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false);
  return fmaxf(x, __int_as_float(y));
}
__device__ __forceinline__ float wave_max(float x) {
  x = dpp_max<0xB1>(x);   // quad_perm [1,0,3,2]
  x = dpp_max<0x4E>(x);   // quad_perm [2,3,0,1]
  x = dpp_max<0x141>(x);  // row_half_mirror
  x = dpp_max<0x140>(x);  // row_mirror
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

template <int CTRL>
__device__ __forceinline__ int dpp_min(int x) {
  return min(x, __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ int wave_min(int x) {
  x = dpp_min<0x140>(dpp_min<0x141>(dpp_min<0x4E>(dpp_min<0xB1>(x))));
  return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

__device__ __forceinline__ float bcast(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

struct WalkLds {
  WalkKp kp[PURSE_MAX_KP];
  float4 pert[kWalkMaxPerturb];  // direction and size of the iteration's perturbations
  float4 kept[kWalkMaxKeep];     // the N_P* kept ones, by rank
  float scale[kWalkMaxScales];   // gamma^m
};

// The iterations of one walk (a whole wavefront); R, t and vel are uniform.
template <int KIND>
__device__ __forceinline__ void walk_steps(WalkLds &L, int n, const float K[4], const WalkParams &wp, float z_min,
                                           int mode, uint64_t seed, uint64_t walk, const float vel[3], float R[9],
                                           float t[3], int32_t *decisions) {
  const int lane = threadIdx.x & 63;
  const int NP = wp.n_perturb, NK = wp.n_keep, NT = wp.n_scales;
  const float pscale = mode == 0 ? wp.t_pert : wp.r_pert;
  // c / NK for c < 512 (NK <= 16) by a 16-bit reciprocal
  const uint32_t inv_k = (65536u + (uint32_t)NK - 1u) / (uint32_t)NK;
  for (int it = 0; it < wp.n_iters; ++it) {
    // ---- N_P perturbations, their boundary distances
    float dq[4];
    int jq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int jj = lane + 64 * q;
      jq[q] = jj;
      dq[q] = -INFINITY;
      if (jj < NP) {
        float dir[3], frac;
        walk_draw(seed, mode, walk, (uint32_t)it, (uint32_t)jj, dir, frac);
        const float s = pscale * frac;
        L.pert[jj] = make_float4(dir[0], dir[1], dir[2], s);
        float Rj[9], tj[3];
        if (mode == 0) {
#pragma unroll
          for (int k = 0; k < 9; ++k) Rj[k] = R[k];
#pragma unroll
          for (int r = 0; r < 3; ++r) tj[r] = fmaf(s, dir[r], t[r]);
        } else {
          const float w[3] = {s * dir[0], s * dir[1], s * dir[2]};
          left_rotate(w, R, Rj);
#pragma unroll
          for (int r = 0; r < 3; ++r) tj[r] = t[r];
        }
        dq[q] = walk_distance<KIND>(L.kp, n, K, Rj, tj);
      }
    }
    // ---- the N_P* largest, in rank order: lane k keeps the k-th's index
    int keep = 0;
    for (int k = 0; k < NK; ++k) {
      float bd = -INFINITY;
      int bj = INT32_MAX;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (jq[q] < NP && (dq[q] > bd || (dq[q] == bd && jq[q] < bj))) {
          bd = dq[q];
          bj = jq[q];
        }
      const float top = wave_max(bd);
      // (equal distances are usual in pose regression: the ball of the part
      // that is not perturbed may be the nearest)
      const int at = bd == top ? bj : INT32_MAX;
      const unsigned long long who = __ballot(at != INT32_MAX);
      const int j = __popcll(who) == 1 ? __builtin_amdgcn_readlane(at, __ffsll(who) - 1) : wave_min(at);
      keep = lane == k ? j : keep;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (jq[q] == j) jq[q] = INT32_MAX;  // picked
    }
    wave_lds_sync();
    if (lane < NK) L.kept[lane] = L.pert[min(keep, NP - 1)];
    wave_lds_sync();
    // ---- candidates (m, k) in order of preference, 64 at a time
    const int C = NT * NK;
    int code = -1;
    for (int c0 = 0; c0 < C; c0 += 64) {
      const int c = c0 + lane;
      const int m = (int)(((uint32_t)min(c, C - 1) * inv_k) >> 16), k = min(c, C - 1) - m * NK;
      const float4 u = L.kept[k];
      const float scale = L.scale[m];
      float Rc[9], tc[3];
      if (mode == 0) {
        const float w[3] = {vel[0] * scale, vel[1] * scale, vel[2] * scale};
        left_rotate(w, R, Rc);
        tc[0] = fmaf(u.w, u.x, t[0]);
        tc[1] = fmaf(u.w, u.y, t[1]);
        tc[2] = fmaf(u.w, u.z, t[2]);
      } else {
        const float w[3] = {u.w * u.x, u.w * u.y, u.w * u.z};
        left_rotate(w, R, Rc);
#pragma unroll
        for (int r = 0; r < 3; ++r) tc[r] = fmaf(vel[r], scale, t[r]);
      }
      const bool in = walk_inside<KIND>(L.kp, n, K, Rc, tc, z_min);
      const unsigned long long hit = __ballot(in && c < C);
      if (hit) {
        const int w = __ffsll(hit) - 1;
#pragma unroll
        for (int k2 = 0; k2 < 9; ++k2) R[k2] = bcast(Rc[k2], w);
#pragma unroll
        for (int r = 0; r < 3; ++r) t[r] = bcast(tc[r], w);
        const int best = c0 + w, bm = (int)(((uint32_t)best * inv_k) >> 16);
        code = (best - bm * NK) * NT + bm;
        break;
      }
    }
    if (decisions && lane == 0) decisions[it] = code;
  }
}

}  // namespace

// Per instance: the average rotation proj_SO3(sum R0) and translation of its
// starts (the parallel samplers' first lines), in float64.
__global__ void __launch_bounds__(64) k_walk_centre(DevBatch b, const int64_t *__restrict__ start_off,
                                                    int64_t total_starts, const float *__restrict__ starts,
                                                    float *centre) {
  const int j = blockIdx.x, lane = threadIdx.x;
  int64_t s0 = start_off[j], s1 = start_off[j + 1];
  if (s0 < 0 || s1 < s0 || s1 > total_starts) s0 = s1 = 0;
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  for (int64_t s = s0 + lane; s < s1; s += 64)
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] += (double)starts[12 * s + k];
#pragma unroll
  for (int k = 0; k < 12; ++k)
    for (int o = 32; o >= 1; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
  if (lane == 0) {
    double Rb[9];
    if (s1 > s0) {
      polar_so3<double>(acc, Rb, 12);
    } else {
      for (int k = 0; k < 9; ++k) Rb[k] = (k % 4 == 0) ? 1.0 : 0.0;
    }
    const double inv = s1 > s0 ? 1.0 / (double)(s1 - s0) : 0.0;
    for (int k = 0; k < 9; ++k) centre[12 * j + k] = (float)Rb[k];
    for (int r = 0; r < 3; ++r) centre[12 * j + 9 + r] = (float)(acc[9 + r] * inv);
  }
}

__global__ void __launch_bounds__(kWalkBlock) k_walk(DevBatch b, DevParams p, WalkParams wp,
                                                     const int64_t *__restrict__ start_off, int64_t total_starts,
                                                     const float *__restrict__ starts,
                                                     const float *__restrict__ centre, float *poses, uint8_t *mask,
                                                     int32_t *decisions) {
  __shared__ WalkLds lds[kWalkWaves];
  // (uniform over the wavefront, and known to be)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mode = blockIdx.y;
  const int64_t n_walks = total_starts * wp.n_walks;
  const int64_t g = (int64_t)blockIdx.x * kWalkWaves + wave;
  if (g >= n_walks) return;  // (whole wavefront)
  const int64_t sg = g / wp.n_walks;
  const int nw = (int)(g % wp.n_walks);
  // instance of start sg: the last j with start_off[j] <= sg
  int lo = 0, hi = b.n_inst - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start_off[mid] <= sg)
      lo = mid;
    else
      hi = mid - 1;
  }
  const int j = lo;
  const int64_t out_i = (int64_t)mode * n_walks + g;
  float *out = poses + 12 * out_i;
  float R[9], t[3];
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = starts[12 * sg + k];
#pragma unroll
  for (int r = 0; r < 3; ++r) t[r] = starts[12 * sg + 9 + r];
  const int kind = b.kind[j], n = b.n_kp[j];
  const int64_t ko = b.kp_off[j];
  const bool valid = (kind == PURSE_KIND_3D3D || kind == PURSE_KIND_2D3D || kind == PURSE_KIND_REG) && n >= 1 &&
                     n <= PURSE_MAX_KP && ko >= 0 && b.kp_off[j + 1] - ko == n && b.kp_off[j + 1] <= b.total_kp;
  if (!valid) {  // (whole wavefront) the start is returned as it is, not in S
    if (lane < 12) out[lane] = starts[12 * sg + lane];
    if (lane == 0) mask[out_i] = 0;
    if (decisions)
      for (int it = lane; it < wp.n_iters; it += 64) decisions[out_i * wp.n_iters + it] = -1;
    return;
  }
  const bool is2d = kind == PURSE_KIND_2D3D, isreg = kind == PURSE_KIND_REG;
  float K[4];
  for (int k = 0; k < 4; ++k) K[k] = is2d ? b.intrinsics[4 * j + k] : 0.f;
  const float tau = is2d ? p.tau2 : p.tau3;
  WalkLds &L = lds[wave];
  if (lane < n) {
    const int64_t q = ko + lane;
    WalkKp k;
    for (int r = 0; r < 3; ++r) {
      k.m[r] = isreg ? 0.f : b.model_pts[3 * q + r];
      k.c[r] = (r < 2 || !is2d) ? b.centres[3 * q + r] : 0.f;
      k.w[r] = 0.f;
    }
    for (int r = 0; r < 9; ++r) k.Ri[r] = 0.f;
    if (is2d) {
      double w[3];
      whiten_factor<double>(b.shapes + 4 * q, w);
      for (int r = 0; r < 3; ++r) k.w[r] = (float)w[r];
    }
    if (isreg) {
      // hypothesis i: rotation from its unit quaternion (shapes), its
      // rotation bound (model_pts x)
      const float *qq = b.shapes + 4 * q;
      const float qn = rsqrtf(qq[0] * qq[0] + qq[1] * qq[1] + qq[2] * qq[2] + qq[3] * qq[3]);
      rot_from_quat(make_float4(qq[0] * qn, qq[1] * qn, qq[2] * qn, qq[3] * qn), k.Ri);
      k.w[0] = b.model_pts[3 * q];
      k.w[1] = radius_limit(b.model_pts[3 * q] + tau);
    }
    k.beta = b.bounds[q];
    k.lim = radius_limit(b.bounds[q] + tau);
    L.kp[lane] = k;
  }
  if (lane < wp.n_scales) {
    float scale = 1.f;
    for (int q = 0; q < lane; ++q) scale *= wp.gamma;
    L.scale[lane] = scale;
  }
  wave_lds_sync();
  const uint64_t seed = b.seed[j];
  const uint64_t walk = (uint64_t)((sg - start_off[j]) * wp.n_walks + nw);  // instance-local walk index
  // initial velocity: radial direction from the centre of the starts plus a
  // random unit vector
  float vel[3];
  {
    float dir[3], frac;
    walk_draw(seed, mode, walk, 0xFFFFFFFFu, 0u, dir, frac);
    const float *C = centre + 12 * j;
    float u[3];
    if (mode == 0) {
      float Y[9];
      // R0 R_bar^T
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) Y[3 * r + c] = R[3 * r] * C[3 * c] + R[3 * r + 1] * C[3 * c + 1] + R[3 * r + 2] * C[3 * c + 2];
      log_so3(Y, u);
    } else {
      for (int r = 0; r < 3; ++r) u[r] = t[r] - C[9 + r];
    }
    const float n2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const float in = n2 > 0.f ? rsqrtf(n2) : 0.f;
    const float mag = mode == 0 ? wp.omega0 : wp.v0;
    for (int r = 0; r < 3; ++r) vel[r] = mag * (u[r] * in + dir[r]);
  }
  int32_t *dec = decisions ? decisions + out_i * wp.n_iters : nullptr;
  bool inside;
  if (is2d) {
    walk_steps<PURSE_KIND_2D3D>(L, n, K, wp, p.z_min, mode, seed, walk, vel, R, t, dec);
    inside = walk_inside<PURSE_KIND_2D3D>(L.kp, n, K, R, t, p.z_min);
  } else if (isreg) {
    walk_steps<PURSE_KIND_REG>(L, n, K, wp, p.z_min, mode, seed, walk, vel, R, t, dec);
    inside = walk_inside<PURSE_KIND_REG>(L.kp, n, K, R, t, p.z_min);
  } else {
    walk_steps<PURSE_KIND_3D3D>(L, n, K, wp, p.z_min, mode, seed, walk, vel, R, t, dec);
    inside = walk_inside<PURSE_KIND_3D3D>(L.kp, n, K, R, t, p.z_min);
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) out[k] = R[k];
#pragma unroll
    for (int r = 0; r < 3; ++r) out[9 + r] = t[r];
    mask[out_i] = inside ? PURSE_MASK_FEASIBLE : 0;
  }
}

void launch_walk(const DevBatch &b, const DevParams &p, const WalkParams &wp, const int64_t *start_off,
                 int64_t total_starts, const float *starts, float *centre, float *poses, uint8_t *mask,
                 int32_t *decisions, hipStream_t stream) {
  hipLaunchKernelGGL(k_walk_centre, dim3(b.n_inst), dim3(64), 0, stream, b, start_off, total_starts, starts, centre);
  const int64_t n_walks = total_starts * wp.n_walks;
  if (n_walks == 0) return;
  const dim3 grid((unsigned)((n_walks + kWalkWaves - 1) / kWalkWaves), 2u);
  hipLaunchKernelGGL(k_walk, grid, dim3(kWalkBlock), 0, stream, b, p, wp, start_off, total_starts, starts, centre,
                     poses, mask, decisions);
}

}  // namespace purse
