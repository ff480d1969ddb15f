// Minimum enclosing geodesic balls of the feasible samples by geodesic
// gradient descent, one workgroup per (instance, chain): chain 0 is the
// rotation ball (unit quaternions, Frobenius key ||C - R||_F^2 =
// 2 |a - b|^2 |a + b|^2), chain 1 the translation ball.
//
// Each step needs the farthest sample from the current centre.  The chain
// keeps a shell of candidates in LDS: at a rescan with reference centre C_ref
// and radius r_ref it keeps every sample with d(C_ref, s) >= theta (theta from
// a histogram, so the shell fits).  By the triangle inequality a sample
// outside the shell is at most theta + d(C, C_ref) from the current centre C,
// so when the shell's best exceeds that bound (with a rounding slack) the
// shell argmax is the argmax over all samples and the step is exact; when it
// does not, the chain rescans around the current centre.  Only undominated
// samples enter the shell (struct Domination): those that can be the farthest
// from some centre within a ball that holds the rest of the descent's path, a
// few per cent of the samples after 16 steps and a few dozen after 256.  Steps
// on the shell run in one wavefront with shuffles only, or, once the winners
// keep coming from a few samples, pipelined: one wavefront runs the descent
// ahead with predicted winners and the others check each step's argmax.
#include <float.h>

#include <type_traits>

#include "purse_bwd_check.hpp"
#include "purse_geodesic.hpp"
#include "purse_launch.hpp"
#include "purse_traj.hpp"

namespace purse {

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kBins = 256;
// Steps of a stage of scan steps; after every rescan that left no shell to step
// on, twice as many, up to kScanMax (samples at one distance from the centre:
// a rescan costs 6 to 15 scans and changes nothing).
constexpr int kScanSteps = 16, kScanMax = 1024;
constexpr int kScanRest = 8;  // last steps that are scanned rather than rescanned for
// samples per thread of the per-sample passes (k_megb_prep, k_megb_radii):
// kPassPer on instances of at least kPassPerMin samples, else one
constexpr int kPassPer = 4;
constexpr int64_t kPassPerMin = 1 << 17;
constexpr int kChainBlock = 512;  // threads of a pipelined chain workgroup (the larger variant)
constexpr int kChainWaves = kChainBlock / 64;
// Variants of the chain workgroup:
//  - kChainWide: eight waves, a shell of 7168 entries and 256 VGPRs (one
//    chain per compute unit);
//  - kChainNarrow: four waves, a shell of 1280 entries and 128 VGPRs, so that
//    four chains share a compute unit (LDS).
constexpr int kChainWide = 1, kChainNarrow = 2;
template <int V>
constexpr int chain_block() { return V == kChainWide ? kChainBlock : 256; }
template <int V>
constexpr int chain_cap() { return V == kChainWide ? 7168 : 1280; }
constexpr int kUnroll = 8;
constexpr int kCap = 7168;
constexpr int kMaxChunks = kCap / 64;
constexpr int kRecentreChunks = 4;  // a step scanning more chunks than this ...
constexpr int kMinShellSteps = 64;   // ... at least this many steps after a rescan triggers a new one
constexpr int kRecentreDiv = 2048;   // (more chunks, up to kRecentreMax, when a rescan streams more
constexpr int kRecentreMax = 32;     //  entries: one chunk per kRecentreDiv of them)
constexpr int kPipeSteps = 64;       // steps per round of a pipelined segment (one per lane)
constexpr int kVerifySkip = 4;       // wave on wave 0's SIMD (waves go round the 4 SIMDs)
constexpr int kPipeMinSeq = 8;       // steps with no new winner before a pipelined segment, doubled after
constexpr int kPipeMaxSeq = 256;     // each failed prediction up to this
static_assert(kCap % 64 == 0, "chunks of 64 tile the shell");

// Chunks a shell step may scan before its stage ends and the chain rescans
// (once kMinShellSteps steps have been taken since the last rescan).  A
// rescan that streams n_src entries costs in proportion to them, so the more
// it streams the more chunks a step may scan first.
__device__ __forceinline__ int recentre_chunks(int n_src) {
  return min(kRecentreMax, max(kRecentreChunks, n_src / kRecentreDiv));
}

__device__ __forceinline__ bool feasible_pt(float4 a, int chain) {
  return chain == 0 ? (a.x >= 0.f) : (a.w != 0.f);
}

// Squared distance: ||R_a - R_b||_F^2 = 2 |a - b|^2 |a + b|^2 for unit
// quaternions a, b (chain 0; both chords are formed directly, so the key stays
// accurate whichever sign b carries); |a - b|^2 for translations (chain 1).
// The sums are written as explicit fused multiply-adds so that every code path
// (shell steps, full scans, the multi-workgroup first phase) rounds a key the
// same way and takes the same argmax decisions.
__device__ __forceinline__ float sqdist(float4 a, float4 b, int chain) {
  if (chain == 0) {
    const float m0 = a.x - b.x, m1 = a.y - b.y, m2 = a.z - b.z, m3 = a.w - b.w;
    const float p0 = a.x + b.x, p1 = a.y + b.y, p2 = a.z + b.z, p3 = a.w + b.w;
    const float x = fmaf(m3, m3, fmaf(m2, m2, fmaf(m1, m1, m0 * m0)));
    const float y = fmaf(p3, p3, fmaf(p2, p2, fmaf(p1, p1, p0 * p0)));
    return (2.f * x) * y;
  }
  const float d0 = a.x - b.x, d1 = a.y - b.y, d2 = a.z - b.z;
  return fmaf(d2, d2, fmaf(d1, d1, d0 * d0));
}

// (key desc, id asc) comparison
__device__ __forceinline__ bool better(float k1, int i1, float k2, int i2) {
  return k1 > k2 || (k1 == k2 && i1 < i2);
}

// Wavefront reductions by DPP row permutes: within each row of 16 lanes
// (quad swaps, half-row and row mirrors), then row broadcasts 15 and 31 carry
// the partial results up, so lane 63 ends with the reduction of all 64 lanes.
__device__ __forceinline__ int wave_max_i32(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x140, 0xF, 0xF, false));  // row_mirror
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int wave_min_i32(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0xB1, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x4E, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x141, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x140, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x142, 0xA, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x143, 0xC, 0xF, false));
  return __builtin_amdgcn_readlane(v, 63);
}

// Keys are squared distances (>= 0) or the sentinel -1: their float bit
// patterns order like the values under signed integer comparison.
__device__ __forceinline__ float wave_max_key(float k) { return __int_as_float(wave_max_i32(__float_as_int(k))); }

// Wavefront argmax (key desc, id asc); every lane gets the winning key and id.
__device__ __forceinline__ void wave_argmax(float k, int id, float &wk, int &wi) {
  wk = wave_max_key(k);
  wi = wave_min_i32(k == wk ? id : INT32_MAX);
}

// Running sum of the last iterates: rotation matrices (chain 0) or centres.
// The rotation of the unit quaternion (w, x, y, z) is written out with
// explicit fused multiply-adds, so that every code path (full scans, shell
// steps) rounds the sum the same way.
__device__ __forceinline__ void accumulate_iterate(float4 C, int chain, float acc[9]) {
  if (chain == 0) {
    const float w = C.x, x = C.y, y = C.z, z = C.w;
    acc[0] += fmaf(-2.f, fmaf(y, y, z * z), 1.f);
    acc[1] = fmaf(2.f, fmaf(x, y, -(w * z)), acc[1]);
    acc[2] = fmaf(2.f, fmaf(x, z, w * y), acc[2]);
    acc[3] = fmaf(2.f, fmaf(x, y, w * z), acc[3]);
    acc[4] += fmaf(-2.f, fmaf(x, x, z * z), 1.f);
    acc[5] = fmaf(2.f, fmaf(y, z, -(w * x)), acc[5]);
    acc[6] = fmaf(2.f, fmaf(x, z, -(w * y)), acc[6]);
    acc[7] = fmaf(2.f, fmaf(y, z, w * x), acc[7]);
    acc[8] += fmaf(-2.f, fmaf(x, x, y * y), 1.f);
  } else {
    acc[0] += C.x;
    acc[1] += C.y;
    acc[2] += C.z;
  }
}

__device__ __forceinline__ float wave_max(float v) { return wave_max_key(v); }

// Streams elements [0, M) of src to the workgroup in rounds of
// BLOCK * kUnroll elements (element s0 + u * BLOCK + tid to thread
// tid, past M the pad value).  The loads of the next round are issued before
// the current round is handed to f(vals, s0), so two rounds are in flight.
// Loads are unconditional at an index clamped to M - 1 (vector loads, and no
// branch that would make the wait counts conservative); the pad is selected
// afterwards.
template <int BLOCK, int U = kUnroll, typename T, typename F>
__device__ __forceinline__ void stream_rounds(const T *__restrict__ src, int M, T pad, F &&f) {
  constexpr int R = BLOCK * U;
  if (M <= 0) return;
  const int tid = threadIdx.x;
  const int last = M - 1;
  T cur[U];
#pragma unroll
  for (int u = 0; u < U; ++u) cur[u] = src[min(u * BLOCK + tid, last)];
  for (int s0 = 0; s0 < M; s0 += R) {
    T nxt[U];  // (the last round reloads in-range elements it does not use)
#pragma unroll
    for (int u = 0; u < U; ++u) nxt[u] = src[min(s0 + R + u * BLOCK + tid, last)];
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = s0 + u * BLOCK + tid < M ? cur[u] : pad;
    f(v, s0);
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
  }
}

}  // namespace

__global__ void k_megb_init(int n_inst, MegbRec *rec) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_inst) return;
  rec[j].first = INT32_MAX;
  rec[j].n_feasible = 0ull;
  rec[j].max_rot = 0ull;
  rec[j].max_trans = 0ull;
  rec[j].dm_n[0] = rec[j].dm_n[1] = 0;
  rec[j].dm_rho[0] = rec[j].dm_rho[1] = 0.f;
  rec[j].ck_hash = 0ull;
  rec[j].ck_T = 0;
  rec[j].ck_every = 0;
}

// Bin of d among kBins bins of width 1 / rw from lo (rw the reciprocal of
// the width, so a pass over every sample takes no division).  The rounding of
// the product can move d by one bin near an edge, which shifts the bins'
// edges as bounds by about 1e-7 of the distance, far inside the shell
// checks' slack; every pass uses this same function, so counts and members
// agree.
__device__ __forceinline__ int bin_of(float d, float lo, float rw) {
  int b = (int)((d - lo) * rw);
  return b < 0 ? 0 : (b >= kBins ? kBins - 1 : b);
}

// ---------------------------------------------------------------------------
// Domination.  In R^4 (unit quaternions a, b, the sign of b such that
// C_ref . b >= 0) and in R^3 (translations) the difference of two samples'
// squared distances |C - b|^2 is affine in the centre C, so for a witness w
//   |C - w|^2 - |C - s|^2 >= |C_ref - w|^2 - |C_ref - s|^2 - 2 rho |s - w|
// for every C within rho of C_ref.  A sample s for which the right side is
// positive (by more than the keys' rounding) is nearer than w to each such
// centre: it is no farthest sample there and can be left out.  The relation
// is transitive, so a witness may itself be left out.  (A bound by the
// triangle inequality instead keeps every sample within 2 rho of the radius:
// 65,536 of 2^20 samples after 32 steps against 6,000-18,000 here, and 7,168
// against 40-1,600 after 128.)
//
// Witnesses are the last distinct winners, at most eight.  C_ref is the mean
// of the iterates of the later half of the steps taken (the iterates zigzag
// about their limit): of the kept ones (checkpoints) for rotations, of at most
// the last 64 for translations, else the current iterate.  rho is a multiple of the next step's length, h / i: the rest of
// the path from step i on stays within 0.6-1.4 such lengths of that mean, and
// within 1.0-2.1 of the iterate itself, on the clouds it was measured on; a
// centre beyond it only ends the stage.
struct Domination {
  float4 w[8];   // witnesses, on C_ref's side
  float xw[8];   // |C_ref - w|^2
  float4 C;      // C_ref
  float xmax;    // largest xw
  float rho, rho_min;  // radius, and the least one worth a pass over the samples
  int n;         // witnesses (0: nothing is dominated and any centre is allowed)
};

// The radius with what a pass over the samples and the step's check take
// from it.  eta covers the rounding of the float32 keys: each is within 8e-7
// of its value relatively (and unit quaternions are so to 2e-7), and xw, xs
// within 4e-7, against 1e-5 here.
struct DomBall {
  float chk;    // a centre is outside from |C - C_ref|^2 > chk on
  float four;   // (2 rho)^2
  float xin;    // samples nearer than this are dominated whatever their direction
  float eta;
};
__device__ __forceinline__ DomBall dom_ball(const Domination &S, float rho) {
  DomBall b;
  if (S.n == 0) return DomBall{INFINITY, FLT_MAX, -1.f, FLT_MAX};
  const float rw = __builtin_amdgcn_sqrtf(S.xmax);
  b.chk = rho * rho * (1.f - 1e-5f);
  b.four = 4.f * rho * rho * (1.f + 4e-5f);
  b.eta = 1e-5f * (rw + rho) * (rw + rho);
  // |s - w| <= |C_ref - s| + |C_ref - w|
  const float in = rw - 2.0002f * rho - b.eta / fmaxf(rw, 1e-30f);
  b.xin = in > 0.f ? in * in : -1.f;
  return b;
}

// |a - b|^2 with the sign of b that makes it smaller (chain 0), which is left in b.
__device__ __forceinline__ float near_sq(float4 a, float4 &b, int chain) {
  if (chain == 0) {
    float x, y;
    rot_chord_sq(a, b, x, y);
    const bool flip = x > y;
    b = flip ? make_float4(-b.x, -b.y, -b.z, -b.w) : b;
    return flip ? y : x;
  }
  return sqdist(a, b, 1);
}

__device__ __forceinline__ float euclid_sq(float4 a, float4 b, int chain) {
  const float d0 = a.x - b.x, d1 = a.y - b.y, d2 = a.z - b.z, d3 = chain == 0 ? a.w - b.w : 0.f;
  return fmaf(d3, d3, fmaf(d2, d2, fmaf(d1, d1, d0 * d0)));
}

// Which of a thread's N samples are dominated, as bits.  A witness is read from
// LDS once for all of them: read for each sample by itself, its latency was the
// time of a rescan over every sample (one workgroup, 65,536 samples 194 -> 90 us,
// 300,000 882 -> 405 us).
constexpr int kDomPer = 4;
template <int N>
__device__ __forceinline__ unsigned dominated(const Domination &S, const DomBall &b, const float4 *a, int chain) {
  float4 s[N];
  float xs[N];
  unsigned dom = 0u;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    s[u] = a[u];
    xs[u] = near_sq(S.C, s[u], chain);
    dom |= xs[u] < b.xin ? 1u << u : 0u;
  }
  for (int k = 0; k < S.n; ++k) {
    const float4 w = S.w[k];
    const float xw = S.xw[k];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const float gap = xw - xs[u] - b.eta;
      dom |= gap > 0.f && gap * gap > b.four * euclid_sq(w, s[u], chain) ? 1u << u : 0u;
    }
  }
  return dom;
}

// Sum over the wavefront, in every lane (a fixed order).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wavefront builds S for the steps from i0 on, at the iterate C: winners
// of the steps before come from the trace tr (the last one given as w_last
// when the trace does not hold it yet, else -1), rotation iterates from the
// checkpoints ckq of spacing ck.
__device__ __forceinline__ void build_domination(Domination &S, float4 C, int i0, int w_last, const int32_t *tr,
                                                 const float4 *D, int M, const float4 *ckq, int ck, int chain) {
  const int lane = threadIdx.x & 63;
  const int taken = i0 - 1;
  int v = -1;
  if (lane < taken) v = lane == 0 && w_last >= 0 ? w_last : tr[2 * (taken - 1 - lane)];
  if (v >= M) v = -1;
  unsigned long long left = __ballot(v >= 0);
  int n = 0, id = -1;
  while (left && n < 8) {
    const int w = __builtin_amdgcn_readlane(v, (int)__ffsll((long long)left) - 1);
    if (lane == n) id = w;
    ++n;
    left &= ~__ballot(v == w);
  }
  const bool mine = lane < n;
  const float4 pw = D[mine ? id : 0];
  // reference centre and the radius in steps
  float4 R = C;
  float f = 2.1f;
  if (chain == 0 && taken >= 2) {
    const int qhi = (taken - 1) / ck, qlo = (taken / 2 + ck - 1) / ck;
    const int nq = min(64, qhi - qlo + 1);
    if (nq >= 2) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
      if (lane < nq) a = ckq[qhi - lane];
      a.x = wave_sum(a.x) + C.x;
      a.y = wave_sum(a.y) + C.y;
      a.z = wave_sum(a.z) + C.z;
      a.w = wave_sum(a.w) + C.w;
      const float nn = __builtin_amdgcn_rsqf(fmaf(a.w, a.w, fmaf(a.z, a.z, fmaf(a.y, a.y, a.x * a.x))));
      R = make_float4(a.x * nn, a.y * nn, a.z * nn, a.w * nn);
      f = i0 < 64 ? 1.5f : 1.3f;
    }
  }
  if (chain == 1 && taken >= 4) {
    // c_m is the mean of the first m winners, so going back from C the sums
    // m c_m lose one winner at a time
    const float4 p = D[v >= 0 ? v : 0];
    float4 a = v >= 0 ? p : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float ux = __shfl_up(a.x, o, 64), uy = __shfl_up(a.y, o, 64), uz = __shfl_up(a.z, o, 64);
      a.x += lane >= o ? ux : 0.f;
      a.y += lane >= o ? uy : 0.f;
      a.z += lane >= o ? uz : 0.f;
    }
    // lane l: a is the sum of the last l + 1 winners, for c_(taken - l - 1)
    const int m = taken - lane - 1, back = min(63, taken / 2);
    const bool use = lane < back && v >= 0 && m >= 1;
    const float im = use ? 1.f / (float)m : 0.f, tk = (float)taken;
    const float inv_n = 1.f / (1.f + wave_sum(use ? 1.f : 0.f));
    R.x = (wave_sum(use ? (tk * C.x - a.x) * im : 0.f) + C.x) * inv_n;
    R.y = (wave_sum(use ? (tk * C.y - a.y) * im : 0.f) + C.y) * inv_n;
    R.z = (wave_sum(use ? (tk * C.z - a.z) * im : 0.f) + C.z) * inv_n;
    f = i0 < 64 ? 1.5f : 1.3f;
  }
  const float inv = 1.f / (float)i0;
  float4 w = pw;
  float x = near_sq(R, w, chain);
  float xmax = wave_max_key(mine ? x : 0.f);
  float step = __builtin_amdgcn_sqrtf(xmax) * inv;
  if (f < 2.f && !(euclid_sq(C, R, chain) < 1.21f * step * step)) {  // (a mean far from the iterate)
    R = C;
    f = 2.1f;
    w = pw;
    x = near_sq(R, w, chain);
    xmax = wave_max_key(mine ? x : 0.f);
    step = __builtin_amdgcn_sqrtf(xmax) * inv;
  }
  const float rho = f * step;
  // (rotations: balls of less than about 100 degrees, where the keys order as
  // the chords do with the margin that eta allows for)
  const bool ok = n > 0 && rho > 0.f && (chain == 1 || xmax + 2.f * rho < 0.75f);
  if (mine) {
    S.w[lane] = w;
    S.xw[lane] = x;
  }
  if (lane == 0) {
    S.C = R;
    S.xmax = xmax;
    S.rho = rho;
    S.rho_min = 1.2f * step;
    S.n = ok ? n : 0;
  }
}

// The first steps move the centre across the whole sample cloud.  For
// instances of at least kBigInstance samples they are spread over kEarlyWG
// workgroups per chain, one launch per step (k_megb_early): kEarlyFull scans of
// every sample, then steps over the undominated ones until those fit a
// chain's shell.  Smaller instances take kEarlyFull full scans inside their
// chain's workgroup.  Host and device apply the same rule.
constexpr int kEarlyBlock = 256;
constexpr int kEarlyList = 4096;  // undominated samples of a workgroup held in LDS before they are written

// Steps of the first phase: until the undominated samples (about 6, 1.5, 0.6
// and 0.3 % of all after 16, 32, 48 and 64 steps of the 2D-3D clouds, up to twice
// that of the 3D-3D ones) are few enough for one workgroup to scan them as fast
// as a launch takes its step (5 us, about 20,000 entries in the wide variant),
// and fit their slots: a chain that starts without them pays rescans over every
// sample, 1.5 us per 1,000 samples each, so the larger the instance the longer
// the phase.  Milliseconds with 17, 25 and 33 steps: one instance of 40,000
// (2D-3D) 0.74, 0.78, 0.81; of 65,536 1.20, 1.24, 1.28 (2D-3D) and 1.50, 1.15, 1.10
// (3D-3D); of 300,000 (3D-3D) 1.43, 1.33, 1.34; eight of 262,144 1.80, 1.76, 1.51;
// 130 of 65,536 (narrow) 3.05, 3.73, 3.67 (2D-3D) and 3.59, 4.09, 4.17 (3D-3D), of
// 100,000 5.27, 5.73, 4.35 and 6.08, 4.60, 4.76.  A short descent ends the phase
// where its last avg iterates begin.
inline int early_steps(int64_t m, bool wide, int T, int avg) {
  int most;
  if (wide)
    most = m < (1 << 16) ? 17 : (m <= (1 << 17) ? 25 : (m <= (1 << 19) ? 33 : (m <= (1 << 21) ? 49 : 65)));
  else
    most = m <= (1 << 16) ? 17 : (m <= (1 << 17) ? 33 : (m <= (1 << 19) ? 49 : 65));
  // (narrow: the chains' own workgroups fill the chip, and scan a short descent as fast)
  return wide || T > 2 * kEarlyFull + avg ? min(most, T - avg) : 0;
}

__host__ __device__ inline bool early_phase_applies(int64_t M, int no_prune, int n_early) {
  return M >= kBigInstance && n_early > 0 && !no_prune;
}

// The step of each turn to gather.
__host__ __device__ constexpr int gather_step(int turn) {
  return turn == 0 ? kEarlyFull + 1 : (turn == 1 ? 25 : (turn == 2 ? 33 : 49));
}

// The undominated samples held before step i: the ball and the number of the
// last turn that gathered any (n = 0: none).
struct Held {
  float4 C;
  float rho;
  int n;
};
__device__ __forceinline__ Held held_before(const EarlyScratch &e, int i) {
  Held h{make_float4(0.f, 0.f, 0.f, 0.f), 0.f, 0};
  if (i > gather_step(0)) {  // (the loads of all turns in flight together)
    Held t[kGathers];
#pragma unroll
    for (int a = 0; a < kGathers; ++a) t[a] = Held{e.dm_c[a], e.dm_rho[a], e.dm_n[a]};
#pragma unroll
    for (int a = 0; a < kGathers; ++a)
      if (gather_step(a) < i && t[a].n > 0) h = t[a];
  }
  return h;
}

// Elements [sb, se) of workgroup b of a chain: kEarlyWG ranges of a multiple
// of kEarlyBlock elements.
__device__ __forceinline__ void early_range(int M, int b, int &sb, int &se) {
  const int span = ((M + kEarlyWG - 1) / kEarlyWG + kEarlyBlock - 1) / kEarlyBlock * kEarlyBlock;
  sb = min(M, b * span);
  se = min(M, sb + span);
}

// Largest 64-bit value of the wavefront (unsigned), in every lane.
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const unsigned long long w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

// (key, id) packed so that an unsigned maximum keeps the larger key and, on
// equal keys, the lower id; keys are >= 0 (a -0 is taken as +0, which it
// equals).  0: no sample.
__device__ __forceinline__ unsigned long long pack_best(float k, int id) {
  return id == INT32_MAX ? 0ull
                         : ((unsigned long long)(__float_as_uint(k) & 0x7fffffffu) << 32) |
                               (unsigned long long)(~(unsigned)id);
}

// Completes step i of a chain's first phase from the kEarlyWG packed argmaxes
// its launch left and the centre it started from (whole wavefront, every lane
// gets the new centre); the winner's id in bi.
__device__ __forceinline__ float4 early_complete(const EarlyScratch &e, int i, const float4 *D, int M, int chain,
                                                 int &bi) {
  static_assert(kEarlyWG == 64, "one partial per lane");
  const unsigned long long best = wave_max_u64(e.part[i & 1][threadIdx.x & 63]);
  bi = best ? (int)~(unsigned)(best & 0xffffffffull) : INT32_MAX;
  const float4 Cp = e.cbuf[(i + 1) & 1];
  return bi < M ? geodesic_step(Cp, D[bi], i, chain) : Cp;
}

// Step i of the first phase for every (instance, chain) the rule selects,
// whose feasible samples outnumber the shell capacity (else the shell holds
// them all and the chain's workgroup needs no scans).  Every workgroup first
// completes step i - 1 itself, so all workgroups hold the same centre with no
// atomic or fence (kernel boundaries order the launches); workgroup 0 records
// the trace, the checkpoint and the centre for the next launch.  Then each
// workgroup finds the farthest of its samples and leaves its packed argmax.
// The chain's workgroup completes the last step.  Buffers alternate between
// consecutive launches, so a launch never writes what it reads.  Launch
// kEarlyFull + 1 also gathers the undominated samples about its centre (in
// LDS, written with one atomic reservation per few thousand), and the later
// ones scan those while the centre is in their ball; when they were too many for
// their slots, or the centre has left the ball, a later turn gathers again (its
// state is a turn's own, so that a launch reads none that it writes).  (2^20 samples: a full
// scan is bound by HBM, 0.36 ms for 64 instances; 64 instances of 2^20 took
// 32 of them and three passes for a shell by distance, 12.6 ms, and take 17
// and 32 over the undominated samples.)
__global__ void __launch_bounds__(kEarlyBlock) k_megb_early(const int64_t *__restrict__ sample_off, int64_t total,
                                                            int64_t max_m, const float4 *__restrict__ quat,
                                                            const float4 *__restrict__ trans, MegbRec *rec,
                                                            EarlyScratch *es, int32_t *trace, float4 *ckpt, int ck,
                                                            int T, int avg, int cap, int no_prune, int n_early,
                                                            DmSlots dms, int i) {
  const int j = blockIdx.z, chain = blockIdx.y, b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t off, M64;
  sample_range(sample_off, j, total, max_m, off, M64);
  if (!early_phase_applies(M64, no_prune, n_early)) return;
  const int M = (int)M64;  // >= kBigInstance here
  const int first = rec[j].first;
  if (first == INT32_MAX || (int64_t)rec[j].n_feasible <= cap) return;
  const float4 *D = (chain ? trans : quat) + off;
  EarlyScratch &e = es[2 * j + chain];
  int32_t *tr = trace + (int64_t)j * T * 2 + chain;
  float4 *ckq = ckpt + (int64_t)j * ckpt_count(T, ck);
  // ---- the centre before step i (every wave reduces the partials itself)
  float4 C;
  int w_last = -1;
  if (i == 1) {
    C = D[first];
  } else {
    C = early_complete(e, i - 1, D, M, chain, w_last);
    if (b == 0 && tid == 0) tr[2 * (i - 2)] = w_last;
  }
  if (b == 0 && tid == 0) {
    e.cbuf[(i + 1) & 1] = C;
    if (chain == 0 && (i - 1) % ck == 0) ckq[(i - 1) / ck] = C;
    if (i == 1)
      for (int a = 0; a < kGathers; ++a) e.dm_n[a] = 0;
  }
  const int slots = M >> dms.shift;
  int32_t *gid = dms.id + chain * dms.stride + (off >> dms.shift);
  float4 *gpt = dms.pt + chain * dms.stride + (off >> dms.shift);
  const Held held = held_before(e, i);
  const bool pruned = held.n > 0 && held.n <= slots &&
                      euclid_sq(C, held.C, chain) <= held.rho * held.rho * (1.f - 1e-5f);
  int turn = -1;
#pragma unroll
  for (int a = 0; a < kGathers; ++a)
    if (i == gather_step(a)) turn = a;
  const bool gather = !pruned && turn >= 0;
  const float4 *src = pruned ? gpt : D;
  const int n_src = pruned ? held.n : M;
  int sb, se;
  early_range(n_src, b, sb, se);
  __shared__ float red_k[kEarlyBlock / 64];
  __shared__ int red_i[kEarlyBlock / 64];
  __shared__ Domination dom;
  __shared__ int list[kEarlyList];
  __shared__ int n_list, base_s;
  if (gather) {
    if (wave == 0) build_domination(dom, C, i, w_last, tr, D, M, ckq, ck, chain);
    if (tid == 0) n_list = 0;
    __syncthreads();
  }
  const bool keep = gather && dom.n > 0;
  DomBall ball = DomBall{0.f, 0.f, 0.f, 0.f};
  if (keep) ball = dom_ball(dom, dom.rho);
  auto flush = [&]() {  // (whole workgroup)
    const int n = n_list;
    if (tid == 0) base_s = n ? atomicAdd(&e.dm_n[turn], n) : 0;
    __syncthreads();
    const int base = base_s;
    for (int p = tid; p < n; p += kEarlyBlock)
      if (base + p < slots) {
        const int s = list[p];
        gid[base + p] = s;
        gpt[base + p] = D[s];
      }
    __syncthreads();
    if (tid == 0) n_list = 0;
    __syncthreads();
  };
  float bk = -1.f;
  int bi = INT32_MAX;
  stream_rounds<kEarlyBlock>(src + sb, se - sb, make_float4(-2.f, 0.f, 0.f, 0.f), [&](const float4 *a, int s0) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int q = sb + s0 + u * kEarlyBlock + tid;
      if (q < se && feasible_pt(a[u], chain)) {
        const float k = sqdist(C, a[u], chain);
        const int s = pruned ? gid[q] : q;
        if (better(k, s, bk, bi)) {
          bk = k;
          bi = s;
        }
      }
    }
    if (keep) {
#pragma unroll
      for (int h = 0; h < kUnroll; h += kDomPer) {
        const unsigned out = dominated<kDomPer>(dom, ball, a + h, chain);
#pragma unroll
        for (int u = 0; u < kDomPer; ++u) {
          const int q = sb + s0 + (h + u) * kEarlyBlock + tid;
          if (q < se && feasible_pt(a[h + u], chain) && !((out >> u) & 1u)) list[atomicAdd(&n_list, 1)] = q;
        }
      }
      static_assert(kEarlyList >= 2 * kEarlyBlock * kUnroll, "a round fits a list at most half full");
      __syncthreads();
      const bool full = n_list > kEarlyList - kEarlyBlock * kUnroll;
      __syncthreads();  // (every thread has read n_list before the next round adds to it)
      if (full) flush();
    }
  });
  if (keep) {
    __syncthreads();
    flush();
    if (b == 0 && tid == 0) {
      e.dm_c[turn] = dom.C;
      e.dm_rho[turn] = dom.rho;
    }
  }
  float wk;
  int wi;
  wave_argmax(bk, bi, wk, wi);
  if (lane == 0) {
    red_k[wave] = wk;
    red_i[wave] = wi;
  }
  __syncthreads();
  if (tid == 0) {
    bk = red_k[0];
    bi = red_i[0];
#pragma unroll
    for (int w = 1; w < kEarlyBlock / 64; ++w)
      if (better(red_k[w], red_i[w], bk, bi)) {
        bk = red_k[w];
        bi = red_i[w];
      }
    e.part[i & 1][b] = pack_best(bk, bi);
  }
}

// Per sample: quaternion (w >= 0; w = -2 marks an infeasible sample) and
// translation (w = 1 feasible, 0 not); first feasible index; feasible count.
template <int PER>
__global__ void __launch_bounds__(kBlock) k_megb_prep(const int64_t *__restrict__ sample_off, int64_t total,
                                                      int64_t max_m, const float *__restrict__ poses,
                                                      const uint8_t *__restrict__ mask, MegbRec *rec,
                                                      float4 *quat, float4 *trans) {
  const int j = blockIdx.y;
  int64_t off, M;
  sample_range(sample_off, j, total, max_m, off, M);
  const int64_t s0 = (int64_t)blockIdx.x * (kBlock * PER) + threadIdx.x;
  __shared__ int cnt[kWaves];
  __shared__ int firsts[kWaves];
  int feas = 0, first = INT32_MAX;
  // PER samples per thread, kBlock apart: the masks first, then the
  // poses of the feasible ones, every load of a round in flight together
  uint8_t m[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t s = s0 + u * kBlock;
    m[u] = s < M ? mask[off + s] : (uint8_t)0;
  }
  float4 a[PER], b[PER], c[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t s = s0 + u * kBlock;
    if (s < M && (m[u] & PURSE_MASK_FEASIBLE)) {
      const float4 *pp = reinterpret_cast<const float4 *>(poses + 12 * (off + s));
      a[u] = pp[0];
      b[u] = pp[1];
      c[u] = pp[2];
    }
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t s = s0 + u * kBlock;
    if (s >= M) continue;
    const int64_t g = off + s;
    if (m[u] & PURSE_MASK_FEASIBLE) {
      float R[9] = {a[u].x, a[u].y, a[u].z, a[u].w, b[u].x, b[u].y, b[u].z, b[u].w, c[u].x};
      quat[g] = quat_from_rot(R);
      trans[g] = make_float4(c[u].y, c[u].z, c[u].w, 1.f);
      ++feas;
      first = min(first, (int)s);
    } else {
      quat[g] = make_float4(-2.f, 0.f, 0.f, 0.f);
      trans[g] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  // block reduction, one atomic per block
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    feas += __shfl_xor(feas, o, 64);
    first = min(first, __shfl_xor(first, o, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    cnt[w] = feas;
    firsts[w] = first;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = 0, f = INT32_MAX;
    for (int k = 0; k < kWaves; ++k) {
      c += cnt[k];
      f = min(f, firsts[k]);
    }
    if (c) {
      atomicAdd(&rec[j].n_feasible, (unsigned long long)c);
      atomicMin(&rec[j].first, f);
    }
  }
}

// ---------------------------------------------------------------------------
// The rotation step with the quaternion's components across lanes, for the
// one wavefront that runs a descent ahead: lane l holds component l & 3 of
// the iterate and of one candidate winner, lanes with bit 2 clear form
// |a - b|^2 and the others |a + b|^2, and every group of eight lanes (row of
// sixteen with four candidates, half with two) takes the step toward its own
// candidate.  The same operations in the same order as
// geodesic_step_inv<true>, so bitwise its results.  A lone wavefront issues one
// instruction every 4 to 6 cycles whatever it does, so the step is bound by
// its instruction count.  Measured alone on a compute unit: 442 cycles with
// eight candidates, 424 with four, 300 with the winner known, against 548 with
// one candidate per lane and the whole quaternion in it.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Sum of the squares of a quad's four lanes, in every lane of the quad.
__device__ __forceinline__ float quad_norm_sq(float m) {
  const float m0 = dpp_f<0x00>(m), m1 = dpp_f<0x55>(m), m2 = dpp_f<0xAA>(m), m3 = dpp_f<0xFF>(m);
  return fmaf(m3, m3, fmaf(m2, m2, fmaf(m1, m1, m0 * m0)));
}

struct RotLane {
  float b, bm;  // candidate's component; +b where |a + b|^2 is formed, else -b
  bool plus;    // (lane & 4) != 0
};
__device__ __forceinline__ RotLane rot_lane(float4 b) {
  const int c = threadIdx.x & 3;
  RotLane r;
  r.b = c == 0 ? b.x : (c == 1 ? b.y : (c == 2 ? b.z : b.w));
  r.plus = (threadIdx.x & 4) != 0;
  r.bm = r.plus ? r.b : -r.b;
  return r;
}

// inv4: 4 / i.  key: the candidate's key (sqdist of chain 0).
__device__ __forceinline__ float rot_lane_step(float a, const RotLane &r, float inv4, float &key) {
  const float v = quad_norm_sq(a + r.bm);
  const float o = dpp_f<0x141>(v);  // row_half_mirror: the group's other quad
  RotChords c;
  c.xs = fminf(v, o);
  const float ys = fmaxf(v, o);
  key = (2.f * c.xs) * ys;
  c.rx = __builtin_amdgcn_sqrtf(c.xs);
  c.ry = __builtin_amdgcn_sqrtf(ys);
  const float bs = (r.plus ? o : v) > c.xs ? -r.b : r.b;  // a . b < 0: |a - b|^2 is the larger
  const float th = atan_eighth(c.rx * __builtin_amdgcn_rcpf(2.f + c.ry)) * inv4;
  float st, ct;
  sincos_small(th, st, ct);
  const float sh = (0.5f * c.rx) * c.ry;
  const float chh = fmaf(-0.5f, c.xs, 1.f);
  const float cb = st * __builtin_amdgcn_rcpf(fmaxf(sh, 1e-30f));
  const float ca = fmaf(-chh, cb, ct);
  const float q = fmaf(cb, bs, ca * a);
  float n = q * __builtin_amdgcn_rsqf(quad_norm_sq(q));
  // (rounded here: the next step's a + bm must not be fused with this product)
  __asm__("" : "+v"(n));
  return n;
}

// The value of the lane group with the larger key, of two rows of sixteen
// lanes (ROW) or two halves of the wavefront; ties take the lower one.
template <bool ROW>
__device__ __forceinline__ void swap_pair(float x, float &lo, float &hi) {
  const unsigned u = __float_as_uint(x);
  const auto p = ROW ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                     : __builtin_amdgcn_permlane32_swap(u, u, false, false);
  lo = __uint_as_float(p[0]);
  hi = __uint_as_float(p[1]);
}

// n steps from the iterate whose component a holds, each toward the candidate
// with the largest key, the one of the lowest lanes among equal keys; the
// starting iterates' components go to rec[4 k].  inv4_tab: 4 / i of step `lane`.
template <int NC>
__device__ __forceinline__ float rot_lane_run(float a, const RotLane &r, float inv4_tab, int n, float *rec) {
  const int upper = (threadIdx.x >> 3) & 1;
#pragma unroll 2
  for (int k = 0; k < n; ++k) {
    rec[4 * k] = a;
    float key;
    float v = rot_lane_step(a, r, readlane_f(inv4_tab, k), key);
    float lo, hi;
    if (NC == 8) {
      // row_ror:8: the row's other group (keys are not negative, so their bits
      // order like the values)
      const float ko = dpp_f<0x128>(key), vo = dpp_f<0x128>(v);
      v = __float_as_int(ko) + upper > __float_as_int(key) ? vo : v;
      key = fmaxf(key, ko);
    }
    if (NC >= 4) {
      swap_pair<true>(key, lo, hi);
      const bool row = hi > lo;
      key = fmaxf(lo, hi);
      swap_pair<true>(v, lo, hi);
      v = row ? hi : lo;
    }
    swap_pair<false>(key, lo, hi);
    const bool half = hi > lo;
    swap_pair<false>(v, lo, hi);
    a = half ? hi : lo;
  }
  return a;
}

// The same with known winners: r0 on even steps, r1 on odd ones.
__device__ __forceinline__ float rot_lane_alternate(float a, const RotLane &r0, const RotLane &r1, float inv4_tab,
                                                    int n, float *rec) {
  float key;
  int k = 0;
  for (; k + 1 < n; k += 2) {
    rec[4 * k] = a;
    a = rot_lane_step(a, r0, readlane_f(inv4_tab, k), key);
    rec[4 * k + 4] = a;
    a = rot_lane_step(a, r1, readlane_f(inv4_tab, k + 1), key);
  }
  if (k < n) {
    rec[4 * k] = a;
    a = rot_lane_step(a, r0, readlane_f(inv4_tab, k), key);
  }
  return a;
}

// A chain's undominated samples in global memory (the state only rescans and
// scan steps read) and its diagnostics.
struct ChainDm {
  int n, n_built;
  float rho;
  float4 C;
};
struct ChainDiag {
  int n_rescan, n_global, n_seg, n_piped, n_fail;
  long long n_groups;
  uint64_t t_start;
};

// One wavefront: entries of the histogram h summed from the top bin down, each
// lane holding four bins (bin kBins - 1 - 4 lane first); returns the sum over
// the bins above the lane's.
__device__ __forceinline__ unsigned int bins_above(const unsigned int *h, unsigned int c[4]) {
  static_assert(kBins == 256, "four bins per lane");
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = h[kBins - 1 - 4 * lane - k];
  const unsigned int own = c[0] + c[1] + c[2] + c[3];
  unsigned int inc = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned int up = __shfl_up(inc, o, 64);
    if (lane >= o) inc += up;
  }
  return inc - own;
}

// One wavefront: the highest bin whose entries no longer fit cap together
// with those of the bins above it (-1: all of them fit).
__device__ __forceinline__ int first_bin_over(const unsigned int *h, unsigned int cap) {
  unsigned int c[4];
  unsigned int cum = bins_above(h, c);
  int over = -1;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    cum += c[k];
    if (over < 0 && cum > cap) over = kBins - 1 - 4 * (int)(threadIdx.x & 63) - k;
  }
  return wave_max_i32(over);
}

// Shared state of one chain's workgroup.
struct ChainShared {
  float4 *pt;             // shell points, [cap]
  int *id;                // shell sample ids, [cap]
  unsigned int *hist;     // [kBins]
  unsigned int *cursor;   // [kBins]
  float *chunk_ub;        // [kMaxChunks]
  float (*red_k)[kChainWaves];
  int (*red_i)[kChainWaves];
};

template <int CHAIN, int V>
__device__ __forceinline__ void chain_run(const ChainShared &S, const int64_t *__restrict__ sample_off,
                                          int64_t max_m, const float4 *__restrict__ pts, MegbRec *rec,
                                          float *dref_all, int64_t total_samples, int32_t *trace,
                                          float4 *ckpt_all, int ck, int T, int avg, int cap, int no_prune,
                                          int n_early, const EarlyScratch *es, DmSlots dms) {
  __shared__ float4 st_C;
  __shared__ int st_i;
  __shared__ float st_theta, st_lo, st_w;
  __shared__ int st_bstar, st_kept;
  __shared__ Domination dom;
  __shared__ int st_mode;  // 0 shell in LDS, 1 scan of every sample
  __shared__ unsigned int sh_n;
  // pipelined shell steps
  __shared__ float4 pl_C[3][kPipeSteps];  // starting iterate of each step of a round (3 rounds in flight)
  __shared__ int pl_W[3][kPipeSteps];     // and its winner, from the check
  __shared__ int pl_cand[8], pl_two;      // the candidates of the predictions
  __shared__ int pl_fail[3];              // first step of a round whose prediction failed
  __shared__ float4 pl_Cend;
  __shared__ int pl_go;

  constexpr int chain = CHAIN;
  constexpr int BLK = chain_block<V>(), NW = BLK / 64;
  // verifier waves of a pipelined segment: every wave but wave 0 and, in the
  // eight-wave group, the one that shares wave 0's SIMD (waves go round the
  // four SIMDs)
  constexpr int kSkipWave = NW > 4 ? kVerifySkip : NW;
  constexpr int kVerifiers = NW > 4 ? NW - 2 : NW - 1;
  // elements per thread and round in the passes over d_ref: the wide variant
  // has the registers to keep more loads in flight, which these
  // latency-bound passes of one workgroup need
  constexpr int UF = V == kChainWide ? 32 : kUnroll;
  // samples of a domination test (four in the narrow variant spill registers of
  // the scan steps: 130 instances of 33,000 samples, 28 steps 0.75 -> 0.81 ms)
  constexpr int kPer = V == kChainWide ? kDomPer : 2;
  const int j = blockIdx.x >> 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t off, M64;
  sample_range(sample_off, j, total_samples, max_m, off, M64);
  const int M = (int)M64;
  const float4 *D = pts + off;
  float *dref = dref_all + chain * total_samples + off;
  int32_t *tr = trace + (int64_t)j * T * 2 + chain;
  // rotation iterates C_{q ck} for the backward (each step's path leaves the
  // ones it starts from)
  float4 *ckq = ckpt_all + (int64_t)j * ckpt_count(T, ck);
  const int first = rec[j].first;
  if (first == INT32_MAX) {
    for (int k = tid; k < T; k += BLK) tr[2 * k] = -1;
    return;
  }
  const int n_feas = (int)rec[j].n_feasible;
  // the first steps were taken by k_megb_early when the rule selects it, which
  // also gathered the undominated samples
  const bool ep = early_phase_applies(M64, no_prune, n_early) && n_feas > cap;
  int32_t *__restrict__ gid = dms.id + chain * dms.stride + (off >> dms.shift);
  float4 *__restrict__ gpt = dms.pt + chain * dms.stride + (off >> dms.shift);
  // Undominated samples whose ball the centre has left are gathered again by
  // the next pass over every sample.  Their state, which only rescans and scan
  // steps read, and the diagnostics live in LDS (thread 0 writes them between
  // barriers), so that the stepping loops keep their registers.
  const int slots = ep ? M >> dms.shift : 0;
  __shared__ ChainDm sg;
  __shared__ ChainDiag sdg;
  if (wave == 0) {
    float4 C1 = D[first];
    if (ep) {
      int bi;
      C1 = early_complete(es[2 * j + chain], n_early, D, M, chain, bi);
      if (lane == 0) tr[2 * (n_early - 1)] = bi;
    }
    if (lane == 0) {
      st_C = C1;
      st_i = ep ? n_early + 1 : 1;
      Held held{make_float4(0.f, 0.f, 0.f, 0.f), 0.f, 0};
      if (ep) held = held_before(es[2 * j + chain], n_early + 1);
      sg.n = held.n <= slots ? held.n : 0;
      sg.rho = held.rho;
      sg.C = held.C;
      sg.n_built = 0;
      sdg = ChainDiag{0, 0, 0, 0, 0, 0ll, __builtin_amdgcn_s_memrealtime()};
    }
  }
  __syncthreads();
  bool use_dm = sg.rho > 0.f && sg.n > 0;
  auto in_dm = [&](float4 c) { return euclid_sq(c, sg.C, chain) <= sg.rho * sg.rho * (1.f - 1e-5f); };
  float acc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.f;
  // (a descent that is over soon after them scans 2 kEarlyFull steps)
  const int n_full = !ep && T <= 2 * kEarlyFull + avg ? 2 * kEarlyFull : kEarlyFull;
  bool stalled = false;
  int scan_len = kScanSteps;
  int recentre = kRecentreChunks;  // chunks a shell step may scan (set by each rescan)
  int stage_groups = 0;

  while (true) {
    const float4 C0 = st_C;  // the centre; distances and bounds are about Cref, near it
    const int i0 = st_i;
    if (i0 > T) break;
    const bool early = i0 <= n_full;
    if (use_dm && !in_dm(C0)) use_dm = false;
    const bool global = (no_prune || stalled || early || (!use_dm && T - i0 < kScanRest)) && n_feas > cap;
    bool barren = stalled;  // scan steps because the last rescan left no shell
    float4 Cref = C0;
    DomBall ball = DomBall{INFINITY, FLT_MAX, -1.f, FLT_MAX};
    float rref = 0.f;
    if (!global) {
      // -------------------------------------------------------------- rescan
      if (wave == 0) build_domination(dom, C0, i0, -1, tr, D, M, ckq, ck, chain);
      if (tid == 0) {
        ++sdg.n_rescan;
        st_kept = 0;
      }
      __syncthreads();
      // entries: the undominated samples (the ball of this rescan then lies
      // within theirs) or every sample
      float rho = dom.rho;
      if (use_dm) {
        const float room = sg.rho - 1.00002f * __builtin_amdgcn_sqrtf(euclid_sq(dom.C, sg.C, chain));
        if (dom.n > 0 && room >= dom.rho_min)
          rho = fminf(rho, room);
        else
          use_dm = false;
      }
      const bool from_dm = use_dm;  // (gathering anew below does not change this rescan's source)
      if (dom.n > 0) {
        ball = dom_ball(dom, rho);
        Cref = dom.C;
      }
      const float4 *src = from_dm ? gpt : D;
      const int n_src = from_dm ? sg.n : M;
      recentre = recentre_chunks(n_src);
      float mx = 0.f, mn = FLT_MAX;
      int kept = 0;
      const bool any_dom = dom.n > 0;
      stream_rounds<BLK>(src, n_src, make_float4(-2.f, 0.f, 0.f, 0.f), [&](const float4 *a, int s0) {
#pragma unroll
        for (int h = 0; h < kUnroll; h += kPer) {
          // (a few entries fill the first lanes of a round only)
          unsigned out = 0u;
          if (any_dom && s0 + h * BLK < n_src)
            out = s0 + (h + 1) * BLK < n_src ? dominated<kPer>(dom, ball, a + h, chain)
                                             : dominated<1>(dom, ball, a + h, chain);
#pragma unroll
          for (int u = 0; u < kPer; ++u) {
            const int s = s0 + (h + u) * BLK + tid;
            if (s < n_src) {
              float d = -1.f;
              if (feasible_pt(a[h + u], chain) && !((out >> u) & 1u)) {
                d = __builtin_amdgcn_sqrtf(sqdist(Cref, a[h + u], chain));  // within the slack
                mx = fmaxf(mx, d);
                mn = fminf(mn, d);
                ++kept;
              }
              dref[s] = d;
            }
          }
        }
      });
      mx = wave_max(mx);
      mn = __int_as_float(wave_min_i32(__float_as_int(mn)));
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) kept += __shfl_xor(kept, o, 64);
      if (lane == 0) {
        S.red_k[0][wave] = mx;
        S.red_k[1][wave] = mn;
        atomicAdd(&st_kept, kept);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        rref = fmaxf(rref, S.red_k[0][k]);
        mn = fminf(mn, S.red_k[1][k]);
      }
      const int n_kept = st_kept;
      if (ep && !from_dm && any_dom && n_kept <= slots) {
        // ------------------------------ gather the undominated samples anew
        if (tid == 0) sh_n = 0u;
        __syncthreads();
        // (a short unroll: this is rare, and its registers would otherwise be
        // taken from the stepping loops)
        stream_rounds<BLK, kUnroll>(dref, M, -1.f, [&](const float *dd, int s0) {
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            const int s = s0 + u * BLK + tid;
            if (dd[u] >= 0.f) {
              const unsigned int pos = atomicAdd(&sh_n, 1u);
              if (pos < (unsigned)slots) {
                gid[pos] = s;
                gpt[pos] = D[s];
              }
            }
          }
        });
        __syncthreads();
        if (tid == 0) {
          sg.n = min((int)sh_n, slots);
          sg.rho = rho;
          sg.C = Cref;
          ++sg.n_built;
        }
        __syncthreads();
        use_dm = sg.n > 0;
      }
      // Shell membership: undominated, and when those do not all fit, d >=
      // theta and (coarse) bin >= bstar of the histogram (lo, w); theta = -1
      // when they fit.
      if (tid == 0) {
        st_mode = 0;
        st_theta = -1.f;
        st_lo = mn;
        st_w = (rref - mn) / (float)kBins;
        st_bstar = 0;
      }
      __syncthreads();
      // Early, when the undominated samples that do not fit the shell will soon
      // be fewer, a few scans of them (3-4 us each) come first.
      const bool scan_first = n_kept > cap && n_kept <= 4 * cap && use_dm && i0 < 8 * kEarlyFull;
      if (scan_first) {
        if (tid == 0) st_mode = 1;
        __syncthreads();
      } else if (n_kept > cap) {
        barren = true;
        for (int level = 0; level < 2; ++level) {
          const float lo = st_lo, wdt = st_w;
          if (!(wdt > 0.f)) {
            if (tid == 0) st_mode = 1;
            __syncthreads();
            break;
          }
          for (int k = tid; k < kBins; k += BLK) S.hist[k] = 0u;
          __syncthreads();
          const float rw = 1.f / wdt;
          stream_rounds<BLK, UF>(dref, n_src, -1.f, [&](const float *dd, int) {
#pragma unroll
            for (int u = 0; u < UF; ++u)
              if (dd[u] >= lo && dd[u] >= 0.f) atomicAdd(&S.hist[bin_of(dd[u], lo, rw)], 1u);
          });
          __syncthreads();
          if (wave == 0) {
            const int bb = first_bin_over(S.hist, (unsigned)cap);
            if (lane == 0) {
              st_theta = -1.f;
              if (bb < 0) {  // everything at or above lo fits
                st_bstar = 0;
                st_theta = level == 0 ? -1.f : lo;
              } else if (bb < kBins - 1) {
                st_bstar = bb + 1;
                st_theta = lo + (float)(bb + 1) * wdt;
              } else if (level == 0) {  // the top bin alone overflows: refine inside it
                st_lo = lo + (float)(kBins - 1) * wdt;
                st_w = wdt / (float)kBins;
                st_theta = -2.f;
              } else {
                st_mode = 1;
              }
            }
          }
          __syncthreads();
          if (st_theta != -2.f || st_mode == 1) break;
        }
      }
      __syncthreads();
      // ---------------- collect, ordered by fine bins over [max(theta,0), rref]
      if (st_mode == 0) {
        const float lo = st_lo, wdt = st_w, theta = st_theta;
        const int bstar = st_bstar;
        const float flo = fmaxf(theta, mn);
        const float fw = (rref - flo) / (float)kBins;
        const bool fine = fw > 0.f;
        const float rw = wdt > 0.f ? 1.f / wdt : 0.f, rfw = fine ? 1.f / fw : 0.f;
        auto member = [&](float d) {
          return d >= 0.f && d >= theta && (theta < 0.f || (d >= lo && bin_of(d, lo, rw) >= bstar));
        };
        auto fbin = [&](float d) { return fine ? bin_of(d, flo, rfw) : kBins - 1; };
        for (int k = tid; k < kBins; k += BLK) S.hist[k] = 0u;
        __syncthreads();
        stream_rounds<BLK, UF>(dref, n_src, -1.f, [&](const float *dd, int) {
#pragma unroll
          for (int u = 0; u < UF; ++u)
            if (member(dd[u])) atomicAdd(&S.hist[fbin(dd[u])], 1u);
        });
        __syncthreads();
        if (wave == 0) {
          // entries in decreasing fine-bin order: cursor[b] = first slot of bin b
          unsigned int c[4];
          unsigned int at = bins_above(S.hist, c);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            S.cursor[kBins - 1 - 4 * lane - k] = at;
            at += c[k];
          }
          if (lane == 63) {
            sh_n = at;
            if (at > (unsigned)cap || at == 0u) st_mode = 1;  // (no entry: no distance is a number)
          }
        }
        __syncthreads();
        if (st_mode == 0) {
          // the ids first; the points are gathered afterwards in one pass
          // over the shell, all loads in flight at once
          stream_rounds<BLK, UF>(dref, n_src, -1.f, [&](const float *dd, int s0) {
#pragma unroll
            for (int u = 0; u < UF; ++u) {
              int s = s0 + u * BLK + tid;
              if (member(dd[u])) {
                unsigned int pos = atomicAdd(&S.cursor[fbin(dd[u])], 1u);
                if (pos < (unsigned)cap) S.id[pos] = s;
              }
            }
          });
          __syncthreads();
          // (undominated samples: the entry index becomes the sample id)
          if (from_dm) {
            for (int e = tid; e < (int)sh_n; e += BLK) {
              const int x = S.id[e];
              S.pt[e] = gpt[x];
              S.id[e] = gid[x];
            }
          } else {
            for (int e = tid; e < (int)sh_n; e += BLK) S.pt[e] = D[S.id[e]];
          }
          __syncthreads();
          // upper bound of d_ref over each chunk of 64 entries: the upper edge
          // of the fine bin holding its first entry (the top bin's is rref);
          // cursor[b] is the end of bin b's entries now
          const int K = (int)sh_n;
          for (int c = tid; c * 64 < K && c < kMaxChunks; c += BLK) {
            const unsigned int e = (unsigned)c * 64u;
            int lo_b = 0, hi_b = kBins - 1;  // the highest bin that ends beyond e
            while (lo_b < hi_b) {
              const int mid = (lo_b + hi_b + 1) >> 1;
              if (S.cursor[mid] > e)
                lo_b = mid;
              else
                hi_b = mid - 1;
            }
            S.chunk_ub[c] = (lo_b >= kBins - 1 || !fine) ? rref : flo + (float)(lo_b + 1) * fw;
          }
        }
        __syncthreads();
      }
    }
    if (global || st_mode == 1) {
      // ------------------------------------------------------------ scan steps
      // every feasible sample (the undominated ones while the centre is in
      // their ball), all waves; a bounded number of steps per stage
      float4 C = C0;
      int i = i0;
      int par = 0;
      if (tid == 0) ++sdg.n_global;
      const bool from_dm = use_dm && !no_prune;
      const int n_src = sg.n;
      const int i_end = no_prune ? T : (early ? min(T, n_full) : min(T, i0 + (barren ? scan_len : kScanSteps) - 1));
      if (barren) scan_len = min(2 * scan_len, kScanMax);
      while (i <= i_end) {
        if (from_dm && !in_dm(C)) break;  // (never on the stage's first step)
        float bk = -1.f;
        int bi = INT32_MAX;
        auto take = [&](float k, int s) {
          if (better(k, s, bk, bi)) {
            bk = k;
            bi = s;
          }
        };
        if (from_dm) {
          stream_rounds<BLK>(gpt, n_src, make_float4(-2.f, 0.f, 0.f, 0.f), [&](const float4 *a, int s0) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
              const int q = s0 + u * BLK + tid;
              if (q < n_src && feasible_pt(a[u], chain)) {
                const float k = sqdist(C, a[u], chain);
                if (k >= bk) take(k, gid[q]);
              }
            }
          });
        } else {
          stream_rounds<BLK>(D, M, make_float4(-2.f, 0.f, 0.f, 0.f), [&](const float4 *a, int s0) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
              const int s = s0 + u * BLK + tid;
              if (s < M && feasible_pt(a[u], chain)) take(sqdist(C, a[u], chain), s);
            }
          });
        }
        float wk;
        int wi;
        wave_argmax(bk, bi, wk, wi);
        if (lane == 0) {
          S.red_k[par][wave] = wk;
          S.red_i[par][wave] = wi;
        }
        __syncthreads();
        bk = S.red_k[par][0];
        bi = S.red_i[par][0];
#pragma unroll
        for (int w = 1; w < NW; ++w)
          if (better(S.red_k[par][w], S.red_i[par][w], bk, bi)) {
            bk = S.red_k[par][w];
            bi = S.red_i[par][w];
          }
        par ^= 1;
        if (CHAIN == 0 && tid == 0 && (i - 1) % ck == 0) ckq[(i - 1) / ck] = C;
        if (bi < M) C = geodesic_step(C, D[bi], i, chain);  // (no winner: no key is a number)
        if (tid == 0) tr[2 * (i - 1)] = bi;
        if (i > T - avg && wave == 0) accumulate_iterate(C, chain, acc);
        ++i;
      }
      if (tid == 0) {
        st_C = C;
        st_i = i;
      }
      __syncthreads();
      stalled = false;
    } else {
      // ---------------------------------------------------------- shell steps
      // Entries sit in chunks of 64 (one entry per lane) in decreasing fine
      // bins of d_ref.  Each lane keeps its own best (key, id, point), one
      // wavefront reduction per step of the scan, and the scan stops once no
      // later chunk can beat the best found.  The first two chunks, which
      // almost every step needs, stay in registers for the whole stage (lanes
      // past the shell's end hold copies of entry 0, which change no argmax);
      // later chunks are read from LDS.  When a step needs many chunks the
      // centre has drifted from C_ref: the stage ends and the next one
      // rescans there.
      //
      // Steps run in segments of two kinds.  Sequential segments run in wave
      // 0 alone.  A single wavefront issues about one instruction every few
      // cycles whatever the dependences, so the common step (the first chunk,
      // or the first two once one has often not sufficed in this stage,
      // bounds all others and one lane holds the maximum) is one straight
      // path: 1/i comes from a per-lane table of the next 64 values, and the
      // winners' ids are collected one per lane and written 64 at a time.
      //
      // Late in the descent the winners cycle among a few samples (the
      // support of the ball).  Wave 0 keeps the last distinct winners (up to
      // 8, one per lane); once no new one has appeared for a while, a
      // pipelined segment takes over: wave 0 runs the descent ahead, taking
      // as the winner of each step the one of those candidates farthest from
      // its iterate (a cheap key that only has to predict), kPipeSteps steps
      // per round, and leaves each step's starting iterate and predicted
      // winner in LDS, while the other waves check the steps of the previous
      // round with the full argmax of a sequential step.  Rounds end at a
      // workgroup barrier.  Every iterate wave 0 computes from verified
      // predictions is the one the sequential descent computes (same inputs,
      // same arithmetic), so the trace and the centre are unchanged; at the
      // first step whose prediction fails, the segment ends with that step's
      // starting iterate and a sequential segment redoes the step.
      const int K = (int)sh_n;
      const float theta = st_theta;
      const float slack = 4e-6f * rref + 1e-30f;
      // a shell of several chunks is cut down again once the steps have become
      // half as long (the first one, which has no witnesses yet, after kEarlyFull steps)
      const int refine_end = (ball.chk < FLT_MAX || early) && (int)sh_n > 64 ? min(T, max(2 * i0, kEarlyFull + 1) - 1)
                                                                             : T;
      const int nchunks = (K + 63) / 64;
      const float4 p0 = S.pt[lane < K ? lane : 0], p1 = S.pt[64 + lane < K ? 64 + lane : 0];
      const int q0 = S.id[lane < K ? lane : 0], q1 = S.id[64 + lane < K ? 64 + lane : 0];
      const float ub1 = nchunks > 1 ? S.chunk_ub[1] : 0.f;
      const float ub2 = nchunks > 2 ? S.chunk_ub[2] : 0.f;
      // the one bound a common step checks: entries past the chunks it
      // scanned, else samples outside the shell, else none
      const bool need_ub1 = nchunks > 1 || theta >= 0.f, need_ub2 = nchunks > 2 || theta >= 0.f;
      const float ubf1 = nchunks > 1 ? ub1 : theta, ubf2 = nchunks > 2 ? ub2 : theta;
      // distance of C from C_ref, compared squared in the bounds (the raw
      // square root is within the slack).  Rotation: |C + C_ref|^2 = 4 -
      // |C - C_ref|^2 for unit quaternions (C stays near C_ref within a stage;
      // the form only feeds bounds).
      // inside: C is in the ball the shell holds for (a centre that is no number,
      // after a sample that is none, counts as inside: every stage takes a step)
      auto drift = [&](float4 Cc, bool &inside) {
        float dC2;
        if (CHAIN == 0) {
          const float e0 = Cc.x - Cref.x, e1 = Cc.y - Cref.y, e2 = Cc.z - Cref.z, e3 = Cc.w - Cref.w;
          const float xc = fmaf(e3, e3, fmaf(e2, e2, fmaf(e1, e1, e0 * e0)));
          inside = !(xc > ball.chk);
          dC2 = (2.f * xc) * (4.f - xc);
        } else {
          dC2 = sqdist(Cc, Cref, chain);
          inside = !(dC2 > ball.chk);
        }
        return __builtin_amdgcn_sqrtf(dC2);
      };
      // wave-0 state carried across the segments of the stage
      float4 C = C0;
      int i = i0;
      int misses = 0;                // one-chunk steps that needed more
      bool wide = false, ended = false;
      int backoff = kPipeMinSeq;     // steps with no new winner before a pipelined segment
      const int last_plain = min(T - avg, refine_end);  // steps after T - avg accumulate their iterate
      // wave 0: candidate winners in lanes 0..7 (id -1: empty, its point C_ref,
      // which is never the farthest), the slot the next new winner takes, and
      // the steps since a new winner appeared
      int cand_id = -1;
      float4 cand_p = Cref;
      int nins = 0, stable = 0;
      int last_w = -1;  // winner of the last sequential step
      int turn_fails = 0;  // two candidates are taken in turn, until that has failed twice
      while (true) {
        if (wave == 0) {
          int ib = i;                                 // first step of the block of 64
          float inv_tab = 1.f / (float)(ib + lane);   // 1/i of step ib + lane
          int trv = 0;                                // winner of step ib + lane
          bool piped = false;
          int next_ck = (i - 1 + ck - 1) / ck * ck;   // next iterate index kept as a checkpoint
          int q_next = next_ck / ck;
          // Steps of the segment up to step `end` with WIDTH chunks in the
          // common step and (SHORT) the short sin/cos series of the geodesic
          // step; returns kStageEnds, kGoWide when one-chunk steps often
          // needed more and the stage should go on with two, kPipe when no
          // new winner has appeared for `backoff` steps and enough steps
          // remain for a pipelined segment, or kRangeDone at `end`.
          constexpr int kStageEnds = 0, kGoWide = 1, kRangeDone = 2, kPipe = 3;
          auto run_steps = [&](auto width, auto short_series, auto accumulate, int end) -> int {
            constexpr int W = decltype(width)::value;
            constexpr bool SHORT = decltype(short_series)::value;
            constexpr bool ACC = decltype(accumulate)::value;  // within the last avg steps
            while (i <= end) {
              if (i - ib == 64) {
                tr[2 * (ib - 1 + lane)] = trv;
                ib = i;
                inv_tab = 1.f / (float)(ib + lane);
              }
              const float inv = readlane_f(inv_tab, i - ib);
              bool inside;
              const float dC = drift(C, inside);
              auto beats = [&](float key, float ub) {
                const float b = ub + dC + slack;
                return key > b * b;
              };
              float bk = sqdist(C, p0, chain), bp_x = p0.x, bp_y = p0.y, bp_z = p0.z, bp_w = p0.w;
              int bi = q0;
              auto take = [&](float k, int q, float4 pp) {
                const bool t = (k > bk) | ((k == bk) & (q < bi));
                bk = t ? k : bk;
                bi = t ? q : bi;
                bp_x = t ? pp.x : bp_x;
                bp_y = t ? pp.y : bp_y;
                bp_z = t ? pp.z : bp_z;
                bp_w = t ? pp.w : bp_w;
              };
              int g = W;  // chunks scanned
              if (W == 2) take(sqdist(C, p1, chain), q1, p1);
              float wk = wave_max_key(bk);
              unsigned long long win = __ballot(bk == wk);
              const bool bounded = W == 2 ? (!need_ub2 || beats(wk, ubf2)) : (!need_ub1 || beats(wk, ubf1));
              if (!(bounded && inside && __popcll(win) == 1)) {
                // -------------------------------------------- uncommon step
                if (!inside) return kStageEnds;  // the shell no longer holds
                if (W == 1 && nchunks > 1 && !beats(wk, ub1)) {
                  take(sqdist(C, p1, chain), q1, p1);
                  wk = wave_max_key(bk);
                  g = 2;
                }
                if (g == 2 && nchunks > 2 && !beats(wk, ub2)) {
                  float4 p = S.pt[2 * 64 + lane];
                  int q = S.id[2 * 64 + lane];
                  while (true) {
                    float4 np;
                    int nq;
                    const bool more = g + 1 < nchunks;
                    if (more) {
                      np = S.pt[(g + 1) * 64 + lane];
                      nq = S.id[(g + 1) * 64 + lane];
                    }
                    const float kk = sqdist(C, p, chain);
                    take(g * 64 + lane < K ? kk : -1.f, q, p);
                    wk = wave_max_key(bk);
                    ++g;
                    if (!more || beats(wk, S.chunk_ub[g])) break;
                    p = np;
                    q = nq;
                  }
                }
                if (theta >= 0.f && !beats(wk, theta)) {
                  stage_groups += g;
                  return kStageEnds;  // the shell no longer suffices
                }
                // winner: the one lane holding the maximum key, else (a tie)
                // the lowest sample id among the lanes that hold it
                win = __ballot(bk == wk);
                if (__popcll(win) > 1) {
                  const int wmin = wave_min_i32(bk == wk ? bi : INT32_MAX);
                  win = __ballot(bk == wk && bi == wmin);
                }
              }
              stage_groups += g;
              const int wl = (int)__ffsll((long long)win) - 1;
              const int wi = __builtin_amdgcn_readlane(bi, wl);
              const float4 pt = make_float4(readlane_f(bp_x, wl), readlane_f(bp_y, wl), readlane_f(bp_z, wl),
                                            readlane_f(bp_w, wl));
              if (CHAIN == 0 && i - 1 == next_ck) {
                if (lane == 0) ckq[q_next] = C;
                next_ck += ck;
                ++q_next;
              }
              C = geodesic_step_inv<SHORT>(C, pt, inv, chain);
              trv = lane == i - ib ? wi : trv;
              if (ACC) accumulate_iterate(C, chain, acc);
              ++i;
              if (SHORT && !ACC) {
                last_w = wi;
                const bool known = (__ballot(cand_id == wi) & 0xFFull) != 0ull;
                const bool ins = !known && lane == nins;
                cand_id = ins ? wi : cand_id;
                cand_p = make_float4(ins ? pt.x : cand_p.x, ins ? pt.y : cand_p.y, ins ? pt.z : cand_p.z,
                                     ins ? pt.w : cand_p.w);
                nins = known ? nins : ((nins + 1) & 7);
                stable = known ? stable + 1 : 0;
              }
              if (g > recentre && i - i0 > kMinShellSteps) return kStageEnds;  // re-centre the shell
              if (W == 1 && g > 1 && ++misses * 4 > i - i0 && i - i0 >= 16) return kGoWide;
              if (SHORT && !ACC && stable >= backoff && end - i + 1 >= 2 * kPipeSteps) return kPipe;
            }
            return kRangeDone;
          };
          // Ranges of steps with no per-step choice of the sin/cos series or
          // of accumulating the iterate: before kShortSeriesStep, then the
          // rest, each split at the last avg steps.
          auto run_range = [&](auto short_series, auto accumulate, int end) {
            if (ended || piped || i > end) return;
            int r = wide ? run_steps(std::integral_constant<int, 2>(), short_series, accumulate, end)
                         : run_steps(std::integral_constant<int, 1>(), short_series, accumulate, end);
            if (r == kGoWide) {
              wide = true;
              r = run_steps(std::integral_constant<int, 2>(), short_series, accumulate, end);
            }
            ended = r == kStageEnds;
            piped = r == kPipe;
          };
          const int long_end = min(T, kShortSeriesStep - 1);
          run_range(std::false_type(), std::false_type(), min(long_end, last_plain));
          if (i > T - avg) run_range(std::false_type(), std::true_type(), min(long_end, refine_end));
          if (i > long_end) run_range(std::true_type(), std::false_type(), last_plain);
          if (i > T - avg && i > long_end) run_range(std::true_type(), std::true_type(), refine_end);
          if (lane < i - ib) tr[2 * (ib - 1 + lane)] = trv;
          if (lane == 0) sdg.n_groups += stage_groups;
          stage_groups = 0;
          if (lane == 0) {
            st_C = C;
            st_i = i;
            pl_go = piped ? 1 : 0;
          }
          for (int k = lane; k < 3; k += 64) pl_fail[k] = INT32_MAX;
        }
        __syncthreads();
        if (!pl_go) break;
        // ------------------------------------------------ pipelined segment
        const int pi0 = st_i, pend = last_plain;
        const int nrounds = (pend - pi0 + kPipeSteps) / kPipeSteps;
        float4 Cs = st_C;                       // wave 0: the iterate ahead
        int fail_step = INT32_MAX;
        float4 fail_C = Cs;
        // wave 0: when only two samples have won since the stage began the
        // winners alternate; the first predicted winner is then the one not
        // taken last
        unsigned long long vm = __ballot(cand_id >= 0) & 0xFFull;
        // (in increasing order of the ids, so that the lowest lane of equal
        // keys is the argmax's choice; empty slots last)
        {
          const int n_cand = __popcll(vm);
          int rank = cand_id >= 0 ? 0 : n_cand + __popcll(~vm & ((1ull << (lane & 7)) - 1ull));
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const int o = __builtin_amdgcn_readlane(cand_id, c);
            rank += cand_id >= 0 && o >= 0 && o < cand_id ? 1 : 0;
          }
          const int to = lane < 8 ? 4 * rank : 4 * lane;
          cand_id = __builtin_amdgcn_ds_permute(to, cand_id);
          cand_p.x = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(cand_p.x)));
          cand_p.y = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(cand_p.y)));
          cand_p.z = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(cand_p.z)));
          cand_p.w = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(cand_p.w)));
          nins = n_cand & 7;
          vm = (1ull << n_cand) - 1ull;
        }
        const bool pair = __popcll(vm) == 2, two = pair && turn_fails < 2;
        const int l0 = (int)__ffsll((long long)vm) - 1, l1 = (int)__ffsll((long long)(vm & (vm - 1ull))) - 1;
        const bool zero_last = __builtin_amdgcn_readlane(cand_id, two ? l0 : 0) == last_w;
        const int la = two ? (zero_last ? l1 : l0) : 0, lb = two ? (zero_last ? l0 : l1) : 0;
        const float4 pA = make_float4(readlane_f(cand_p.x, la), readlane_f(cand_p.y, la), readlane_f(cand_p.z, la),
                                      readlane_f(cand_p.w, la));
        const float4 pB = make_float4(readlane_f(cand_p.x, lb), readlane_f(cand_p.y, lb), readlane_f(cand_p.z, lb),
                                      readlane_f(cand_p.w, lb));
        // the candidates of a round's prediction, for its check: the two in
        // turn, or eight (empty ones -1)
        const bool four = __popcll(vm) <= 4;
        if (wave == 0) {
          if (lane < 8) pl_cand[lane] = two ? (lane == 0 ? __builtin_amdgcn_readlane(cand_id, la)
                                                         : (lane == 1 ? __builtin_amdgcn_readlane(cand_id, lb) : -1))
                                            : cand_id;
          if (lane == 0) pl_two = two ? 1 : 0;
        }
        // rotation chain: the iterate's component and the lanes' candidates
        // (candidates fill the slots from 0 on, so at most four are in 0..3)
        RotLane rl = rot_lane(pA), rl1 = rot_lane(pB);
        float al = 0.f;
        if (CHAIN == 0) {
          al = (lane & 3) == 0 ? Cs.x : ((lane & 3) == 1 ? Cs.y : ((lane & 3) == 2 ? Cs.z : Cs.w));
          if (!two) {
            const int slot_of = pair ? lane >> 5 : (four ? lane >> 4 : lane >> 3);
            rl = rot_lane(make_float4(__shfl(cand_p.x, slot_of, 64), __shfl(cand_p.y, slot_of, 64),
                                      __shfl(cand_p.z, slot_of, 64), __shfl(cand_p.w, slot_of, 64)));
          }
        }
        for (int r = 0; r <= nrounds; ++r) {
          const int s_r = pi0 + r * kPipeSteps;
          const int slot = r % 3;
          if (tid == 0) pl_fail[slot] = INT32_MAX;  // (read last at the start of round r - 2)
          if (wave == 0) {
            if (r < nrounds) {
              const int n_r = min(kPipeSteps, pend - s_r + 1);
              const float pinv_tab = 1.f / (float)(s_r + lane);  // 1/i of step s_r + lane
              // (kPipeSteps is even: step k of every round takes A when k is even)
              float *rec_c = reinterpret_cast<float *>(&pl_C[slot][0]) + (lane & 3);
              if constexpr (CHAIN == 0) {
                const float inv4 = 4.f * pinv_tab;
                al = two ? rot_lane_alternate(al, rl, rl1, inv4, n_r, rec_c)
                         : (pair ? rot_lane_run<2>(al, rl, inv4, n_r, rec_c)
                                 : (four ? rot_lane_run<4>(al, rl, inv4, n_r, rec_c)
                                         : rot_lane_run<8>(al, rl, inv4, n_r, rec_c)));
              } else if (two) {
                for (int k = 0; k < n_r; ++k) {
                  const float inv = readlane_f(pinv_tab, k);
                  if (lane == 0) pl_C[slot][k] = Cs;
                  Cs = geodesic_step_inv<true>(Cs, (k & 1) ? pB : pA, inv, chain);
                }
              } else {
                for (int k = 0; k < n_r; ++k) {
                  const float inv = readlane_f(pinv_tab, k);
                  // predicted winner: the argmax over the candidates (lanes
                  // 0..7) with the keys of the full argmax; the step toward
                  // every candidate, one per lane, alongside it
                  const float u = sqdist(Cs, cand_p, chain);
                  const float4 Cn = geodesic_step_inv<true>(Cs, cand_p, inv, chain);
                  int ub = __float_as_int(u);
                  ub = max(ub, __builtin_amdgcn_update_dpp(INT32_MIN, ub, 0xB1, 0xF, 0xF, false));
                  ub = max(ub, __builtin_amdgcn_update_dpp(INT32_MIN, ub, 0x4E, 0xF, 0xF, false));
                  ub = max(ub, __builtin_amdgcn_update_dpp(INT32_MIN, ub, 0x141, 0xF, 0xF, false));
                  const int umax = __builtin_amdgcn_readlane(ub, 0);
                  const unsigned long long at_max = __ballot(__float_as_int(u) == umax) & 0xFFull;
                  const int wl = at_max ? (int)__ffsll((long long)at_max) - 1 : 0;
                  if (lane == 0) pl_C[slot][k] = Cs;
                  Cs = make_float4(readlane_f(Cn.x, wl), readlane_f(Cn.y, wl), readlane_f(Cn.z, wl),
                                   readlane_f(Cn.w, wl));
                }
              }
              // (a checkpoint from a step found wrong later is rewritten
              // when the step is redone)
              if (CHAIN == 0 && lane < n_r && (s_r + lane - 1) % ck == 0)
                ckq[(s_r + lane - 1) / ck] = pl_C[slot][lane];
              if (CHAIN == 0) {
                if (r == nrounds - 1 && lane < 4) reinterpret_cast<float *>(&pl_Cend)[lane] = al;
              } else
              if (r == nrounds - 1 && lane == 0) pl_Cend = Cs;
            }
          } else if (r >= 1 && wave != kSkipWave) {
            // check the steps of round r - 1, sixteen at a time: four lanes
            // per step, each scanning every fourth entry of a chunk, until the
            // bounds rule out the rest for all sixteen
            const int s_p = s_r - kPipeSteps, n_p = min(kPipeSteps, pend - s_p + 1);
            const int pslot = (r + 2) % 3;
            const int vw = wave < kSkipWave ? wave - 1 : wave - 2;
            const int sub = lane & 3;
            for (int k0 = 16 * vw; k0 < n_p; k0 += 16 * kVerifiers) {
              const int k = min(k0 + (lane >> 2), n_p - 1);
              const float4 Cv = pl_C[pslot][k];
              bool inside;
              const float dC = drift(Cv, inside);
              auto beats = [&](float key, float ub) {
                const float b = ub + dC + slack;
                return key > b * b;
              };
              // argmax (key desc, id asc) over the lane's entries, then the quad's
              float bk = -1.f, wk = -1.f;
              int bi = INT32_MAX, wi = INT32_MAX;
              bool ok = inside;
              for (int g = 0;;) {
                const int e1 = min(K, 64 * g + 64);
#pragma unroll 4
                for (int e = 64 * g + sub; e < e1; e += 4) {
                  const float kk = sqdist(Cv, S.pt[e], chain);
                  const int q = S.id[e];
                  const bool t = (kk > bk) | ((kk == bk) & (q < bi));
                  bi = t ? q : bi;
                  bk = t ? kk : bk;
                }
                wk = bk;
                wi = bi;
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                  const float ko = st ? dpp_f<0x4E>(wk) : dpp_f<0xB1>(wk);
                  const int io = __float_as_int(st ? dpp_f<0x4E>(__int_as_float(wi)) : dpp_f<0xB1>(__int_as_float(wi)));
                  const bool t = better(ko, io, wk, wi);
                  wi = t ? io : wi;
                  wk = t ? ko : wk;
                }
                ++g;
                const float rest = g < nchunks ? S.chunk_ub[g] : theta;
                const bool open = (g < nchunks || theta >= 0.f) && !beats(wk, rest);
                if (__ballot(open) == 0ull) break;
                if (g >= nchunks || (g > recentre && s_p + k0 - i0 > kMinShellSteps)) {
                  // (samples outside the shell may win, or a step needs many
                  // chunks: a sequential segment redoes it and re-centres)
                  ok = ok && !open;
                  break;
                }
              }
              // the winner is the predicted one if it is among the candidates,
              // which were compared by the same keys and rule
              bool hit = false;
              if (pl_two) {
                hit = wi == pl_cand[k & 1];
              } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) hit = hit || wi == pl_cand[c];
              }
              if (!(ok && hit) && sub == 0) atomicMin(&pl_fail[pslot], k);
              if (sub == 0) pl_W[pslot][k] = wi;
            }
          }
          __syncthreads();
          if (r >= 1) {
            const int s_p = s_r - kPipeSteps, n_p = min(kPipeSteps, pend - s_p + 1);
            const int pslot = (r + 2) % 3;
            const int f = pl_fail[pslot];
            // the verified steps of round r - 1 enter the trace
            if (wave == 1 && lane < min(n_p, f)) tr[2 * (s_p + lane - 1)] = pl_W[pslot][lane];
            if (f != INT32_MAX) {
              fail_step = s_p + f;
              fail_C = pl_C[pslot][f];
              break;
            }
          }
        }
        if (tid == 0) {
          ++sdg.n_seg;
          sdg.n_piped += (fail_step == INT32_MAX ? pend + 1 : fail_step) - pi0;
          sdg.n_fail += fail_step == INT32_MAX ? 0 : 1;
        }
        if (fail_step == INT32_MAX) {
          C = pl_Cend;
          i = pend + 1;
        } else {
          C = fail_C;
          i = fail_step;
          if (two)
            ++turn_fails;
          else
            backoff = min(2 * backoff, kPipeMaxSeq);
          stable = 0;
        }
        // (pl_Cend and the failing slot are read before any later write:
        // the next write to either follows the barrier that ends the next
        // sequential segment)
      }
      // after a stage that made no step, a stage of scan steps
      stalled = st_i == i0;
      if (!stalled) scan_len = kScanSteps;
    }
  }
  // ------------------------------------------------------------------ centre
  if (tid == 0) {
    if (ep) {  // (as they may have been gathered anew)
      rec[j].dm_n[chain] = sg.n;
      rec[j].dm_rho[chain] = sg.rho;
      rec[j].dm_c[chain] = sg.C;
    }
    rec[j].n_rescan[chain] = sdg.n_rescan;
    rec[j].n_global[chain] = sdg.n_global | (sg.n_built << 16);
    rec[j].n_groups[chain] = sdg.n_groups;
    // (the real-time clock runs at 100 MHz)
    rec[j].chain_us[chain] = (int32_t)((__builtin_amdgcn_s_memrealtime() - sdg.t_start) / 100ull);
    if (chain == 0) {
      rec[j].n_piped = sdg.n_piped;
      rec[j].n_pipe_fail = sdg.n_fail;
      rec[j].n_pipe_seg = sdg.n_seg;
    }
    if (chain == 0) {
      double Md[9], Rd[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) Md[k] = (double)acc[k];
      polar_so3<double>(Md, Rd, 12);
#pragma unroll
      for (int k = 0; k < 9; ++k) rec[j].centre[k] = (float)Rd[k];
    } else {
      const int na = avg < T ? avg : T;
#pragma unroll
      for (int k = 0; k < 3; ++k) rec[j].centre[9 + k] = acc[k] / (float)na;
    }
  }
}

// One workgroup of chain_block<V>() threads per (instance, chain): even blocks
// run the rotation chain, odd blocks the translation chain.
// The narrow variant is held to 128 VGPRs (a few spills outside the step
// loops), so that four chains share a compute unit: a chain's steps run in
// one wavefront, which leaves most issue slots to the other chains' waves.
template <int V>
__global__ void __launch_bounds__(chain_block<V>(), V == kChainWide ? 1 : 4) k_megb_chain(const int64_t *__restrict__ sample_off, int64_t max_m,
                                                            const float4 *__restrict__ quat,
                                                            const float4 *__restrict__ trans, MegbRec *rec,
                                                            float *dref_all, int64_t total_samples,
                                                            int32_t *trace, float4 *ckpt, int ck, int T, int avg,
                                                            int cap, int no_prune, int n_early,
                                                            const EarlyScratch *es, DmSlots dms) {
  extern __shared__ float4 sh_pt[];
  __shared__ unsigned int hist[kBins];
  __shared__ unsigned int cursor[kBins];
  __shared__ float chunk_ub[kMaxChunks];
  __shared__ float red_k[2][kChainWaves];
  __shared__ int red_i[2][kChainWaves];
  const ChainShared S{sh_pt, reinterpret_cast<int *>(sh_pt + cap), hist, cursor, chunk_ub, red_k, red_i};
  if (blockIdx.x & 1)
    chain_run<1, V>(S, sample_off, max_m, trans, rec, dref_all, total_samples, trace, ckpt, ck, T, avg, cap,
                       no_prune, n_early, es, dms);
  else
    chain_run<0, V>(S, sample_off, max_m, quat, rec, dref_all, total_samples, trace, ckpt, ck, T, avg, cap,
                       no_prune, n_early, es, dms);
}

// Signature of an instance's descent, stored with the checkpoints it left, so
// that the backward uses them only for this descent: the sum of a term per
// step of (step, winner, the bits of the winner's rotation), and one for the
// start (the first feasible sample), which determine the iterates.  One
// workgroup, beside those of the radii (its 4,096 gathers are all latency:
// 17 us as a launch of its own).
__device__ __forceinline__ void sign_descent(int64_t off, int64_t M, const float *__restrict__ poses,
                                             const int32_t *__restrict__ tr, MegbRec &rec, int T, int ck) {
  const int first = rec.first;
  unsigned long long h = 0ull;
  if (first != INT32_MAX)
    for (int i = (int)threadIdx.x; i <= T; i += kBlock) {
      const int id = i == 0 ? first : tr[2 * (i - 1)];
      if (id >= 0 && id < M) {
        uint32_t R[9];
        const float *P = poses + 12 * (off + id);
        for (int k = 0; k < 9; ++k) R[k] = __float_as_uint(P[k]);
        h += step_sig_term(i, id, R);
      } else {
        h += trace_mix(i, id);
      }
    }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) h += __shfl_xor(h, o, 64);
  __shared__ unsigned long long part[kWaves];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0ull;
    for (int w = 0; w < kWaves; ++w) t += part[w];
    rec.ck_hash = t;
    rec.ck_T = first != INT32_MAX ? T : 0;
    rec.ck_every = ck;
  }
}

// float64 radii about the centre: max ||R* - R_s||_F^2 and ||t* - t_s||^2
// (the first workgroup of each instance signs its descent instead).
template <int PER>
__global__ void __launch_bounds__(kBlock) k_megb_radii(const int64_t *__restrict__ sample_off, int64_t total,
                                                       int64_t max_m, const float *__restrict__ poses,
                                                       const uint8_t *__restrict__ mask, MegbRec *rec,
                                                       const int32_t *__restrict__ trace, int T, int ck) {
  const int j = blockIdx.y;
  int64_t off, M;
  sample_range(sample_off, j, total, max_m, off, M);
  if (blockIdx.x == 0) {
    sign_descent(off, M, poses, trace + (int64_t)j * T * 2, rec[j], T, ck);
    return;
  }
  const int64_t s0 = (int64_t)(blockIdx.x - 1) * (kBlock * PER) + threadIdx.x;
  __shared__ double red[2][kWaves];
  double fr = 0.0, ft = 0.0;
  if (rec[j].first != INT32_MAX) {
    // PER samples per thread, kBlock apart, loads in flight together
    uint8_t m[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int64_t s = s0 + u * kBlock;
      m[u] = s < M ? mask[off + s] : (uint8_t)0;
    }
    float4 pa[PER], pb[PER], pc[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int64_t s = s0 + u * kBlock;
      if (s < M && (m[u] & PURSE_MASK_FEASIBLE)) {
        const float4 *pp = reinterpret_cast<const float4 *>(poses + 12 * (off + s));
        pa[u] = pp[0];
        pb[u] = pp[1];
        pc[u] = pp[2];
      }
    }
    const float *C = rec[j].centre;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int64_t s = s0 + u * kBlock;
      if (s < M && (m[u] & PURSE_MASK_FEASIBLE)) {
        const float P[12] = {pa[u].x, pa[u].y, pa[u].z, pa[u].w, pb[u].x, pb[u].y,
                             pb[u].z, pb[u].w, pc[u].x, pc[u].y, pc[u].z, pc[u].w};
        double r = 0.0, t = 0.0;
        for (int k = 0; k < 9; ++k) {
          double d = (double)C[k] - (double)P[k];
          r += d * d;
        }
        for (int k = 9; k < 12; ++k) {
          double d = (double)C[k] - (double)P[k];
          t += d * d;
        }
        fr = fmax(fr, r);
        ft = fmax(ft, t);
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    fr = fmax(fr, __shfl_xor(fr, o, 64));
    ft = fmax(ft, __shfl_xor(ft, o, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][w] = fr;
    red[1][w] = ft;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kWaves; ++k) {
      fr = fmax(fr, red[0][k]);
      ft = fmax(ft, red[1][k]);
    }
    fr = fmax(fr, red[0][0]);
    ft = fmax(ft, red[1][0]);
    if (fr > 0.0) atomicMax(&rec[j].max_rot, (unsigned long long)__double_as_longlong(fr));
    if (ft > 0.0) atomicMax(&rec[j].max_trans, (unsigned long long)__double_as_longlong(ft));
  }
}

// ---------------------------------------------------------------------------
// Step III of the paper ("The CLOSURE Algorithm"): the exact minimum enclosing
// ball of the feasible samples, translations in R^3 and rotations as unit
// quaternions in R^4 put on one hemisphere (the quaternions of the descent's
// centre and of every sample with a non-negative inner product), replacing
// the descent's centre.  One workgroup per (instance, chain), float64.
//
// The support of the exact ball lies among the samples farthest from the
// descent's centre, which is close to the exact one: a shell of the
// farthest samples (a 256-bin histogram of their distance picks a threshold
// that keeps at most kExactShell of them) is staged in LDS and its exact
// ball found by support-set iteration: the support set B (at most dim + 1
// points) and its ball; the shell's farthest point p from the centre, if
// outside, gives the new ball as the smallest ball enclosing B and p whose
// boundary holds p and some subset of B (the lanes try the 2^|B| subsets,
// each by the circumsphere of its points in their affine hull).  The radius
// grows at every step and the support sets are finite, so this ends; the
// last ball encloses the shell and is the ball of a subset of it, hence the
// shell's minimum ball.  Every sample is then checked against it; any sample
// outside is added to the shell and the iteration resumes, so the final ball
// encloses all samples and is the minimum ball of a subset: the exact one.
//
// Where the descent left undominated samples in global memory (instances of
// the first phase), "all samples" are those: any other one is nearer than one
// of them to every centre in their ball, so a ball around such a centre that
// encloses them encloses it too.  A centre outside it (checked at the end)
// restarts the search over every sample.  (One workgroup's passes over
// 262,144 samples took 1.36 ms, over 10,000-20,000 undominated ones 0.2 ms.)
constexpr int kExactShell = 1024;   // staged at first
constexpr int kExactCap = 2048;     // shell capacity including samples added by the checks
constexpr int kExactRounds = 16;    // check-and-add rounds before giving up (the descent's centre is kept)
constexpr int kExactBins = 256;

__device__ __forceinline__ void exact_point(const float4 *D, int64_t s, int chain, const double ref[4], double x[4]) {
  const float4 a = D[s];
  if (chain == 0) {
    x[0] = a.x;
    x[1] = a.y;
    x[2] = a.z;
    x[3] = a.w;
    const double dot = x[0] * ref[0] + x[1] * ref[1] + x[2] * ref[2] + x[3] * ref[3];
    if (dot < 0.0)
      for (int k = 0; k < 4; ++k) x[k] = -x[k];
  } else {
    x[0] = a.x;
    x[1] = a.y;
    x[2] = a.z;
    x[3] = 0.0;
  }
}

__device__ __forceinline__ double exact_d2(const double x[4], const double c[4]) {
  double d = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) d += (x[k] - c[k]) * (x[k] - c[k]);
  return d;
}

// Circumsphere of k points P[0..k) (rows of 4) in their affine hull:
// c = P0 + sum lam_i (P_i - P0) with 2 (P_i - P0).(c - P0) = |P_i - P0|^2.
// Returns false for affinely dependent points.
__device__ __forceinline__ bool exact_circumsphere(const double P[5][4], int k, double c[4], double &r2) {
  double A[4][4], G[4][4], b[4], lam[4];
  const int m = k - 1;
  for (int i = 0; i < m; ++i)
    for (int q = 0; q < 4; ++q) A[i][q] = P[i + 1][q] - P[0][q];
  for (int i = 0; i < m; ++i) {
    b[i] = 0.0;
    for (int q = 0; q < 4; ++q) b[i] += 0.5 * A[i][q] * A[i][q];
    for (int jj = 0; jj < m; ++jj) {
      double g = 0.0;
      for (int q = 0; q < 4; ++q) g += A[i][q] * A[jj][q];
      G[i][jj] = g;
    }
  }
  // Cholesky of the Gram matrix (positive definite iff independent)
  double scale = 0.0;
  for (int i = 0; i < m; ++i) scale = fmax(scale, G[i][i]);
  for (int i = 0; i < m; ++i) {
    for (int jj = 0; jj <= i; ++jj) {
      double v = G[i][jj];
      for (int q = 0; q < jj; ++q) v -= G[i][q] * G[jj][q];
      if (i == jj) {
        if (!(v > 1e-14 * scale)) return false;
        G[i][i] = sqrt(v);
      } else {
        G[i][jj] = v / G[jj][jj];
      }
    }
  }
  for (int i = 0; i < m; ++i) {
    double v = b[i];
    for (int q = 0; q < i; ++q) v -= G[i][q] * lam[q];
    lam[i] = v / G[i][i];
  }
  for (int i = m - 1; i >= 0; --i) {
    double v = lam[i];
    for (int q = i + 1; q < m; ++q) v -= G[q][i] * lam[q];
    lam[i] = v / G[i][i];
  }
  for (int q = 0; q < 4; ++q) {
    double v = P[0][q];
    for (int i = 0; i < m; ++i) v += lam[i] * A[i][q];
    c[q] = v;
  }
  r2 = exact_d2(P[0], c);
  return true;
}

__global__ void __launch_bounds__(kBlock) k_megb_exact(const int64_t *__restrict__ sample_off, int64_t total,
                                                       int64_t max_m, const float4 *__restrict__ quat,
                                                       const float4 *__restrict__ trans, MegbRec *rec,
                                                       DmSlots dms) {
  const int j = blockIdx.x >> 1, chain = blockIdx.x & 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t off, M64;
  sample_range(sample_off, j, total, max_m, off, M64);
  if (rec[j].first == INT32_MAX) return;  // empty instance (whole workgroup)
  const float dm_rho = rec[j].dm_rho[chain];
  const int dm_n = rec[j].dm_n[chain];
  const float4 dm_c = rec[j].dm_c[chain];
  bool pruned = dm_rho > 0.f && dm_n > 0 && dm_n <= (int)(M64 >> dms.shift);
  const int dim = chain ? 3 : 4;
  __shared__ double pts[kExactCap][4];
  __shared__ int hist[kExactBins];
  __shared__ int n_s, fail_s, nb_s, add_s;
  __shared__ double B_s[5][4], c_s[4], r2_s, thr_s;
  __shared__ double red_v[kWaves];
  __shared__ int red_i[kWaves];
  // the descent's centre (and the hemisphere's reference)
  double ref[4];
  {
    const float *C = rec[j].centre;
    if (chain == 0) {
      const float4 q = quat_from_rot(C);
      ref[0] = q.x;
      ref[1] = q.y;
      ref[2] = q.z;
      ref[3] = q.w;
    } else {
      ref[0] = C[9];
      ref[1] = C[10];
      ref[2] = C[11];
      ref[3] = 0.0;
    }
  }
  // ---- largest distance from the descent's centre, then the shell threshold
  auto block_max = [&](double v, int i, double &bv, int &bi) {
    for (int o = 32; o >= 1; o >>= 1) {
      const double v2 = __shfl_xor(v, o, 64);
      const int i2 = __shfl_xor(i, o, 64);
      if (v2 > v || (v2 == v && i2 < i)) {
        v = v2;
        i = i2;
      }
    }
    if (lane == 0) {
      red_v[wave] = v;
      red_i[wave] = i;
    }
    __syncthreads();
    bv = red_v[0];
    bi = red_i[0];
    for (int w = 1; w < kWaves; ++w)
      if (red_v[w] > bv || (red_v[w] == bv && red_i[w] < bi)) {
        bv = red_v[w];
        bi = red_i[w];
      }
    __syncthreads();
  };
  for (;;) {
    const float4 *D = pruned ? dms.pt + chain * dms.stride + (off >> dms.shift) : (chain ? trans : quat) + off;
    const int M = pruned ? dm_n : (int)M64;
    double dmax = -1.0;
    int imax = INT32_MAX;
    for (int s = tid; s < M; s += kBlock) {
      if (!feasible_pt(D[s], chain)) continue;
      double x[4];
      exact_point(D, s, chain, ref, x);
      const double d = exact_d2(x, ref);
      if (d > dmax) {
        dmax = d;
        imax = s;
      }
    }
    double r2hat;
    int ihat;
    block_max(dmax, imax, r2hat, ihat);
    if (ihat == INT32_MAX) {  // no distance is a number: the descent's centre is kept
      if (tid == 0) fail_s = 1;
      break;
    }
    const double rhat = sqrt(fmax(r2hat, 0.0));
    for (int k = tid; k < kExactBins; k += kBlock) hist[k] = 0;
    __syncthreads();
    // bins of the distance over [0, rhat]; the threshold keeps at most
    // kExactShell samples (all of them when there are fewer)
    const double binw = rhat > 0.0 ? rhat / kExactBins : 1.0;
    for (int s = tid; s < M; s += kBlock) {
      if (!feasible_pt(D[s], chain)) continue;
      double x[4];
      exact_point(D, s, chain, ref, x);
      const int bin = max(0, min(kExactBins - 1, (int)(sqrt(exact_d2(x, ref)) / binw)));
      atomicAdd(&hist[bin], 1);
    }
    __syncthreads();
    if (tid == 0) {
      int acc = 0, b = kExactBins;
      while (b > 0 && acc + hist[b - 1] <= kExactShell) acc += hist[--b];
      thr_s = b == kExactBins ? rhat : b * binw;  // (a top bin over capacity: its farthest sample only)
      n_s = 0;
      fail_s = 0;
    }
    __syncthreads();
    const double thr = thr_s;
    for (int s = tid; s < M; s += kBlock) {
      if (!feasible_pt(D[s], chain)) continue;
      double x[4];
      exact_point(D, s, chain, ref, x);
      if (sqrt(exact_d2(x, ref)) >= thr || s == ihat) {
        const int k = atomicAdd(&n_s, 1);
        if (k < kExactShell)
          for (int q = 0; q < 4; ++q) pts[k][q] = x[q];
      }
    }
    __syncthreads();
    if (tid == 0) {
      n_s = min(n_s, kExactShell);
      // start: the ball of the single farthest sample
      double x[4];
      exact_point(D, ihat, chain, ref, x);
      for (int q = 0; q < 4; ++q) {
        B_s[0][q] = x[q];
        c_s[q] = x[q];
      }
      nb_s = 1;
      r2_s = 0.0;
    }
    __syncthreads();
    const double eps = 1e-12;
    for (int round = 0; round < kExactRounds; ++round) {
      // ---- support-set iteration on the shell
      for (int step = 0; step < 4 * kExactCap; ++step) {
        const double c[4] = {c_s[0], c_s[1], c_s[2], c_s[3]};
        const double r2 = r2_s;
        double bv = -1.0;
        int bi = INT32_MAX;
        for (int k = tid; k < n_s; k += kBlock) {
          const double d = exact_d2(pts[k], c);
          if (d > bv) {
            bv = d;
            bi = k;
          }
        }
        double fv;
        int fi;
        block_max(bv, bi, fv, fi);
        if (fi == INT32_MAX || fv <= r2 * (1.0 + eps) + 1e-300) break;
        // smallest ball with p on its boundary enclosing B and p (wave 0: one
        // subset of B per lane)
        if (wave == 0) {
          const int nb = nb_s;
          double best_r2 = INFINITY, best_c[4] = {0, 0, 0, 0};
          int best_m = -1;
          if (lane < (1 << nb)) {
            double P[5][4];
            int k = 0;
            for (int q = 0; q < 4; ++q) P[k][q] = pts[fi][q];
            ++k;
            for (int i = 0; i < nb; ++i)
              if ((lane >> i) & 1) {
                if (k < dim + 1)
                  for (int q = 0; q < 4; ++q) P[k][q] = B_s[i][q];
                ++k;
              }
            double cc[4], rr2;
            if (k <= dim + 1 && exact_circumsphere(P, k, cc, rr2)) {
              bool encl = true;
              for (int i = 0; i < nb; ++i) encl = encl && exact_d2(B_s[i], cc) <= rr2 * (1.0 + 1e-10) + 1e-300;
              if (encl) {
                best_r2 = rr2;
                best_m = lane;
                for (int q = 0; q < 4; ++q) best_c[q] = cc[q];
              }
            }
          }
          // smallest radius, then the lower subset index
          double v = -best_r2;
          int m = best_m < 0 ? INT32_MAX : best_m;
          for (int o = 32; o >= 1; o >>= 1) {
            const double v2 = __shfl_xor(v, o, 64);
            const int m2 = __shfl_xor(m, o, 64);
            if (v2 > v || (v2 == v && m2 < m)) {
              v = v2;
              m = m2;
            }
          }
          if (m == INT32_MAX) {
            if (lane == 0) fail_s = 1;
          } else if (lane == m) {
            double nB[5][4];
            int k = 0;
            for (int q = 0; q < 4; ++q) nB[k][q] = pts[fi][q];
            ++k;
            for (int i = 0; i < nb; ++i)
              if ((m >> i) & 1) {
                for (int q = 0; q < 4; ++q) nB[k][q] = B_s[i][q];
                ++k;
              }
            for (int i = 0; i < k; ++i)
              for (int q = 0; q < 4; ++q) B_s[i][q] = nB[i][q];
            nb_s = k;
            for (int q = 0; q < 4; ++q) c_s[q] = best_c[q];
            r2_s = best_r2;
          }
        }
        __syncthreads();
        if (fail_s) break;
      }
      if (fail_s) break;
      // ---- every sample against the ball; samples outside join the shell
      if (tid == 0) add_s = 0;
      __syncthreads();
      {
        const double c[4] = {c_s[0], c_s[1], c_s[2], c_s[3]};
        const double lim = r2_s * (1.0 + 1e-9) + 1e-300;
        for (int s = tid; s < M; s += kBlock) {
          if (!feasible_pt(D[s], chain)) continue;
          double x[4];
          exact_point(D, s, chain, ref, x);
          if (exact_d2(x, c) > lim) {
            const int k = atomicAdd(&add_s, 1);
            const int slot = n_s + k;
            if (slot < kExactCap)
              for (int q = 0; q < 4; ++q) pts[slot][q] = x[q];
          }
        }
      }
      __syncthreads();
      if (add_s == 0) break;
      if (tid == 0) {
        if (n_s + add_s > kExactCap) fail_s = 1;  // (the shell is full: the descent's centre is kept)
        n_s = min(kExactCap, n_s + add_s);
      }
      __syncthreads();
      if (fail_s) break;
      if (round == kExactRounds - 1 && tid == 0) fail_s = 1;
    }
    __syncthreads();
    if (!pruned) break;
    // the centre lies in the undominated samples' ball (quaternions up to sign)
    const double dc[4] = {dm_c.x, dm_c.y, dm_c.z, chain ? 0.0 : dm_c.w};
    const double nc[4] = {-dc[0], -dc[1], -dc[2], -dc[3]}, cc[4] = {c_s[0], c_s[1], c_s[2], c_s[3]};
    const double d2 = chain ? exact_d2(cc, dc) : fmin(exact_d2(cc, dc), exact_d2(cc, nc));
    const bool inside = d2 <= (double)dm_rho * dm_rho * (1.0 - 1e-5);
    __syncthreads();  // (every thread has read the centre)
    if (!fail_s && inside) break;
    pruned = false;
  }
  __syncthreads();
  if (tid == 0 && !fail_s) {
    if (chain == 0) {
      double q[4] = {c_s[0], c_s[1], c_s[2], c_s[3]};
      const double n = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
      if (n > 0.0) {
        const float4 qf = make_float4((float)(q[0] / n), (float)(q[1] / n), (float)(q[2] / n), (float)(q[3] / n));
        float Rr[9];
        rot_from_quat(qf, Rr);
        for (int k = 0; k < 9; ++k) rec[j].centre[k] = Rr[k];
      }
    } else {
      for (int k = 0; k < 3; ++k) rec[j].centre[9 + k] = (float)c_s[k];
    }
  }
}

__global__ void k_megb_final(int n_inst, const MegbRec *rec, float *centre, double *radii, int64_t *n_feasible,
                             int32_t *inst_status) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_inst) return;
  const MegbRec r = rec[j];
  n_feasible[j] = (int64_t)r.n_feasible;
  if (r.first == INT32_MAX) {
    const float nanf_ = __int_as_float(0x7fc00000);
    for (int k = 0; k < 12; ++k) centre[12 * j + k] = nanf_;
    radii[2 * j] = radii[2 * j + 1] = __longlong_as_double(0x7ff8000000000000ll);
    if ((inst_status[j] & 0xFF) == PURSE_INST_OK) inst_status[j] = (inst_status[j] & ~0xFF) | PURSE_INST_EMPTY;
    return;
  }
  for (int k = 0; k < 12; ++k) centre[12 * j + k] = r.centre[k];
  double fr = __longlong_as_double((long long)r.max_rot);
  double ft = __longlong_as_double((long long)r.max_trans);
  double x = sqrt(fr) / (2.0 * sqrt(2.0));
  radii[2 * j] = 2.0 * asin(x < 1.0 ? x : 1.0);
  radii[2 * j + 1] = sqrt(ft);
}

void launch_megb(const DevBatch &b, const DevParams &p, const float *poses, const uint8_t *mask, MegbRec *rec,
                 float4 *quat, float4 *trans, float *dref, float4 *ckpt, EarlyScratch *es, DmSlots dms, float *centre,
                 double *radii, int64_t *n_feasible, int32_t *trace, int32_t *inst_status, int64_t max_samples,
                 int64_t total_samples, hipStream_t stream) {
  const int ck = ckpt_spacing(p.ckpt_every);
  const int n = b.n_inst;
  hipLaunchKernelGGL(k_megb_init, dim3((n + 255) / 256), dim3(256), 0, stream, n, rec);
  // (several samples per thread on large instances: fewer workgroups and
  // atomics; one on small ones, whose passes are latency-bound)
  const bool per4 = max_samples >= kPassPerMin;
  const int per = per4 ? kPassPer : 1;
  const dim3 grid((unsigned)((max_samples + kBlock * per - 1) / (kBlock * per)), (unsigned)n);
  const dim3 rgrid(grid.x + 1, grid.y);  // (and one workgroup per instance for its signature)
  if (per4)
    hipLaunchKernelGGL(k_megb_prep<kPassPer>, grid, dim3(kBlock), 0, stream, b.sample_off, total_samples,
                       max_samples, poses, mask, rec, quat, trans);
  else
    hipLaunchKernelGGL(k_megb_prep<1>, grid, dim3(kBlock), 0, stream, b.sample_off, total_samples, max_samples,
                       poses, mask, rec, quat, trans);
  // The wide variant while there are at most as many chains as compute
  // units, else the narrow one (measured on batches of 256-1,024 uneven
  // instances: 1.4-2.3 times faster than the shell steps of one wave with no
  // pipelined segments, which ran at the same four chains per compute unit).
  // The variants keep shells of different capacities, which the first-phase
  // kernel must know.
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    n_cu = 0;
  const bool wide = 2 * n <= n_cu;
  const int cap = wide ? chain_cap<kChainWide>() : chain_cap<kChainNarrow>();
  const size_t lds = (size_t)cap * (sizeof(float4) + sizeof(int));
  const int no_prune = (p.flags & PURSE_FLAG_NO_PRUNING) ? 1 : 0;
  const int n_early = early_steps(max_samples, wide, p.megb_iters, p.megb_avg);
  if (early_phase_applies(max_samples, no_prune, n_early)) {
    const dim3 eg((unsigned)kEarlyWG, 2u, (unsigned)n);
    for (int i = 1; i <= n_early; ++i)
      hipLaunchKernelGGL(k_megb_early, eg, dim3(kEarlyBlock), 0, stream, b.sample_off, total_samples, max_samples,
                         quat, trans, rec, es, trace, ckpt, ck, p.megb_iters, p.megb_avg, cap, no_prune, n_early,
                         dms, i);
  }
  if (wide)
    hipLaunchKernelGGL(k_megb_chain<kChainWide>, dim3(2 * n), dim3(chain_block<kChainWide>()), lds, stream,
                       b.sample_off, max_samples, quat, trans, rec, dref, total_samples, trace, ckpt, ck, p.megb_iters,
                       p.megb_avg, cap, no_prune, n_early, es, dms);
  else
    hipLaunchKernelGGL(k_megb_chain<kChainNarrow>, dim3(2 * n), dim3(chain_block<kChainNarrow>()), lds, stream,
                       b.sample_off, max_samples, quat, trans, rec, dref, total_samples, trace, ckpt, ck, p.megb_iters,
                       p.megb_avg, cap, no_prune, n_early, es, dms);
  if (p.flags & PURSE_FLAG_EXACT_MEB)
    hipLaunchKernelGGL(k_megb_exact, dim3(2 * n), dim3(kBlock), 0, stream, b.sample_off, total_samples, max_samples,
                       quat, trans, rec, dms);
  if (per4)
    hipLaunchKernelGGL(k_megb_radii<kPassPer>, rgrid, dim3(kBlock), 0, stream, b.sample_off, total_samples,
                       max_samples, poses, mask, rec, trace, p.megb_iters, ck);
  else
    hipLaunchKernelGGL(k_megb_radii<1>, rgrid, dim3(kBlock), 0, stream, b.sample_off, total_samples, max_samples,
                       poses, mask, rec, trace, p.megb_iters, ck);
  hipLaunchKernelGGL(k_megb_final, dim3((n + 255) / 256), dim3(256), 0, stream, n, rec, centre, radii,
                     n_feasible, inst_status);
}

}  // namespace purse
