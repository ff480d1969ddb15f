// The sampler: one trajectory per lane.  A workgroup covers one tile of
// blockDim consecutive samples of one instance, so every wave reads the same
// keypoint records (wave-uniform loads) and runs one code path; one launch
// per kind keeps each kind's register allocation separate.
//
// Tiles of a ragged batch are dealt from a schedule: per kind, the instances in
// decreasing per-trajectory cost (the keypoint count orders it within a kind),
// each contributing ceil(M_j / tile) consecutive tiles.  The hardware dispatches
// workgroups in index order, so the heaviest tiles start first and the tail of
// the launch is made of light ones (longest-processing-time-first list
// scheduling).  Up to 64 instances, every wavefront works its tile out from the
// records itself (few_tile); larger batches, and the work queue, have the
// schedule built on the device after the prologue (k_schedule).  A launch that
// the chip holds at once anyway runs all kinds in one kernel (k_sample_few).
#include <algorithm>
#include <mutex>

#include "purse_launch.hpp"
#include "purse_traj.hpp"

namespace purse {

constexpr int kSmallN = 16;  // keypoint bound of the unrolled 2D-3D variant

// Keypoints of the general 2D-3D loop whose targets stay in LDS: the 7.5 KB a
// wavefront that 160 KB allows at the five wavefronts per SIMD of its registers
// (four wavefronts with 20 keypoints, and three with 26, are slower).
constexpr int kHeldKp = 15;

constexpr int kSchedBlock = 1024;

// Launch group of an instance: 0 for 3D-3D (an invalid kind goes there too,
// and its flagged outputs are written as zeros), 1 for 2D-3D with the
// general keypoint loop, 2 for 2D-3D instances of at most kSmallN keypoints
// (the unrolled loop, unless the flags ask for the general one).  The group
// depends on the instance alone, so an instance computes bitwise the same
// samples in any batch.
__device__ __forceinline__ int launch_group(const InstRec &I, int flags) {
  if (I.kind != PURSE_KIND_2D3D) return 0;
  return (I.n_kp <= kSmallN && !(flags & PURSE_FLAG_GENERIC_LOOP)) ? 2 : 1;
}

// Lanes per trajectory of launch group 2.
__host__ __device__ inline int group_lanes(int flags) {
  return (flags & PURSE_FLAG_QUAD_LANES) ? 4 : ((flags & PURSE_FLAG_PAIR_LANES) ? 2 : 1);
}

template <int KIND, int NMAX>
constexpr int group_of() {
  return KIND == PURSE_KIND_3D3D ? 0 : (NMAX > 0 ? 2 : 1);
}

constexpr int kMaxSorted = 8192;  // larger batches keep instance order

// Samples per tile of a launch group (a power of two), for workgroups of
// `lanes`: one per lane, or one per lane group in the lane-group modes.
__device__ __forceinline__ int tile_shift(int group, int lanes, int flags) {
  return 31 - __clz(group == 2 ? lanes / group_lanes(flags) : lanes);
}

__device__ __forceinline__ uint32_t tiles_of(const InstRec &I, int group, int lanes, int flags) {
  const int sh = tile_shift(group, lanes, flags);
  return (uint32_t)((I.n_samples + (((int64_t)1 << sh) - 1)) >> sh);
}

// Cost class of an instance's trajectories, 0 the heaviest.
__device__ __forceinline__ int cost_class(const InstRec &I, int flags) {
  return (flags & PURSE_FLAG_INSTANCE_ORDER) ? 0 : PURSE_MAX_KP - min(max(I.n_kp, 0), PURSE_MAX_KP);
}

constexpr int kSchedKeys = kSchedGroups * (PURSE_MAX_KP + 1);  // (group, cost class)

// Builds the groups' schedules in one workgroup.  A stable counting sort by
// (group, cost class, index): totals per key, then each chunk of kSchedBlock
// instances takes its places from the keys' bases, the counts of the
// wavefronts before its own, and its rank among the equal keys of its
// wavefront; then one prefix sum of tile counts over the whole order, from
// which each group takes the differences to its own start.  (Ranking every
// instance against every other, one group after the other, took 102 us for
// 512 instances, between the prologue and the first trajectory.)
__global__ void __launch_bounds__(kSchedBlock) k_schedule(const InstRec *__restrict__ inst, int n, int tile_lanes,
                                                          int flags, int32_t *__restrict__ sched) {
  constexpr int kWaves = kSchedBlock / 64;
  __shared__ uint32_t tl[kMaxSorted];            // tile counts in order
  __shared__ uint32_t cnt[kWaves][kSchedKeys];   // a chunk's counts per wavefront, then places
  __shared__ uint32_t base[kSchedKeys];          // next place of each key
  __shared__ uint32_t part[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t stride = sched_ints(n);
  // exclusive prefix sum of one value per thread
  auto scan = [&](uint32_t v, uint32_t &total) {
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)x, o, 64);
      if (lane >= o) x += y;
    }
    __syncthreads();  // (part is free)
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t q = part[w];
      before += w < wave ? q : 0u;
      all += q;
    }
    total = all;
    return before + x - v;
  };
  if (n <= kMaxSorted) {
    for (int k = tid; k < kSchedKeys; k += kSchedBlock) base[k] = 0u;
    __syncthreads();
    auto key_of = [&](const InstRec &I) {
      return launch_group(I, flags) * (PURSE_MAX_KP + 1) + cost_class(I, flags);
    };
    for (int j = tid; j < n; j += kSchedBlock) atomicAdd(&base[key_of(inst[j])], 1u);
    __syncthreads();
    {
      const uint32_t v = tid < kSchedKeys ? base[tid] : 0u;
      uint32_t total;
      const uint32_t x = scan(v, total);
      if (tid < kSchedKeys) base[tid] = x;
      __syncthreads();
    }
    uint32_t g0[kSchedGroups + 1];  // first place of each group
    for (int g = 0; g < kSchedGroups; ++g) g0[g] = base[g * (PURSE_MAX_KP + 1)];
    g0[kSchedGroups] = (uint32_t)n;
    __syncthreads();
    for (int j0 = 0; j0 < n; j0 += kSchedBlock) {
      for (int k = tid; k < kWaves * kSchedKeys; k += kSchedBlock) (&cnt[0][0])[k] = 0u;
      __syncthreads();
      const int j = j0 + tid;
      const bool in = j < n;
      int grp = 0, key = 0;
      uint32_t tiles = 0;
      if (in) {
        const InstRec &I = inst[j];
        grp = launch_group(I, flags);
        key = key_of(I);
        tiles = tiles_of(I, grp, tile_lanes, flags);
      }
      unsigned long long same = __ballot(in);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const unsigned long long m = __ballot((key >> bit) & 1);
        same &= ((key >> bit) & 1) ? m : ~m;
      }
      const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
      if (in && rank == 0u) cnt[wave][key] = (uint32_t)__popcll(same);
      __syncthreads();
      if (tid < kSchedKeys) {
        uint32_t at = base[tid];
        for (int w = 0; w < kWaves; ++w) {
          const uint32_t c = cnt[w][tid];
          cnt[w][tid] = at;
          at += c;
        }
        base[tid] = at;
      }
      __syncthreads();
      if (in) {
        const uint32_t r = cnt[wave][key] + rank;
        tl[r] = tiles;
        sched[grp * stride + (r - g0[grp])] = j;
      }
      __syncthreads();
    }
    const int per = (n + kSchedBlock - 1) / kSchedBlock;
    const int b0 = min(n, tid * per), b1 = min(n, b0 + per);
    uint32_t acc = 0, total;
    for (int k = b0; k < b1; ++k) acc += tl[k];
    uint32_t run = scan(acc, total);
    __syncthreads();
    for (int k = b0; k < b1; ++k) {
      const uint32_t t = tl[k];
      tl[k] = run;
      run += t;
    }
    __syncthreads();
    for (int g = 0; g < kSchedGroups; ++g) {
      // places beyond the group's instances start at its end: no tile of theirs
      int32_t *tstart = sched + g * stride + n;
      const uint32_t first = g0[g] < (uint32_t)n ? tl[g0[g]] : total;
      const uint32_t end = (g0[g + 1] < (uint32_t)n ? tl[g0[g + 1]] : total) - first;
      const int m = (int)(g0[g + 1] - g0[g]);
      for (int k = tid; k <= n; k += kSchedBlock) tstart[k] = (int32_t)(k < m ? tl[g0[g] + k] - first : end);
    }
  } else {
    // instance order, one group after the other
    const int per = (n + kSchedBlock - 1) / kSchedBlock;
    const int b0 = min(n, tid * per), b1 = min(n, b0 + per);
    for (int g = 0; g < kSchedGroups; ++g) {
      int32_t *order = sched + g * stride, *tstart = order + n;
      auto tiles = [&](int j) {
        const InstRec &I = inst[j];
        return launch_group(I, flags) == g ? tiles_of(I, g, tile_lanes, flags) : 0u;
      };
      uint32_t acc = 0, total;
      for (int j = b0; j < b1; ++j) acc += tiles(j);
      uint32_t run = scan(acc, total);
      for (int j = b0; j < b1; ++j) {
        order[j] = j;
        tstart[j] = (int32_t)run;
        run += tiles(j);
      }
      if (tid == 0) tstart[n] = (int32_t)total;
    }
  }
  // the work-queue counters of the three groups
  if (tid < kSchedGroups) sched[kSchedGroups * stride + tid] = 0;
}

// Tile b of launch group `group` (all of them for -1) of at most kFewInst
// instances: its instance j and its place t among that instance's tiles; false
// beyond the last tile.  Lane l holds instance l's tile count and cost, and
// sums the counts of the instances before it; whole wavefronts call it.  (A
// schedule built by a kernel of its own cost a launch, 10 us of the 0.2 ms of
// the smallest calls; the sums are some 6 instructions per instance.)
constexpr int kFewInst = 64;

__device__ __forceinline__ bool few_tile(const InstRec *__restrict__ inst, int n, int lanes, int flags, int group,
                                         uint32_t b, int &j, uint32_t &t) {
  const int lane = threadIdx.x & 63;
  int key = INT32_MAX;
  uint32_t tiles = 0;
  if (lane < n) {
    const InstRec &I = inst[lane];
    const int g = launch_group(I, flags);
    if (group < 0 || g == group) {
      tiles = tiles_of(I, g, lanes, flags);
      // (a 2D-3D trajectory takes longer than any 3D-3D one)
      key = cost_class(I, flags) + (g == 0 && !(flags & PURSE_FLAG_INSTANCE_ORDER) ? PURSE_MAX_KP + 1 : 0);
    }
  }
  uint32_t start = 0;
  for (int i = 0; i < n; ++i) {
    const int ki = __builtin_amdgcn_readlane(key, i);
    const uint32_t ti = (uint32_t)__builtin_amdgcn_readlane((int)tiles, i);
    start += (ki < key || (ki == key && i < lane)) ? ti : 0u;
  }
  const unsigned long long hit = __ballot(b >= start && b - start < tiles);
  if (hit == 0ull) return false;
  j = __ffsll(hit) - 1;
  t = b - (uint32_t)__builtin_amdgcn_readlane((int)start, j);
  return true;
}

// The tile of schedule entry b: the entry k of the order with
// tstart[k] <= b < tstart[k + 1].
__device__ __forceinline__ int tile_entry(const int32_t *__restrict__ tstart, int n_inst, int b) {
  int lo = 0, hi = n_inst - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tstart[mid] <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Sample s of instance j, one per lane.
template <int KIND, int NMAX>
__device__ __forceinline__ void sample_at(int j, int64_t s, const InstRec *__restrict__ inst,
                                          const KpRec *__restrict__ kprec, const DevParams &p,
                                          float *__restrict__ poses, uint8_t *__restrict__ mask) {
  const InstRec &I = inst[j];
  if (launch_group(I, p.flags) != group_of<KIND, NMAX>() || s >= I.n_samples) return;
  const int64_t g = I.sample_off + s;
  float4 *out = reinterpret_cast<float4 *>(poses + 12 * g);
  if ((I.status & 0xFF) != PURSE_INST_OK) {
    out[0] = make_float4(0.f, 0.f, 0.f, 0.f);
    out[1] = make_float4(0.f, 0.f, 0.f, 0.f);
    out[2] = make_float4(0.f, 0.f, 0.f, 0.f);
    mask[g] = 0;
    return;
  }
  const FrameRef F = frame_ref(I);
  Pose x = initial_pose<float>(F, I.seed, (uint64_t)s, p);
  int n_fb = 0;
  uint8_t m;
  if constexpr (KIND == PURSE_KIND_2D3D && NMAX == 0) {
    // this lane's column of its wave's kHeldKp x 64 targets
    extern __shared__ float2 held_s[];
    const KpHeld kpl{kprec + I.kp_off, held_s + (threadIdx.x >> 6) * (kHeldKp * 64) + (threadIdx.x & 63),
                     min(I.n_kp, kHeldKp)};
    m = run_trajectory<KIND, NMAX>(I, F, kpl, x, p, true, n_fb);
  } else {
    const KpPlain kpl{kprec + I.kp_off};
    m = run_trajectory<KIND, NMAX>(I, F, kpl, x, p, true, n_fb);
  }
  out[0] = make_float4(x.R[0], x.R[1], x.R[2], x.R[3]);
  out[1] = make_float4(x.R[4], x.R[5], x.R[6], x.R[7]);
  out[2] = make_float4(x.R[8], x.t[0], x.t[1], x.t[2]);
  mask[g] = m;
}

// This workgroup's tile of a launch group: instance j and the tile's place t
// among its tiles, from the schedule or (none: at most kFewInst instances) the
// records.
__device__ __forceinline__ bool tile_of(const InstRec *__restrict__ inst, const int32_t *__restrict__ sched,
                                        int n_inst, int flags, int grp, int &j, uint32_t &t) {
  if (!sched) return few_tile(inst, n_inst, blockDim.x, flags, grp, blockIdx.x, j, t);
  const int32_t *order = sched + (size_t)grp * sched_ints(n_inst);
  const int32_t *tstart = order + n_inst;
  const int b = blockIdx.x;
  if (b >= tstart[n_inst]) return false;
  const int lo = tile_entry(tstart, n_inst, b);
  j = order[lo];
  t = (uint32_t)(b - tstart[lo]);
  return true;
}

// Work-queue mode: each workgroup takes the next tile of the group's
// schedule from the counter k_schedule cleared, until none is left (every
// workgroup reaches the end of the schedule and leaves).
template <typename F>
__device__ __forceinline__ void tile_queue(int32_t *counter, int total, F &&run) {
  __shared__ int sh_b;
  for (;;) {
    if (threadIdx.x == 0) sh_b = atomicAdd(counter, 1);
    __syncthreads();
    const int b = sh_b;
    __syncthreads();  // (sh_b is read before the next tile's atomic overwrites it)
    if (b >= total) break;
    run(b);
  }
}

// (3D-3D: 128 registers, four wavefronts per SIMD)
template <int KIND, int NMAX, bool QUEUE>
__global__ void __launch_bounds__(256, KIND == PURSE_KIND_3D3D ? 4 : 1) k_sample(const InstRec *__restrict__ inst, const KpRec *__restrict__ kprec,
                                                int32_t *__restrict__ sched, int n_inst, DevParams p,
                                                float *__restrict__ poses, uint8_t *__restrict__ mask) {
  constexpr int grp = group_of<KIND, NMAX>();
  if (QUEUE) {
    const int32_t *order = sched + (size_t)grp * sched_ints(n_inst);
    const int32_t *tstart = order + n_inst;
    tile_queue(sched + (size_t)kSchedGroups * sched_ints(n_inst) + grp, tstart[n_inst], [&](int b) {
      const int lo = tile_entry(tstart, n_inst, b);
      sample_at<KIND, NMAX>(order[lo], (int64_t)(b - tstart[lo]) * blockDim.x + threadIdx.x, inst, kprec, p, poses,
                            mask);
    });
  } else {
    int j;
    uint32_t t;
    if (!tile_of(inst, sched, n_inst, p.flags, grp, j, t)) return;
    sample_at<KIND, NMAX>(j, (int64_t)t * blockDim.x + threadIdx.x, inst, kprec, p, poses, mask);
  }
}

// Lane-group modes of the unrolled 2D-3D group (PURSE_FLAG_PAIR_LANES: G = 2,
// PURSE_FLAG_QUAD_LANES: G = 4): a workgroup of blockDim lanes runs blockDim / G
// trajectories, G lanes each; the instance's keypoint records are staged in
// LDS first.
template <int NMAX, int G>
__device__ __forceinline__ void sample_lanes_at(int j, int64_t s0, KpRec *kp_s, const InstRec *__restrict__ inst,
                                                const KpRec *__restrict__ kprec, const DevParams &p,
                                                float *__restrict__ poses, uint8_t *__restrict__ mask) {
  const InstRec &I = inst[j];
  if (launch_group(I, p.flags) != 2) return;  // (whole workgroup)
  const bool valid = (I.status & 0xFF) == PURSE_INST_OK;
  if (valid && (int)threadIdx.x < I.n_kp) kp_s[threadIdx.x] = kprec[I.kp_off + threadIdx.x];
  __syncthreads();
  const int64_t s = s0 + (threadIdx.x / G);
  const int q = threadIdx.x % G;
  if (s >= I.n_samples) return;  // the lanes of a group leave together
  const int64_t g = I.sample_off + s;
  float4 *out = reinterpret_cast<float4 *>(poses + 12 * g);
  if (!valid) {
    if (q == 0) {
      out[0] = make_float4(0.f, 0.f, 0.f, 0.f);
      out[1] = make_float4(0.f, 0.f, 0.f, 0.f);
      out[2] = make_float4(0.f, 0.f, 0.f, 0.f);
      mask[g] = 0;
    }
    return;
  }
  const FrameRef F = frame_ref(I);
  Pose x = initial_pose<float>(F, I.seed, (uint64_t)s, p);
  const uint8_t m = run_trajectory_lanes<NMAX, G>(I, F, kp_s, q, x, p);
  if (q == 0) {
    out[0] = make_float4(x.R[0], x.R[1], x.R[2], x.R[3]);
    out[1] = make_float4(x.R[4], x.R[5], x.R[6], x.R[7]);
    out[2] = make_float4(x.R[8], x.t[0], x.t[1], x.t[2]);
    mask[g] = m;
  }
}

template <int NMAX, int G, bool QUEUE>
__global__ void __launch_bounds__(256, G == 4 ? 4 : 1) k_sample2d_lanes(const InstRec *__restrict__ inst,
                                                        const KpRec *__restrict__ kprec,
                                                        int32_t *__restrict__ sched, int n_inst, DevParams p,
                                                        float *__restrict__ poses, uint8_t *__restrict__ mask) {
  __shared__ KpRec kp_s[NMAX];
  if (QUEUE) {
    // (the queue's barriers also keep a tile's keypoint records until every
    // lane is done with them)
    const int32_t *order = sched + (size_t)2 * sched_ints(n_inst);
    const int32_t *tstart = order + n_inst;
    tile_queue(sched + (size_t)kSchedGroups * sched_ints(n_inst) + 2, tstart[n_inst], [&](int b) {
      const int lo = tile_entry(tstart, n_inst, b);
      sample_lanes_at<NMAX, G>(order[lo], (int64_t)(b - tstart[lo]) * (blockDim.x / G), kp_s, inst, kprec, p, poses,
                               mask);
    });
  } else {
    int j;
    uint32_t t;
    if (!tile_of(inst, sched, n_inst, p.flags, 2, j, t)) return;
    sample_lanes_at<NMAX, G>(j, (int64_t)t * (blockDim.x / G), kp_s, inst, kprec, p, poses, mask);
  }
}

// All launch groups of at most kFewInst instances in one launch, for batches
// that the chip holds at once (few_waves): a launch per group, on streams of
// their own with a fork and a join, costs 25 us that the groups of a large
// batch win back by overlapping and a small batch does not.
template <int G>
__global__ void __launch_bounds__(256) k_sample_few(const InstRec *__restrict__ inst, const KpRec *__restrict__ kprec,
                                                    int n_inst, DevParams p, float *__restrict__ poses,
                                                    uint8_t *__restrict__ mask) {
  __shared__ KpRec kp_s[G > 1 ? kSmallN : 1];
  int j;
  uint32_t t;
  if (!few_tile(inst, n_inst, blockDim.x, p.flags, -1, blockIdx.x, j, t)) return;
  const int64_t s = (int64_t)t * blockDim.x + threadIdx.x;
  const int grp = launch_group(inst[j], p.flags);
  if (grp == 0)
    sample_at<PURSE_KIND_3D3D, 0>(j, s, inst, kprec, p, poses, mask);
  else if (grp == 1)
    sample_at<PURSE_KIND_2D3D, 0>(j, s, inst, kprec, p, poses, mask);
  else if constexpr (G > 1)
    sample_lanes_at<kSmallN, G>(j, (int64_t)t * (blockDim.x / G), kp_s, inst, kprec, p, poses, mask);
  else
    sample_at<PURSE_KIND_2D3D, kSmallN>(j, s, inst, kprec, p, poses, mask);
}

// Wavefronts that k_sample_few holds at once: three per SIMD at its registers.
int64_t few_waves(int n_cu) { return (int64_t)n_cu * 4 * 3; }

int64_t sample_grid(int64_t total_samples, int n_inst, int tile) {
  // sum_j ceil(M_j / tile) <= total / tile + n_inst
  return total_samples / tile + n_inst;
}

namespace {

// Two auxiliary streams (default priority) and three events per device for
// the concurrent launch groups, created on first use and kept until the
// process ends.
struct GroupAux {
  hipStream_t s[2] = {nullptr, nullptr};
  hipEvent_t fork = nullptr, join[2] = {nullptr, nullptr};
  bool ok = false, tried = false;
};
std::mutex g_group_mu;
GroupAux g_group[64];

GroupAux *group_aux() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  GroupAux &a = g_group[dev];
  if (!a.tried) {
    a.tried = true;
    bool ok = hipEventCreateWithFlags(&a.fork, hipEventDisableTiming) == hipSuccess;
    for (int k = 0; k < 2 && ok; ++k)
      ok = hipStreamCreateWithFlags(&a.s[k], hipStreamNonBlocking) == hipSuccess &&
           hipEventCreateWithFlags(&a.join[k], hipEventDisableTiming) == hipSuccess;
    a.ok = ok;
  }
  return a.ok ? &a : nullptr;
}

}  // namespace

hipError_t launch_sample(const DevBatch &b, const DevParams &p, const InstRec *inst, const KpRec *kp,
                         int32_t *sched, float *poses, uint8_t *mask, int asked_tile, int64_t grid_samples,
                         int waves_per_simd, hipStream_t stream) {
  const int tile = asked_tile ? asked_tile : 256;
  const bool queue = (p.flags & PURSE_FLAG_WORK_QUEUE) != 0;
  int dev = 0, n_cu = 256, lds_cu = 163840, lds_block = 65536;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    n_cu = 256;
  if (hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
      lds_cu <= 0)
    lds_cu = 163840;
  if (hipDeviceGetAttribute(&lds_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
      lds_block <= 0)
    lds_block = 65536;
  // LDS that keeps a compute unit from taking more than its share of a launch's
  // workgroups: the dispatcher otherwise doubles up on some while others stay
  // empty, one way or the other from call to call (262144 samples of 24
  // keypoints, four wavefronts per SIMD: 0.77 or 0.89 ms)
  auto even_lds = [&](int64_t wgs) {
    const int64_t share = std::max<int64_t>(1, (wgs + n_cu - 1) / n_cu);
    return (size_t)std::max<int64_t>(0, std::min<int64_t>(lds_cu / (share + 1) + 512, lds_block - 2048));
  };
  if (b.n_inst <= kFewInst && !queue) {
    sched = nullptr;
    const int lanes = group_lanes(p.flags);
    const int64_t waves = sample_grid(grid_samples * lanes, b.n_inst, 64);
    if (waves_per_simd == 0 && !(p.flags & PURSE_FLAG_SERIAL_GROUPS) && waves <= few_waves(n_cu)) {
      // the smallest workgroups, unless the caller asked for a size, that
      // still leave each its own compute unit: a wavefront runs up to 1.4
      // times as fast there
      const int wg = asked_tile ? asked_tile : (waves <= n_cu ? 64 : (waves <= 2 * n_cu ? 128 : 256));
      // sum_j ceil(M_j / t) <= (sum_j M_j + n (t - 1)) / t, t = wg / lanes
      const int t = wg / lanes;
      const int64_t wgs = (grid_samples + (int64_t)b.n_inst * (t - 1)) / t;
      const size_t held = std::max((size_t)wg * kHeldKp * sizeof(float2), even_lds(wgs));
      const dim3 g((unsigned)wgs);
      if (lanes == 4)
        hipLaunchKernelGGL((k_sample_few<4>), g, dim3(wg), held, stream, inst, kp, b.n_inst, p, poses, mask);
      else if (lanes == 2)
        hipLaunchKernelGGL((k_sample_few<2>), g, dim3(wg), held, stream, inst, kp, b.n_inst, p, poses, mask);
      else
        hipLaunchKernelGGL((k_sample_few<1>), g, dim3(wg), held, stream, inst, kp, b.n_inst, p, poses, mask);
      return hipSuccess;
    }
  } else {
    hipLaunchKernelGGL(k_schedule, dim3(1), dim3(kSchedBlock), 0, stream, inst, b.n_inst, tile, p.flags, sched);
  }
  // The three launch groups write disjoint samples and read only the
  // prologue's records and the schedules: they run concurrently on the
  // caller's stream and two auxiliary streams (a fork and a join by events,
  // which graph capture records as edges), so one group's tail overlaps the
  // others' work.  Serially on the caller's stream when asked or when the
  // auxiliary streams could not be created or forked to.
  std::unique_lock<std::mutex> lk(g_group_mu);
  GroupAux *aux = (p.flags & PURSE_FLAG_SERIAL_GROUPS) ? nullptr : group_aux();
  hipStream_t gs[3] = {stream, stream, stream};
  if (aux && hipEventRecord(aux->fork, stream) == hipSuccess &&
      hipStreamWaitEvent(aux->s[0], aux->fork, 0) == hipSuccess &&
      hipStreamWaitEvent(aux->s[1], aux->fork, 0) == hipSuccess) {
    gs[1] = aux->s[0];
    gs[2] = aux->s[1];
  } else {
    aux = nullptr;
  }
  // waves per SIMD: at most 8 resident (the hardware's limit), or the cap,
  // which each workgroup's LDS padding enforces: just over the share of the
  // compute unit's LDS that would admit one more workgroup, within the
  // per-workgroup limit less room for the kernels' own LDS (under 1 KB).  The
  // allocation granularity can leave one workgroup fewer than the cap.
  const int wg_waves = tile / 64;
  const int cap = waves_per_simd > 0 ? waves_per_simd : 8;
  const int wg_per_cu = std::max(1, (4 * cap + wg_waves - 1) / wg_waves);
  size_t lds = waves_per_simd > 0 ? (size_t)std::max(0, std::min(lds_cu / (wg_per_cu + 1) + 512, lds_block - 2048)) : 0;
  // (one instance is one launch group, whose workgroups may all be resident)
  if (waves_per_simd == 0 && b.n_inst == 1 && !queue) {
    const int t = tile / group_lanes(p.flags);
    const int64_t wgs = (grid_samples + t - 1) / t;
    if (wgs <= (int64_t)n_cu * 8) lds = even_lds(wgs);
  }
  // the general 2D-3D loop's held targets
  const size_t lds_held = std::max(lds, (size_t)tile * kHeldKp * sizeof(float2));
  auto grid_of = [&](int t) {
    const int64_t g = sample_grid(grid_samples, b.n_inst, t);
    return dim3((unsigned)(queue ? std::min<int64_t>(g, (int64_t)n_cu * wg_per_cu) : g));
  };
  const dim3 grid = grid_of(tile);
  if (p.flags & PURSE_FLAG_QUAD_LANES) {
    if (queue)
      hipLaunchKernelGGL((k_sample2d_lanes<kSmallN, 4, true>), grid_of(tile / 4), dim3(tile), lds, stream, inst, kp,
                         sched, b.n_inst, p, poses, mask);
    else
      hipLaunchKernelGGL((k_sample2d_lanes<kSmallN, 4, false>), grid_of(tile / 4), dim3(tile), lds, stream, inst, kp,
                         sched, b.n_inst, p, poses, mask);
  } else if (p.flags & PURSE_FLAG_PAIR_LANES) {
    if (queue)
      hipLaunchKernelGGL((k_sample2d_lanes<kSmallN, 2, true>), grid_of(tile / 2), dim3(tile), lds, stream, inst, kp,
                         sched, b.n_inst, p, poses, mask);
    else
      hipLaunchKernelGGL((k_sample2d_lanes<kSmallN, 2, false>), grid_of(tile / 2), dim3(tile), lds, stream, inst, kp,
                         sched, b.n_inst, p, poses, mask);
  } else if (queue) {
    hipLaunchKernelGGL((k_sample<PURSE_KIND_2D3D, kSmallN, true>), grid, dim3(tile), lds, stream, inst, kp, sched,
                       b.n_inst, p, poses, mask);
  } else {
    hipLaunchKernelGGL((k_sample<PURSE_KIND_2D3D, kSmallN, false>), grid, dim3(tile), lds, stream, inst, kp, sched,
                       b.n_inst, p, poses, mask);
  }
  if (queue) {
    hipLaunchKernelGGL((k_sample<PURSE_KIND_2D3D, 0, true>), grid, dim3(tile), lds_held, gs[1], inst, kp, sched, b.n_inst,
                       p, poses, mask);
    hipLaunchKernelGGL((k_sample<PURSE_KIND_3D3D, 0, true>), grid, dim3(tile), lds, gs[2], inst, kp, sched, b.n_inst,
                       p, poses, mask);
  } else {
    hipLaunchKernelGGL((k_sample<PURSE_KIND_2D3D, 0, false>), grid, dim3(tile), lds_held, gs[1], inst, kp, sched,
                       b.n_inst, p, poses, mask);
    hipLaunchKernelGGL((k_sample<PURSE_KIND_3D3D, 0, false>), grid, dim3(tile), lds, gs[2], inst, kp, sched,
                       b.n_inst, p, poses, mask);
  }
  if (aux) {
    for (int k = 0; k < 2; ++k) {
      hipError_t e = hipEventRecord(aux->join[k], aux->s[k]);
      if (e == hipSuccess) e = hipStreamWaitEvent(stream, aux->join[k], 0);
      if (e != hipSuccess) return e;  // the caller's stream is not joined to that group
    }
  }
  return hipSuccess;
}

}  // namespace purse
