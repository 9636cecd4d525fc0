// kernels.hip -- the plan evaluator's kernels other than the evaluation
// passes (those are in eval_pass.hip): packing and checking, bucketing,
// per-stage records, device memory, the u64 redo and the argmin; and the
// launchers the C ABI calls.  The data flow is described in device.h.
#include <mutex>

#include "launch.h"

namespace hetsim {

// ---------------------------------------------------------------- allocation-free workspace
// The workspace of sim_eval_plans_noalloc: one chunk's buffers (kNoAllocBytes,
// about 82 MiB) in a static device array.  Every GPU the library runs on holds
// its own copy until the process ends; host code reaches it only through the
// address hipGetSymbolAddress returns for the current device (the array's
// name in host code is a host-side stand-in, not a device address).
static __device__ __align__(256) uint8_t scratch[kNoAllocBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices];
}  // namespace

int noalloc_scratch(int device, void** ptr) {
  if (device < 0 || device >= kMaxDevices || !ptr) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(scratch_mu);
  if (!scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t r = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (r != hipSuccess) return (int)r;
    if (!p) return (int)hipErrorInvalidSymbol;
    scratch_ptr[device] = p;
  }
  *ptr = scratch_ptr[device];
  return 0;
}

// ---------------------------------------------------------------- bucketing
__global__ void k_fill32(uint32_t* p, uint32_t n, uint32_t v) {
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) p[j] = v;
}

// Inclusive sum over a block of 1024 threads (16 wavefronts).
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* part) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const uint32_t x = __shfl_up(v, o);
    v += lane >= o ? x : 0;
  }
  if (lane == 63) part[wave] = v;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < 16; ++w) before += w < wave ? part[w] : 0;
  __syncthreads();
  return v + before;
}

// Bucket offsets: cursor[b] the first entry of bucket b in order[], gstart and
// tstart each group's first entry and tile (grouped: shared layout, plans;
// otherwise pipelines), and the continuation lists' places and capacities in a
// buffer of `units` units, all of it: in proportion to (S + 2) / 48 of the tiles
// of S stages in the first list -- about twice what the first pass leaves on the
// random sweeps -- and a quarter of that in the second.  Lists of no more than
// that overflowed over links an eighth as fast, and a pipeline that finds its
// list full keeps its wavefront: 240000 plans of Llama-7B 608 us, 385 with the
// whole buffer; 2^20 plans of Mixtral at a 32nd 1507 and 1235.
// Four threads per group, eight buckets each.
__global__ void __launch_bounds__(1024) k_scan(const uint32_t* __restrict__ hist, uint32_t* __restrict__ cursor,
                                               uint32_t* __restrict__ gstart, uint32_t* __restrict__ tstart,
                                               uint32_t* __restrict__ cinfo, uint32_t grouped, uint32_t units) {
  constexpr uint32_t kPer = 8, kThreads = kBuckets / kPer;
  static_assert(kThreads <= 1024 && kBucketsM / kPer == 4, "four threads per group");
  __shared__ uint32_t part[16], stiles[kMaxStages];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, grp = tid >> 2;
  const bool has = tid < kThreads, head = has && (tid & 3) == 0;
  if (tid < (uint32_t)kMaxStages) stiles[tid] = 0;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j) {
    v[j] = has ? hist[tid * kPer + j] : 0;
    sum += v[j];
  }
  const uint32_t incl = block_scan(sum, part);
  uint32_t run = incl - sum;
  if (has) {
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      cursor[tid * kPer + j] = run;
      run += v[j];
    }
  }
  uint32_t n = sum + __shfl_xor(sum, 1);
  n += __shfl_xor(n, 2);   // the group's entries
  const uint32_t per = grouped ? plans_per_tile(kMaxClasses - grp % kMaxClasses) : 64u;
  const uint32_t tiles = head ? (n + per - 1) / per : 0;
  const uint32_t tincl = block_scan(tiles, part);
  if (head) {
    gstart[grp] = incl - sum;
    tstart[grp] = tincl - tiles;
    if (grp < kPlainGroups && tiles) atomicAdd(&stiles[grp / kMaxClasses % kMaxStages], tiles);
  }
  if (tid == kThreads - 1) {
    gstart[kGroups] = incl;
    tstart[kGroups] = tincl;
  }
  __syncthreads();
  if (tid < 64) {
    const bool on = tid < (uint32_t)kMaxStages;
    const uint32_t S = on ? kMaxStages - tid : 0;
    // the first list's tiles, in up to kContSubs equal parts
    uint32_t cap1 = on ? (stiles[tid] * (S + 2) + 47) / 48 : 0, cap2 = (cap1 + 3) / 4;
    auto total = [&](uint32_t x) {   // sum over the wavefront
#pragma unroll
      for (uint32_t o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
      return x;
    };
    auto before = [&](uint32_t x) {   // sum over the lower lanes
      uint32_t y = x;
#pragma unroll
      for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t z = __shfl_up(y, o);
        y += lane >= o ? z : 0;
      }
      return y - x;
    };
    const uint32_t all = total((cap1 + cap2) * S);
    if (all && all <= units) {
      // what is left of the buffer too, in the same proportions: over slow
      // links more of the shorter pipelines stay aperiodic.  (Rounded down, the
      // factor's own error included; a list needs no more than its tiles.)
      const double f = (double)units / (double)all * (1 - 0x1p-20);
      const uint32_t most = on ? stiles[tid] : 0;
      cap1 = (uint32_t)((double)cap1 * f) < most ? (uint32_t)((double)cap1 * f) : most;
      cap2 = (uint32_t)((double)cap2 * f) < most ? (uint32_t)((double)cap2 * f) : most;
    } else if (all) {
      // the first lists in proportion, so that the second ones fit in their quarter
      const uint64_t want = (uint64_t)total(cap1 * S) * 5;
      cap1 = (uint32_t)((uint64_t)cap1 * units * 4 / want);
      cap2 = cap1 / 4;
    }
    uint32_t subs = 1;
    while (subs < kContSubs && 4 * subs <= cap1) subs *= 2;
    const uint32_t part = cap1 / subs;
    const uint32_t b1 = before(cap1 * S), b2 = total(cap1 * S) + before(cap2 * S);
    if (on) {
      cinfo[tid] = b1;
      cinfo[16 + tid] = part;
      cinfo[64 + tid] = subs;
      cinfo[32 + tid] = b2;
      cinfo[48 + tid] = cap2;
    }
  }
}

// Place every plan (or pipeline) at its bucket's next free entry.  kPer entries
// per thread: 16, or 2 in smaller calls (a call of 29470 plans 128 us with 16,
// 121 with 2, 262144 plans 250 and 260; even at 60000).
constexpr uint32_t kScatterSmall = 1 << 16;
template <int kPer>
__global__ void __launch_bounds__(256) k_scatter(const uint16_t* __restrict__ keys, uint32_t n,
                                                 uint32_t* __restrict__ cursor, uint32_t* __restrict__ order) {
  __shared__ uint32_t lc[kBuckets];
  for (uint32_t j = threadIdx.x; j < kBuckets; j += blockDim.x) lc[j] = 0;
  __syncthreads();
  uint32_t key[kPer], rank[kPer];
  const uint32_t first = blockIdx.x * blockDim.x * kPer + threadIdx.x;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t i = first + j * blockDim.x;
    key[j] = i < n ? keys[i] : kNoKey;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) rank[j] = key[j] != kNoKey ? atomicAdd(&lc[key[j]], 1u) : 0;
  __syncthreads();
  if (kPer <= 2) {
    // few entries: the first one of each bucket takes the block's places
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (key[j] != kNoKey && rank[j] == 0) lc[key[j]] = atomicAdd(&cursor[key[j]], lc[key[j]]);
  } else {
    for (uint32_t j = threadIdx.x; j < kBuckets; j += blockDim.x)
      if (lc[j]) lc[j] = atomicAdd(&cursor[j], lc[j]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (key[j] != kNoKey) order[lc[key[j]] + rank[j]] = first + j * blockDim.x;
}

// ---------------------------------------------------------------- per-class layout: plan order
// k_plan_syncs walks each plan's layer segments, one plan per lane, so a
// wavefront lasts as long as its longest walk.  The valid plans are first
// counting-sorted by (classes, total stages over the classes), a close proxy
// for the number of segments (the union of the classes' cuts), into perm;
// pc as kPlanSortWords describes.  The key comes from the pipeline metadata
// k_prep wrote (S | G << 5 | ..., per class; zero past the classes and for
// invalid plans).
__device__ __forceinline__ uint32_t plan_key(uint4 m) {
  const uint32_t G = (m.x >> 5) & 7, st = (m.x & 31) + (m.y & 31) + (m.z & 31) + (m.w & 31);
  return (G - 1) * 64 + st - 1;
}
constexpr int kPlanPer = 8;   // plans per thread of the plan-order kernels
__global__ void __launch_bounds__(256) k_plan_hist(const uint4* __restrict__ meta, uint32_t n,
                                                   uint32_t* __restrict__ pc) {
  __shared__ uint32_t lh[kPlanBuckets];
  lh[threadIdx.x] = 0;
  __syncthreads();
  for (int j = 0; j < kPlanPer; ++j) {
    const uint32_t i = (blockIdx.x * kPlanPer + j) * 256 + threadIdx.x;
    if (i >= n) break;
    const uint4 m = meta[i];
    if (m.x) atomicAdd(&lh[plan_key(m)], 1u);
  }
  __syncthreads();
  if (lh[threadIdx.x]) atomicAdd(&pc[threadIdx.x], lh[threadIdx.x]);
}
__global__ void __launch_bounds__(256) k_plan_scatter(const uint4* __restrict__ meta, uint32_t n,
                                                      uint32_t* __restrict__ pc, uint32_t* __restrict__ perm) {
  static_assert(kPlanBuckets == 256, "one bucket per thread");
  __shared__ uint32_t base[kPlanBuckets], lc[kPlanBuckets];
  const uint32_t b = threadIdx.x;
  base[b] = pc[b];
  lc[b] = 0;
  __syncthreads();
  for (uint32_t off = 1; off < kPlanBuckets; off <<= 1) {   // inclusive scan of the counts
    const uint32_t x = b >= off ? base[b - off] : 0;
    __syncthreads();
    base[b] += x;
    __syncthreads();
  }
  if (blockIdx.x == 0 && b == kPlanBuckets - 1) pc[2 * kPlanBuckets] = base[b];   // valid plans
  const uint32_t excl = base[b] - pc[b];
  __syncthreads();
  base[b] = excl;
  uint32_t key[kPlanPer], rank[kPlanPer];
  for (int j = 0; j < kPlanPer; ++j) {
    const uint32_t i = (blockIdx.x * kPlanPer + j) * 256 + threadIdx.x;
    key[j] = kNoKey;
    if (i < n) {
      const uint4 m = meta[i];
      if (m.x) {
        key[j] = plan_key(m);
        rank[j] = atomicAdd(&lc[key[j]], 1u);
      }
    }
  }
  __syncthreads();
  if (lc[b]) lc[b] = atomicAdd(&pc[kPlanBuckets + b], lc[b]);
  __syncthreads();
  for (int j = 0; j < kPlanPer; ++j)
    if (key[j] != kNoKey) perm[base[key[j]] + lc[key[j]] + rank[j]] = (blockIdx.x * kPlanPer + j) * 256 + threadIdx.x;
}

// ---------------------------------------------------------------- continuation passes
// The first list: tiles dealt round-robin to the waves of the grid.  Bound by
// the serial chain of each lane's iterations (a wave of 16 stages takes 0.12 us
// for one of them alone); most of a tile's lanes end after a few, so a sixth of
// the lane slots is busy.  (The rates of 16 stages beside their state do not fit
// the 256 registers: 148 bytes per lane are in private memory.)  Redoing such pipelines from the start with the
// whole loop, as a list of slots instead of states would need, took 446 us per
// 2M-plan chunk of a random 512-device sweep where this takes 303 (126 with no
// other kernel beside it) and k_power 149 (54).
__global__ void __launch_bounds__(256, 2) k_cont(EvalBufs e) {
  __shared__ ContIndex<1, 64> ix;
  ix.fill(e);
  if (ix.entries <= kContFew) return;   // k_power's
  const uint32_t lane = threadIdx.x & 63u, waves = gridDim.x * (blockDim.x >> 6);
  uint32_t S, at, count, first;
  for (uint32_t q = blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       ix.find(e, q, S, at, count, first); q += waves) {
    if (at * 64 + lane >= count) continue;
    const double* base = e.cont + (size_t)first * (kContUnit / 8) + (size_t)at * (256 * S) + lane;
    switch (S) {
#define X(S_) \
  case S_: cont_one<S_>(e, base); break;
      X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#undef X
      default: break;
    }
  }
}

// The second list, and the first one when it is short: one pipeline per
// wavefront.  A steady iteration is a
// max-plus linear map of the state; its matrix is squared, and applied to the
// state at the set bits of the number of iterations left, so a pipeline takes
// log2(left) steps however its schedule behaves.  Every entry is the weight of
// a path the schedule contains, so exact like the times.  All stage counts run
// in a frame of 16 stages, the S stages of the pipeline last: the ones before
// them hold kNoPath (below every sum of real times), and the frame's shorter
// steady part (its first stages drain earlier) takes 16 - S iterations off the
// loop -- hence kPowerMin.  Measured alone: about 8 us for 1000 iterations of
// 16 stages, where one lane takes 120 us.
constexpr double kNoPath = -1e30;
constexpr uint32_t kPowerRow = 17;   // doubles per matrix row: the row groups hit different banks
// p: the entry; A, A2: two matrices and v: 64 doubles of the wavefront's LDS
__device__ __forceinline__ void power_one(const EvalBufs& e, const double* p, uint32_t S, double* A, double* A2,
                                          double* v) {
  constexpr int N = kMaxStages;
  const uint32_t lane = threadIdx.x & 63u, j = lane & 15u, g = lane >> 4;
  const uint2 ls = *(const uint2*)&p[64 * (3 * S - 1)];
  uint32_t left = ls.x - (N - S);
  if (lane == 0) count_skipped(e, (int)S, (int)left);
  // lanes 0-15 the state, 16-31 a, 32-47 d, 48-63 e of frame stage j
  {
    const int s = (int)j - (int)(N - S);
    const bool real = s >= 0 && !(g == 2 && s == (int)S - 1);
    v[lane] = real ? p[64 * ((g == 3 ? 3 * S : g * S) + s)] : g == 0 || g == 3 ? kNoPath : 0;
  }
  wave_sync_lds();
  Chain<N, double> h;
#pragma unroll
  for (int s = 0; s < N; ++s) {
    h.f[s] = s == (int)j ? 0 : kNoPath;
    h.a[s] = v[N + s];
    h.d[s] = v[2 * N + s];
    h.e[s] = v[3 * N + s];
  }
  double x = v[j];   // the state, one component per lane (four copies)
  // column j of the matrix, and the longest path from state component j to the end
  Chain<N, double> u = h;
  const double last = chain_end<N, double, false>(u, u.a, N);
  chain_iter<N, double, false>(h, h.a, 0, 0);
  if (g == 0) {
#pragma unroll
    for (int s = 0; s < N; ++s) A[s * kPowerRow + j] = h.f[s];
  }
  wave_sync_lds();
  while (true) {
    if (left & 1) {
      v[lane] = x;
      wave_sync_lds();
      double y = kNoPath;
#pragma unroll
      for (int k = 0; k < 4; ++k) y = vmax(y, A[j * kPowerRow + 4 * g + k] + v[4 * g + k]);
      y = vmax(y, __shfl_xor(y, 16));
      x = vmax(y, __shfl_xor(y, 32));
    }
    left >>= 1;
    if (!left) break;
    double c[4] = {kNoPath, kNoPath, kNoPath, kNoPath};
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const double w = A[k * kPowerRow + j];
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = vmax(c[i], A[(4 * g + i) * kPowerRow + k] + w);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) A2[(4 * g + i) * kPowerRow + j] = c[i];
    wave_sync_lds();
    double* t = A;
    A = A2;
    A2 = t;
  }
  double T = x + last;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) T = vmax(T, __shfl_xor(T, o));
  if (lane == 0) raise_time(e, ls.y, T);
  wave_sync_lds();
}

// (A second list of more than kPowerLong entries is taken by tiles of 64: the
// entries with little left to their end on their lanes, then the others.)
__global__ void __launch_bounds__(256) k_power(EvalBufs e) {
  __shared__ double mats[4][2][kMaxStages * kPowerRow];
  __shared__ double vec[4][4 * kMaxStages];
  __shared__ ContIndex<2, 1> ix;
  __shared__ ContIndex<2, 64> tiles;
  __shared__ ContIndex<1, 1> ix1;
  ix.fill(e);
  ix1.fill(e);
  const bool by_tile = ix.entries > kPowerLong;
  if (by_tile) tiles.fill(e);
  const uint32_t n1 = ix1.entries <= kContFew ? ix1.entries : 0;   // (the second list is empty then)
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t waves = gridDim.x * 4;
  uint32_t S, at, count, first;
  for (uint32_t q = blockIdx.x * 4 + wave;
       by_tile ? tiles.find(e, q, S, at, count, first)
               : q < n1 ? ix1.find(e, q, S, at, count, first) : ix.find(e, q - n1, S, at, count, first);
       q += waves) {
    const double* base = e.cont + (size_t)first * (kContUnit / 8);
    if (!by_tile) {
      power_one(e, base + (size_t)(at >> 6) * (256 * S) + (at & 63u), S, mats[wave][0], mats[wave][1], vec[wave]);
      continue;
    }
    base += (size_t)at * (256 * S);
    const uint32_t n = count - 64 * at < 64 ? count - 64 * at : 64;
    const uint32_t left = lane < n ? ((const uint2*)&base[64 * (3 * S - 1) + lane])->x : 0;
    const bool far = left * S >= kPowerCost * n;
    if (lane < n && !far) {
      switch (S) {
#define X(S_) \
  case S_: cont_rest<S_>(e, base + lane); break;
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#undef X
        default: break;
      }
    }
    for (uint64_t todo = __ballot(far); todo; todo &= todo - 1)
      power_one(e, base + __builtin_ctzll(todo), S, mats[wave][0], mats[wave][1], vec[wave]);
  }
}

// ---------------------------------------------------------------- argmin
__global__ void k_best_init(sim_best* b) {
  b->time_ps = kInvalid;
  b->index = INT64_MAX;
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    uint64_t w = __shfl_xor(v, o);
    v = w < v ? w : v;
  }
  return v;
}

__global__ void __launch_bounds__(256) k_min_time(const uint64_t* __restrict__ t, int64_t n, sim_best* b) {
  __shared__ uint64_t part[4];
  uint64_t v = kInvalid;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    v = t[i] < v ? t[i] : v;
  v = wave_min_u64(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) v = part[w] < v ? part[w] : v;
    if (v != kInvalid) atomicMin((unsigned long long*)&b->time_ps, (unsigned long long)v);
  }
}

__global__ void __launch_bounds__(256) k_min_index(const uint64_t* __restrict__ t, int64_t n, int64_t base,
                                                   sim_best* b) {
  __shared__ uint64_t part[4];
  const uint64_t best = b->time_ps;
  uint64_t v = kInvalid;
  if (best != kInvalid)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
      if (t[i] == best) { v = (uint64_t)i; break; }
  v = wave_min_u64(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) v = part[w] < v ? part[w] : v;
    if (v != kInvalid) atomicMin((long long*)&b->index, (long long)(base + (int64_t)v));
  }
}

__global__ void k_best_fix(sim_best* b) {
  if (b->time_ps == kInvalid) b->index = -1;
}

// The whole reduction by one block: up to kMinSmall times it takes 5-10 us,
// the four kernels above 17 us and more whatever the size.
constexpr int64_t kMinSmall = 1 << 16;
__global__ void __launch_bounds__(1024) k_min_small(const uint64_t* __restrict__ t, uint32_t n, int64_t base,
                                                    sim_best* b) {
  __shared__ uint64_t tpart[16], ipart[16];
  uint64_t bt = kInvalid, bi = kInvalid;
  for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 8 * 1024) {   // (a later index never beats an equal time)
    uint64_t v[8];
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) v[j] = i0 + 1024 * j < n ? t[i0 + 1024 * j] : kInvalid;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j)
      if (v[j] < bt) {
        bt = v[j];
        bi = i0 + 1024 * j;
      }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t t2 = __shfl_xor(bt, o), i2 = __shfl_xor(bi, o);
    if (t2 < bt || (t2 == bt && i2 < bi)) { bt = t2; bi = i2; }
  }
  if ((threadIdx.x & 63) == 0) { tpart[threadIdx.x >> 6] = bt; ipart[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w)
      if (tpart[w] < bt || (tpart[w] == bt && ipart[w] < bi)) { bt = tpart[w]; bi = ipart[w]; }
    b->time_ps = bt;
    b->index = bt == kInvalid ? -1 : base + (int64_t)bi;
  }
}

__global__ void __launch_bounds__(256) k_best_reduce(const sim_best* __restrict__ in, int64_t n, sim_best* out) {
  __shared__ uint64_t tpart[4], ipart[4];
  uint64_t bt = kInvalid, bi = kInvalid;
  for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
    const uint64_t tt = in[j].time_ps;
    const int64_t ii = in[j].index;
    if (tt == kInvalid || ii < 0) continue;
    if (tt < bt || (tt == bt && (uint64_t)ii < bi)) { bt = tt; bi = (uint64_t)ii; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    uint64_t t2 = __shfl_xor(bt, o), i2 = __shfl_xor(bi, o);
    if (t2 < bt || (t2 == bt && i2 < bi)) { bt = t2; bi = i2; }
  }
  if ((threadIdx.x & 63) == 0) { tpart[threadIdx.x >> 6] = bt; ipart[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w)
      if (tpart[w] < bt || (tpart[w] == bt && ipart[w] < bi)) { bt = tpart[w]; bi = ipart[w]; }
    out->time_ps = bt;
    out->index = bt == kInvalid ? -1 : (int64_t)bi;
  }
}


// ---------------------------------------------------------------- launchers
static int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

hipError_t launch_fill32(uint32_t* p, uint32_t n, uint32_t v, hipStream_t s) {
  k_fill32<<<blocks_for(n, 256) < 1024 ? blocks_for(n, 256) : 1024, 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}
hipError_t launch_prep(const Tab& t, const Tab* dtab, const sim_plans& p, int64_t n, uint64_t* out, PackedPlan* packed,
                       uint4* pcut, uint32_t* meta, uint32_t* hist, uint16_t* keys, hipStream_t s) {
  const uint32_t per = n < kPrepSmall ? 1 : kPrepPerThread;
  const int g = blocks_for(n, 256 * per);
  if (p.chdr) k_prep<true><<<g, 256, 0, s>>>(t, dtab, p, n, out, packed, pcut, meta, hist, keys, per);
  else k_prep<false><<<g, 256, 0, s>>>(t, dtab, p, n, out, packed, pcut, meta, hist, keys, per);
  return hipGetLastError();
}
hipError_t launch_memory(const Tab& t, const Tab* dtab, const sim_plans& p, int64_t n, uint64_t* out, hipStream_t s) {
  if (p.chdr) k_memory<true><<<blocks_for(n, 256), 256, 0, s>>>(t, dtab, p, n, out);
  else k_memory<false><<<blocks_for(n, 256), 256, 0, s>>>(t, dtab, p, n, out);
  return hipGetLastError();
}

// pc: the plan-order counters (zero on entry); perm: n words
hipError_t launch_plan_syncs(const Tab& t, const uint4* pcut, const uint32_t* meta,
                             int64_t n, double* hdp, uint32_t* pc, uint32_t* perm, hipStream_t s) {
  const int go = blocks_for(n, 256 * kPlanPer);
  k_plan_hist<<<go, 256, 0, s>>>((const uint4*)meta, (uint32_t)n, pc);
  k_plan_scatter<<<go, 256, 0, s>>>((const uint4*)meta, (uint32_t)n, pc, perm);
  const int g = blocks_for(n, 256);
  const size_t lds = (t.mode < 2 ? t.lds_bytes : 0) + 4 * (256 * t.K) * 4;   // and the lanes' counters
  if (t.mode == 0) k_plan_syncs<0><<<g, 256, lds, s>>>(t, pcut, perm, pc, n, hdp);
  else if (t.mode == 1) k_plan_syncs<1><<<g, 256, lds, s>>>(t, pcut, perm, pc, n, hdp);
  else k_plan_syncs<2><<<g, 256, lds, s>>>(t, pcut, perm, pc, n, hdp);
  return hipGetLastError();
}

hipError_t launch_stages(const Tab& t, const PackedPlan* packed, const uint4* pcut, const uint32_t* meta, int64_t n,
                         uint64_t* out_stage, hipStream_t s) {
  const int g = blocks_for(n * kMaxClasses * kMaxStages, 256);
  if (pcut) k_stages<true><<<g, 256, 0, s>>>(t, packed, pcut, meta, n, out_stage);
  else k_stages<false><<<g, 256, 0, s>>>(t, packed, pcut, meta, n, out_stage);
  return hipGetLastError();
}
hipError_t launch_scan(const Work& w, bool grouped, hipStream_t s) {
  k_scan<<<1, 1024, 0, s>>>(w.hist, w.cursor, w.gstart, w.tstart, w.cinfo, grouped ? 1u : 0u, w.cont_units);
  return hipGetLastError();
}
hipError_t launch_scatter(const Work& w, uint32_t n, hipStream_t s) {
  if (n < kScatterSmall) k_scatter<2><<<blocks_for(n, 512), 256, 0, s>>>(w.keys, n, w.cursor, w.order);
  else k_scatter<16><<<blocks_for(n, 4096), 256, 0, s>>>(w.keys, n, w.cursor, w.order);
  return hipGetLastError();
}
// ---------------------------------------------------------------- node-rate probe
// Peak rate of the recurrence's schedule-node operation on this device:
// end = max(end, input + hop) + duration, in fp64 (add, max, add), over
// kProbeChains independent chains per lane so that issue, not latency,
// bounds it.  The result feeds roofline reports; it is not part of any
// evaluation.
constexpr int kProbeChains = 8;
__global__ void __launch_bounds__(256) k_node_probe(double* __restrict__ sink, int iters, double c, double d) {
  double a[kProbeChains];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
#pragma unroll
  for (int j = 0; j < kProbeChains; ++j) a[j] = (double)(i + j);
  for (int k = 0; k < iters; ++k) {
#pragma unroll
    for (int j = 0; j < kProbeChains; ++j) a[j] = __builtin_fmax(a[j], a[(j + 1) % kProbeChains] + c) + d;
  }
  double t = 0;
#pragma unroll
  for (int j = 0; j < kProbeChains; ++j) t += a[j];
  sink[i] = t;
}

hipError_t launch_node_probe(double* sink, int blocks, int iters, hipStream_t s) {
  k_node_probe<<<blocks, 256, 0, s>>>(sink, iters, 3.0, 1.0);
  return hipGetLastError();
}

// ---------------------------------------------------------------- evaluation passes
// Blocks of each evaluation kernel that fit the device at once.
int eval_grids(Tab* t) {
  int cus = 0, dev = 0;
  hipError_t r = hipGetDevice(&dev);
  if (r == hipSuccess) r = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (r != hipSuccess) return (int)r;
  const size_t lds = t->mode < 2 ? t->lds_bytes : 0;
  int nb[6] = {0, 0, 0, 0, 0, 0};
  if (t->mode == 0) r = occupancy_v<0>(nb, lds, t->K);
  else if (t->mode == 1) r = occupancy_v<1>(nb, lds, t->K);
  else r = occupancy_v<2>(nb, lds, t->K);
  if (r == hipSuccess) {
    if (t->mode == 0) r = occupancy_all_v<0>(nb + 4, lds, t->K);
    else if (t->mode == 1) r = occupancy_all_v<1>(nb + 4, lds, t->K);
    else r = occupancy_all_v<2>(nb + 4, lds, t->K);
  }
  if (r == hipSuccess)
    r = hipOccupancyMaxActiveBlocksPerMultiprocessor(nb + 5, (const void*)k_cont, 256, 0);
  if (r != hipSuccess) return (int)r;
  for (int i = 0; i < 4; ++i) t->grid_eval[i] = (uint32_t)((nb[i] > 0 ? nb[i] : 1) * cus);
  t->grid_all = (uint32_t)((nb[4] > 0 ? nb[4] : 1) * cus);
  t->grid_cont = (uint32_t)((nb[5] > 0 ? nb[5] : 1) * cus);
  return 0;
}

// first pass of one stage-count group (g = 0..3) over a chunk (with two-level
// collectives the shared layout's plans are all k_all's)
hipError_t launch_group(const Tab& t, const EvalBufs& e, uint32_t max_tiles, int g, hipStream_t s) {
  const bool het = e.pcut != nullptr;
  if (!het && t.ccl_hier) return hipSuccess;
  if (t.mode == 0)
    return het ? launch_group_v<0, true>(t, e, max_tiles, g, s) : launch_group_v<0, false>(t, e, max_tiles, g, s);
  if (t.mode == 1)
    return het ? launch_group_v<1, true>(t, e, max_tiles, g, s) : launch_group_v<1, false>(t, e, max_tiles, g, s);
  return het ? launch_group_v<2, true>(t, e, max_tiles, g, s) : launch_group_v<2, false>(t, e, max_tiles, g, s);
}

// the plans k_eval does not take, and in a small call all of them (none with
// the per-class layout)
hipError_t launch_all(const Tab& t, const EvalBufs& e, uint32_t max_tiles, bool plain, hipStream_t s) {
  if (e.pcut) return hipSuccess;
  if (t.mode == 0) return launch_all_v<0>(t, e, max_tiles, plain || t.ccl_hier, s);
  if (t.mode == 1) return launch_all_v<1>(t, e, max_tiles, plain || t.ccl_hier, s);
  return launch_all_v<2>(t, e, max_tiles, plain || t.ccl_hier, s);
}

// after the first passes: the continuation lists, and the u64
// redo of the overflowed pipelines
hipError_t launch_rest(const Tab& t, const EvalBufs& e, uint32_t max_tiles, hipStream_t s) {
  const uint32_t need = (max_tiles + 3) / 4, grid = need < 1 ? 1 : need < t.grid_cont ? need : t.grid_cont;
  k_cont<<<grid, 256, 0, s>>>(e);
  k_power<<<grid, 256, 0, s>>>(e);
  if (e.pcut) k_redo_u64<true><<<32, 64, 0, s>>>(t, e);
  else k_redo_u64<false><<<32, 64, 0, s>>>(t, e);
  return hipGetLastError();
}

hipError_t launch_argmin(const uint64_t* t, int64_t n, int64_t base, sim_best* b, hipStream_t s) {
  if (n <= kMinSmall) {
    k_min_small<<<1, 1024, 0, s>>>(t, (uint32_t)n, base, b);
    return hipGetLastError();
  }
  int g = blocks_for(n, 256 * 8);
  g = g < 1 ? 1 : (g > 2048 ? 2048 : g);
  k_best_init<<<1, 1, 0, s>>>(b);
  k_min_time<<<g, 256, 0, s>>>(t, n, b);
  k_min_index<<<g, 256, 0, s>>>(t, n, base, b);
  k_best_fix<<<1, 1, 0, s>>>(b);
  return hipGetLastError();
}
hipError_t launch_best_reduce(const sim_best* in, int64_t n, sim_best* out, hipStream_t s) {
  k_best_reduce<<<1, 256, 0, s>>>(in, n, out);
  return hipGetLastError();
}

}  // namespace hetsim

