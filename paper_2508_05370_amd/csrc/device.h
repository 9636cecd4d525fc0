// device.h -- device code of the plan evaluator, shared by the library's
// translation units (kernels.hip and the evaluation-pass variants).
//
// Data flow of one chunk of plans (all in HBM):
//   k_prep     one plan per lane: decode and check the plan, pack it (with
//              the per-class layout into one 128-byte line), and count it per
//              bucket: in the shared layout the whole plan by (kind of
//              schedule or interleaved shape, stages, classes, longest
//              micro-batch count), with the per-class layout each pipeline
//              (one per replica class).
//   k_scan     one block: first entry of each bucket, entry and tile of each
//              group, places of the continuation lists.
//   k_scatter  places the plans (pipelines) in that order.
//   k_plan_hist, k_plan_scatter, k_plan_syncs (per-class layout only) the
//              syncs of every (class, stage), once per plan, plans sorted by
//              the length of their segment walks.
//   k_eval     one tile of a group per wavefront, a pipeline per lane, the G
//              pipelines of a plan on adjacent lanes; one launch per four
//              stage counts, 1F1B plans.  Setup: place the class on its device
//              pools, read stage compute from the layer prefix tables, find
//              each group's slowest link with range-max tables, and cost the
//              TP/EP/PP collectives and (shared over a plan's lanes) the DP
//              syncs.  Then the 1F1B recurrence, unrolled per stage count so
//              that all per-stage state stays in VGPRs.  Once a steady
//              iteration advances the whole state by one constant, the
//              remaining ones are added in one step (periodic shortcut); lanes
//              still aperiodic after a fixed budget leave for a continuation
//              list.  One store of the plan's time.
//   k_all      one launch for every other kind of the shared layout -- overlap,
//              zero-bubble and interleaved plans -- and in small calls for
//              all plans.
//   k_cont     the first continuation list, with full wavefronts of it.
//   k_power    what is still left, and a first list too short for k_cont, a
//              pipeline per wavefront, by powers of the iteration's max-plus
//              matrix (where very much is left, a pipeline per lane).
//   k_redo_u64 pipelines whose time reached 2^53 ps, again in u64.
//              Later passes raise a plan's time with atomic max.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stddef.h>

#include <type_traits>

#include "internal.h"

namespace hetsim {

constexpr uint64_t kInvalid = ~0ull;

// ---------------------------------------------------------------- helpers
// Stage and sync times are integers below 2^52 and messages below 2^48 bytes
// (sim_create checks both), carried in fp64: sums and products of them are
// exact, and fp64 runs at the full VALU rate, where a 64-bit integer product
// takes several quarter-rate instructions.
//
// ceil(bytes * bq / 2^16): the product with its rounding error, and one more
// where the rounded product is an integer and the error positive (a rounded
// product is never above an integer that the exact one does not exceed).
__device__ __forceinline__ double link_ps(double bytes, uint32_t bq) {
  const double y = (double)bq * 0x1p-16, h = bytes * y, l = __builtin_fma(bytes, y, -h), c = __builtin_ceil(h);
  return c + (l > c - h ? 1.0 : 0.0);
}

// ceil(x / p) for x / p < 2^50 and p >= 1, given rp = RN(1/p): the rounded
// product is within 1/2 + 2^-2 of x/p, so its remainder's sign decides.
__device__ __forceinline__ double ceil_div(double x, double p, double rp) {
  const double q = __builtin_rint(x * rp);
  return q + (__builtin_fma(-q, p, x) > 0 ? 1.0 : 0.0);
}

// Order of LDS accesses within a wavefront: its lanes' accesses complete in
// order; the fences keep the compiler from moving one lane's reads above other
// lanes' writes.
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// max over [lo, hi] of a range-max table with row length n
__device__ __forceinline__ uint32_t range_max(const uint32_t* __restrict__ tb, uint32_t n, uint32_t lo, uint32_t hi) {
  uint32_t j = 31u - __clz(hi - lo + 1);
  uint32_t a = tb[j * n + lo], b = tb[j * n + hi + 1 - (1u << j)];
  return a > b ? a : b;
}

// number of the nibbles selected by `sel` that equal k (in 32-bit halves: the
// shifts bring a nibble's bits down to its lowest one, which no neighbour
// reaches)
__device__ __forceinline__ uint32_t count_type(uint64_t types, uint32_t k, uint64_t sel) {
  const uint32_t ones = 0x11111111u, kk = ones * k;
  uint32_t lo = (uint32_t)types ^ kk, hi = (uint32_t)(types >> 32) ^ kk;
  lo |= lo >> 1;
  hi |= hi >> 1;
  lo |= lo >> 2;
  hi |= hi >> 2;
  return (uint32_t)__popc(~lo & (ones & (uint32_t)sel)) + (uint32_t)__popc(~hi & (ones & (uint32_t)(sel >> 32)));
}

// ceil(a / b) for a < 2^16 and 1 <= b < 2^16: the fp32 quotient's floor is
// within one of the true one, and the remainder says which.
__device__ __forceinline__ uint32_t ceil_div16(uint32_t a, uint32_t b) {
  const uint32_t q = (uint32_t)((float)a * __builtin_amdgcn_rcpf((float)b));
  const int r = (int)(a - q * b);
  return q + (r > 0 ? 1u : 0u) + (r > (int)b ? 1u : 0u);
}

// ceil(x / p) for x < 2^53 and p >= 1, given rp = RN(1/p): the rounded
// product is within 1 of x/p, so one correction each way makes it exact
// (two are applied).
__device__ __forceinline__ uint64_t div_up(uint64_t x, uint64_t p, double rp) {
  uint64_t q = (uint64_t)((double)x * rp);
  int64_t r = (int64_t)(x - q * p);
  const int64_t ps = (int64_t)p;
  if (r < 0) { --q; r += ps; }
  if (r < 0) { --q; r += ps; }
  if (r >= ps) { ++q; r -= ps; }
  if (r >= ps) { ++q; r -= ps; }
  return q + (r != 0);
}

// ceil(x / p) for any x: div_up below 2^53, the integer division above
// (never on the workloads here; a branch the wavefront skips when no lane
// takes it)
__device__ __forceinline__ uint64_t div_up_u64(uint64_t x, uint64_t p, double rp) {
  if (x < (1ull << 53)) return div_up(x, p, rp);
  return x / p + (x % p != 0);
}

// DP gradient sync of one stage over a ring of p members.  tree: an
// all-reduce takes the faster of the ring and a pipelined binary tree
// (reduce up, broadcast down: 2 ceil(log2 p) latencies, each member's
// gradient twice over the slowest link); ZeRO's reduce-scatter and
// all-gather stay rings.
__device__ __forceinline__ double ring_sync(uint32_t p, double rp, uint32_t zero, double grads, double params,
                                            double alpha, uint32_t bq, uint32_t tree) {
  const double g = ceil_div(grads, (double)p, rp), steps = (double)(p - 1);
  if (!zero) {
    double r = 2 * steps * alpha + link_ps(2 * steps * g, bq);
    if (tree && p > 1) {
      const double tt = (double)(2 * (32 - __builtin_clz(p - 1))) * alpha + link_ps(2 * grads, bq);
      r = tt < r ? tt : r;
    }
    return r;
  }
  return 2 * steps * alpha + link_ps(steps * g, bq) + link_ps(steps * ceil_div(params, (double)p, rp), bq);
}

// The same sync as latency steps and link time (the part that concurrent
// syncs over the same links share); the tree only when strictly faster.
__device__ __forceinline__ void ring_parts(uint32_t p, double rp, uint32_t zero, double grads, double params,
                                           double alpha, uint32_t bq, uint32_t tree, double& lat, double& bw) {
  const double g = ceil_div(grads, (double)p, rp), steps = (double)(p - 1);
  lat = 2 * steps * alpha;
  if (!zero) {
    bw = link_ps(2 * steps * g, bq);
    if (tree && p > 1) {
      const double tl = (double)(2 * (32 - __builtin_clz(p - 1))) * alpha, tb = link_ps(2 * grads, bq);
      if (tl + tb < lat + bw) {
        lat = tl;
        bw = tb;
      }
    }
  } else {
    bw = link_ps(steps * g, bq) + link_ps(steps * ceil_div(params, (double)p, rp), bq);
  }
}

// micro-batch counts: exact up to 20, then two buckets per power of two, and
// one for 768 and more.  A plain pipeline leaves its tile for a continuation
// list after its first budget of steady iterations, so larger counts need no
// finer sort for it.  The zero-bubble order's S - 1 iterations before that, and
// interleaved pipelines, which stay until they are periodic or at their end,
// are bounded by the bucket only.
__device__ __forceinline__ uint32_t m_bucket(uint32_t M) {
  if (M <= 20) return M - 1;
  const uint32_t e = 31u - __clz(M), j = 2 * (e - 4) + ((M >> (e - 1)) & 1);
  return 20 + (j < 11 ? j : 11);
}
__device__ __forceinline__ uint32_t bucket(uint32_t group, uint32_t M) {
  return group * kBucketsM + (kBucketsM - 1 - m_bucket(M));
}
__host__ __device__ constexpr uint32_t plain_group(uint32_t kind, uint32_t S, uint32_t G) {
  return (kind * kMaxStages + kMaxStages - S) * kMaxClasses + kMaxClasses - G;
}
// (S, v) shapes of interleaved pipelines: S v <= 16 virtual stages
#define HETSIM_IL_SHAPES(X) \
  X(2, 2) X(2, 3) X(2, 4) X(3, 2) X(3, 3) X(3, 4) X(4, 2) X(4, 3) X(4, 4) X(5, 2) X(5, 3) X(6, 2) X(7, 2) X(8, 2)
// their index in that list
__host__ __device__ constexpr uint32_t il_shape(uint32_t S, uint32_t v) {
  return S <= 4 ? (S - 2) * 3 + v - 2 : S == 5 ? 7 + v : S + 5;
}
static_assert(il_shape(4, 4) == 8 && il_shape(5, 2) == 9 && il_shape(5, 3) == 10 && il_shape(8, 2) == kIlShapes - 1,
              "interleaved shapes");
__host__ __device__ constexpr uint32_t il_group(uint32_t S, uint32_t v, uint32_t G) {
  return kPlainGroups + il_shape(S, v) * kMaxClasses + kMaxClasses - G;
}

// pipeline metadata word: S | G << 5 | M << 8 | (v - 1) << 24 (0 = no pipeline);
// bucket keys travel as u16, kNoKey = no plan (or pipeline)
constexpr uint32_t kNoKey = 0xffff;
static_assert(kBuckets < kNoKey, "bucket keys fit 16 bits");

// ---------------------------------------------------------------- plan validation
// Decoded plan fields used by every pipeline of the plan.
struct Plan {
  uint32_t tpl, epl, S, G, zero, mi, tp, ep, psum;
  uint32_t overlap;         // gradient sync overlapped with the last backward pass
  uint32_t v;               // model chunks per device: 1, or 2..4 for interleaved 1F1B
  uint32_t zb;              // zero-bubble order: backward split into input and weight gradients
  uint64_t cut_lo, cut_hi;  // cut bytes of stages 0-7 and 8-15, eight per word (virtual stages when v > 1)
  uint32_t reps[4], nmb[4];
  uint64_t tv[4];           // stage types, nibbles past S cleared
  // the class a pipeline evaluates: index, replicas, micro-batches, types.
  // Read here, from the packed plan in memory, so that no per-lane class
  // index ever selects among the fields above (that would put them in
  // private memory).
  uint32_t c, rc, nc;
  uint64_t tc;
  // per-class layout: byte c = log2 TP | (PP - 1) << 2 | micro-batch size
  // index << 6 of class c (0 with the shared layout, where tpl, S, mi and
  // the cuts above hold for every class; with the per-class layout they are
  // the pipeline's own class's)
  uint32_t chdr;
};

__device__ __forceinline__ uint32_t cls_tpl(uint32_t chdr, uint32_t c) { return (chdr >> (8 * c)) & 3; }
__device__ __forceinline__ uint32_t cls_S(uint32_t chdr, uint32_t c) { return ((chdr >> (8 * c + 2)) & 15) + 1; }
__device__ __forceinline__ uint32_t cls_mi(uint32_t chdr, uint32_t c) { return (chdr >> (8 * c + 6)) & 3; }
__device__ __forceinline__ uint64_t stage_sel(uint32_t S) { return S == 16 ? ~0ull : ((1ull << (4 * S)) - 1); }

// cut of stage s (a run-time index): mask arithmetic rather than a select,
// which the compiler may turn into an indexed load of the plan in private
// memory
__device__ __forceinline__ uint32_t cut_at(const Plan& p, uint32_t s) {
  const uint64_t m = 0ull - (uint64_t)(s >> 3);
  const uint64_t w = (p.cut_lo & ~m) | (p.cut_hi & m);
  return (uint32_t)(w >> (8 * (s & 7))) & 0xff;
}

__device__ __forceinline__ Plan unpack(const PackedPlan& q, uint32_t c = 0) {
  Plan p;
  p.c = c;
  const uint32_t cc = q.cls[c];
  p.rc = cc & 0xffff;
  p.nc = cc >> 16;
  p.tc = q.types[c];
  const uint32_t hdr = q.hdr;
  p.tpl = hdr & 3; p.epl = (hdr >> 2) & 3; p.S = ((hdr >> 4) & 15) + 1; p.G = ((hdr >> 8) & 3) + 1;
  p.zero = (hdr >> 10) & 1; p.mi = (hdr >> 11) & 3; p.tp = 1u << p.tpl; p.ep = 1u << p.epl; p.psum = q.psum;
  p.overlap = (hdr >> 13) & 1;
  p.v = ((hdr >> 14) & 3) + 1;
  p.zb = (hdr >> 16) & 1;
  p.chdr = q.pad0;
  const uint64_t* cw = reinterpret_cast<const uint64_t*>(q.cut);
  p.cut_lo = cw[0];
  p.cut_hi = cw[1];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    p.reps[j] = q.cls[j] & 0xffff;
    p.nmb[j] = q.cls[j] >> 16;
    p.tv[j] = q.types[j];
  }
  return p;
}

// A per-class-layout plan without its cut rows, seen as class c of the layout's
// header; tpl, tp, S, mi and the cuts are the pipeline's own class's.
__device__ __forceinline__ PackedPlan het_record(const uint4* line) {
  PackedPlan q;
  const uint4 a = line[0], b = line[1], x = line[2], y = line[3];
  q.hdr = a.x; q.psum = a.y; q.pad0 = a.z; q.pad1 = 0;
  uint32_t* z = reinterpret_cast<uint32_t*>(q.cut);
  z[0] = z[1] = z[2] = z[3] = 0;
  q.cls[0] = b.x; q.cls[1] = b.y; q.cls[2] = b.z; q.cls[3] = b.w;
  q.types[0] = (uint64_t)x.y << 32 | x.x; q.types[1] = (uint64_t)x.w << 32 | x.z;
  q.types[2] = (uint64_t)y.y << 32 | y.x; q.types[3] = (uint64_t)y.w << 32 | y.z;
  return q;
}

// The plan of pipeline `slot` (plan slot / 4, class slot % 4).  With the
// per-class layout the own class's TP degree, depth and cuts replace the
// header's.
template <bool kHet>
__device__ __forceinline__ Plan load_plan(const PackedPlan* packed, const uint4* pcut, uint32_t slot) {
  if constexpr (!kHet) return unpack(packed[slot >> 2], slot & 3);
  const uint4* line = pcut + (size_t)(slot >> 2) * kHetWords;
  const uint32_t c = slot & 3;
  Plan p = unpack(het_record(line), 0);
  // (the class's own fields from memory, so that no per-lane index selects among the fields above)
  const uint32_t cc = reinterpret_cast<const uint32_t*>(line + 1)[c];
  p.c = c;
  p.rc = cc & 0xffff;
  p.nc = cc >> 16;
  p.tc = reinterpret_cast<const uint64_t*>(line + 2)[c];
  p.tpl = cls_tpl(p.chdr, c);
  p.tp = 1u << p.tpl;
  p.S = cls_S(p.chdr, c);
  p.mi = cls_mi(p.chdr, c);
  const uint4 r = line[4 + c];
  p.cut_lo = (uint64_t)r.y << 32 | r.x;
  p.cut_hi = (uint64_t)r.w << 32 | r.z;
  return p;
}
// a per-class-layout plan's four cut rows
__device__ __forceinline__ const uint4* cut_rows(const uint4* pcut, uint32_t plan) {
  return pcut + (size_t)plan * kHetWords + 4;
}

// micro-batches per replica of the pipeline's class (its M)
__device__ __forceinline__ uint32_t class_mb(const Plan& p) { return ceil_div16(p.nc, p.rc); }

// plans per thread of k_prep: one in smaller calls, which would leave most of
// the chip without a block (29470 plans 133 us with four, 128 with one, 262144
// plans 242 and 250; even at 131072)
constexpr uint32_t kPrepPerThread = 4;
constexpr int64_t kPrepSmall = 1 << 17;

__device__ __forceinline__ void load_check_tab(CheckTab& ct, const Tab* dtab) {
  const uint32_t* src = (const uint32_t*)static_cast<const CheckTab*>(dtab);
  for (uint32_t j = threadIdx.x; j < sizeof(CheckTab) / 4; j += blockDim.x) ((uint32_t*)&ct)[j] = src[j];
}

// Plan i as loaded and checked by one lane: every rule of the plan layout
// except the memory check.  Per-class quantities are kept per class; with
// the shared layout every class has the header's.
struct Checked {
  bool ok;
  uint32_t hdr, psum, chdr;
  uint32_t tpl[4], S[4];   // per class (devices per replica)
  uint32_t v;              // model chunks per device (interleaved 1F1B when > 1)
  uint32_t cw[4][4];       // per class: cut bytes, four per word, 0 past the class's (virtual) stages
  uint32_t cls[4];         // 0 past the class count
  uint64_t tv[4];          // stage types, nibbles past the class's stages cleared; 0 past the class count
};

template <bool kHet>
__device__ __forceinline__ Checked check_plan(const Tab& t, const CheckTab& ct, const sim_plans& pl, int64_t i) {
  Checked r;
  const int64_t st = pl.stride;
  // every plane exists: load before any use
  const uint32_t hdr = pl.hdr[i];
  uint32_t cb[kHet ? 64 : 16];
#pragma unroll
  for (int s = 0; s < (kHet ? 64 : 16); ++s) cb[s] = kHet ? pl.ccut[s * st + i] : pl.cut[s * st + i];
  const uint32_t chdr = kHet ? pl.chdr[i] : 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    r.cls[c] = pl.cls[c * st + i];
    r.tv[c] = pl.types[c * st + i];
  }
  const uint32_t epl = (hdr >> 2) & 3, G = ((hdr >> 8) & 3) + 1, mi = (hdr >> 11) & 3;
  const uint32_t ep = 1u << epl, v = ((hdr >> 14) & 3) + 1;
  bool ok = (hdr >> 17) == 0 && mi < t.n_mbs && ((t.ep_ok >> epl) & 1);
  // the per-class layout leaves the header's TP and PP fields unused (0) and
  // has no overlap, interleaving or zero-bubble order
  if (kHet) ok = ok && (hdr & 0x1f8f3) == 0;   // and its micro-batch size: every class has its own
  // the zero-bubble order goes with neither overlap nor interleaving
  if (!kHet && ((hdr >> 16) & 1)) ok = ok && (hdr & 0xe000) == 0;
  // interleaving: no overlap, at least two devices, at most 16 virtual stages
  if (!kHet && v > 1) {
    const uint32_t S0 = ((hdr >> 4) & 15) + 1;
    ok = ok && ((hdr >> 13) & 1) == 0 && S0 >= 2 && S0 * v <= (uint32_t)kMaxStages;
  }
  uint32_t batch = 0, psum = 0;
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) {
    const uint32_t lay = kHet ? (chdr >> (8 * c)) & 0xff : (hdr & 3) | (((hdr >> 4) & 15) << 2);
    const uint32_t tpl = lay & 3, S = ((lay >> 2) & 15) + 1;
    r.tpl[c] = tpl;
    r.S[c] = S;
#pragma unroll
    for (int j = 0; j < 4; ++j) r.cw[c][j] = 0;
    if (c < G) {
      const uint32_t mic = kHet ? lay >> 6 : mi;   // the class's micro-batch size index
      if (kHet) ok = ok && mic < t.n_mbs;
      if (kHet || c == 0) {   // the shared layout's cuts are checked once
        ok = ok && ((t.tp_ok >> tpl) & 1);
        const uint32_t ncut = kHet ? S : S * v;
        uint32_t prev = 0;
#pragma unroll
        for (uint32_t s = 0; s < 16; ++s) {
          if (s < ncut) {
            const uint32_t v = cb[(kHet ? 16 * c : 0) + s];
            ok = ok && v > prev;
            prev = v;
            r.cw[c][s >> 2] |= v << (8 * (s & 3));
          }
        }
        ok = ok && prev == t.L;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) r.cw[c][j] = r.cw[0][j];
      }
      r.tv[c] &= stage_sel(S);
      const uint32_t reps = r.cls[c] & 0xffff, nmb = r.cls[c] >> 16;
      ok = ok && reps >= 1 && nmb >= reps && (reps & (ep - 1)) == 0;
      if (!kHet && v > 1 && ok) {   // interleaving: M a multiple of S and at least 2 S
        const uint32_t M = ceil_div16(nmb, reps);
        ok = M % S == 0 && M >= 2 * S;
      }
      batch += nmb * ct.mbs[mic];
      psum += reps;
    } else {
      r.cls[c] = 0;
      r.tv[c] = 0;
    }
  }
  ok = ok && batch == t.gbs;
  // every stage's type exists and holds whole TP groups in a node, and the
  // capacity of every pool under the packing (blocks aligned to their TP degree)
  uint32_t bad[4];   // stages of class c not yet found on a type that it may use
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) bad[c] = c < G ? r.S[c] : 0;
  for (uint32_t k = 0; k < t.K; ++k) {
    uint32_t need = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c) {
      const uint32_t nk = c < G ? count_type(r.tv[c], k, stage_sel(r.S[c])) : 0;
      if (nk) need = ((need + (1u << r.tpl[c]) - 1) >> r.tpl[c] << r.tpl[c]) + (((r.cls[c] & 0xffff) * nk) << r.tpl[c]);
      bad[c] -= (ct.type_ok[r.tpl[c]] >> k) & 1 ? nk : 0;
    }
    ok = ok && need <= t.cap[k];
  }
  ok = ok && (bad[0] | bad[1] | bad[2] | bad[3]) == 0;
  r.ok = ok;
  r.hdr = hdr;
  r.psum = psum;
  r.chdr = chdr;
  r.v = kHet ? 1 : v;
  return r;
}

// Peak bytes of one device of a stage of ns layers at TP 2^tpl apart from
// its stored activations: weights and gradients of the parameters its TP
// rank holds, and the optimizer state, split with ZeRO over the DP group
// (all replicas for the non-expert parameters, replicas / EP for the
// experts).
__device__ __forceinline__ uint64_t state_bytes(const Tab& t, const CheckTab& ct, uint32_t tpl, uint32_t epl,
                                                uint32_t zero,
                                                uint32_t psum, bool first, bool last, uint32_t ns, double rp,
                                                double rpx) {
  uint64_t pd = (uint64_t)ns * ct.par_layer[tpl];
  if (first) pd += ct.par_embed[tpl];
  if (last) pd += ct.par_head[tpl];
  const uint64_t pe = (uint64_t)ns * ct.par_expert[tpl][epl];
  uint64_t od = t.opt_bytes * pd, oe = t.opt_bytes * pe;
  if (zero) {
    od = div_up_u64(od, psum, rp);
    if (oe) oe = div_up_u64(oe, psum >> epl, rpx);
  }
  return (t.param_bytes + t.grad_bytes) * (pd + pe) + od + oe;
}

// cut byte of stage s (run-time index) of class c (a compile-time index) of a checked plan
__device__ __forceinline__ uint32_t checked_cut(const Checked& r, uint32_t c, uint32_t s) {
  const uint64_t lo = (uint64_t)r.cw[c][0] | ((uint64_t)r.cw[c][1] << 32);
  const uint64_t hi = (uint64_t)r.cw[c][2] | ((uint64_t)r.cw[c][3] << 32);
  const uint64_t m = 0ull - (uint64_t)(s >> 3);
  return (uint32_t)(((lo & ~m) | (hi & m)) >> (8 * (s & 7))) & 0xff;
}

// State bytes of stage s (ns layers) of class c of a checked plan.
__device__ __forceinline__ uint64_t class_state_bytes(const Tab& t, const CheckTab& ct, const Checked& r, uint32_t c,
                                                      uint32_t s,
                                                      uint32_t ns) {
  const uint32_t epl = (r.hdr >> 2) & 3, zero = (r.hdr >> 10) & 1;
  // (the reciprocals are the same for every stage of the plan)
  return state_bytes(t, ct, r.tpl[c], epl, zero, r.psum, s == 0, s == r.S[c] - 1, ns, 1.0 / (double)r.psum,
                     1.0 / (double)(r.psum >> epl));
}

// Peak bytes of the devices of stage s (ns layers) of class c: its state plus
// the activations of the min(PP - s, M) micro-batches 1F1B keeps in flight
// there (min(PP, M) on every stage under the zero-bubble order, where a
// micro-batch's activations stay until its weight-gradient pass).
__device__ __forceinline__ uint64_t class_stage_bytes(const CheckTab& ct, const Checked& r, uint32_t c, uint32_t s,
                                                      uint32_t ns, uint64_t state) {
  // the micro-batch size: the header's (shared layout) or the class's (per-class layout, header field 0)
  const uint32_t mi = ((r.hdr >> 11) & 3) | cls_mi(r.chdr, c), S = r.S[c];
  const uint32_t reps = r.cls[c] & 0xffff, M = ceil_div16(r.cls[c] >> 16, reps);
  const uint32_t held = ((r.hdr >> 16) & 1) ? S : S - s;
  const uint32_t fly = held < M ? held : M;
  return state + (uint64_t)ns * fly * ct.act_layer[r.tpl[c]][mi];
}

// Interleaved 1F1B: device s holds virtual stages j S + s (j < v), so its
// state covers the layers of all of them (ns; the embedding on device 0, the
// head on device S - 1), and its activations are those of its
// 2 (S - 1 - s) + (v - 1) S warm-up passes plus one (at most M v passes),
// each counted at the device's largest chunk (nmax layers).
__device__ __forceinline__ void il_device_layers(const Checked& r, uint32_t s, uint32_t& ns, uint32_t& nmax) {
  const uint32_t S = r.S[0];
  ns = 0;
  nmax = 0;
  for (uint32_t j = 0; j < r.v; ++j) {
    const uint32_t vs = j * S + s;
    const uint32_t n = checked_cut(r, 0, vs) - (vs ? checked_cut(r, 0, vs - 1) : 0);
    ns += n;
    nmax = n > nmax ? n : nmax;
  }
}
__device__ __forceinline__ uint64_t il_stage_bytes(const CheckTab& ct, const Checked& r, uint32_t c, uint32_t s,
                                                   uint32_t nmax, uint64_t state) {
  const uint32_t mi = (r.hdr >> 11) & 3, S = r.S[c], v = r.v;
  const uint32_t reps = r.cls[c] & 0xffff, M = ceil_div16(r.cls[c] >> 16, reps);
  const uint32_t w = 2 * (S - 1 - s) + (v - 1) * S + 1;
  const uint32_t fly = w < M * v ? w : M * v;
  return state + (uint64_t)nmax * fly * ct.act_layer[r.tpl[c]][mi];
}

// Every device of a checked plan fits its type's memory.  With one layout
// for all classes a stage's state is the same for every class: computed once.
template <bool kHet>
__device__ __forceinline__ bool fits_memory(const Tab& t, const CheckTab& ct, const Checked& r) {
  const uint32_t G = ((r.hdr >> 8) & 3) + 1;
  bool ok = true;
  if (!kHet && r.v > 1) {
    for (uint32_t s = 0; s < r.S[0]; ++s) {
      uint32_t ns, nmax;
      il_device_layers(r, s, ns, nmax);
      const uint64_t state = class_state_bytes(t, ct, r, 0, s, ns);
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c)
        if (c < G)
          ok = ok && il_stage_bytes(ct, r, c, s, nmax, state) <= ct.mem_cap[(uint32_t)(r.tv[c] >> (4 * s)) & 15];
    }
    return ok;
  }
  if (!kHet) {
    uint32_t prev = 0;
    for (uint32_t s = 0; s < r.S[0]; ++s) {
      const uint32_t cut = checked_cut(r, 0, s), ns = cut - prev;
      prev = cut;
      const uint64_t state = class_state_bytes(t, ct, r, 0, s, ns);
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c)
        if (c < G)
          ok = ok && class_stage_bytes(ct, r, c, s, ns, state) <= ct.mem_cap[(uint32_t)(r.tv[c] >> (4 * s)) & 15];
    }
    return ok;
  }
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) {
    if (c >= G) continue;
    uint32_t prev = 0;
    for (uint32_t s = 0; s < r.S[c]; ++s) {
      const uint32_t cut = checked_cut(r, c, s), ns = cut - prev;
      prev = cut;
      const uint64_t v = class_stage_bytes(ct, r, c, s, ns, class_state_bytes(t, ct, r, c, s, ns));
      ok = ok && v <= ct.mem_cap[(uint32_t)(r.tv[c] >> (4 * s)) & 15];
    }
  }
  return ok;
}

// Decode and check plan i (every rule of the plan layout); on success pack it
// (with the per-class layout into its line at pcut).  Writes out[i] (0 = valid,
// to be raised by the pipelines; else invalid), and when given the per-pipeline
// metadata S | G << 5 | M << 8 | (v - 1) << 24 with the class's own S (0 = no
// pipeline) and the bucket keys, counted in hist.  Bound by instruction issue
// and the 150-odd bytes per plan: 2M plans of a sweep, beside the evaluation
// kernels, 227 us with the rules checked class by class over the packed types,
// 132 in one pass over them (106 with no other kernel beside it).
template <bool kHet>
__global__ void __launch_bounds__(256) k_prep(Tab t, const Tab* __restrict__ dtab, sim_plans pl, int64_t n,
                                              uint64_t* __restrict__ out,
                                              PackedPlan* __restrict__ packed, uint4* __restrict__ pcut,
                                              uint32_t* __restrict__ meta, uint32_t* __restrict__ hist,
                                              uint16_t* __restrict__ keys, uint32_t per) {
  __shared__ uint32_t lh[kBuckets];
  __shared__ CheckTab ct;
  load_check_tab(ct, dtab);
  if (hist)
    for (uint32_t j = threadIdx.x; j < kBuckets; j += blockDim.x) lh[j] = 0;
  __syncthreads();
  for (uint32_t rep = 0; rep < per; ++rep) {
    const int64_t i = ((int64_t)blockIdx.x * per + rep) * blockDim.x + threadIdx.x;
    if (i >= n) break;
    const Checked r = check_plan<kHet>(t, ct, pl, i);
    const bool ok = r.ok && (!t.mem_check || fits_memory<kHet>(t, ct, r));
    const uint32_t G = ((r.hdr >> 8) & 3) + 1;
    if (out) out[i] = ok ? 0 : kInvalid;
    if (ok && !kHet) {
      PackedPlan q;
      q.hdr = r.hdr; q.psum = r.psum; q.pad0 = 0; q.pad1 = 0;
      uint32_t* qc = reinterpret_cast<uint32_t*>(q.cut);
#pragma unroll
      for (int j = 0; j < 4; ++j) { qc[j] = r.cw[0][j]; q.cls[j] = r.cls[j]; q.types[j] = r.tv[j]; }
      packed[i] = q;
    }
    if (ok && kHet) {
      uint4* q = pcut + i * kHetWords;
      auto lo = [](uint64_t x) { return (uint32_t)x; };
      auto hi = [](uint64_t x) { return (uint32_t)(x >> 32); };
      q[0] = make_uint4(r.hdr, r.psum, r.chdr, 0);
      q[1] = make_uint4(r.cls[0], r.cls[1], r.cls[2], r.cls[3]);
      q[2] = make_uint4(lo(r.tv[0]), hi(r.tv[0]), lo(r.tv[1]), hi(r.tv[1]));
      q[3] = make_uint4(lo(r.tv[2]), hi(r.tv[2]), lo(r.tv[3]), hi(r.tv[3]));
#pragma unroll
      for (int c = 0; c < 4; ++c) q[4 + c] = make_uint4(r.cw[c][0], r.cw[c][1], r.cw[c][2], r.cw[c][3]);
    }
    uint32_t m[4], Mmax = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c) {
      m[c] = 0;
      if (ok && c < G) {
        const uint32_t reps = r.cls[c] & 0xffff, M = ceil_div16(r.cls[c] >> 16, reps);
        m[c] = r.S[c] | (G << 5) | (M << 8) | ((r.v - 1) << 24);
        Mmax = M > Mmax ? M : Mmax;
      }
    }
    // bucket keys: of the plan, ranked by its longest class, or with the
    // per-class layout of each pipeline
    if (keys && !kHet) {
      uint32_t key = kNoKey;
      if (ok) {
        const uint32_t S = r.S[0], kind = (r.hdr >> 16) & 1 ? 2 : (r.hdr >> 13) & 1;
        // (interleaved: Mmax is a multiple of S below 2^16, so its product with
        // the approximate reciprocal rounds to the quotient)
        key = r.v > 1 ? bucket(il_group(S, r.v, G), (uint32_t)((float)Mmax * __builtin_amdgcn_rcpf((float)S) + 0.5f))
                      : bucket(plain_group(kind, S, G), Mmax);
        if (hist) atomicAdd(&lh[key], 1u);
      }
      keys[i] = (uint16_t)key;
    }
    if (keys && kHet) {
      uint32_t key[4];
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c) {
        key[c] = m[c] ? bucket(plain_group(0, r.S[c], G), m[c] >> 8 & 0xffff) : kNoKey;
        if (hist && m[c]) atomicAdd(&lh[key[c]], 1u);
      }
      reinterpret_cast<uint2*>(keys)[i] = make_uint2(key[0] | key[1] << 16, key[2] | key[3] << 16);
    }
    // one 16-byte store per plan (the workspace is 256-byte aligned; a
    // caller's class array may be aligned to 4 bytes only)
    if (meta) {
      if (((uintptr_t)meta & 15) == 0) {
        reinterpret_cast<uint4*>(meta)[i] = make_uint4(m[0], m[1], m[2], m[3]);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) meta[i * 4 + c] = m[c];
      }
    }
  }
  if (hist) {
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < kBuckets; j += blockDim.x)
      if (lh[j]) atomicAdd(&hist[j], lh[j]);
  }
}

// Peak memory of every (class, stage) device, one plan per lane.  A lane's 512
// bytes of results are four rows of 128: each class's go through LDS, so that
// the wavefront stores whole rows (one lane's stores, 512 bytes from its
// neighbour's, would be a partial line each).  250000 plans, 145 MB: 204 us with
// one lane's stores, 64 by rows.
constexpr uint32_t kMemRow = kMaxStages + 1;   // words per row in LDS
template <bool kHet>
__global__ void __launch_bounds__(256) k_memory(Tab t, const Tab* __restrict__ dtab, sim_plans pl, int64_t n,
                                                uint64_t* __restrict__ out) {
  __shared__ CheckTab ct;
  __shared__ uint64_t rows[4][64 * kMemRow];
  load_check_tab(ct, dtab);
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + 64 * wave;
  if (first >= n) return;
  const int64_t i = first + lane < n ? first + lane : n - 1;   // (lanes past the end repeat the last plan)
  const uint32_t live = n - first < 64 ? (uint32_t)(n - first) : 64u;
  const Checked r = check_plan<kHet>(t, ct, pl, i);
  const uint32_t G = ((r.hdr >> 8) & 3) + 1;
  uint64_t* const row = &rows[wave][lane * kMemRow];
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) {
    uint32_t prev = 0;
    for (uint32_t s = 0; s < (uint32_t)kMaxStages; ++s) {
      uint64_t v = kInvalid;
      if (r.ok) {
        v = 0;
        if (c < G && s < r.S[c] && r.v > 1) {
          uint32_t ns, nmax;
          il_device_layers(r, s, ns, nmax);
          v = il_stage_bytes(ct, r, c, s, nmax, class_state_bytes(t, ct, r, c, s, ns));
        } else if (c < G && s < r.S[c]) {
          const uint32_t cut = checked_cut(r, c, s);
          v = class_stage_bytes(ct, r, c, s, cut - prev, class_state_bytes(t, ct, r, c, s, cut - prev));
          prev = cut;
        }
      }
      row[s] = v;
    }
    wave_sync_lds();
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q) {   // four rows at a time
      const uint32_t a = 4 * q + (lane >> 4), s = lane & 15u;
      if (a < live) out[(first + a) * (kMaxClasses * kMaxStages) + c * kMaxStages + s] = rows[wave][a * kMemRow + s];
    }
    wave_sync_lds();
  }
}

// ---------------------------------------------------------------- table image
// Reads of the setup tables (the image described with Tab).  kMode 0: the
// whole image is in LDS; 1: all but the device range-max rows; 2: all in
// device memory.
template <int kMode>
struct Hot {
  const uint8_t* b;       // image base for every section but the device rows
  const uint32_t* rmn;    // device range-max rows
  const Tab& t;
  __device__ __forceinline__ Hot(const Tab& tab, const uint4* lds)
      : b(kMode < 2 ? (const uint8_t*)lds : (const uint8_t*)tab.img),
        rmn((const uint32_t*)((kMode == 0 ? (const uint8_t*)lds : (const uint8_t*)tab.img) + tab.o_rmn)),
        t(tab) {}
  __device__ __forceinline__ TypeInfo type(uint32_t k) const {
    const uint4* q = (const uint4*)(b + k * sizeof(TypeInfo));
    const uint4 x = q[0], y = q[1];
    TypeInfo r;
    r.node_off = x.x; r.dev_off = x.y; r.dpl = x.z; r.bq_pcie = x.w;
    r.a_intra = __hiloint2double((int)y.y, (int)y.x);
    r.a_side = __hiloint2double((int)y.w, (int)y.z);
    return r;
  }
  __device__ __forceinline__ const SizeInfo& size() const { return *(const SizeInfo*)(b + t.o_size); }
  __device__ __forceinline__ const SpeedInfo& speed(uint32_t k) const { return ((const SpeedInfo*)(b + t.o_speed))[k]; }
  __device__ __forceinline__ double side_alpha(uint32_t k) const {
    return *(const double*)(b + k * sizeof(TypeInfo) + offsetof(TypeInfo, a_side));
  }
  __device__ __forceinline__ double intra_alpha(uint32_t k) const {
    return *(const double*)(b + k * sizeof(TypeInfo) + offsetof(TypeInfo, a_intra));
  }
  // {forward, backward} prefix entry
  __device__ __forceinline__ double2 pfb(uint32_t i) const { return ((const double2*)(b + t.o_pfb))[i]; }
  __device__ __forceinline__ double2 emb(uint32_t i) const { return ((const double2*)(b + t.o_emb))[i]; }
  __device__ __forceinline__ double2 head(uint32_t i) const { return ((const double2*)(b + t.o_head))[i]; }
  __device__ __forceinline__ double pa(uint32_t i) const { return ((const double*)(b + t.o_pa))[i]; }
  __device__ __forceinline__ const uint32_t* rmi() const { return (const uint32_t*)(b + t.o_rmi); }
};

// Copy the LDS part of the image (every thread of the block takes part).
template <int kMode>
__device__ __forceinline__ void fill_lds(const Tab& t, uint4* lds) {
  if (kMode < 2) {
    const uint32_t n = t.lds_bytes >> 4;
    const uint4* img = (const uint4*)t.img;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) lds[i] = img[i];
    __syncthreads();
  }
}

// ---------------------------------------------------------------- per-pipeline setup
// Stage quantities of class c of a valid plan: rec[s] = {forward and backward
// time of one micro-batch on stage s, hop s -> s+1, DP sync of stage s}.
//
// Placement: every pool is filled in (class, stage) order, reps*tp devices per
// (class, stage), so a (class, stage) of type k starts after the devices of
// type k used by earlier classes and by earlier stages of its own class.
// Devices of type k taken before (class c2, stage s) for a class index c2
// that is a compile-time constant once the callers' class loops unroll.
__device__ __forceinline__ uint32_t placed_before(const Plan& p, uint32_t c2, uint32_t s, uint32_t k) {
  const uint64_t sel = p.S == 16 ? ~0ull : ((1ull << (4 * p.S)) - 1);
  uint32_t below = 0;
#pragma unroll
  for (uint32_t c3 = 0; c3 < 4; ++c3)
    if (c3 < c2) below += p.reps[c3] * count_type(p.tv[c3], k, sel);
  return below + p.reps[c2] * count_type(p.tv[c2], k, (1ull << (4 * s)) - 1);
}

// The same for the pipeline's own class (a per-lane index).
__device__ __forceinline__ uint32_t placed_before_own(const Plan& p, uint32_t s, uint32_t k) {
  const uint64_t sel = p.S == 16 ? ~0ull : ((1ull << (4 * p.S)) - 1);
  uint32_t below = 0;
#pragma unroll
  for (uint32_t c3 = 0; c3 < 4; ++c3)
    if (c3 < p.c) below += p.reps[c3] * count_type(p.tv[c3], k, sel);
  return below + p.rc * count_type(p.tc, k, (1ull << (4 * s)) - 1);
}

// Devices of type k taken before (class c2, stage s), and the same for the
// pipeline's own class, under either layout.  With the per-class layout each
// class takes reps * its own TP degree devices per stage, and its blocks
// start at a multiple of that degree (so no TP group spans two nodes): a
// class's blocks in a pool are contiguous after its first one is aligned.
__device__ __forceinline__ uint32_t align_up(uint32_t x, uint32_t tpl) { return ((x + (1u << tpl) - 1) >> tpl) << tpl; }

template <bool kHet>
__device__ __forceinline__ uint32_t dev_before(const Plan& p, uint32_t c2, uint32_t s, uint32_t k) {
  if (!kHet) return placed_before(p, c2, s, k) * p.tp;
  uint32_t ptr = 0;
#pragma unroll
  for (uint32_t c3 = 0; c3 < 4; ++c3) {
    if (c3 < c2) {
      const uint32_t tl = cls_tpl(p.chdr, c3), nk = count_type(p.tv[c3], k, stage_sel(cls_S(p.chdr, c3)));
      if (nk) ptr = align_up(ptr, tl) + ((p.reps[c3] * nk) << tl);
    }
  }
  const uint32_t tl = cls_tpl(p.chdr, c2);
  return align_up(ptr, tl) + ((p.reps[c2] * count_type(p.tv[c2], k, (1ull << (4 * s)) - 1)) << tl);
}
template <bool kHet>
__device__ __forceinline__ uint32_t dev_before_own(const Plan& p, uint32_t s, uint32_t k) {
  if (!kHet) return placed_before_own(p, s, k) * p.tp;
  uint32_t ptr = 0;
#pragma unroll
  for (uint32_t c3 = 0; c3 < 4; ++c3) {
    if (c3 < p.c) {
      const uint32_t tl = cls_tpl(p.chdr, c3), nk = count_type(p.tv[c3], k, stage_sel(cls_S(p.chdr, c3)));
      if (nk) ptr = align_up(ptr, tl) + ((p.reps[c3] * nk) << tl);
    }
  }
  return align_up(ptr, p.tpl) + ((p.rc * count_type(p.tc, k, (1ull << (4 * s)) - 1)) << p.tpl);
}

// Parameters one TP rank holds of a layer (and of its experts), the embedding
// and the head, in fp64.
struct Params {
  double layer, expert, embed, head;
  __device__ __forceinline__ Params(const SizeInfo& z, uint32_t tpl, uint32_t epl)
      : layer(z.layer[tpl]), expert(z.expert[tpl][epl]), embed(z.embed[tpl]), head(z.head[tpl]) {}
  __device__ __forceinline__ double stage(uint32_t ns, bool first, bool last) const {
    return (double)ns * layer + (first ? embed : 0.0) + (last ? head : 0.0);
  }
};

// DP sync of a stage over every replica of every class: one ring across all
// replicas on the slowest NIC of the participating devices, or inside one
// node when every replica of the stage sits in the same node; MoE models add
// the expert ring over the EP-sized groups.  The same for every class of the
// plan.  Its link is put together from each class's share of the stage: the
// slowest NIC or PCIe rate of the class's devices, and type << 24 | the node
// that holds them all (kNoNode: several).
constexpr uint32_t kNoNode = 0xffffff;
struct DpLink {
  double alpha;
  uint32_t bq;
};

// With two-level collectives enabled, hs is the group's shape for them:
// usable when every class's devices of the stage fill whole nodes with the
// same number g > 1 of TP groups per node, over N > 1 nodes in all; a_in
// and bq_in are the worst node latency and fabric rate over them.
struct HierShape {
  bool ok;
  uint32_t g, N, bq_in;
  double a_in;
};

// The link of stage s found from the plan alone.
template <int kMode>
__device__ __forceinline__ DpLink stage_link(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s,
                                             HierShape& hs) {
  const uint32_t G = p.G, tp = p.tp;
  bool same = true;
  uint32_t k0 = 0, nmin = 0xffffffffu, nmax = 0, bq_dp = 0;
  double a_dp = 0;
  hs.ok = t.ccl_hier != 0;
  hs.g = 0; hs.N = 0; hs.bq_in = 0; hs.a_in = 0;
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2) {
    if (c2 >= G) continue;
    const uint32_t k2 = (uint32_t)(p.tv[c2] >> (4 * s)) & 15;
    const TypeInfo t2 = h.type(k2);
    const uint32_t b2 = placed_before(p, c2, s, k2) * tp, n2 = p.reps[c2] * tp, d2 = t2.dpl;
    const uint32_t l2 = t2.node_off + (b2 >> d2), h2 = t2.node_off + ((b2 + n2 - 1) >> d2);
    const uint32_t dl2 = t2.dev_off + b2;
    const uint32_t nic2 = range_max(h.rmn, t.D, dl2, dl2 + n2 - 1);
    if (c2 == 0) k0 = k2; else same = same && k2 == k0;
    nmin = l2 < nmin ? l2 : nmin;
    nmax = h2 > nmax ? h2 : nmax;
    const uint32_t bx = nic2 > t2.bq_pcie ? nic2 : t2.bq_pcie;
    bq_dp = bx > bq_dp ? bx : bq_dp;
    a_dp = 2 * t2.a_side > a_dp ? 2 * t2.a_side : a_dp;
    if (t.ccl_hier) {
      const uint32_t dm = (1u << d2) - 1, gm = (1u << d2) >> p.tpl;
      hs.ok = hs.ok && (b2 & dm) == 0 && (n2 & dm) == 0 && (c2 == 0 || gm == hs.g);
      hs.g = gm;
      hs.N += n2 >> d2;
      hs.a_in = t2.a_intra > hs.a_in ? t2.a_intra : hs.a_in;
      const uint32_t bi = range_max(h.rmi(), t.N, l2, h2);
      hs.bq_in = bi > hs.bq_in ? bi : hs.bq_in;
    }
  }
  hs.ok = hs.ok && hs.g > 1 && hs.N > 1;
  const bool intra = same && nmin == nmax;
  return {intra ? h.intra_alpha(k0) : a_dp, intra ? h.rmi()[nmin] : bq_dp};
}

// The same link from the classes' shares that the plan's lanes left in LDS
// (link: class 0's, the others after it).
template <int kMode>
__device__ __forceinline__ DpLink exchanged_link(const Hot<kMode>& h, uint32_t G, const uint2* link) {
  uint32_t w0 = 0, bq_dp = 0;
  bool same = true;
  double a = 0;
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2) {
    if (c2 >= G) continue;
    const uint2 l = link[c2];
    if (c2 == 0) w0 = l.y; else same = same && l.y == w0;
    bq_dp = l.x > bq_dp ? l.x : bq_dp;
    const double a2 = h.side_alpha(l.y >> 24);
    a = a2 > a ? a2 : a;
  }
  const bool intra = same && (w0 & kNoNode) != kNoNode;
  return {intra ? h.intra_alpha(w0 >> 24) : 2 * a, intra ? h.rmi()[w0 & kNoNode] : bq_dp};
}

// A dense all-reduce of `grads` bytes per member over the group, with the
// two-level algorithm when the shape allows it and it is faster: the
// node-local ring over the whole gradient (g members), then the ring
// across the N nodes over a 1/g shard (g is a power of two).
__device__ __forceinline__ double with_hier(double ring, const HierShape& hs, uint32_t zero, double grads,
                                            const DpLink& l) {
  if (!hs.ok || zero) return ring;
  const double g1 = 2.0 * (double)(hs.g - 1), n1 = 2.0 * (double)(hs.N - 1);
  const double sh = __builtin_ceil(grads / (double)hs.g);
  const double intra = g1 * hs.a_in + link_ps(g1 * sh, hs.bq_in);
  const double inter = n1 * l.alpha + link_ps(n1 * ceil_div(sh, (double)hs.N, 1.0 / (double)hs.N), l.bq);
  return intra + inter < ring ? intra + inter : ring;
}

// The sync of pd parameters (and px expert parameters of a MoE model) per rank
// over a link.
template <bool kHier>
__device__ __forceinline__ double link_dp(const Tab& t, const Plan& p, const DpLink& l, const HierShape& hs,
                                          double rp, double rpe, double pd, double px) {
  const double gb = (double)t.grad_bytes, pb = (double)t.param_bytes;
  double tdp = ring_sync(p.psum, rp, p.zero, gb * pd, pb * pd, l.alpha, l.bq, t.ccl_tree);
  if (kHier) tdp = with_hier(tdp, hs, p.zero, gb * pd, l);
  const uint32_t pe = p.psum >> p.epl;
  if (t.E && pe > 1) tdp += ring_sync(pe, rpe, p.zero, gb * px, pb * px, l.alpha, l.bq, t.ccl_tree);
  return tdp;
}

// The DP sync of stage s (ns layers) from the plan alone.
template <int kMode>
__device__ __forceinline__ double stage_dp(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s,
                                           uint32_t ns, double rp, double rpe) {
  if (p.psum <= 1) return 0;
  HierShape hs;
  const DpLink l = stage_link<kMode>(t, h, p, s, hs);
  const Params par(h.size(), p.tpl, p.epl);
  return link_dp<true>(t, p, l, hs, rp, rpe, par.stage(ns, s == 0, s == p.S - 1), (double)ns * par.expert);
}

// Gradient sync overlapped with stage s's last backward pass (shared layout;
// stage s holds layers [lo, hi) on device type k in the pipeline's class).
// Buckets -- the head on the last stage, the layers from the top, the
// embedding on the first stage -- each start once their backward is done,
// one after another on the stage's ring.  Bucket j is ready at
// r_j = end - R_j (R_j: backward compute of the buckets after it), so the
// queue completes at end + max_j (D_j - R_j) (D_j: syncs of bucket j and
// the later ones); that tail is returned, walked from the last bucket.
// The plan-level part of stage s's overlapped sync: the sync of one layer's
// bucket (dl; every layer bucket of the stage has the same size) and, on
// the first and last stages, of the embedding's and the head's buckets.
struct OvlSyncs {
  double dl, demb, dhead;
};
template <int kMode>
__device__ __forceinline__ OvlSyncs overlap_syncs(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s,
                                                  const DpLink& l, const HierShape& hs, double rp, double rpe) {
  OvlSyncs r = {0, 0, 0};
  const Params par(h.size(), p.tpl, p.epl);
  const double gb = (double)t.grad_bytes, pb = (double)t.param_bytes;
  auto ring = [&](double n) {
    return with_hier(ring_sync(p.psum, rp, p.zero, gb * n, pb * n, l.alpha, l.bq, t.ccl_tree), hs, p.zero, gb * n, l);
  };
  r.dl = link_dp<true>(t, p, l, hs, rp, rpe, par.layer, par.expert);
  if (s == 0) r.demb = ring(par.embed);
  if (s == p.S - 1) r.dhead = ring(par.head);
  return r;
}

// The class's part: its buckets' readiness from its own backward compute on
// device type k, walked against the syncs.  (In fp64 the result is exact
// where it is below 2^53; the u64 redo takes int64.)
template <int kMode, typename V>
__device__ __forceinline__ V overlap_walk(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s,
                                          uint32_t lo, uint32_t hi, uint32_t k, const OvlSyncs& y) {
  if (p.psum <= 1) return 0;
  const uint32_t tpl = p.tpl, mi = p.mi;
  const uint32_t L1 = t.L + 1, epq = t.E ? p.epl : 0;
  const uint32_t row = ((k * 4 + tpl) * t.n_mbs + mi) * t.nep + epq;
  V D = 0, R = 0, X = 0;
  if (s == 0) {
    D += (V)y.demb;
    X = D;
    R += (V)h.emb(k * t.n_mbs + mi).y;
  }
  if (t.uniform_layers) {
    // every layer's backward costs the same r: after layer i of the n the
    // value D - R is (D + dl - R) + i (dl - r), linear in i, so its largest
    // is at the first or the last layer
    const V n = (V)(hi - lo), dl = (V)y.dl, r = (V)h.pfb(row).y;
    const V v0 = D + dl - R, v1 = v0 + (n - 1) * (dl - r);
    X = v0 > X ? v0 : X;
    X = v1 > X ? v1 : X;
    D += n * dl;
    R += n * r;
  } else {
    for (uint32_t l = lo; l < hi; ++l) {
      D += (V)y.dl;
      X = D - R > X ? D - R : X;
      R += (V)(h.pfb(row * L1 + l + 1).y - h.pfb(row * L1 + l).y);
    }
  }
  if (s == p.S - 1) {
    D += (V)y.dhead;
    X = D - R > X ? D - R : X;
  }
  return X;
}

// The sync that follows stage s of the pipeline's class (shared layout), from
// the plan alone: the stage's whole ring, or with overlap the part of its
// bucket syncs left after its last backward pass.
template <int kMode>
__device__ __forceinline__ uint64_t stage_sync(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s,
                                               uint32_t lo, uint32_t hi, double rp, double rpe) {
  if (!p.overlap) return (uint64_t)stage_dp(t, h, p, s, hi - lo, rp, rpe);
  if (p.psum <= 1) return 0;
  HierShape hs;
  const DpLink l = stage_link<kMode>(t, h, p, s, hs);
  return (uint64_t)overlap_walk<kMode, int64_t>(t, h, p, s, lo, hi, (uint32_t)(p.tc >> (4 * s)) & 15,
                                                overlap_syncs(t, h, p, s, l, hs, rp, rpe));
}

// Per-class layout.  The gradients of layers [a, e) -- a segment between
// consecutive cuts of any class, so inside one stage of every class -- sync
// in one ring over every replica, on the coarsest TP layout among the
// classes; before it, each class with finer shards gathers the coarse shard
// inside its TP groups (ring all-gather over 2^(tpl - tpl_min) members of
// the class's own shard, on the node fabric; classes at the same time, so
// the slowest counts).  rows: the plan's four class cut rows.
__device__ __forceinline__ uint32_t row_word(const uint4 (&rows)[4], uint32_t c, uint32_t j) {
  const uint4 v = rows[c];
  return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
}

// Weighting of a gradient shard of n elements by the class's share of the
// global batch, on a device of type k: one multiply per element, the fp32
// shard read and written (the roofline time of one elementwise op)
// (the ceilings through fp64 reciprocals: a 64-bit integer division is a
// long instruction loop on this ISA)
__device__ __forceinline__ uint64_t weigh_ps(const Tab& t, const SpeedInfo& v, uint64_t n) {
  const uint64_t by = 2000 * t.grad_bytes * n;
  const uint64_t tc = div_up_u64(n, v.tflops, v.rtflops), tm = div_up_u64(by, v.hbm, v.rhbm);
  return tc > tm ? tc : tm;
}

template <int kMode>
__device__ __forceinline__ uint64_t seg_dp(const Tab& t, const Hot<kMode>& h, const Plan& p, const uint4 (&rows)[4],
                                           uint32_t a, uint32_t e, double rp, double rpe, uint64_t& lat,
                                           uint64_t& bw) {
  const uint32_t G = p.G, epl = p.epl, ns = e - a;
  uint32_t tmin = 3;
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2)
    if (c2 < G) tmin = cls_tpl(p.chdr, c2) < tmin ? cls_tpl(p.chdr, c2) : tmin;
  // classes at different micro-batch sizes weight their gradients first
  bool mixed = false;
#pragma unroll
  for (uint32_t c2 = 1; c2 < 4; ++c2)
    if (c2 < G) mixed = mixed || cls_mi(p.chdr, c2) != cls_mi(p.chdr, 0);
  bool same = true;
  uint32_t k0 = 0, nmin = 0xffffffffu, nmax = 0, bq_dp = 0;
  double a_dp = 0;
  uint64_t rs = 0, rs_l = 0, rs_b = 0;
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2) {
    if (c2 >= G) continue;
    const uint32_t tpl2 = cls_tpl(p.chdr, c2);
    // the stage of class c2 holding layer a: its cuts in (0, a] (bytes past its stages are 0)
    uint32_t s2 = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t w = row_word(rows, c2, j);
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t v = (w >> (8 * q)) & 0xff;
        s2 += (v != 0 && v <= a) ? 1u : 0u;
      }
    }
    const uint32_t k2 = (uint32_t)(p.tv[c2] >> (4 * s2)) & 15;
    const TypeInfo t2 = h.type(k2);
    const uint32_t b2 = dev_before<true>(p, c2, s2, k2), n2 = p.reps[c2] << tpl2, d2 = t2.dpl;
    const uint32_t l2 = t2.node_off + (b2 >> d2), h2 = t2.node_off + ((b2 + n2 - 1) >> d2);
    const uint32_t dl2 = t2.dev_off + b2;
    const uint32_t nic2 = range_max(h.rmn, t.D, dl2, dl2 + n2 - 1);
    if (c2 == 0) k0 = k2; else same = same && k2 == k0;
    nmin = l2 < nmin ? l2 : nmin;
    nmax = h2 > nmax ? h2 : nmax;
    const uint32_t bx = nic2 > t2.bq_pcie ? nic2 : t2.bq_pcie;
    bq_dp = bx > bq_dp ? bx : bq_dp;
    a_dp = 2 * t2.a_side > a_dp ? 2 * t2.a_side : a_dp;
    if (tpl2 > tmin || mixed) {
      // the class's shard: weighted (one multiply per element, read and
      // written at the device's HBM rate) when micro-batch sizes differ,
      // then gathered to the coarsest TP layout inside each TP group
      const uint64_t g1 = (1u << (tpl2 - tmin)) - 1;
      const Params p2(h.size(), tpl2, epl);
      const uint64_t sh = (uint64_t)(p2.stage(ns, a == 0, e == t.L) + (double)ns * p2.expert);
      const uint64_t sc = mixed ? weigh_ps(t, h.speed(k2), sh) : 0;
      const uint32_t bq_in = range_max(h.rmi(), t.N, l2, h2);
      const uint64_t rl = sc + g1 * (uint64_t)t2.a_intra,
                     rb = (uint64_t)link_ps((double)(g1 * t.grad_bytes * sh), bq_in), r = rl + rb;
      if (r > rs) {
        rs = r;
        rs_l = rl;
        rs_b = rb;
      }
    }
  }
  const bool intra = same && nmin == nmax;
  const double alpha = intra ? h.intra_alpha(k0) : a_dp;
  const uint32_t bq = intra ? h.rmi()[nmin] : bq_dp;
  const Params par(h.size(), tmin, epl);
  const double pd = par.stage(ns, a == 0, e == t.L), gb = (double)t.grad_bytes, pb = (double)t.param_bytes;
  double ld = 0, bd = 0, le = 0, be = 0;
  if (p.psum > 1) ring_parts(p.psum, rp, p.zero, gb * pd, pb * pd, alpha, bq, t.ccl_tree, ld, bd);
  const uint32_t pe = p.psum >> epl;
  if (t.E && pe > 1) {
    const double px = (double)ns * par.expert;
    ring_parts(pe, rpe, p.zero, gb * px, pb * px, alpha, bq, t.ccl_tree, le, be);
  }
  lat = (uint64_t)(ld + le) + rs_l;
  bw = (uint64_t)(bd + be) + rs_b;
  return lat + bw;
}

// The sync a stage [lo, hi) of the pipeline's class waits for: the longest
// of the segments inside it, or with contention the largest latency part
// plus the sum of the link-time parts.
template <int kMode>
__device__ __forceinline__ uint64_t het_stage_dp(const Tab& t, const Hot<kMode>& h, const Plan& p,
                                                 const uint4 (&rows)[4], uint32_t lo, uint32_t hi, double rp,
                                                 double rpe) {
  uint64_t best = 0, lmax = 0, bsum = 0;
  for (uint32_t a = lo; a < hi;) {
    uint32_t e = hi;   // the next cut of any class above a
#pragma unroll
    for (uint32_t c2 = 0; c2 < 4; ++c2)
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t w = row_word(rows, c2, j);
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          const uint32_t v = (w >> (8 * q)) & 0xff;
          e = (v > a && v < e) ? v : e;
        }
      }
    uint64_t sl, sb;
    const uint64_t x = seg_dp(t, h, p, rows, a, e, rp, rpe, sl, sb);
    best = x > best ? x : best;
    lmax = sl > lmax ? sl : lmax;
    bsum += sb;
    a = e;
  }
  return t.contention ? lmax + bsum : best;
}

__device__ __forceinline__ void load_rows(const uint4* prow, uint4 (&rows)[4]) {
#pragma unroll
  for (int c = 0; c < 4; ++c) rows[c] = prow[c];
}

// cut byte of stage s (run-time index) of class c of the plan's cut rows
__device__ __forceinline__ uint32_t row_cut(const uint4 (&rows)[4], uint32_t c, uint32_t s) {
  const uint4 r = rows[c];
  const uint64_t lo = (uint64_t)r.y << 32 | r.x, hi = (uint64_t)r.w << 32 | r.z;
  const uint64_t m = 0ull - (uint64_t)(s >> 3);
  return (uint32_t)(((lo & ~m) | (hi & m)) >> (8 * (s & 7))) & 0xff;
}

// Per-class layout: where class c's stages of type k start in their pool (each
// class's blocks are contiguous from a multiple of its TP degree on), for
// classes 0 .. last, handed to put(c, k, first device).
template <typename Put>
__device__ __forceinline__ void class_starts(const Tab& t, const Plan& p, uint32_t last, Put put) {
  for (uint32_t k = 0; k < t.K; ++k) {
    uint32_t ptr = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c) {
      const uint32_t tl = cls_tpl(p.chdr, c), first = align_up(ptr, tl);
      if (c <= last) put(c, k, first);
      const uint32_t n = c < p.G ? count_type(p.tv[c], k, stage_sel(cls_S(p.chdr, c))) : 0;
      ptr = n ? first + ((p.reps[c] * n) << tl) : ptr;
    }
  }
}
// The next devices from a lane's counter in LDS.
__device__ __forceinline__ uint32_t draw(uint32_t* counter, uint32_t devices) {
  return __hip_atomic_fetch_add(counter, devices, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Per-class layout: the sync each (class, stage) of a valid plan waits for
// -- the same values as het_stage_dp -- found by one walk over the segments
// of the whole model.  Each class's stage holding the current segment, with
// its placement and links, is recomputed only when the walk crosses one of
// that class's cuts; a class's running max is stored when it leaves a stage.
// drow: the plan's four rows of 16 entries (class c, stage s at c*16 + s);
// cnt: the lane's column of 4 K counters in LDS (class c, type k at 64 (c K + k)).  In
// fp64: exact below 2^53, and a pipeline that waits for a longer sync is
// redone in u64.
template <int kMode>
__device__ __forceinline__ void het_plan_syncs(const Tab& t, const Hot<kMode>& h, const Plan& p,
                                               const uint4 (&rows)[4], double* __restrict__ drow,
                                               uint32_t* cnt) {
  const uint32_t G = p.G, epl = p.epl;
  const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> epl);
  uint32_t tmin = 3;
  bool mixed = false;   // classes at different micro-batch sizes weight their gradients first
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2)
    if (c2 < G) {
      tmin = cls_tpl(p.chdr, c2) < tmin ? cls_tpl(p.chdr, c2) : tmin;
      mixed = mixed || cls_mi(p.chdr, c2) != cls_mi(p.chdr, 0);
    }
  // per class: current stage and its end, and that stage's type, node range,
  // worst NIC/PCIe rate, inter-node latency, node latency, worst node fabric;
  // classes enter their first stage at the walk's first step
  // cur: the stage's sync so far -- the longest segment, or with contention
  // the largest latency part (cur) and the summed link times (curb)
  uint32_t stg[4], nxt[4], kk[4], nl[4], nh[4], bx[4], bin[4];
  double as2[4], ain[4], cur[4], curb[4];
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2) {
    stg[c2] = 0xffffffffu; nxt[c2] = c2 < G ? 0 : 0xffffffffu; kk[c2] = 0; nl[c2] = 0; nh[c2] = 0; bx[c2] = 0;
    bin[c2] = 0; as2[c2] = 0; ain[c2] = 0; cur[c2] = 0; curb[c2] = 0;
  }
  class_starts(t, p, 3, [&](uint32_t c, uint32_t k, uint32_t first) { cnt[64 * (c * t.K + k)] = first; });
  const Params par(h.size(), tmin, epl);
  const double gb = (double)t.grad_bytes, pb = (double)t.param_bytes;
  double sl[4];   // parameters of a layer on one TP rank of each class
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2) {
    const uint32_t tpl2 = cls_tpl(p.chdr, c2);
    sl[c2] = h.size().layer[tpl2] + h.size().expert[tpl2][epl];
  }
  for (uint32_t a = 0; a < t.L;) {
#pragma unroll
    for (uint32_t c2 = 0; c2 < 4; ++c2) {
      if (nxt[c2] == a) {   // the walk crossed one of class c2's cuts (or starts)
        if (a > 0) drow[c2 * kMaxStages + stg[c2]] = cur[c2] + curb[c2];
        cur[c2] = 0;
        curb[c2] = 0;
        const uint32_t s2 = ++stg[c2], tpl2 = cls_tpl(p.chdr, c2);
        const uint32_t k2 = (uint32_t)(p.tv[c2] >> (4 * s2)) & 15;
        const TypeInfo t2 = h.type(k2);
        const uint32_t n2 = p.reps[c2] << tpl2, b2 = draw(&cnt[64 * (c2 * t.K + k2)], n2), d2 = t2.dpl;
        const uint32_t l2 = t2.node_off + (b2 >> d2), h2 = t2.node_off + ((b2 + n2 - 1) >> d2);
        const uint32_t dl2 = t2.dev_off + b2;
        const uint32_t nic2 = range_max(h.rmn, t.D, dl2, dl2 + n2 - 1);
        nxt[c2] = row_cut(rows, c2, s2);
        kk[c2] = k2;
        nl[c2] = l2;
        nh[c2] = h2;
        bx[c2] = nic2 > t2.bq_pcie ? nic2 : t2.bq_pcie;
        as2[c2] = 2 * t2.a_side;
        ain[c2] = t2.a_intra;
        bin[c2] = tpl2 > tmin ? range_max(h.rmi(), t.N, l2, h2) : 0;
      }
    }
    uint32_t e = t.L;
#pragma unroll
    for (uint32_t c2 = 0; c2 < 4; ++c2)
      if (c2 < G) e = nxt[c2] < e ? nxt[c2] : e;
    // the sync of layers [a, e)
    const uint32_t ns = e - a;
    bool same = true;
    uint32_t nmin = 0xffffffffu, nmax = 0, bq_dp = 0;
    double a_dp = 0, rs = 0, rs_l = 0, rs_b = 0;
#pragma unroll
    for (uint32_t c2 = 0; c2 < 4; ++c2) {
      if (c2 >= G) continue;
      same = same && kk[c2] == kk[0];
      nmin = nl[c2] < nmin ? nl[c2] : nmin;
      nmax = nh[c2] > nmax ? nh[c2] : nmax;
      bq_dp = bx[c2] > bq_dp ? bx[c2] : bq_dp;
      a_dp = as2[c2] > a_dp ? as2[c2] : a_dp;
      const uint32_t tpl2 = cls_tpl(p.chdr, c2);
      if (tpl2 > tmin || mixed) {
        const double g1 = (double)((1u << (tpl2 - tmin)) - 1);
        const double sh = (double)ns * sl[c2] + (a == 0 ? h.size().embed[tpl2] : 0.0) +
                          (e == t.L ? h.size().head[tpl2] : 0.0);
        const double rl = (mixed ? (double)weigh_ps(t, h.speed(kk[c2]), (uint64_t)sh) : 0.0) + g1 * ain[c2];
        const double rb = link_ps(g1 * gb * sh, bin[c2]), r = rl + rb;
        if (r > rs) {
          rs = r;
          rs_l = rl;
          rs_b = rb;
        }
      }
    }
    const bool intra = same && nmin == nmax;
    const double alpha = intra ? ain[0] : a_dp;
    const uint32_t bq = intra ? h.rmi()[nmin] : bq_dp;
    const double pd = par.stage(ns, a == 0, e == t.L), px = (double)ns * par.expert;
    if (!t.contention) {
      double x = p.psum <= 1 ? 0 : ring_sync(p.psum, rp, p.zero, gb * pd, pb * pd, alpha, bq, t.ccl_tree);
      const uint32_t pe = p.psum >> epl;
      if (t.E && pe > 1) x += ring_sync(pe, rpe, p.zero, gb * px, pb * px, alpha, bq, t.ccl_tree);
      x += rs;
#pragma unroll
      for (uint32_t c2 = 0; c2 < 4; ++c2)
        if (c2 < G) cur[c2] = x > cur[c2] ? x : cur[c2];
    } else {
      double ld = 0, bd = 0, le = 0, be = 0;
      if (p.psum > 1) ring_parts(p.psum, rp, p.zero, gb * pd, pb * pd, alpha, bq, t.ccl_tree, ld, bd);
      const uint32_t pe = p.psum >> epl;
      if (t.E && pe > 1) ring_parts(pe, rpe, p.zero, gb * px, pb * px, alpha, bq, t.ccl_tree, le, be);
      const double l = ld + le + rs_l, b = bd + be + rs_b;
#pragma unroll
      for (uint32_t c2 = 0; c2 < 4; ++c2)
        if (c2 < G) {
          cur[c2] = l > cur[c2] ? l : cur[c2];
          curb[c2] += b;
        }
    }
    a = e;
  }
#pragma unroll
  for (uint32_t c2 = 0; c2 < 4; ++c2)
    if (c2 < G) drow[c2 * kMaxStages + stg[c2]] = cur[c2] + curb[c2];
}

// Where the devices of stage s of the pipeline's class sit: type k, its
// pool's info, the first device in the pool, the stage's nodes, and the
// slowest node fabric and NIC rates over the stage's reps * tp devices.
struct StagePlace {
  uint32_t k, base, nl, nh, bq_in, bq_nic;
  TypeInfo ti;
};
template <int kMode>
__device__ __forceinline__ StagePlace stage_place(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t k,
                                                  uint32_t base) {
  StagePlace r;
  r.k = k;
  r.base = base;
  r.ti = h.type(k);
  const uint32_t nd = p.rc * p.tp, dpl = r.ti.dpl, j = 31u - __clz(nd);
  r.nl = r.ti.node_off + (base >> dpl);
  r.nh = r.ti.node_off + ((base + nd - 1) >> dpl);
  r.bq_in = range_max(h.rmi(), t.N, r.nl, r.nh);
  // (range_max with the level the same for every stage)
  const uint32_t* row = h.rmn + j * t.D + r.ti.dev_off + base;
  const uint32_t a = row[0], b = row[nd - (1u << j)];
  r.bq_nic = a > b ? a : b;
  return r;
}

// Forward and backward time of one micro-batch over layers [lo, hi) on a stage
// of the pipeline's class (act: bytes of its activation): the layers, the embedding if `first`, the head if
// `last`, the TP all-reduces exposed in the forward pass and the MoE
// all-to-all in both passes.  wc: the weight-gradient pass of the zero-bubble
// order, half of the backward compute rounded down (the all-to-all carries
// input gradients: it stays in the input-gradient pass).
template <int kMode, bool kHet>
__device__ __forceinline__ void stage_cost(const Tab& t, const Hot<kMode>& h, const Plan& p, const StagePlace& sp,
                                           double act, uint32_t lo, uint32_t hi, bool first, bool last, double& fc,
                                           double& bc, double& wc) {
  const uint32_t tp = p.tp, ep = p.ep, tpl = p.tpl, epl = p.epl, mi = p.mi, ns = hi - lo, dpl = sp.ti.dpl, k = sp.k;
  const uint32_t L1 = t.L + 1, epq = t.E ? p.epl : 0;
  const uint32_t row = ((k * 4 + tpl) * t.n_mbs + mi) * t.nep + epq;
  if (t.uniform_layers) {
    const double2 lc = h.pfb(row);
    fc = lc.x * (double)ns;
    bc = lc.y * (double)ns;
  } else {
    const double2 ph = h.pfb(row * L1 + hi), pl = h.pfb(row * L1 + lo);
    fc = ph.x - pl.x;
    bc = ph.y - pl.y;
  }
  if (first) {
    const double2 em = h.emb(k * t.n_mbs + mi);
    fc += em.x;
    bc += em.y;
  }
  if (last) {
    const double2 hd = h.head((k * 4 + tpl) * t.n_mbs + mi);
    fc += hd.x;
    bc += hd.y;
  }
  wc = __builtin_floor(bc * 0.5);
  if (tp > 1) {  // TP all-reduces of this stage, exposed in the forward pass
    const double steps = (double)((2 * ns + first) * 2 * (tp - 1));
    const double act_tp = __builtin_ceil(__builtin_ldexp(act, -(int)tpl));   // a TP rank's share
    fc += steps * sp.ti.a_intra + link_ps(steps * act_tp, sp.bq_in);
  }
  if (t.E && ep > 1) {  // dispatch + combine all-to-all in each pass
    // EP groups are blocks of ep*tp devices from base on.  With one TP
    // degree for all classes base is a multiple of ep*tp, and the groups
    // are inside nodes iff one fits a node.  With per-class degrees, a
    // group of E = ep*tp <= node size starting at offset r in its node
    // fits iff r <= node - E; the offsets of the successive groups are
    // base's in-node offset plus multiples of E, so with b = base mod E
    // != 0 the first group to cross is number node/E - 1 - (in-node offset div E).
    const uint32_t E = ep * tp;
    bool intra = E <= (1u << dpl);
    if (kHet && intra && (sp.base & (E - 1)) != 0) {
      const uint32_t q = (sp.base & ((1u << dpl) - 1)) / E;
      intra = p.rc / ep <= (1u << dpl) / E - 1 - q;
    }
    const double alpha = intra ? sp.ti.a_intra : 2 * sp.ti.a_side;
    const uint32_t bq = intra ? sp.bq_in : (sp.bq_nic > sp.ti.bq_pcie ? sp.bq_nic : sp.ti.bq_pcie);
    const uint32_t pa = (epl * t.n_mbs + mi) * L1;
    const double e = (double)(ns * 2 * (ep - 1)) * alpha + link_ps(2 * (h.pa(pa + hi) - h.pa(pa + lo)), bq);
    fc += e;
    bc += e;
  }
}

// Rail-only network (Fig. 2): the NIC of local rank r of every node joins
// rail r and rails do not meet.  A pipeline hop between nodes pairs device i
// of the sending stage (n = reps * tp devices) with device i of the receiving
// one; a pair at different local ranks is
// forwarded over a node's fabric first -- the sender's, or the receiver's
// when the sender's nodes hold one device -- which adds that node's latency
// and the activation at its slowest fabric rate (over the
// stage's nodes).  Offsets os, or in their nodes: every pair shares a rank
// iff os == or and, with different node sizes, the n pairs do not reach the
// end of the smaller node (past it one rank wraps and the other does not).
__device__ __forceinline__ double rail_extra(uint32_t n, const StagePlace& from, const StagePlace& to, double act) {
  const uint32_t ds = 1u << from.ti.dpl, dr = 1u << to.ti.dpl, os = from.base & (ds - 1), orr = to.base & (dr - 1);
  const bool same = os == orr && (ds == dr || os + n <= (ds < dr ? ds : dr));
  if (same) return 0;
  const bool at_s = from.ti.dpl > 0;
  return (at_s ? from.ti.a_intra : to.ti.a_intra) + link_ps(act, at_s ? from.bq_in : to.bq_in);
}

// Hop between two stages of one class, a placed before b when they share a
// pool: inside a node iff every replica's pair is, i.e. iff a's first device
// and b's last one share a node.
__device__ __forceinline__ double hop_ps(const Tab& t, const Plan& p, const StagePlace& a, const StagePlace& b,
                                         double act, bool a_sends) {
  const uint32_t dpl = b.ti.dpl, n = p.rc * p.tp;
  const bool intra = a.k == b.k && (a.base >> dpl) == ((b.base + n - p.tp) >> dpl);
  const double alpha = intra ? b.ti.a_intra : a.ti.a_side + b.ti.a_side;
  const uint32_t in = a.bq_in > b.bq_in ? a.bq_in : b.bq_in, nic = a.bq_nic > b.bq_nic ? a.bq_nic : b.bq_nic;
  const uint32_t pcie = a.ti.bq_pcie > b.ti.bq_pcie ? a.ti.bq_pcie : b.ti.bq_pcie;
  double hop = alpha + link_ps(act, intra ? in : nic > pcie ? nic : pcie);
  if (t.rail_only && !intra) hop += a_sends ? rail_extra(n, a, b, act) : rail_extra(n, b, a, act);
  return hop;
}

// Setup of a pipeline: the costs of its stages into `sink`.  first_device(s, k)
// places stage s (of type k) in its pool; placed(s, place) sees where it went.
// Stage s - 1 of the same pool ends where stage s begins, so hop_ps's order
// holds.
template <int kMode, bool kHet, typename Sink, typename First, typename Placed>
__device__ __forceinline__ void class_setup(const Tab& t, const Hot<kMode>& h, const Plan& p, Sink& sink,
                                            First first_device, Placed placed) {
  // register sinks fix the stage count at compile time (the plan's S equals it)
  const uint32_t S = Sink::kS ? (uint32_t)Sink::kS : p.S;
  const double act = h.size().act[p.mi];
  uint32_t lo = 0;
  StagePlace prev = {};
#pragma unroll Sink::kUnroll
  for (uint32_t s = 0; s < S; ++s) {
    const uint32_t hi = cut_at(p, s), k = (uint32_t)(p.tc >> (4 * s)) & 15;
    const StagePlace sp = stage_place<kMode>(t, h, p, k, first_device(s, k));
    placed(s, sp);
    double fc, bc, wc;
    stage_cost<kMode, kHet>(t, h, p, sp, act, lo, hi, s == 0, s == S - 1, fc, bc, wc);
    const double hop = s > 0 ? hop_ps(t, p, prev, sp, act, true) : 0;
    prev = sp;
    sink.put(s, fc, bc, wc, hop, lo, hi);
    lo = hi;
  }
}

// Stage records {forward, backward, hop, sync} in memory order (the hop of the
// last stage is 0), with the pipeline's syncs found from the plan alone, and,
// given `w`, each stage's weight-gradient pass.
template <int kMode, bool kHet>
struct RecSink {
  static constexpr int kS = 0, kUnroll = 1;   // stage count taken from the plan
  const Tab& t;
  const Hot<kMode>& h;
  const Plan& p;
  const uint4* prow;   // per-class layout: the plan's four cut rows
  uint64_t (&rec)[kMaxStages][kRecWords];
  uint64_t* w;
  __device__ __forceinline__ void put(uint32_t s, double fc, double bc, double wc, double hop, uint32_t lo,
                                      uint32_t hi) {
    const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> p.epl);
    uint64_t tdp;
    if (kHet) {
      uint4 rows[4];
      load_rows(prow, rows);
      tdp = het_stage_dp(t, h, p, rows, lo, hi, rp, rpe);
    } else {
      tdp = stage_sync(t, h, p, s, lo, hi, rp, rpe);
    }
    rec[s][0] = (uint64_t)fc;
    rec[s][1] = (uint64_t)bc;
    rec[s][2] = 0;
    rec[s][3] = tdp;
    if (w) w[s] = (uint64_t)wc;
    if (s > 0) rec[s - 1][2] = (uint64_t)hop;
  }
};
template <int kMode, bool kHet>
__device__ __forceinline__ void class_records(const Tab& t, const Hot<kMode>& h, const Plan& p, const uint4* prow,
                                              uint64_t (&rec)[kMaxStages][kRecWords], uint64_t* w) {
  RecSink<kMode, kHet> sink{t, h, p, prow, rec, w};
  class_setup<kMode, kHet>(t, h, p, sink, [&](uint32_t s, uint32_t k) { return dev_before_own<kHet>(p, s, k); },
                           [](uint32_t, const StagePlace&) {});
}

// RegSink keeps forward, backward and hop times of an S-stage pipeline in
// registers: each stage shifts the arrays down by one and appends, so after S stages stage s
// sits at index s; a runtime-indexed array would go through private memory.
// The stage loop runs S (a compile-time count) times, unrolled by
// kSetupUnroll: within an unrolled body the shifts are register renames, so
// the copies are paid once per kSetupUnroll stages.
constexpr int kSetupUnroll = 4;

template <int S>
struct RegSink {
  static constexpr int kS = S, kUnroll = kSetupUnroll;
  double f[S], b[S], c[S];
  __device__ __forceinline__ RegSink() {
#pragma unroll
    for (int i = 0; i < S; ++i) f[i] = b[i] = c[i] = 0;
  }
  __device__ __forceinline__ void put(uint32_t s, double fc, double bc, double, double hop, uint32_t, uint32_t) {
#pragma unroll
    for (int i = 0; i + 1 < S; ++i) {
      f[i] = f[i + 1];
      b[i] = b[i + 1];
      c[i] = c[i + 1];
    }
    f[S - 1] = fc;
    b[S - 1] = bc;
    c[S - 1] = 0;
    if (S > 1 && s > 0) c[S - 2] = hop;
  }
};

// ZbSink: the same with the backward split for the zero-bubble order: bi,
// the input-gradient pass, and w, the weight-gradient pass.
template <int S>
struct ZbSink {
  static constexpr int kS = S, kUnroll = kSetupUnroll;
  double f[S], bi[S], w[S], c[S];
  __device__ __forceinline__ ZbSink() {
#pragma unroll
    for (int i = 0; i < S; ++i) f[i] = bi[i] = w[i] = c[i] = 0;
  }
  __device__ __forceinline__ void put(uint32_t s, double fc, double bc, double wc, double hop, uint32_t, uint32_t) {
#pragma unroll
    for (int i = 0; i + 1 < S; ++i) {
      f[i] = f[i + 1];
      bi[i] = bi[i + 1];
      w[i] = w[i + 1];
      c[i] = c[i + 1];
    }
    f[S - 1] = fc;
    bi[S - 1] = bc - wc;
    w[S - 1] = wc;
    c[S - 1] = 0;
    if (S > 1 && s > 0) c[S - 2] = hop;
  }
};

// Per (class, stage) quantities of every plan, in plan order: one (virtual)
// stage per lane, so that the sixteen lanes of a pipeline store its records
// side by side.  For an interleaved pipeline per virtual stage, hops and syncs
// per device, in the first PP records, the last hop being the wrap hop.
// 20011 plans: a pipeline per lane, its records in private memory, 97 us, a
// stage per lane 30.
template <bool kHet>
__global__ void __launch_bounds__(256) k_stages(Tab t, const PackedPlan* __restrict__ packed,
                                                const uint4* __restrict__ pcut, const uint32_t* __restrict__ meta,
                                                int64_t n, uint64_t* __restrict__ out_stage) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, slot = id / kMaxStages;
  const uint32_t s = (uint32_t)(id % kMaxStages);
  if (slot >= n * kMaxClasses) return;
  const uint32_t m = meta[slot], S = m & 31, v = (m >> 24) + 1;
  if (s >= S * v) return;   // (S = 0: no pipeline)
  const Plan p = load_plan<kHet>(packed, pcut, (uint32_t)slot);
  const Hot<2> h(t, nullptr);
  const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> p.epl), act = h.size().act[p.mi];
  const uint32_t d = v > 1 ? s % S : s, lo = s ? cut_at(p, s - 1) : 0, hi = cut_at(p, s);   // device d, layers [lo, hi)
  auto place = [&](uint32_t x) {
    const uint32_t k = (uint32_t)(p.tc >> (4 * x)) & 15;
    return stage_place<2>(t, h, p, k, dev_before_own<kHet>(p, x, k));
  };
  const StagePlace sp = place(d);
  double fc, bc, wc;
  stage_cost<2, kHet>(t, h, p, sp, act, lo, hi, s == 0, s == S * v - 1, fc, bc, wc);
  double hop = 0;
  uint64_t sync = 0;
  if (s < S) {
    if (s + 1 < S) hop = hop_ps(t, p, sp, place(s + 1), act, true);
    else if (v > 1) hop = hop_ps(t, p, place(0), sp, act, false);   // to device 0, placed before it
    if (kHet) {
      uint4 rows[4];
      load_rows(cut_rows(pcut, (uint32_t)(slot >> 2)), rows);
      sync = het_stage_dp(t, h, p, rows, lo, hi, rp, rpe);
    } else if (v > 1) {
      uint32_t ns = 0;
      for (uint32_t j = 0; j < v; ++j) ns += cut_at(p, j * S + s) - (j * S + s ? cut_at(p, j * S + s - 1) : 0);
      sync = (uint64_t)stage_dp(t, h, p, s, ns, rp, rpe);
    } else {
      sync = stage_sync(t, h, p, s, lo, hi, rp, rpe);
    }
  }
  ulonglong2* o = reinterpret_cast<ulonglong2*>(out_stage + (slot * kMaxStages + s) * kRecWords);
  if (((uintptr_t)out_stage & 15) == 0) {
    o[0] = make_ulonglong2((uint64_t)fc, (uint64_t)bc);
    o[1] = make_ulonglong2((uint64_t)hop, sync);
  } else {
    uint64_t* q = out_stage + (slot * kMaxStages + s) * kRecWords;
    q[0] = (uint64_t)fc;
    q[1] = (uint64_t)bc;
    q[2] = (uint64_t)hop;
    q[3] = sync;
  }
}

// Per-class layout: the syncs of every (class, stage) of every valid plan
// (one plan per lane), once per plan rather than once per pipeline; lane j
// takes plan perm[j] of the pc[512] valid plans (sorted by the length of
// their walks).  Bound by instruction issue; 3M plans 1203 us with u64 links
// and earlier devices counted over the packed types, 951 with exact fp64
// links, 846 with the counts in LDS, 736 with a plan in one 128-byte line.
template <int kMode>
__global__ void __launch_bounds__(256) k_plan_syncs(Tab t, const uint4* __restrict__ pcut,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ pc, int64_t n,
                                                    double* __restrict__ hdp) {
  extern __shared__ uint4 lds[];
  fill_lds<kMode>(t, lds);
  const Hot<kMode> h(t, lds);
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n || j >= (int64_t)pc[2 * kPlanBuckets]) return;
  const uint32_t i = perm[j];
  const Plan p = unpack(het_record(pcut + (size_t)i * kHetWords));
  uint4 rows[4];
  load_rows(cut_rows(pcut, i), rows);
  uint32_t* const cnt = (uint32_t*)((char*)lds + (kMode < 2 ? t.lds_bytes : 0)) + (threadIdx.x >> 6) * (256 * t.K) +
                        (threadIdx.x & 63u);
  het_plan_syncs(t, h, p, rows, hdp + (size_t)i * (kMaxClasses * kMaxStages), cnt);
}


// ---------------------------------------------------------------- 1F1B pipeline
// Schedule of one class (S stages, M micro-batches per replica): stage s runs
// W_s = min(S-1-s, M) forwards, then pairs (forward, backward), then its last
// W_s backwards.  F(s, m), B(s, i) are the ends of forward m and backward i:
//   F(s, m) = max(previous op's end on s, F(s-1, m) + c_{s-1}) + f_s
//   B(s, i) = max(previous op's end on s, B(s+1, i) + c_s) + b_s,
// and the pipeline's time is T = max_s B(s, M-1) + x_s (x_s: the gradient
// sync that waits for stage s), the longest path of a graph whose nodes are
// the ops.  Times are integers carried exactly in fp64.
//
// Four things make that path cheap:
//  * Potentials.  Measured from phi_s = f_0 + sum_{j<s} (c_j + f_{j+1}) -- the
//    end of F(s, 0) -- and B from phi_s + b_s, the edges F(s-1,m) -> F(s,m) and
//    F(s,.) -> B(s,.) cost nothing, B(s,.) -> F(s,.) costs a_s = f_s + b_s and
//    B(s+1,i) -> B(s,i) costs d_s = 2 c_s + f_{s+1} + b_{s+1}.  A steady
//    iteration (a backward, then a forward, on every stage, from the last to
//    the first) is then
//      B = max(F_s, B + d_s);  F_s = max(B + a_s, F_{s-1})
//    -- 4 fp64 operations per stage (6 on the times themselves), with the S
//    values F_s as the whole state; B is carried from stage to stage.
//  * Warm-up in closed form.  Forward m <= W_s of stage s follows forwards
//    only, and its longest path spends its m micro-batches at the slowest of
//    the stages 0..s: F(s, m) = m max_{j<=s} f_j.  The iteration above starts
//    from F_s = F(s, min(S-1-s, M-1)).
//  * Drain from the end.  After F(s, M-1) a stage runs backwards only: e_s is
//    the longest path from B(s, M-1-min(S-1-s, M-1)) to the end of the
//    iteration, syncs included, found backwards before the loop; the schedule
//    ends with T = max_s B_s + e_s.
//  * Periodic regime.  One iteration maps the state to maxima of (component +
//    constant) terms, so adding a constant lam to every component adds lam to
//    every component of the result: once an iteration advances every
//    component by the same lam, every later one does too, and the remaining r
//    steady iterations collapse into F += r lam, exactly.
// In fp64 every value is at most T: if T stays below 2^53 nothing was rounded,
// otherwise the pipeline is redone in u64.
typedef uint64_t StageRec[kMaxStages][kRecWords];

__device__ __forceinline__ double vmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ uint64_t vmax(uint64_t a, uint64_t b) { return a > b ? a : b; }

// Steady iterations k_cont gives a pipeline before it moves to the second
// list, and how many must be left for a pipeline to go on elsewhere (k_power
// needs 16 minus the stage count).
constexpr int kContBudget = 48, kPowerMin = 16;
// With so few entries in the first list k_cont leaves them to k_power: their
// tiles would not fill the chip, and a tile takes 15-60 us, an entry 6.  A
// call of 60000 random plans takes 226 us with the line at 4096 entries and 196
// at 16384, one of 131072 plans 242 and 259: the line lies between.
constexpr uint32_t kContFew = 12288;
// A second list of more entries than this goes on lane by lane, a tile per
// wavefront: a matrix power takes a SIMD about 6.8 us however many there are,
// an iteration of a tile 7.5 ns per stage, so the entries of a full tile of n
// share a run of up to kPowerCost n iterations and stages for what n powers
// would cost; those with more left keep to the powers.  Random sweeps leave
// 3000-10000 entries there, and gain nothing (a line at 16384 took sweeps that
// leave 20000 from 660 to 805 us, behind the tiles' longest runs); sweeps over
// links an eighth or a sixteenth as fast leave 70000-90000: 2^20 plans of
// Llama-7B 1189 -> 794 us, of Mixtral 1031 -> 741.
constexpr uint32_t kPowerLong = 32768, kPowerCost = 1000;

// A wavefront of the first pass waits this many steady iterations for its
// lanes, then the aperiodic ones leave for the continuation lists.  Most
// schedules are periodic after a few iterations, later with more stages; at
// S + 8, 16-18 % of the random sweeps' 16-stage pipelines leave, 6-9 % of the
// 8-stage and 2-4 % of the 4-stage ones.
__host__ __device__ constexpr int first_budget(int S) { return S + 8; }

template <int S, typename V>
struct Chain {
  V a[S], d[S], e[S], f[S];   // d[S-1] unused
};

// The chain of a pipeline from its stages' forward, backward and hop times and
// syncs.  kZb, the zero-bubble order (ZB-H1, Qi et al. 2024): b is the
// input-gradient pass, w the weight-gradient pass; stage s runs W(s, i - s)
// right after B(s, i) once i >= s, and its last min(s, M) W passes at the end.
// A W only delays its stage, so it adds w to a_s (from iteration s on), to the
// backwards-only edges of the drain and, min(s + 1, M) times, to the end.
template <int S, typename V, bool kZb>
__device__ __forceinline__ void reduce_chain(const V (&f)[S], const V (&b)[S], const V (&w)[S], const V (&c)[S],
                                             const V (&x)[S], uint32_t M, Chain<S, V>& h) {
  const int m_ = (int)M;
#pragma unroll
  for (int s = 0; s < S; ++s) h.d[s] = s + 1 < S ? c[s] + c[s] + f[s + 1] + b[s + 1] : (V)0;
  V phi = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    phi += s ? c[s - 1] + f[s] : f[0];
    V y = phi + b[s] + x[s];
    if (kZb) y += (V)(s + 1 < m_ ? s + 1 : m_) * w[s];
    h.e[s] = s ? vmax(y, h.e[s - 1] + h.d[s - 1]) : y;
  }
#pragma unroll
  for (int k = 1; k < S; ++k) {
    if (k < m_) {
#pragma unroll
      for (int s = 0; s <= S - 1 - k; ++s) {
        V y = h.e[s] + b[s];
        if (kZb) y += m_ - 1 - k >= s ? w[s] : (V)0;
        h.e[s] = s ? vmax(y, h.e[s - 1] + h.d[s - 1]) : y;
      }
    }
  }
  V fm = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    fm = vmax(fm, f[s]);
    h.a[s] = f[s] + b[s] + (kZb ? w[s] : (V)0);
    h.f[s] = (V)(S - 1 - s < m_ - 1 ? S - 1 - s : m_ - 1) * fm;
  }
}

// Iteration i on stages S-1 .. lo (lo = 0: a steady iteration).  kZb: before
// iteration s stage s has no W to run yet.
template <int S, typename V, bool kZb>
__device__ __forceinline__ V chain_iter(Chain<S, V>& h, const V (&w)[S], int i, int lo) {
  V B = 0;
#pragma unroll
  for (int s = S - 1; s >= 0; --s) {
    if (s >= lo) {
      B = s == S - 1 ? h.f[s] : vmax(h.f[s], B + h.d[s]);
      const V n = B + (kZb ? (i >= s ? h.a[s] : h.a[s] - w[s]) : h.a[s]);
      h.f[s] = s ? vmax(n, h.f[s - 1]) : n;
    }
  }
  return B;
}

// The steady iterations with the periodic shortcut, checked on the second
// iteration of each pair: `left` iterations on entry, those not run on return
// (0 unless the budget ran out).
template <int S, typename V>
__device__ __forceinline__ void chain_jump(Chain<S, V>& h, int& left, int budget, int& skipped) {
  while (left >= 2 && budget > 0) {
    chain_iter<S, V, false>(h, h.a, 0, 0);
    bool same = true;
    V lam = 0, B = 0;
#pragma unroll
    for (int s = S - 1; s >= 0; --s) {
      B = s == S - 1 ? h.f[s] : vmax(h.f[s], B + h.d[s]);
      const V n = s ? vmax(B + h.a[s], h.f[s - 1]) : B + h.a[s];
      if (s == S - 1) lam = n - h.f[s];
      else same = same & (n - h.f[s] == lam);
      h.f[s] = n;
    }
    left -= 2;
    budget -= 2;
    if (same) {
      const V k = (V)left * lam;
#pragma unroll
      for (int s = 0; s < S; ++s) h.f[s] += k;
      skipped = left;
      left = 0;
    }
  }
  if (left == 1) {
    chain_iter<S, V, false>(h, h.a, 0, 0);
    left = 0;
  }
}

// After the steady iterations: stage t runs its last pair in step t, and the
// iteration ends with e_t after its next backward.  With M < S the first
// stages have run all their forwards before their first backward: their
// backwards follow step S - M's.
template <int S, typename V, bool kZb>
__device__ __forceinline__ V chain_end(Chain<S, V>& h, const V (&w)[S], uint32_t M) {
  const int m_ = (int)M;
  V T = 0;
#pragma unroll
  for (int t = 0; t < S; ++t) {
    if (t >= S - m_) {
      V B = t == S - 1 ? (V)0 : chain_iter<S, V, kZb>(h, w, m_ - S + t, t + 1);
      B = t == S - 1 ? h.f[t] : vmax(h.f[t], B + h.d[t]);
      T = vmax(T, B + h.e[t]);
      if (t > 0 && t == S - m_) {
#pragma unroll
        for (int s = S - 2; s >= 0; --s)
          if (s < t) {
            B = vmax(h.f[s], B + h.d[s]);
            T = vmax(T, B + h.e[s]);
          }
      }
    }
  }
  return T;
}

// The time of a chain of M micro-batches with the periodic shortcut, the
// whole loop in place where it stays aperiodic; `skipped` returns the steady
// iterations it skipped.
template <int S, typename V, bool kZb>
__device__ __forceinline__ V chain_time(Chain<S, V>& h, const V (&w)[S], uint32_t M, int& skipped) {
  int left = (int)M - S;
  skipped = 0;
  if (kZb) {   // from iteration S - 1 on every stage runs its W
    int i = 0;
    for (; i < left && i < S - 1; ++i) chain_iter<S, V, true>(h, w, i, 0);
    left -= i;
  }
  chain_jump<S, V>(h, left, INT_MAX, skipped);
  return chain_end<S, V, kZb>(h, w, M);
}

// If T < 2^53 no rounding ever happened (every value the fp64 pass computes is
// the length of a path, at most T).  Otherwise the pipeline goes on the redo
// list and k_redo_u64 evaluates it again in u64, outside the hot kernels.
constexpr double kExact = 9007199254740992.0;

// ---------------------------------------------------------------- continuation lists
// Offer a pipeline's chain with `left` steady iterations to run to list kList
// (1 or 2) of its stage count; false if the list is full.
template <int S, int kList>
__device__ __forceinline__ bool cont_push(const EvalBufs& e, const Chain<S, double>& h, int left, uint32_t slot) {
  constexpr uint32_t j = kMaxStages - S;
  uint32_t first, cap, ctr;
  if (kList == 1) {
    const uint32_t sub = blockIdx.x & (e.cinfo[64 + j] - 1);
    cap = e.cinfo[16 + j];
    first = e.cinfo[j] + sub * cap * S;
    ctr = cont1_ctr(j, sub);
  } else {
    first = e.cinfo[32 + j];
    cap = e.cinfo[48 + j];
    ctr = cont2_ctr(j);
  }
  const uint32_t pos = atomicAdd(&e.ctr[ctr], 1u);
  if (pos >= cap * 64u) return false;
  double* q = e.cont + (size_t)first * (kContUnit / 8) + (size_t)(pos >> 6) * (256 * S) + (pos & 63u);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    q[64 * s] = h.f[s];
    q[64 * (S + s)] = h.a[s];
    if (s < S - 1) q[64 * (2 * S + s)] = h.d[s];
    q[64 * (3 * S + s)] = h.e[s];
  }
  *(uint2*)&q[64 * (3 * S - 1)] = make_uint2((uint32_t)left, slot);
  return true;
}

__device__ __forceinline__ void count_skipped(const EvalBufs& e, int S, int skipped) {
  if (e.skipped_ops && skipped > 0)
    atomicAdd(e.skipped_ops + ((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % kSkipSlots) * kSkipStride,
              (unsigned long long)skipped * (unsigned long long)(6 * (S - 1) + 2));
}

// Raise a plan's time (the result word is in place since k_prep).
__device__ __forceinline__ void raise_time(const EvalBufs& e, uint32_t slot, double T) {
  if (T < kExact) atomicMax((unsigned long long*)&e.out[slot >> 2], (unsigned long long)T);
  else e.ovf[atomicAdd(&e.ctr[0], 1u)] = slot;
}

// Schedules that are not periodic after a few iterations mostly drift, often
// with a period of two iterations: each stage advances at its own rate, and a
// queue between two of them fills or drains until the order of a max changes.
// Let q iterations advance the state by a vector D.  If, in q further
// iterations, every max's argument carries its rate on so that the rates come
// out as D again, and the state has moved by D, then the state moves by D
// every q iterations for as long as no argument is overtaken: at least
// J = min lead / (rate of the other - rate of the argument) times.  All of
// them are taken in one step.  (A periodic schedule is the case of equal
// rates, J without bound.)
//
// For how many steps x stays on its side of max(x, y) when x - y = dx changes by
// dr per step (whole numbers): -dx / dr where that is positive, as the bits of
// an fp32 number read unsigned, so that what sets no bound is larger than any
// bound: a negative quotient, a tie (a tiny negative number), and equal rates.
// Those divide by 2^-60, which is lost beside any other rate: the quotient is
// negative or at least 2^60 and, as |dx| < 2^62, finite.  (This file is compiled
// with -ffinite-math-only, under which an infinity or a NaN is an undefined
// value.)  rcp: an fp32 reciprocal within one unit in the last place.
template <typename Rcp>
__host__ __device__ __forceinline__ uint32_t lead_bits(double dx, double dr, Rcp rcp) {
  const float j = __builtin_fmaf(-(float)dx, rcp((float)dr + 0x1p-60f), -1e-30f);
  return __builtin_bit_cast(uint32_t, j);
}

// One iteration with the rates r of the state (on return of the new state).
// The argument of max(x, y) is x if the difference x - y, or at a tie that of
// the rates, is positive: the sign of (x - y) + 2^-60 (rx - ry), as all are
// integers below 2^53.  J: lowered to the bits of each max's bound (lead_bits).
template <int S>
__device__ __forceinline__ void rate_iter(Chain<S, double>& h, double (&r)[S], uint32_t& J) {
  double B = 0, rB = 0;
  auto pick = [&](double x, double rx, double y, double ry, double& v, double& rv) {
    const double dx = x - y, dr = rx - ry;
    v = vmax(x, y);
    rv = __builtin_fma(dr, 0x1p-60, dx) > 0 ? rx : ry;
    const uint32_t b = lead_bits(dx, dr, [](float y) { return __builtin_amdgcn_rcpf(y); });
    J = b < J ? b : J;
  };
#pragma unroll
  for (int s = S - 1; s >= 0; --s) {
    if (s == S - 1) {
      B = h.f[s];
      rB = r[s];
    } else {
      pick(h.f[s], r[s], B + h.d[s], rB, B, rB);
    }
    if (s) {
      pick(B + h.a[s], rB, h.f[s - 1], r[s - 1], h.f[s], r[s]);
    } else {
      h.f[0] = B + h.a[0];
      r[0] = rB;
    }
  }
}

// Go on with a pipeline of the first list, q = 1, 2 in turn: q iterations find
// D; if all its components are equal the schedule has period q.  Otherwise the
// next q iterations say whether D repeats, and where it does q more follow the
// rates.  (A plain 16-stage iteration takes 0.12 us, one with rates 1 us.  On
// the random sweeps 9 in 10 of these pipelines end within 30 iterations; in a
// sweep of a million plans the slowest would take all of its 500-1100.)
template <int S>
__device__ __forceinline__ void cont_one(const EvalBufs& e, const double* tile) {
  Chain<S, double> h;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    h.f[s] = tile[64 * s];
    h.a[s] = tile[64 * (S + s)];
    h.d[s] = s < S - 1 ? tile[64 * (2 * S + s)] : 0;
  }
  const uint2 ls = *(const uint2*)&tile[64 * (3 * S - 1)];
  int left = (int)ls.x, skipped = 0, q = 1, budget = kContBudget;
  const uint32_t slot = ls.y;
  while (left >= 3 * q && budget > 0) {
    double o[S], D[S];
#pragma unroll
    for (int s = 0; s < S; ++s) o[s] = h.f[s];
    for (int i = 0; i < q; ++i) chain_iter<S, double, false>(h, h.a, 0, 0);
    left -= q;
    budget -= q;
    bool same = true;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      D[s] = h.f[s] - o[s];
      same = same & (D[s] == D[0]);
    }
    if (same) {
      const int k = left / q;
#pragma unroll
      for (int s = 0; s < S; ++s) h.f[s] += (double)k * D[0];
      left -= k * q;
      skipped += k * q;
    } else {
#pragma unroll
      for (int s = 0; s < S; ++s) o[s] = h.f[s];
      for (int i = 0; i < q; ++i) chain_iter<S, double, false>(h, h.a, 0, 0);
      left -= q;
      budget -= q;
      bool ok = true;
#pragma unroll
      for (int s = 0; s < S; ++s) ok = ok & (h.f[s] - o[s] == D[s]);
      if (ok) {
        double r[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          o[s] = h.f[s];
          r[s] = D[s];
        }
        uint32_t J = __float_as_uint(1e9f);
        for (int i = 0; i < q; ++i) rate_iter<S>(h, r, J);
        left -= q;
        budget -= q;
#pragma unroll
        for (int s = 0; s < S; ++s) ok = ok & (r[s] == D[s]) & (h.f[s] - o[s] == D[s]);
        if (ok) {
          // (the fp32 quotient, shortened by more than its error)
          const float bound = __uint_as_float(J) * 0.99999f;
          const int room = left / q, k = bound < (float)room ? (int)bound : room;
#pragma unroll
          for (int s = 0; s < S; ++s) h.f[s] += (double)k * D[s];
          left -= k * q;
          skipped += k * q;
        }
      }
    }
    q = 3 - q;
  }
#pragma unroll
  for (int s = 0; s < S; ++s) h.e[s] = tile[64 * (3 * S + s)];
  // out of budget: the second list, or the rest here if little is left or the list is full
  if (left >= 2 * kPowerMin && cont_push<S, 2>(e, h, left, slot)) {
    count_skipped(e, S, skipped);
    return;
  }
  for (; left > 0; --left) chain_iter<S, double, false>(h, h.a, 0, 0);
  // (M enters the end only where it is below S: never here)
  raise_time(e, slot, chain_end<S, double, false>(h, h.a, S));
  count_skipped(e, S, skipped);
}

// An entry of the second list to its end, on its lane.
template <int S>
__device__ __forceinline__ void cont_rest(const EvalBufs& e, const double* tile) {
  Chain<S, double> h;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    h.f[s] = tile[64 * s];
    h.a[s] = tile[64 * (S + s)];
    h.d[s] = s < S - 1 ? tile[64 * (2 * S + s)] : 0;
  }
  const uint2 ls = *(const uint2*)&tile[64 * (3 * S - 1)];
  int left = (int)ls.x, skipped = 0;
  chain_jump<S, double>(h, left, INT_MAX, skipped);
#pragma unroll
  for (int s = 0; s < S; ++s) h.e[s] = tile[64 * (3 * S + s)];
  raise_time(e, ls.y, chain_end<S, double, false>(h, h.a, S));   // (M enters only where it is below S)
  count_skipped(e, S, skipped);
}

// The parts of a list, by the block: entries and units (a tile of 64 entries,
// or one entry) up to the end of each part, most stages first; find() takes
// unit q of the whole list to its part.
template <int kList, uint32_t kPer>
struct ContIndex {
  static constexpr int kHalves = kList == 1 ? 2 : 1;
  static constexpr uint32_t kPerList = kList == 1 ? kContSubs : 1;
  static_assert(kMaxStages * kPerList <= 64 * kHalves, "a lane per part");
  uint32_t n[64 * kHalves], incl[64 * kHalves], entries;   // in LDS
  __device__ __forceinline__ void fill(const EvalBufs& e) {
    if (threadIdx.x < 64) {
      const uint32_t lane = threadIdx.x;
      uint32_t run = 0, sum = 0;
#pragma unroll
      for (int h = 0; h < kHalves; ++h) {
        const uint32_t x = 64 * h + lane, j = x / kPerList, sub = x % kPerList;
        const bool on = j < (uint32_t)kMaxStages && (kList == 2 || sub < e.cinfo[64 + j]);
        const uint32_t cap = on ? e.cinfo[(kList == 1 ? 16 : 48) + j] * 64u : 0;
        const uint32_t c = on ? e.ctr[kList == 1 ? cont1_ctr(j, sub) : cont2_ctr(j)] : 0;
        n[x] = c < cap ? c : cap;
        sum += n[x];
        uint32_t y = (n[x] + kPer - 1) / kPer;
#pragma unroll
        for (uint32_t o = 1; o < 64; o <<= 1) {
          const uint32_t z = __shfl_up(y, o);
          y += lane >= o ? z : 0;
        }
        incl[x] = run + y;
        run = __shfl(run + y, 63);
      }
#pragma unroll
      for (uint32_t o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
      entries = sum;
    }
    __syncthreads();
  }
  // S: stage count; at: the unit in its part; count: the part's entries; base: its first 2 KiB unit
  __device__ __forceinline__ bool find(const EvalBufs& e, uint32_t q, uint32_t& S, uint32_t& at, uint32_t& count,
                                       uint32_t& base) const {
    const uint32_t lane = threadIdx.x & 63u;
    for (int h = 0; h < kHalves; ++h) {
      const uint64_t past = __ballot(incl[64 * h + lane] > q);
      if (past) {
        const uint32_t x = 64 * h + (uint32_t)__builtin_ctzll(past), j = x / kPerList, sub = x % kPerList;
        count = __builtin_amdgcn_readfirstlane(n[x]);
        at = q - (__builtin_amdgcn_readfirstlane(incl[x]) - (count + kPer - 1) / kPer);
        S = kMaxStages - j;
        base = kList == 1 ? e.cinfo[j] + sub * e.cinfo[16 + j] * S : e.cinfo[32 + j];
        return true;
      }
    }
    return false;
  }
};

// The time of a plan whose G pipelines sit on adjacent lanes from `lead` on,
// all of them here: the first one stores the largest result of the finished
// ones (one store per plan; later passes raise it with atomicMax).  G is the
// same in the whole wavefront.
__device__ __forceinline__ void store_plan_time(const EvalBufs& e, uint32_t slot, uint32_t G, uint32_t lead, bool done,
                                                double T) {
  const uint32_t lane = threadIdx.x & 63u;
  const bool mine = done && T < kExact;
  double v = mine ? T : 0;
  for (uint32_t c = 1; c < G; ++c) {
    const double u = __shfl(v, (int)(lead + c));
    if (lane == lead) v = u > v ? u : v;
  }
  if (lane == lead && v > 0) e.out[slot >> 2] = (uint64_t)v;
  if (done && !mine) e.ovf[atomicAdd(&e.ctr[0], 1u)] = slot;
}

// What the G lanes of a plan-sorted plan (classes 0 .. G - 1 from `lead` on)
// share in their wavefront's LDS, a column of 64 entries per stage and one of
// counters per device type:
//  * placement: cnt[64 k + lane], the devices of type k (in units of the TP
//    degree) placed before the lane's next stage of that type.  Every lane
//    counts its own class, takes the sum of the classes before it as its
//    start, and then draws each stage's first device by an atomic add on its
//    own counter -- a few LDS accesses per stage, where counting over the
//    packed types takes some twenty operations per earlier class;
//  * links: every lane leaves its class's share of each stage's DP link;
//  * syncs: the lane of class c puts stages c, c + G, ... together and leaves
//    each stage's sync in the entry of class 0, for all lanes of the plan.
template <int S>
struct PlanLanes {
  uint32_t G, lane, lead;
  double* col;      // [64 s + lane]
  uint32_t* cnt;    // [64 k + lane]
  __device__ __forceinline__ PlanLanes(const Plan& p, double* xw, uint32_t* cw)
      : G(p.G), lane(threadIdx.x & 63u), lead((threadIdx.x & 63u) - p.c), col(xw), cnt(cw) {}
  __device__ __forceinline__ uint32_t& counter(const Plan& p, uint32_t s) {
    return cnt[((uint32_t)(p.tc >> (4 * s)) & 15) * 64 + lane];
  }
  __device__ __forceinline__ void start(const Tab& t, const Plan& p) {
    for (uint32_t k = 0; k < t.K; ++k) cnt[64 * k + lane] = 0;
    if (G == 1) return;
#pragma unroll
    for (uint32_t s = 0; s < (uint32_t)S; ++s) draw(&counter(p, s), p.rc);
    wave_sync_lds();
    for (uint32_t k = 0; k < t.K; ++k) {
      uint32_t before = 0;
      for (uint32_t c = 0; c + 1 < G; ++c) {
        const uint32_t n = cnt[64 * k + lead + c];
        before += c < p.c ? n : 0;
      }
      wave_sync_lds();
      cnt[64 * k + lane] = before;
    }
  }
  __device__ __forceinline__ uint32_t first_device(const Plan& p, uint32_t k) {
    return draw(&cnt[64 * k + lane], p.rc) * p.tp;
  }
  __device__ __forceinline__ void placed(uint32_t s, const StagePlace& sp) {
    reinterpret_cast<uint2*>(col)[64 * s + lane] =
        make_uint2(sp.bq_nic > sp.ti.bq_pcie ? sp.bq_nic : sp.ti.bq_pcie,
                   sp.k << 24 | (sp.nl == sp.nh ? sp.nl : kNoNode));
  }
  template <int kMode, bool kHier>
  __device__ __forceinline__ DpLink link(const Tab& t, const Hot<kMode>& h, const Plan& p, uint32_t s, HierShape& hs) {
    hs.ok = false;
    if (kHier && t.ccl_hier) return stage_link<kMode>(t, h, p, s, hs);
    return exchanged_link(h, G, reinterpret_cast<const uint2*>(col) + 64 * s + lead);
  }
  // the stages' syncs into col[64 s + lead]; ns(s): the stage's layers
  template <int kMode, bool kHier, typename Layers>
  __device__ __forceinline__ void syncs(const Tab& t, const Hot<kMode>& h, const Plan& p, Layers ns) {
    wave_sync_lds();
    const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> p.epl);
    const Params par(h.size(), p.tpl, p.epl);
    for (uint32_t s = p.c; s < (uint32_t)S; s += G) {
      double x = 0;
      if (p.psum > 1) {
        HierShape hs;
        const DpLink l = link<kMode, kHier>(t, h, p, s, hs);
        const uint32_t n = ns(s);
        x = link_dp<kHier>(t, p, l, hs, rp, rpe, par.stage(n, s == 0, s == (uint32_t)S - 1), (double)n * par.expert);
      }
      col[64 * s + lead] = x;
    }
    wave_sync_lds();
  }
  // the same for an overlapped plan: one layer's bucket sync per stage, the
  // embedding's and the head's in columns S and S + 1; then every lane walks
  // its own buckets' readiness against them and leaves the tail of stage s in
  // its own entry
  template <int kMode>
  __device__ __forceinline__ void overlap(const Tab& t, const Hot<kMode>& h, const Plan& p) {
    wave_sync_lds();
    const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> p.epl);
    for (uint32_t s = p.c; s < (uint32_t)S; s += G) {
      OvlSyncs y = {0, 0, 0};
      if (p.psum > 1) {
        HierShape hs;
        const DpLink l = link<kMode, true>(t, h, p, s, hs);
        y = overlap_syncs(t, h, p, s, l, hs, rp, rpe);
      }
      col[64 * s + lead] = y.dl;
      if (s == 0) col[64 * S + lead] = y.demb;
      if (s == (uint32_t)S - 1) col[64 * (S + 1) + lead] = y.dhead;
    }
    wave_sync_lds();
    const double demb = col[64 * S + lead], dhead = col[64 * (S + 1) + lead];
    uint32_t lo = 0;
    for (uint32_t s = 0; s < (uint32_t)S; ++s) {
      const uint32_t hi = cut_at(p, s);
      const double x = overlap_walk<kMode, double>(t, h, p, s, lo, hi, (uint32_t)(p.tc >> (4 * s)) & 15,
                                                   OvlSyncs{col[64 * s + lead], demb, dhead});
      wave_sync_lds();   // every lane of the plan has read stage s's bucket
      col[64 * s + lane] = x;
      lo = hi;
    }
  }
};

// One pipeline of the first pass (kKind 0) or of the variant pass (overlapped
// sync, zero-bubble order; with two-level collectives, kHier, also plain
// ones): setup, syncs, chain, and the recurrence with the first pass's budget.
// xw, cw: the wavefront's columns and counters (shared layout).
template <int S, int kMode, bool kHet, int kKind, bool kHier>
__device__ __forceinline__ void eval_one(const Tab& t, const Hot<kMode>& h, const EvalBufs& e, uint32_t slot,
                                         double* xw, uint32_t* cw) {
  constexpr bool kZb = kKind == 2, kOvl = kKind == 1;
  typename std::conditional<kZb, ZbSink<S>, RegSink<S>>::type r;
  const Plan p = load_plan<kHet>(e.packed, e.pcut, slot);
  const uint32_t M = class_mb(p), G = p.G, lead = (threadIdx.x & 63u) - p.c;
  Chain<S, double> ch;
  {
    double x[S];
    if constexpr (!kHet) {
      PlanLanes<S> pl(p, xw, cw);
      pl.start(t, p);
      class_setup<kMode, false>(t, h, p, r, [&](uint32_t, uint32_t k) { return pl.first_device(p, k); },
                                [&](uint32_t s, const StagePlace& sp) { pl.placed(s, sp); });
      if constexpr (kOvl) pl.template overlap<kMode>(t, h, p);
      else
        pl.template syncs<kMode, kHier>(t, h, p,
                                        [&](uint32_t s) { return cut_at(p, s) - (s ? cut_at(p, s - 1) : 0); });
#pragma unroll
      for (int s = 0; s < S; ++s) x[s] = xw[s * 64 + (kOvl ? pl.lane : lead)];
      wave_sync_lds();
    } else {
      uint32_t* const cnt = cw + (threadIdx.x & 63u);
      class_starts(t, p, p.c, [&](uint32_t c, uint32_t k, uint32_t first) {
        if (c == p.c) cnt[64 * k] = first;
      });
      const uint32_t nd = p.rc * p.tp;
      class_setup<kMode, true>(t, h, p, r, [&](uint32_t, uint32_t k) { return draw(&cnt[64 * k], nd); },
                               [](uint32_t, const StagePlace&) {});
      // per-class layout: the syncs the plan pass stored for this pipeline's stages
      const double* drow = e.hdp + (size_t)slot * kMaxStages;
#pragma unroll
      for (int s = 0; s < S; ++s) x[s] = drow[s];
    }
    if constexpr (kZb) reduce_chain<S, double, true>(r.f, r.bi, r.w, r.c, x, M, ch);
    else reduce_chain<S, double, false>(r.f, r.b, r.b, r.c, x, M, ch);
  }
  int left = (int)M - S, skipped = 0, budget = first_budget(S);
  if constexpr (kZb) {   // from iteration S - 1 on every stage runs its W
    int i = 0;
    for (; i < left && i < S - 1; ++i) chain_iter<S, double, true>(ch, r.w, i, 0);
    left -= i;
  }
  bool done = true;
  while (true) {
    chain_jump<S, double>(ch, left, budget, skipped);
    if (left <= 0) break;
    if (left >= kPowerMin && cont_push<S, 1>(e, ch, left, slot)) {
      done = false;
      break;
    }
    budget = INT_MAX;
  }
  double T = 0;
  if (done) {
    if constexpr (kZb) T = chain_end<S, double, true>(ch, r.w, M);
    else T = chain_end<S, double, false>(ch, ch.a, M);
    count_skipped(e, S, skipped);
  }
  if constexpr (kHet) {
    if (done) raise_time(e, slot, T);
  } else {
    store_plan_time(e, slot, G, lead, done, T);
  }
}

// ---------------------------------------------------------------- interleaved 1F1B
// Schedule (Narayanan et al. 2021): device s of an S-device pipeline holds
// chunks j = 0..v-1 of the model, virtual stage j S + s.  It runs
// W_s = 2 (S-1-s) + (v-1) S warm-up forwards, then (forward, backward) pairs,
// then its last W_s backwards; its k-th forward runs chunk (k mod S v) / S,
// its k-th backward chunk v-1 - (k mod S v) / S, both on micro-batch
// (k div S v) S + k mod S.  With M a multiple of S and M >= 2 S the devices
// advance in lockstep: at step t device s runs forward k = t - s, then
// backward k = t - s - W_s (each where 0 <= k < M v), and each op's input is
// an op of a neighbouring device at step t - 1: for a forward on device
// s > 0 the forward of device s - 1, on device 0 (chunk j > 0) the forward
// of device S - 1 across the wrap hop; for a backward on device s < S - 1
// the backward of device s + 1, on device S - 1 (chunk j < v - 1) the
// backward of device 0 across the wrap hop; the last virtual stage's
// backward takes its own forward of the same step.  Steps run
// t = 0 .. M v + W_0 - 1.  Within a trip of S v steps starting at a multiple
// of S v, the chunk of every op is a compile-time constant, so every
// duration is a register.

// Per virtual stage forward and backward time (f, b), hops between devices
// (c[s]: s -> s + 1, c[S - 1]: the wrap hop S - 1 -> 0).
template <int S, int v, int kMode, typename V, typename First, typename Placed>
__device__ __forceinline__ void il_setup(const Tab& t, const Hot<kMode>& h, const Plan& p, V (&f)[S * v],
                                         V (&b)[S * v], V (&c)[S], First first_device, Placed placed) {
  constexpr int NV = S * v;
  const double act = h.size().act[p.mi];
  StagePlace first = {}, prev = {};
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t k = (uint32_t)(p.tc >> (4 * s)) & 15;
    const StagePlace sp = stage_place<kMode>(t, h, p, k, first_device((uint32_t)s, k));
    placed((uint32_t)s, sp);
#pragma unroll
    for (int j = 0; j < v; ++j) {
      const int vs = j * S + s;
      const uint32_t lo = vs ? cut_at(p, vs - 1) : 0, hi = cut_at(p, vs);
      double fc, bc, wc;
      stage_cost<kMode, false>(t, h, p, sp, act, lo, hi, vs == 0, vs == NV - 1, fc, bc, wc);
      f[vs] = (V)fc;
      b[vs] = (V)bc;
    }
    if (s > 0) c[s - 1] = (V)hop_ps(t, p, prev, sp, act, true);
    if (s == 0) first = sp;
    if (s == S - 1)   // the wrap hop: device S - 1 sends to device 0, placed before it
      c[S - 1] = (V)hop_ps(t, p, first, sp, act, false);
    prev = sp;
  }
}
template <int S, int v, int kMode, typename V>
__device__ __forceinline__ void il_setup_own(const Tab& t, const Hot<kMode>& h, const Plan& p, V (&f)[S * v],
                                             V (&b)[S * v], V (&c)[S]) {
  il_setup<S, v, kMode, V>(t, h, p, f, b, c, [&](uint32_t s, uint32_t k) { return dev_before_own<false>(p, s, k); },
                           [](uint32_t, const StagePlace&) {});
}

// One trip of S v steps from a step that is a multiple of S v.  n = M v is
// such a multiple too and at least 2 S v, and W_0 <= 2 S v, so which ops of
// a trip exist is known at compile time: kOff is the trip's first step in a
// warm-up trip (kPhase < 0), its first step minus n in a cool-down trip
// (kPhase > 0), and in a steady trip every device runs a forward and a
// backward at every step.  Against one trip with each op predicated at run
// time for both ends: k_all over 2M plans 1149 -> 658 us.
// F[s], B[s]: end of device s's latest forward / backward; busy[s]: of its
// latest op.
template <int S, int v, typename V, int kPhase, int kOff>
__device__ __forceinline__ void il_trip(const V (&f)[S * v], const V (&b)[S * v], const V (&c)[S], V (&F)[S],
                                        V (&B)[S], V (&busy)[S]) {
  constexpr int NV = S * v;
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    V nF[S], nB[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int W = 2 * (S - 1 - s) + (v - 1) * S;
      const int jf = ((u - s) % NV + NV) % NV / S, vf = jf * S + s;
      const int jb = v - 1 - ((u - s - W) % NV + NV) % NV / S, vb = jb * S + s;
      const int kf = kOff + u - s, kb = kf - W;   // op numbers (in cool-down: minus n)
      const bool has_f = kPhase < 0 ? kf >= 0 : kPhase == 0 || kf < 0;
      const bool has_b = kPhase < 0 ? kb >= 0 : kPhase == 0 || kb < 0;
      nF[s] = F[s];
      nB[s] = B[s];
      if (has_f) {
        const V rf = s > 0 ? F[s - 1] + c[s - 1] : jf > 0 ? F[S - 1] + c[S - 1] : (V)0;
        busy[s] = nF[s] = vmax(busy[s], rf) + f[vf];
      }
      if (has_b) {
        const V rb = vb == NV - 1 ? nF[s] : s < S - 1 ? B[s + 1] + c[s] : B[0] + c[S - 1];
        busy[s] = nB[s] = vmax(busy[s], rb) + b[vb];
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      F[s] = nF[s];
      B[s] = nB[s];
    }
  }
}

// The whole schedule; busy[s] = end of device s's last op.  kJump: a trip
// in the steady part maps the state (F, B; busy = B there) to a max of
// (component + constant) terms, so once a steady trip advances every
// component by one constant lam the later steady trips do too, and they are
// taken in one step (the argument of the plain pipeline's shortcut).
template <int S, int v, typename V, bool kJump>
__device__ __forceinline__ void il_pipe(const V (&f)[S * v], const V (&b)[S * v], const V (&c)[S], uint32_t M,
                                        V (&busy)[S]) {
  constexpr int NV = S * v, W0 = 2 * (S - 1) + (v - 1) * S;
  static_assert(W0 <= 2 * NV, "at most two trips of warm-up and of cool-down");
  const int n = (int)M * v;   // (a multiple of NV, at least 2 NV)
  V F[S], B[S], pF[S], pB[S];
#pragma unroll
  for (int s = 0; s < S; ++s) F[s] = B[s] = busy[s] = 0;
  il_trip<S, v, V, -1, 0>(f, b, c, F, B, busy);
  if (W0 > NV) il_trip<S, v, V, -1, NV>(f, b, c, F, B, busy);
  bool first = true;
  for (int t0 = W0 > NV ? 2 * NV : NV; t0 < n; t0 += NV) {
    if (kJump) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        pF[s] = F[s];
        pB[s] = B[s];
      }
    }
    il_trip<S, v, V, 0, 0>(f, b, c, F, B, busy);
    if (kJump && !first) {
      const V lam = B[0] - pB[0];
      bool same = true;
#pragma unroll
      for (int s = 0; s < S; ++s) same = same && F[s] - pF[s] == lam && B[s] - pB[s] == lam;
      const int r = (n - (t0 + NV)) / NV;
      if (same && r > 0) {
        const V k = (V)r * lam;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          F[s] += k;
          B[s] += k;
          busy[s] += k;
        }
        t0 += r * NV;
      }
    }
    first = false;
  }
  il_trip<S, v, V, 1, 0>(f, b, c, F, B, busy);
  if (W0 > NV) il_trip<S, v, V, 1, NV>(f, b, c, F, B, busy);
}

// Layers on device s: the sum over its chunks.
template <int S, int v>
__device__ __forceinline__ uint32_t il_device_ns(const Plan& p, int s) {
  uint32_t ns = 0;
#pragma unroll
  for (int j = 0; j < v; ++j) {
    const int vs = j * S + s;
    ns += cut_at(p, vs) - (vs ? cut_at(p, vs - 1) : 0);
  }
  return ns;
}

// The iteration time of one interleaved pipeline: the latest device end
// plus that device's DP sync over the parameters of all its chunks.
template <int S, int v, int kMode, typename V>
__device__ __forceinline__ V il_tail(const Tab& t, const Hot<kMode>& h, const Plan& p, const V (&busy)[S]) {
  const double rp = 1.0 / (double)p.psum, rpe = 1.0 / (double)(p.psum >> p.epl);
  V T = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) T = vmax(T, busy[s] + (V)stage_dp(t, h, p, s, il_device_ns<S, v>(p, s), rp, rpe));
  return T;
}

template <int S, int v, int kMode, typename V, bool kJump>
__device__ __forceinline__ V il_time(const Tab& t, const Hot<kMode>& h, const Plan& p) {
  V f[S * v], b[S * v], c[S], busy[S];
  il_setup_own<S, v, kMode, V>(t, h, p, f, b, c);
  il_pipe<S, v, V, kJump>(f, b, c, class_mb(p), busy);
  return il_tail<S, v, kMode, V>(t, h, p, busy);
}

// One plan-sorted interleaved pipeline.
template <int S, int v, int kMode>
__device__ __forceinline__ void eval_il(const Tab& t, const Hot<kMode>& h, const EvalBufs& e, uint32_t slot,
                                        double* x, uint32_t* cw) {
  const uint32_t lane = threadIdx.x & 63u;
  double busy[S];
  uint32_t G, lead;
  {
    double f[S * v], b[S * v], c[S];
    uint32_t M;
    {
      const Plan p = load_plan<false>(e.packed, e.pcut, slot);
      G = p.G;
      lead = lane - p.c;
      PlanLanes<S> pl(p, x, cw);
      pl.start(t, p);
      il_setup<S, v, kMode, double>(t, h, p, f, b, c, [&](uint32_t, uint32_t k) { return pl.first_device(p, k); },
                                    [&](uint32_t s, const StagePlace& sp) { pl.placed(s, sp); });
      pl.template syncs<kMode, true>(t, h, p, [&](uint32_t s) { return il_device_ns<S, v>(p, (int)s); });
      M = class_mb(p);
    }
    il_pipe<S, v, double, true>(f, b, c, M, busy);
  }
  double T = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) T = vmax(T, busy[s] + x[s * 64 + lead]);
  wave_sync_lds();
  store_plan_time(e, slot, G, lead, true, T);
}

// Blocks of four waves share one LDS copy of the table image.
constexpr uint32_t kEvalThreads = 256;

// A wavefront's columns and counters (PlanLanes) after the table image.
struct WaveLds {
  double* col;
  uint32_t* cnt;
  __device__ __forceinline__ WaveLds(const Tab& t, uint4* lds, uint32_t image, uint32_t cols, uint32_t wave) {
    char* const p = (char*)lds + image + wave * wave_lds_bytes(cols, t.K);
    col = (double*)p;
    cnt = (uint32_t*)(p + cols * 64 * 8);
  }
};

// Words that an earlier kernel wrote and this one only reads at uniform
// indices: in the constant address space they are scalar loads.
__device__ __forceinline__ uint32_t fixed_word(const uint32_t* p, uint32_t i) {
  return ((const __attribute__((address_space(4))) uint32_t*)(uintptr_t)p)[i];
}

// The group of tile q, which is one of groups [g0, g0 + n) (q is uniform in the
// wavefront, so this is scalar code).
__device__ __forceinline__ uint32_t tile_group(const EvalBufs& e, uint32_t q, uint32_t g0, uint32_t n) {
  uint32_t g = g0;
  for (uint32_t j = 1; j < n; ++j) g += q >= fixed_word(e.tstart, g0 + j) ? 1u : 0u;
  return g;
}

// This lane's pipeline of tile q of group g: false if it has none.
template <bool kHet>
__device__ __forceinline__ bool tile_slot(const EvalBufs& e, uint32_t q, uint32_t g, uint32_t& slot) {
  const uint32_t lane = threadIdx.x & 63u, G = kHet ? 1 : kMaxClasses - g % kMaxClasses;
  const uint32_t per = kHet ? 64 : plans_per_tile(G), j = lane / G, r = (q - fixed_word(e.tstart, g)) * per + j;
  const uint32_t first = fixed_word(e.gstart, g);
  if (j >= per || r >= fixed_word(e.gstart, g + 1) - first) return false;
  const uint32_t x = e.order[first + r];
  slot = kHet ? x : x * kMaxClasses + (lane - j * G);
  return true;
}

// First pass over the four stage counts of group GRP, 1F1B plans.  One kernel
// per four stage counts keeps the register footprint, and so the occupancy, of
// small pipelines independent of the 16-stage code.  The grid is capped at a
// few times the blocks that fit at once (each block holds a copy of the table
// image); its waves take the group's tiles in a fixed stride, heaviest first.
// Bound by instruction issue.  Per 2M-plan chunk of the 512-device sweep the
// four took 805, 714, 269 and 148 us with the recurrence on the times, u64
// setup and 40 iterations of waiting, and take 593, 216, 268 and 91.
template <int GRP, int kMode, bool kHet>
__global__ void __launch_bounds__(kEvalThreads) k_eval(const Tab* __restrict__ tp, EvalBufs e) {
  const Tab& t = *tp;
  constexpr int kTop = kMaxStages - 4 * GRP;   // stage counts kTop-3 .. kTop
  constexpr uint32_t g0 = 16 * GRP;
  extern __shared__ uint4 lds[];
  const uint32_t lo = fixed_word(e.tstart, g0), hi = fixed_word(e.tstart, g0 + 16);
  if (lo + blockIdx.x * (kEvalThreads / 64) >= hi) return;   // the whole block, before any barrier
  fill_lds<kMode>(t, lds);
  const Hot<kMode> h(t, lds);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const WaveLds w(t, lds, kMode < 2 ? t.lds_bytes : 0, kHet ? 0 : plan_cols(GRP, false), wave);
  for (uint32_t q = lo + blockIdx.x * (kEvalThreads / 64) + wave; q < hi; q += gridDim.x * (kEvalThreads / 64)) {
    const uint32_t g = tile_group(e, q, g0, 16), S = kTop - (g - g0) / kMaxClasses;
    uint32_t slot;
    if (!tile_slot<kHet>(e, q, g, slot)) continue;
    if (S == kTop) eval_one<kTop, kMode, kHet, 0, false>(t, h, e, slot, w.col, w.cnt);
    else if (S == kTop - 1) eval_one<kTop - 1, kMode, kHet, 0, false>(t, h, e, slot, w.col, w.cnt);
    else if (S == kTop - 2) eval_one<kTop - 2, kMode, kHet, 0, false>(t, h, e, slot, w.col, w.cnt);
    else eval_one<kTop - 3, kMode, kHet, 0, false>(t, h, e, slot, w.col, w.cnt);
  }
}

// Plans of every kind and stage count in one kernel: the overlap, zero-bubble
// and interleaved ones of every call, and with two-level collectives (whose
// sync code k_eval lacks) or in a small call also the plain ones.  One launch,
// where one per kind and stage-count group costs 4-5 us each even if it has
// nothing to do.  The price is occupancy: the whole kernel takes 256 registers,
// two wavefronts per SIMD for every kind and stage count, where compiled apart
// the kinds of up to four stages would take 167 and those of five to eight
// 187-209 (117-153 without the two-level collectives: three and four
// wavefronts), and it keeps a few registers in private memory.
// Bound by instruction issue and the chains' latency at that occupancy: the
// two thirds of 2.5M plans that overlap or run the zero-bubble order take 553
// us, where kernels fed with tiles a third full took 2460; 2^20 overlapped plans
// of at most four stages 308 us in all, and 787 with kernels of their own.
template <int S, int kMode>
__device__ __forceinline__ void eval_kind(const Tab& t, const Hot<kMode>& h, const EvalBufs& e, uint32_t kind,
                                          uint32_t slot, const WaveLds& w) {
  if (kind == 2) eval_one<S, kMode, false, 2, true>(t, h, e, slot, w.col, w.cnt);
  else if (kind == 1) eval_one<S, kMode, false, 1, true>(t, h, e, slot, w.col, w.cnt);
  else eval_one<S, kMode, false, 0, true>(t, h, e, slot, w.col, w.cnt);
}
template <int kMode>
__global__ void __launch_bounds__(kEvalThreads, 2) k_all(const Tab* __restrict__ tp, EvalBufs e, uint32_t plain) {
  const Tab& t = *tp;
  const uint32_t lo = plain ? 0 : fixed_word(e.tstart, kMaxStages * kMaxClasses), hi = fixed_word(e.tstart, kGroups);
  if (lo + blockIdx.x * (kEvalThreads / 64) >= hi) return;   // the whole block, before any barrier
  extern __shared__ uint4 lds[];
  fill_lds<kMode>(t, lds);
  const Hot<kMode> h(t, lds);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const WaveLds w(t, lds, kMode < 2 ? t.lds_bytes : 0, plan_cols(0, true), wave);
  for (uint32_t q = lo + blockIdx.x * (kEvalThreads / 64) + wave; q < hi; q += gridDim.x * (kEvalThreads / 64)) {
    uint32_t g = 0;   // the last group that starts at or before tile q
    for (uint32_t step = 128; step > 0; step >>= 1)
      if (g + step < kGroups && fixed_word(e.tstart, g + step) <= q) g += step;
    uint32_t slot;
    if (!tile_slot<false>(e, q, g, slot)) continue;
    if (g >= kPlainGroups) {
      switch ((g - kPlainGroups) / kMaxClasses) {
#define X(S_, V_)                                        \
  case il_shape(S_, V_):                                 \
    eval_il<S_, V_, kMode>(t, h, e, slot, w.col, w.cnt); \
    break;
        HETSIM_IL_SHAPES(X)
#undef X
        default: break;
      }
    } else {
      const uint32_t kind = g / (kMaxStages * kMaxClasses);
      switch (kMaxStages - g / kMaxClasses % kMaxStages) {
#define X(S_)                                        \
  case S_:                                           \
    eval_kind<S_, kMode>(t, h, e, kind, slot, w);    \
    break;
        X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#undef X
        default: break;
      }
    }
  }
}

// Pipelines whose fp64 time reached 2^53 ps, again in u64 (exact below 2^64).
// zb: the zero-bubble order, W[s] each stage's weight-gradient pass.
template <int S>
__device__ __forceinline__ uint64_t redo_one(const StageRec& R, const uint64_t (&W)[kMaxStages], bool zb,
                                             uint32_t M) {
  uint64_t f[S], b[S], w[S], c[S], x[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    f[s] = R[s][0];
    w[s] = zb ? W[s] : 0;
    b[s] = R[s][1] - w[s];
    c[s] = R[s][2];
    x[s] = R[s][3];
  }
  // the zero-bubble chain with w = 0 is the plain one; the periodic shortcut
  // holds in any exact arithmetic
  Chain<S, uint64_t> h;
  int skipped;
  reduce_chain<S, uint64_t, true>(f, b, w, c, x, M, h);
  return chain_time<S, uint64_t, true>(h, w, M, skipped);
}

template <bool kHet>
__global__ void __launch_bounds__(64) k_redo_u64(Tab t, EvalBufs e) {
  const uint32_t n = e.ctr[0];
  for (uint32_t j = blockIdx.x * 64u + threadIdx.x; j < n; j += gridDim.x * 64u) {
    const uint32_t slot = e.ovf[j];
    const Plan p = load_plan<kHet>(e.packed, e.pcut, slot);
    const uint32_t S = p.S, M = class_mb(p);
    const Hot<2> h(t, nullptr);
    if (!kHet && p.v > 1) {
      uint64_t r = 0;
      switch (il_shape(S, p.v)) {
#define X(S_, V_)                                                    \
  case il_shape(S_, V_):                                             \
    r = il_time<S_, V_, 2, uint64_t, true>(t, h, p);                 \
    break;
        HETSIM_IL_SHAPES(X)
#undef X
        default: break;
      }
      atomicMax((unsigned long long*)&e.out[slot >> 2], (unsigned long long)r);
      continue;
    }
    StageRec R;
    uint64_t W[kMaxStages];
    const bool w = !kHet && p.zb;
    class_records<2, kHet>(t, h, p, kHet ? cut_rows(e.pcut, slot >> 2) : nullptr, R, W);
    uint64_t r;
    switch (S) {
      case 1: r = redo_one<1>(R, W, w, M); break;
      case 2: r = redo_one<2>(R, W, w, M); break;
      case 3: r = redo_one<3>(R, W, w, M); break;
      case 4: r = redo_one<4>(R, W, w, M); break;
      case 5: r = redo_one<5>(R, W, w, M); break;
      case 6: r = redo_one<6>(R, W, w, M); break;
      case 7: r = redo_one<7>(R, W, w, M); break;
      case 8: r = redo_one<8>(R, W, w, M); break;
      case 9: r = redo_one<9>(R, W, w, M); break;
      case 10: r = redo_one<10>(R, W, w, M); break;
      case 11: r = redo_one<11>(R, W, w, M); break;
      case 12: r = redo_one<12>(R, W, w, M); break;
      case 13: r = redo_one<13>(R, W, w, M); break;
      case 14: r = redo_one<14>(R, W, w, M); break;
      case 15: r = redo_one<15>(R, W, w, M); break;
      default: r = redo_one<16>(R, W, w, M); break;
    }
    atomicMax((unsigned long long*)&e.out[slot >> 2], (unsigned long long)r);
  }
}
}  // namespace hetsim
