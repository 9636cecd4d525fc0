// internal.h -- context tables shared by the host builder and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <vector>

#include "hetsim.h"

namespace hetsim {

constexpr int kMaxTypes = 16;
constexpr int kMaxStages = 16;
constexpr int kMaxClasses = 4;
constexpr int kRecWords = 4;                    // per (plan, class, stage): fwd, bwd, hop, dp
// Order of a chunk.  Shared-layout plans are sorted by plan into groups of one
// kind of schedule, stage count S and class count G, and inside a group into
// micro-batch buckets (most micro-batches first); with the per-class layout
// the pipelines are sorted one by one (kind 0).  Groups: 64 per kind (more
// stages first, then more classes), then four per interleaved shape (S, v).
// A group's plans are dealt to tiles of one wavefront each: the G pipelines of
// a plan on G adjacent lanes, 64 / G plans per tile (21 when G = 3); the
// per-class layout has one pipeline per lane.  order[] holds the plans (or
// pipelines) group by group, gstart[g] the first of group g, tstart[g] its
// first tile.
constexpr int kKinds = 3;                       // 0: 1F1B; 1: overlapped gradient sync; 2: zero-bubble order
constexpr int kBucketsM = 32;
constexpr int kIlShapes = 14;                   // (S, v) of interleaved plans: S v <= 16
constexpr uint32_t kPlainGroups = kKinds * kMaxStages * kMaxClasses;
constexpr uint32_t kGroups = kPlainGroups + kIlShapes * kMaxClasses;
constexpr uint32_t kBuckets = kGroups * kBucketsM;
__host__ __device__ constexpr uint32_t plans_per_tile(uint32_t G) { return G == 3 ? 21 : 64 / G; }
// LDS of the passes over plan-sorted pipelines: per wavefront one column of 64
// doubles per stage (up to the kernel's largest stage count, and where
// overlapped plans run two more for the embedding's and the head's buckets),
// and one column of 64 counters per device type.
__host__ __device__ constexpr uint32_t plan_cols(int group, bool overlap) {
  return (uint32_t)(kMaxStages - 4 * group) + (overlap ? 2u : 0u);
}
__host__ __device__ constexpr uint32_t wave_lds_bytes(uint32_t cols, uint32_t types) {
  return cols * 64 * 8 + types * 64 * 4;
}
__host__ __device__ constexpr uint32_t block_lds_bytes(uint32_t cols, uint32_t types) {
  return 4 * wave_lds_bytes(cols, types);
}

// A validated plan packed into 80 contiguous bytes, so that the pipelines of
// one plan gather it with five 16-byte loads.
struct __attribute__((aligned(16))) PackedPlan {
  uint32_t hdr, psum, pad0, pad1;   // header; replicas summed over classes
  uint8_t cut[16];
  uint32_t cls[4];
  uint64_t types[4];
};

// With the per-class layout a plan takes one 128-byte line, gathered whole:
// {header, replicas, class header, 0}, the four class words, the stage types
// and the four classes' cut rows, as eight 16-byte words.
constexpr uint32_t kHetWords = 8;

// Per-device-type fields a kernel reads together (32 bytes, two loads).
struct TypeInfo {
  uint32_t node_off, dev_off;     // first global node / device of the pool
  uint32_t dpl;                   // log2 devices per node
  uint32_t bq_pcie;               // PCIe ps/byte in 2^-16 units, 0 = absent
  double a_intra;                 // intra-node message latency (ps; integers below 2^43)
  double a_side;                  // one end of an inter-node path: two PCIe trips + NIC
};

// Device speed of a pool (TFLOP/s, GB/s of HBM) and the reciprocals rounded to
// nearest (for exact ceilings): the gradient weighting of classes with
// different micro-batch sizes.
struct SpeedInfo {
  uint32_t tflops, hbm, pad0, pad1;
  double rtflops, rhbm;
};

// Quantities by TP degree, EP degree and micro-batch size (log2 or index), in
// fp64: parameters of one layer (non-expert, expert), the embedding and the
// head on one TP rank, and the bytes of one micro-batch activation.
struct SizeInfo {
  double layer[4], embed[4], head[4], expert[4][4], act[4];
};

// The tables of the per-pipeline setup form one byte image in device memory
// that the evaluation kernels copy into LDS, where lanes gather from it at
// LDS rather than vector-cache rates.  Times are whole numbers in fp64.
// Sections, each 16-byte aligned:
//   TypeInfo [K]; SizeInfo; SpeedInfo [K]; {forward, backward} layer prefix sums
//   [K][4 log2 TP][n_mbs][nep][L+1] (nep = 4 EP slots for MoE models, 1 for
//   dense ones), or, when every layer costs the same (dense models), one
//   {forward, backward} layer cost [K][4][n_mbs] (uniform_layers);
//   {fwd, bwd} embedding [K][n_mbs]; {fwd, bwd} head
//   [K][4][n_mbs]; all-to-all bytes prefix [4][n_mbs][L+1] (MoE only);
//   range-max rows of the node fabric rates [lvl_node][N]; range-max rows
//   of the device NIC rates [lvl_dev][D] (last, the largest).
// mode 0: the whole image fits the LDS budget; 1: all but the device rows
// fit; 2: nothing is copied and every table is read from device memory.
constexpr uint32_t kLdsBudget = 64 * 1024;

// What the plan check gathers by per-lane indices (k_prep keeps a copy in LDS:
// a gather from the kernel argument block goes to host memory).
struct CheckTab {
  uint32_t type_ok[4];            // [log2 TP] bit k: type k exists and TP 2^j divides its node size
  uint32_t mbs[4];
  uint64_t par_layer[4];          // non-expert parameters of one layer on one TP rank, by log2 TP
  uint64_t par_expert[4][4];      // expert parameters of one layer per rank [log2 TP][log2 EP]
  uint64_t par_embed[4], par_head[4];
  uint64_t act_layer[4][4];       // bytes one layer stores for backward per micro-batch [log2 TP][mbs index]
  uint64_t mem_cap[kMaxTypes];    // device memory of type k, bytes
};

// Everything a kernel needs about one (model, cluster) pair.  Scalars travel
// by value in the kernel argument block; tables live in device memory.
struct Tab : CheckTab {
  uint32_t L, K, E, n_mbs, gbs;
  uint32_t tp_ok;                 // bit j: TP 2^j divides heads, kv heads and MLP widths
  uint32_t ep_ok;                 // bit j: EP 2^j allowed (dense models: EP 1 only)
  uint32_t D, N;                  // total devices, total nodes
  uint32_t lvl_dev, lvl_node;     // levels of the range-max tables
  uint32_t dpn_log2[kMaxTypes];
  uint32_t cap[kMaxTypes];        // devices per pool
  uint32_t dev_off[kMaxTypes];    // first global device of pool k
  uint32_t node_off[kMaxTypes];   // first global node of pool k
  uint32_t bq_pcie[kMaxTypes];    // PCIe ps/byte in 2^-16 units, 0 = absent
  uint64_t a_intra[kMaxTypes];    // intra-node message latency
  uint64_t a_side[kMaxTypes];     // one end of an inter-node path: two PCIe trips + NIC
  uint32_t tflops[kMaxTypes];     // device speed of pool k (TFLOP/s, GB/s of HBM)
  uint32_t hbm[kMaxTypes];
  uint64_t act[4];                // bytes of one micro-batch activation per mbs index
  uint64_t grad_bytes, param_bytes;
  uint32_t mem_check;             // 1: device memory capacities given; plans must fit them
  uint32_t rail_only;             // 1: rail-only inter-node network (cross-rail hops forwarded in a node)
  uint32_t ccl_tree;              // 1: all-reduces take the faster of ring and tree
  uint32_t contention;            // 1: a stage's concurrent segment syncs share its links
  uint32_t ccl_hier;              // 1: whole-node DP groups may take the two-level all-reduce
  uint64_t opt_bytes;             // optimizer-state bytes per parameter
  uint32_t nep;                   // EP slots of the prefix tables
  uint32_t uniform_layers;        // 1: the layer table holds one layer's cost per row
  uint32_t o_size, o_speed, o_pfb, o_emb, o_head, o_pa, o_rmi, o_rmn;   // section byte offsets (TypeInfo at 0)
  uint32_t img_bytes;             // whole image
  uint32_t lds_bytes;             // prefix copied to LDS: img_bytes, o_rmn or 0 by mode
  uint32_t mode;
  const void* img;                // the image in device memory (16-byte aligned)
  uint32_t grid_eval[4];          // blocks of each first-pass kernel that fit the device at once
  uint32_t grid_all;              // blocks of k_all that fit the device at once
  uint32_t grid_cont;             // blocks of the continuation kernels that fit the device at once
};

// Continuation lists.  A pipeline whose schedule is still aperiodic after the
// first pass's budget leaves its recurrence state -- 4 S words: F_s, a_s, d_s,
// e_s and the iterations left with the pipeline's slot -- in a list of its
// stage count, in tiles of 64 (word r of entry l of a tile at [64 r + l]), and
// k_cont goes on with full wavefronts of them; what is left after its budget
// moves on to a second list and k_power.  A pipeline that finds its list full
// goes on where it is.  Most wavefronts of the first pass offer something, and
// atomics on one address are served one by one (about 12 ns each, which alone
// was 80-100 us of a group's pass over a million plans): the first list of a
// stage count is cut into up to kContSubs lists, picked by the block, and
// every counter has a cache line of its own.
// cinfo, j = 16 - S: [j] the first list's first 2 KiB unit in the continuation
// buffer, [16 + j] the capacity of each of its [64 + j] parts in tiles (S
// units each); [32 + j] and [48 + j] place and capacity of the second list.
constexpr uint32_t kContUnit = 2048;            // bytes
constexpr uint32_t kContSubs = 8;
constexpr uint32_t kContWords = 80;
// Counters of a chunk, kCtrStep words apart: pipelines to redo in u64, those
// offered to the parts of the first and to the second continuation list of
// 16 - j stages; the per-class layout's plan-order counters (kPlanSortWords)
// follow them, then the redo list.
constexpr uint32_t kCtrStep = 32;
__host__ __device__ constexpr uint32_t cont1_ctr(uint32_t j, uint32_t sub) {
  return (1 + j * kContSubs + sub) * kCtrStep;
}
__host__ __device__ constexpr uint32_t cont2_ctr(uint32_t j) { return (1 + kMaxStages * kContSubs + j) * kCtrStep; }
constexpr uint32_t kEvalCounters = cont2_ctr(kMaxStages);
// Per-class layout: plans counting-sorted by (classes, total stages) before
// the plan-level sync pass -- counts [0, 256), cursors [256, 512), the
// number of valid plans at 512.
constexpr uint32_t kPlanBuckets = 256;
constexpr uint32_t kPlanSortWords = 2 * kPlanBuckets + 1;
// The skipped-work counter is spread over slots on separate cache lines so
// that the waves of a launch do not serialise on one address.
constexpr uint32_t kSkipSlots = 512, kSkipStride = 16;

// Device buffers of one evaluation pass over a chunk.
struct EvalBufs {
  const PackedPlan* packed;    // shared layout
  const uint4* pcut;           // per-class layout: kHetWords per plan; nullptr for the shared layout
  const double* hdp;           // per-class layout: the syncs of pipeline slot's stages at [16 slot, + 16)
  const uint32_t* order;       // plans (shared layout) or pipeline slots (per-class layout) by group
  const uint32_t* gstart;      // [kGroups + 1]
  const uint32_t* tstart;      // [kGroups + 1]
  const uint32_t* cinfo;       // [kContWords]
  uint64_t* out;
  uint32_t* ctr;
  uint32_t* ovf;               // pipelines whose fp64 time reached 2^53
  double* cont;                // the continuation lists
  unsigned long long* skipped_ops;   // optional: kSkipSlots counters, kSkipStride words apart
  const Tab* dtab;             // the context's Tab in device memory
};

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace of one chunk: packed plans, their order, bucket counts followed by
// the evaluation counters and the redo list (counts and counters cleared
// together), bucket cursors, group and tile starts, the bucket key of each
// plan (u16; of each pipeline with the per-class layout), the continuation
// lists, and with the per-class layout the pipeline metadata, the plan order
// of the sync pass, the plans' lines (in place of the packed plans) and the
// syncs each pipeline's stages wait for (16 u64 per pipeline slot, 512 bytes
// per plan).
constexpr uint32_t kCounters = kBuckets + kEvalCounters + kPlanSortWords;
struct Work {
  PackedPlan* packed;
  uint4* pcut;
  double* hdp;
  uint32_t *meta, *perm, *order, *hist, *ctr, *ovf, *cursor, *gstart, *tstart, *cinfo;
  uint16_t* keys;
  double* cont;
  uint32_t cont_units;         // size of cont in kContUnit
};
// Bytes of the continuation lists: about what k_scan would take for a random
// sweep's chunk (two to three pipelines per plan), at least one tile of every
// list.  Small calls get up to four times as much: over slow links up to a half
// of their pipelines stay aperiodic, and an overfull list keeps wavefronts to
// the end (60000 per-class plans over links a 16th as fast 602 us with
// kContPerPlan).
constexpr size_t cont_bytes(int64_t ch, size_t per_plan) {
  const size_t b = (size_t)ch * per_plan;
  return ((b > (1u << 20) ? b : (1u << 20)) + kContUnit - 1) / kContUnit * kContUnit;
}
constexpr size_t kContPerPlan = 224;
constexpr size_t kContSmall = (size_t)64 << 20;   // bytes below which a call's lists may exceed kContPerPlan
constexpr size_t cont_per_plan(int64_t ch) {
  const size_t n = (size_t)ch, most = kContSmall / n;
  return most <= kContPerPlan ? kContPerPlan : most < 4 * kContPerPlan ? most : 4 * kContPerPlan;
}
// Where the device has no room for that, the lists of a chunk get this instead:
// less in all than a call took before there were lists (168 B per plan in the
// shared layout, 744 in the per-class layout), at up to three times the time of
// a random sweep.
constexpr size_t kContPerPlanLow = 32;
struct Carver {   // running offset
  size_t off = 0;
  constexpr size_t take(size_t bytes) {
    const size_t r = off;
    off += align256(bytes);
    return r;
  }
};
struct WorkOffsets {
  size_t cont, pcut, hdp, meta, perm, packed, order, hist, cursor, gstart, tstart, cinfo, keys, total;
};
constexpr WorkOffsets work_offsets(int64_t ch, bool het, size_t cont) {
  const size_t n = (size_t)ch, np = het ? 4 * n : n, nh = het ? n : 0;
  Carver c;
  WorkOffsets o = {};
  o.cont = c.take(cont);
  o.pcut = c.take(nh * kHetWords * 16);
  o.hdp = c.take(nh * kMaxClasses * kMaxStages * 8);
  o.meta = c.take(nh * 16);
  o.perm = c.take(nh * 4);
  o.packed = c.take(het ? 0 : n * sizeof(PackedPlan));
  o.order = c.take(np * 4);
  o.hist = c.take(kCounters * 4 + n * 16);
  o.cursor = c.take(kBuckets * 4);
  o.gstart = c.take((kGroups + 1) * 4);
  o.tstart = c.take((kGroups + 1) * 4);
  o.cinfo = c.take(kContWords * 4);
  o.keys = c.take(np * 2);
  o.total = c.off;
  return o;
}
// (cont: bytes of the continuation lists, whole units)
constexpr size_t work_bytes(int64_t ch, bool het, size_t cont) { return work_offsets(ch, het, cont).total; }
inline Work carve(void* base, int64_t ch, bool het, size_t cont) {
  const WorkOffsets o = work_offsets(ch, het, cont);
  char* p = (char*)base;
  Work w;
  w.cont = (double*)(p + o.cont);
  w.cont_units = (uint32_t)(cont / kContUnit);
  w.pcut = het ? (uint4*)(p + o.pcut) : nullptr;
  w.hdp = het ? (double*)(p + o.hdp) : nullptr;
  w.meta = het ? (uint32_t*)(p + o.meta) : nullptr;
  w.perm = het ? (uint32_t*)(p + o.perm) : nullptr;
  w.packed = (PackedPlan*)(p + o.packed);
  w.order = (uint32_t*)(p + o.order);
  w.hist = (uint32_t*)(p + o.hist);
  w.ctr = w.hist + kBuckets;
  w.ovf = w.hist + kCounters;
  w.cursor = (uint32_t*)(p + o.cursor);
  w.gstart = (uint32_t*)(p + o.gstart);
  w.tstart = (uint32_t*)(p + o.tstart);
  w.cinfo = (uint32_t*)(p + o.cinfo);
  w.keys = (uint16_t*)(p + o.keys);
  return w;
}

// nbuf chunks' workspace from alloc (nullptr: no room); *cont: the bytes of each
// one's lists.
template <typename Alloc>
inline auto alloc_work(Alloc alloc, int nbuf, int64_t ch, bool het, size_t* cont) {
  for (const size_t per : {cont_per_plan(ch), kContPerPlanLow}) {
    *cont = cont_bytes(ch, per);
    if (auto p = alloc(nbuf * work_bytes(ch, het, *cont))) return p;
  }
  return decltype(alloc((size_t)0))();
}

// The allocation-free entry point's workspace, a static device array (one per
// GPU): one chunk of at most kNoAllocPlans plans in the shared layout or
// kNoAllocPlansHet in the per-class layout, with lists of at least kContPerPlan
// bytes per plan; they take what the chunk's other buffers leave.  A pipeline
// that finds its list full keeps its wavefront to the end: with 46 MiB, and a
// call whose lists would have less than 96 bytes per plan in two chunks, 262144
// plans took 390 us and take 255, and 240000 plans over links a 16th as fast
// took 1310 and take 380.
constexpr int64_t kNoAllocPlans = 1 << 18;
constexpr int64_t kNoAllocPlansHet = 1 << 16;
constexpr size_t larger(size_t a, size_t b) { return a > b ? a : b; }
constexpr size_t kNoAllocBytes = larger(work_bytes(kNoAllocPlans, false, cont_bytes(kNoAllocPlans, kContPerPlan)),
                                        work_bytes(kNoAllocPlansHet, true, cont_bytes(kNoAllocPlansHet, kContPerPlan)));
constexpr size_t noalloc_cont(int64_t n, bool het) {
  return (kNoAllocBytes - work_bytes(n, het, 0)) / kContUnit * kContUnit;
}
// Address of this device's copy of that array (the current device); 0 or a
// HIP error code.
int noalloc_scratch(int device, void** ptr);

// Host side: validate descriptors and build the tables (host copies).
struct HostTables {
  Tab tab;
  // pf, pb [K][4][n_mbs][4][L+1]; emb [K][n_mbs][2]; head [K][4][n_mbs][2]; pa [4][n_mbs][L+1]
  std::vector<uint64_t> pf, pb, emb, head, pa;
  std::vector<uint32_t> rm_nic, rm_intra;
  std::vector<TypeInfo> ty;
  std::vector<uint8_t> img;       // the device image built from the above
};

// Blocks of each evaluation kernel that fit the current device at once (they
// size the capped grids).  Returns a HIP error code.
int eval_grids(Tab* t);

// Returns 0 (SIM_OK), SIM_EINVAL or SIM_ERANGE.
int build_tables(const sim_model_desc* model, const sim_cluster_desc* cluster, HostTables* out);

}  // namespace hetsim
