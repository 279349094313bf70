// Internal declarations of the FMM library (host side).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <exception>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/fmm.h"

namespace fmm {

// Status carried through host code; converted to fmm_status at the ABI.
struct Error {
  fmm_status code;
  std::string msg;
};

void set_error(const std::string& msg);
void clear_error();

#define FMM_HIP(call)                                                      \
  do {                                                                     \
    hipError_t e_ = (call);                                                \
    if (e_ != hipSuccess)                                                  \
      throw ::fmm::Error{e_ == hipErrorOutOfMemory ? FMM_ENOMEM            \
                                                   : FMM_EDEVICE,          \
                         std::string(#call) + ": " + hipGetErrorString(e_)}; \
  } while (0)

// Device buffer owned by a plan.
struct DevBuf {
  void* ptr = nullptr;
  size_t bytes = 0;
};

// Part of a device block that is handed out in 256-byte aligned pieces: a
// plan is some dozens of small arrays, and each hipMalloc and hipFree takes
// about 10 us.
struct Arena {
  char* at = nullptr;
  size_t left = 0;
  // the next piece, or NULL when the block has no room for it
  void* take(size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    if (bytes > left) return nullptr;
    char* p = at;
    at += bytes;
    left -= bytes;
    return p;
  }
};

// Constant operator tables of one expansion order (values in double; the
// float path keeps a rounded copy).  Layouts are shared with the kernels in
// eval.hip and batch.hip through the index helpers of tables.h.
struct Tables {
  int p = -1;
  std::vector<double> host;  // all tables, concatenated
  void* dev64 = nullptr;     // device copy (double)
  void* dev32 = nullptr;     // device copy (float)
};

// Boxes whose final local one launch forms: box[g] (own[g]: add its own
// M2L sum) receives the translations of sources anc[g * gs + j] (-1: none),
// gs a power of two covering the most sources of any box.
struct FinList {
  int32_t* box = nullptr;
  int32_t* own = nullptr;
  int32_t* anc = nullptr;
  int gs = 1;
  int64_t n = 0;
};

// Centre and length scale of a box in one 32-byte record.
struct alignas(32) BoxGeo {
  double x, y, z, scale;
};

// Lanes of one M2L block (every wave of it), and how many of them hold an
// item: all, except in FP64 at p = 8, where 63 rows of 81 accumulators let
// four blocks of two waves share a CU's LDS (160 KB).
constexpr int kM2LBlock = 64;
constexpr int m2l_lanes(int p, bool fp64) { return fp64 && p == 8 ? 63 : kM2LBlock; }

// Near-field work items: item j covers direct pairs [kb[j], ke[j]) of target
// leaf leaf[j]; every target leaf has at least one.  out[j] < 0: the leaf's
// only item, written to the near field; otherwise the element offset of the
// item's partial sums (4 rows of the leaf's point count: potential, field x,
// y, z) in part.  The split leaves split_leaf[i] add the partials of their
// split_cnt[i] items from split_first[i] on, in item order.
struct NearItems {
  int32_t* leaf = nullptr;
  int32_t* kb = nullptr;
  int32_t* ke = nullptr;
  int64_t* out = nullptr;
  int32_t* split_leaf = nullptr;
  int32_t* split_first = nullptr;
  int32_t* split_cnt = nullptr;
  void* part = nullptr;  // one buffer of both directions (make_work)
  int64_t n = 0, n_split = 0, part_elems = 0;
  // items of leaves of the wide forms (near_form) come first, those of more
  // threads (256, 128, 64) before those of fewer
  int64_t n_wide256 = 0, n_wide = 0, n_wide64 = 0;
  // form of the remaining items in passes without a field (near_form)
  int rest_pot = 0;
};

// Interaction lists of one direction, CSR by target.  M2L work items: lane
// i covers pairs [item_begin[i], item_end[i]) of target item_tgt[i] (-1 for
// an idle lane); the items are packed into blocks of kM2LBlock lanes, the
// items of one target consecutive inside one block (item_first[t],
// item_cnt[t]).  Block b holds the target segments seg_ptr[b] ..
// seg_ptr[b+1]-1: segment g covers lanes [seg_lanes[g] & 255,
// seg_lanes[g] >> 8) of target seg_tgt[g].
struct ListSet {
  int32_t* m2l_ptr = nullptr;  // [nbox+1]
  int32_t* m2l_src = nullptr;  // [n_m2l]
  int32_t* p2p_ptr = nullptr;  // [nleaf+1]
  int32_t* p2p_src = nullptr;  // [n_p2p]
  int32_t* item_tgt = nullptr;    // [n_items]
  int32_t* item_begin = nullptr;  // [n_items]
  int32_t* item_end = nullptr;    // [n_items]
  int32_t* item_first = nullptr;  // [nbox]
  int32_t* item_cnt = nullptr;    // [nbox]
  int32_t* seg_ptr = nullptr;     // [n_blocks+1]
  int32_t* seg_tgt = nullptr;
  int32_t* seg_lanes = nullptr;
  // Final locals of the target side in two launches (FinList): fin[0] over
  // the leaves' parent boxes, each receiving its own M2L sum and the
  // translations of the M2L sums of all its ancestors with M2L pairs;
  // fin[1] over the leaves, each receiving its own M2L sum and the
  // translation of its parent's final local (when the parent has one).
  FinList fin[2];
  int64_t n_m2l = 0, n_p2p = 0, n_items = 0, n_blocks = 0;
  NearItems near;  // make_p2p_items
};

// Near-field work items (make_p2p_items): items wanted, shortest and longest
// item in interactions, and the number of target leaves that fill the chip.
constexpr int64_t kP2PItems = 16384, kP2PItemMin = 1 << 12, kP2PItemMax = 1 << 16;
constexpr int64_t kP2PLeaves = 8192;

// Per-evaluation device buffers (all but the M2L partial rows of the
// batched form): leaf-ordered source records, expansions, the near field,
// the adjoint's field and the 32-vector copies.
struct Workspace {
  void* src = nullptr;      // [n] {x, y, z, q} in leaf order
  void* C = nullptr;        // [nbox][K]   multipoles (normalised)
  void* D = nullptr;        // [nbox][K]   locals (normalised)
  void* near = nullptr;     // [4n] near field in leaf order: pot [n], field [n][3]
  void* field_t = nullptr;  // [n][3] field of the transposed pass (adjoint)
  // multi-vector workspace (FP32 plans with max_rhs > 1), vectors innermost
  void* bq = nullptr;    // [n][32]
  void* bC = nullptr;    // [nbox][K][32]
  void* bD = nullptr;    // [nbox][K][32]
  void* bpot = nullptr;  // [n][32]
  void* bfld = nullptr;  // [n][3][32]
  bool stages = true;    // record stage-timing events when the plan profiles
};

// Byte offsets of the workspace buffers inside one allocation, each
// aligned to 256 bytes, in the order of Workspace; `forward` is the size of
// the leading part one single-vector evaluation uses (src, C, D, near).
struct WorkspaceLayout {
  size_t off[10] = {0};
  size_t size[10] = {0};
  size_t forward = 0;
  size_t total = 0;
};
WorkspaceLayout workspace_layout(int64_t n, int64_t nbox, const fmm_params& prm, bool batched);
// Point the buffers of ws at base + offsets (the first `count` buffers).
void bind_workspace(Workspace& ws, char* base, const WorkspaceLayout& L, int count);

// One level step of the upward (M2M) or downward (L2L) pass: n boxes a[i]
// with b[i] = first child (M2M; the 2^s children are consecutive) or parent
// (L2L; -1 for a root).
struct Step {
  int32_t* a = nullptr;
  int32_t* b = nullptr;
  int64_t n = 0;
};

// One side of a plan: the charges (sources) or the evaluation points
// (targets).  A plan over one point set has one side that plays both
// roles; a plan with separate sources and targets (Sec. II.B) has the
// sources as side 0 and the targets as side 1, each with its own tree.
// Slots [pt0, pt0 + npt) and leaves [leaf0, leaf0 + nleaf) of the plan's
// concatenated arrays are the side's; its boxes are those of its trees.
struct Side {
  int64_t pt0 = 0, npt = 0;
  int64_t leaf0 = 0, nleaf = 0;
  std::vector<Step> m2m_steps;  // bottom-up, parents of one level per step
  std::vector<Step> l2l_steps;  // top-down, boxes of one level with a parent local
  Step l2l_sum;                 // every box whose local is formed (b unused)
};

}  // namespace fmm

struct fmm_plan {
  int device = 0;
  fmm_params prm{};
  int64_t n = 0;
  int L = 0, s = 0, nch = 0;
  int64_t nbox = 0, nleaf = 0;
  std::vector<int64_t> level_off;  // host, size L+2

  // tree (device)
  int32_t* perm = nullptr;        // [n]
  int32_t* leaf_start = nullptr;  // [nleaf+1]
  double* xs = nullptr;           // leaf-ordered positions [n] x3 (SoA)
  double* ys = nullptr;
  double* zs = nullptr;
  double* cx = nullptr;  // box centres [nbox] (SoA)
  double* cy = nullptr;
  double* cz = nullptr;
  double* radius = nullptr;  // [nbox]
  double* scale = nullptr;   // [nbox] length scale of the box's expansions
  fmm::BoxGeo* geo = nullptr;  // [nbox] cx, cy, cz, scale
  int32_t max_leaf_count = 0;
  // some two points coincide or cannot be told apart in the plan's precision
  // (set by the tree build)
  bool has_dup = true;
  // launch tiles (0: the default rule from max_leaf_count; set by
  // fmm_plan_autotune): P2P source groups, P2M/L2P leaves per wave
  int p2p_groups = 0;
  int leaves_per_wave = 0;
  // 1: one lane per M2L translation; 0: the shared form where it is built
  // (m2l_shared_built), else one lane
  int m2l_waves = 0;
  // 1: one lane per M2M / L2L translation; 0: shared by four waves from
  // order kChainShareMinOrder on
  int chain_waves = 0;
  // waves per block of the batched near field (1, 2, 4, 8; 0: by the
  // plan's largest leaf)
  int batch_p2p_waves = 0;
  // 1: the near field on the caller's stream after the far-field chain; 0:
  // on the plan's second stream beside it
  int near_stream = 0;
  int32_t* leaf_box = nullptr;  // [nleaf] global box id of each leaf
  int nsides = 1;               // 2: separate sources (side 0) and targets (side 1)
  fmm::Side side[2];
  int n_problems = 1;           // > 1: union of independent trees

  // lists (device): [0] forward, [1] transposed (every pair reversed; the
  // adjoint operator)
  fmm::ListSet lists[2];
  int64_t p2p_inter = 0;

  // evaluation workspace: one device allocation of workspace_bytes carved
  // into the buffers below (workspace_layout); empty for plans created with
  // FMM_PLAN_NO_WORKSPACE
  fmm::Workspace ws;
  size_t workspace_bytes = 0;
  unsigned flags = 0;  // fmm_plan_create_ex flags
  // batched M2L partial rows [n_items][K][32] (FP32 plans with max_rhs > 1);
  // sized by the lists, so held with them
  void* bpart = nullptr;
  // batched plans: leaf position of every input index (inverse of perm)
  int32_t* iperm = nullptr;
  const void* tables = nullptr;  // device operator tables for (p, precision)

  std::vector<fmm::DevBuf> bufs;
  fmm::Arena arena;  // small arrays (plans with a caller's allocator: none)
  fmm_plan* memory = nullptr;  // plan whose blocks this one's arrays are part of
  size_t device_bytes = 0;
  // device memory source of the plan (fmm_plan_create_ex), also used for
  // temporaries during the build; stream passed to the callbacks
  fmm_allocator allocator{nullptr, nullptr, nullptr};
  hipStream_t alloc_stream = nullptr;

  // second stream of the evaluation: the near field runs on it beside the
  // far-field chain (forked after P2M, joined before L2P; events without
  // timing; default priority)
  hipStream_t side_stream = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;

  // stage timing (fmm_plan_set_profiling)
  bool profiling = false;
  std::vector<hipEvent_t> ev_pool;               // free events
  std::vector<std::vector<hipEvent_t>> ev_rows;  // 2 FMM_NSTAGES per pass
};

// Captured evaluation (fmm_graph_create).
struct fmm_graph {
  int device = 0;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace fmm {

// Device memory for the plan (kept until fmm_plan_destroy), through the
// plan's allocator.
void* plan_alloc(fmm_plan* pl, size_t bytes);
void plan_free_all(fmm_plan* pl);
// Temporary device memory during the build, through the plan's allocator.
void* dev_alloc(fmm_plan* pl, size_t bytes);
void dev_free(fmm_plan* pl, void* p);
// Temporaries of one build step, released when it goes out of scope.  Taken
// in blocks, to save calls of hipMalloc and hipFree (one by one from a caller's
// allocator): the first of the bytes that the step expects to need, later ones
// each twice as large up to kStep (blocks of 64 MB and allocations of their own
// above 16 MB: plan of 2^20 points 19.0 -> 19.8 ms, destroyed 1.4 -> 1.9).  The
// largest plan that fits must not shrink for it: beyond kExpect nothing is taken
// in advance, requests above kOwn that do not fit the first block are
// allocations of their own (so that a later block leaves at most a quarter
// unused), and where the device has no room for a block the request alone is
// tried.
struct Scratch {
  static constexpr size_t kFirst = (size_t)4 << 20, kOwn = (size_t)256 << 20,
                          kStep = (size_t)1 << 30, kExpect = (size_t)1 << 30;
  fmm_plan* pl;
  std::vector<void*> ptrs;
  Arena arena;
  size_t block;  // size of the next block
  // (a multiple of a piece's 256 bytes, so that a request of up to a block fits)
  explicit Scratch(fmm_plan* p, size_t expect = 0)
      : pl(p), block((kFirst + (expect <= kExpect ? expect : 0) + 255) / 256 * 256) {}
  void* get(size_t bytes) {
    bytes = bytes ? bytes : 16;
    if (!pl->allocator.alloc) {
      if (void* p = arena.take(bytes)) return p;
      if (bytes <= (ptrs.empty() ? block : std::min(block, kOwn)))
        if (void* b = try_block()) {
          arena = Arena{(char*)b, block};
          block = std::min(2 * block, kStep);
          return arena.take(bytes);
        }
    }
    void* p = dev_alloc(pl, bytes);
    ptrs.push_back(p);
    return p;
  }
  // a block, or NULL where there is no room for it
  void* try_block() {
    try {
      void* b = dev_alloc(pl, block);
      ptrs.push_back(b);
      return b;
    } catch (const Error&) {
      block = kFirst;
      return nullptr;
    }
  }
  ~Scratch() {
    // the build's kernels may still read them: wait for the stream first
    if (!ptrs.empty()) (void)hipStreamSynchronize(pl->alloc_stream);
    for (void* p : ptrs) dev_free(pl, p);
  }
};

// Index arrays of a plan gathered on the host and sent in one copy: add()
// names the pointer to set, flush() allocates, copies (the host buffer is
// free again when it returns) and sets them.
struct Upload {
  std::vector<int32_t> host;
  std::vector<std::pair<int32_t**, size_t>> dst;
  void add(const std::vector<int32_t>& v, int32_t** p) {
    dst.emplace_back(p, host.size());
    host.insert(host.end(), v.begin(), v.end());
    host.resize((host.size() + 63) / 64 * 64);  // 256-byte aligned pieces
  }
  void flush(fmm_plan* pl, hipStream_t st) {
    int32_t* d = (int32_t*)plan_alloc(pl, sizeof(int32_t) * host.size());
    if (!host.empty()) {
      FMM_HIP(hipMemcpyAsync(d, host.data(), sizeof(int32_t) * host.size(), hipMemcpyHostToDevice,
                             st));
      FMM_HIP(hipStreamSynchronize(st));
    }
    for (auto& e : dst) *e.first = d + e.second;
    host.clear();
    dst.clear();
  }
};

// One tree inside a plan: depth, level offsets, first global box id and
// first global leaf.
struct TreeDesc {
  int L;
  std::vector<int64_t> level_off;
  int64_t box_base;
  int64_t leaf_base = 0;
};
// Leaf boxes and level steps of each side over its trees (api.cpp): side k
// takes trees[k] (a plan with one side passes one group).  M2M step h takes
// the parents h+1 levels above each tree's leaves; L2L step l takes level l
// of every tree at least that deep.  Boxes outside every M2L pair and
// without such an ancestor are left out (their expansions are never read,
// or are zero), except that every leaf gets its local.  Also, per list
// direction, the ancestors of every target-side leaf whose M2L sums reach it.
void make_steps(fmm_plan* pl, const std::vector<std::vector<TreeDesc>>& trees, hipStream_t st);
// Side whose charges a pass in direction dir (0: G-hat, 1: G-hat^T) reads,
// and side whose points it evaluates.
inline const Side& src_side(const fmm_plan* pl, int dir) {
  return pl->side[pl->nsides == 1 ? 0 : dir];
}
inline const Side& tgt_side(const fmm_plan* pl, int dir) {
  return pl->side[pl->nsides == 1 ? 0 : 1 - dir];
}
// Union of independent plans (multi.hip): every per-point, per-box and
// per-leaf array concatenated, indices shifted to global numbering.
// With lists = false the sub-plans carry trees only, and perm stays local
// to each sub-plan (input indices of its own point set).
void build_union(fmm_plan* U, const std::vector<const fmm_plan*>& subs, hipStream_t st,
                 bool lists = true);

// Tree build (tree.hip): fills perm, leaf_start, xs/ys/zs, centres, radii.
void build_tree(fmm_plan* pl, const double* pos, hipStream_t st);
// Lists (lists.hip): fills m2l_*, p2p_*, items, from the level march
// between the source tree src and the target tree tgt of the plan (the
// same tree for a plan over one point set).
void build_lists(fmm_plan* pl, const TreeDesc& src, const TreeDesc& tgt, hipStream_t st);
// Plan with the 32-vector form.
inline bool batched_plan(const fmm_plan* pl) {
  return pl->prm.precision == FMM_FP32 && pl->prm.max_rhs > 1 && pl->nsides == 1;
}
// Work distribution of both directions (lists.hip): M2L items, near-field items.
void make_work(fmm_plan* pl, hipStream_t st);
// Operator tables for order p (tables.cpp), cached per process/device.
const void* get_tables(int p, int precision, int device);
// Evaluation (pass.hip): dir 0 = G-hat, dir 1 = G-hat^T.
void evaluate(fmm_plan* pl, const Workspace& ws, int dir, const void* q, int nrhs, void* pot,
              void* field, hipStream_t st);
// Up to kBatchWidth FP32 charge vectors in one pass (batch.hip, compiled once
// per order; batch_near.hip).
constexpr int kBatchWidth = 32;
int batch_width();
void batch_gather(const fmm_plan* pl, const float* q, int R, float* qL, hipStream_t st);
void batch_near(const fmm_plan* pl, const ListSet& Ls, int R, const float* qL, float* potL,
                float* fldL, hipStream_t st);
void batch_scatter(const fmm_plan* pl, int R, const float* potL, const float* fldL, float* pot,
                   float* field, hipStream_t st);
template <int P>
void run_batch(fmm_plan* pl, const ListSet& Ls, const float* q, int R, float* pot, float* field,
               hipStream_t st);
// waves per block of the batched near field for this plan
int batch_p2p_waves(const fmm_plan* pl);
// Whether R vectors (1 <= R <= kBatchWidth) are taken one by one.
bool vectors_one_by_one(const fmm_plan* pl, int R);
// iperm of a batched plan from its perm (on st)
void make_iperm(fmm_plan* pl, hipStream_t st);
void evaluate_batch(fmm_plan* pl, int dir, const float* q, int R, float* pot, float* field,
                    hipStream_t st);
// Adjoint combine: grad_x = -(g * field_fwd + q * field_t) (pass.hip).
void adjoint_combine(fmm_plan* pl, const void* q, const void* g, const void* field_fwd,
                     const void* field_t, void* grad_x, hipStream_t st);

// Direct summation (direct.hip).
void direct_sum(int64_t n, const double* pos, const void* q, int precision,
                const int64_t* targets, int64_t nt, void* pot, void* field,
                hipStream_t st);
// Launch tiles in effect (pass.hip): P2P source groups G (1, 2, 4; G > 1
// needs max_leaf_count <= 64 / G) and P2M/L2P leaves per wave (1, 2, 4, 8;
// needs max_leaf_count <= 64 / leaves).
int p2p_groups(const fmm_plan* pl);
int default_p2p_groups(const fmm_plan* pl);
// Near-field form of the target leaves of nt points, whose direct lists have
// `list` source leaves per work item on average, in a plan of `items` items:
// the largest product of
//   - the share of busy lanes (of the waves that have work: a round of the
//     list that leaves whole waves without a leaf costs nothing),
//   - the form's rate with all lanes busy against k_p2p's, and
//   - x / (x + 1) for x waves per SIMD (1024 SIMDs), the fill of the chip.
// The rates are those measured on cubes of 2^12 leaves of 16 to 250 points
// (FP32); a pass without a field has the higher ones, since a pair is cheaper
// there and a record's read is shared by two.  The product then orders the
// forms as measured from 2^6 leaves on, e.g. (pass in us, one wave | 64 | 128
// | 256 threads): 2^8 leaves of 56 points 129 | 103 | 85 | 84, of 150 220 | -
// | - | 215; 2^12 leaves of 48 366 | 349 | 305 | 305, of 72 825 | - | 577 |
// 571, of 112 1103 | - | 1196 | 1292; potential of 2^12 leaves of 56 312 |
// 287 | 295 | 303, of 104 847 | - | 802 | 900.  256 threads serve to fill the
// chip only: with 16 waves a SIMD and more they gain 0 to 4% by themselves
// (9% for 132 to 140 points) but hold up the far field beside them (16
// problems of 22 to 109 points a leaf, pass: 1.65 | 1.76 ms without and with).
// The items that keep one wave with a field never take 256 threads without one
// (rate 0): their lists of one to four leaves leave groups without a leaf, which
// the product rates too high (near field, one wave | 128 in two rounds of
// targets | 256 threads: 2^8 leaves of 200 points 148 | 178 | 162 us, of 256 187
// | 221 | 204; 2^9 of 160 139 | 145 | 131).
// FP64 leaves of a plan with two or four source groups (32 points and fewer)
// always take the wide form; in FP32 the wide forms reproduce the sums of one
// source group, so such plans keep k_p2p.
enum { kNearWide256 = 0, kNearWide = 1, kNearWide64 = 2, kNearWave = 3 };
struct WideRates {
  double w64, w128, w256;
};
constexpr WideRates kWideField{1.0, 0.97, 0.88}, kWidePot{1.12, 1.05, 0.0};
constexpr double kWideFillWaves = 16.0;
// FP64: the flat form's rate, and what 128 threads have to gain on 64
constexpr double kFlatRate = 0.9, kFlatGain = 1.08;
int near_form(const fmm_plan* pl, int nt, double list, int64_t items, bool field);
int leaves_per_wave(const fmm_plan* pl);
int m2l_waves(const fmm_plan* pl);
int chain_waves(const fmm_plan* pl);
// waves per translation of the shared forms
constexpr int kShareWaves = 4;
// lowest order with the shared M2M / L2L forms
constexpr int kChainShareMinOrder = 5;
// Values of the m2l_waves tile besides 1 for order p and precision (1: none).
// 4 asks for the form whose translations are shared by four waves; it is
// built (m2l_shared_built) where it is the faster one, and both values run
// the one-lane form elsewhere.
constexpr int m2l_share_waves(int p, bool fp64) {
  return fp64 ? ((p == 6 || p == 7) ? 4 : 1) : (p >= 9 ? 4 : 1);
}
constexpr bool m2l_shared_built(int p, bool fp64) { return !fp64 && p == 10; }
bool valid_p2p_groups(const fmm_plan* pl, int g);
bool valid_leaves_per_wave(const fmm_plan* pl, int l);

// Stage-timing helpers (api.cpp).
hipEvent_t take_event(fmm_plan* pl);
void release_profile(fmm_plan* pl);
enum { kStSort = 0, kStP2M, kStM2M, kStM2L, kStL2L, kStL2P, kStP2P };
// Begin/end events of every stage of one pass (when profiling is on), each
// pair recorded on the stream the stage runs on.
struct StageMarks {
  std::vector<hipEvent_t>* row = nullptr;
  explicit StageMarks(fmm_plan* pl, bool enabled = true) {
    if (!pl->profiling || !enabled) return;
    pl->ev_rows.emplace_back();
    row = &pl->ev_rows.back();
    for (int k = 0; k < 2 * FMM_NSTAGES; ++k) row->push_back(take_event(pl));
  }
  void begin(int k, hipStream_t s) const {
    if (row) FMM_HIP(hipEventRecord((*row)[2 * k], s));
  }
  void end(int k, hipStream_t s) const {
    if (row) FMM_HIP(hipEventRecord((*row)[2 * k + 1], s));
  }
};

// Near field over the direct lists Ls (near.hip): src holds the leaf-ordered
// source records of this pass, near receives potential [n] and field [n][3]
// in leaf order, both of the plan's precision.
void near_field(fmm_plan* pl, const ListSet& Ls, const void* src, int64_t n, void* near, bool field,
                hipStream_t sp, const StageMarks& mk);
// One pass of expansion order P (eval.hip, compiled once per order).
template <int P, typename T>
void run_pass(fmm_plan* pl, const Workspace& ws, int dir, const T* q, T* pot, T* field,
              hipStream_t st);

// Runs f, turning exceptions into a status and the thread's error message
// (every C entry point).
template <typename F>
fmm_status guard(F&& f) {
  try {
    clear_error();
    f();
    return FMM_OK;
  } catch (const Error& e) {
    set_error(e.msg);
    return e.code;
  } catch (const std::bad_alloc&) {
    set_error("host allocation failed");
    return FMM_ENOMEM;
  } catch (const std::exception& e) {
    set_error(e.what());
    return FMM_EDEVICE;
  } catch (...) {
    set_error("unknown error");
    return FMM_EDEVICE;
  }
}

// Sorting primitives (sort.hip).
size_t sort_pairs_u64_i32_temp(int n);
void sort_pairs_u64_i32(void* temp, size_t temp_bytes, const uint64_t* kin,
                        uint64_t* kout, const int32_t* vin, int32_t* vout,
                        int n, hipStream_t st);
size_t sort_keys_u64_temp(int64_t n);
void sort_keys_u64(void* temp, size_t temp_bytes, const uint64_t* kin,
                   uint64_t* kout, int64_t n, int end_bit, hipStream_t st);
size_t scan_i32_temp(int64_t n);
void exclusive_scan_i32(void* temp, size_t temp_bytes, const int32_t* in,
                        int32_t* out, int64_t n, hipStream_t st);

}  // namespace fmm
