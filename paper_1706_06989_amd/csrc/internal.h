// Internal declarations of libamfmm_hip.so (host orchestration + kernels).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <stdexcept>
#include <string>
#include <vector>

#include "amfmm.h"

namespace amfmm {

constexpr int kMaxLevel = 21;  // Morton key resolution per coordinate
constexpr int kGeo = 4;        // per cell: Zx, Zy, Zz, R_max
constexpr int kMom = 18;       // per cell: M, M_ij (6), M_ijk (10), pad
constexpr int kLoc = 24;       // per cell: C (1), C_k (3), C_kl (6), C_klm (10), g_c (3), pad
constexpr int kLocGen = 40;    // expansion order 4: 35 local coefficients, g_c (3), pad

// words of the pinned read-back buffer: walk totals, bounding box and input
// flags (8 doubles), cells per level (2 per level)
constexpr int kPinWalk = 0, kPinBox = 16, kPinTree = 24, kPinWords = 24 + 2 * (kMaxLevel + 1);

// index of a symmetric pair / triple inside the packed arrays
//   pairs   xx xy xz yy yz zz
//   triples xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz

struct Error : std::runtime_error {
  int code;
  Error(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

// the walk of a batch would exceed the list budget: retry with a smaller batch
struct BudgetExceeded : Error {
  BudgetExceeded() : Error(AMFMM_E_OOM, "interaction lists exceed the list budget") {}
};

#define AMFMM_HIP(call)                                                                   \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess)                                                                 \
      throw ::amfmm::Error(AMFMM_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

// phases of a solve (amfmm_get_phase_times order)
// kPhWalkPass: the walk's one pass over the pairs (its staging kernel), a part
// of the walk that is also reported on its own
enum Phase { kPhValidate = 0, kPhSort, kPhTree, kPhMoments, kPhWalk, kPhFar, kPhPush, kPhNear, kPhWalkPass, kPhEnd };
constexpr int kMaxStamps = 1 << 15;  // clock words of a timeline (see mark)

// Grow-only device buffer owned by a context.
struct DevBuf {
  void* p = nullptr;
  size_t cap = 0;
};

struct Ctx {
  amfmm_options opt;
  hipStream_t stream = nullptr;
  int device = 0;
  std::string last_error;
  size_t bytes = 0;  // device bytes currently held
  std::vector<DevBuf*> bufs;

  // particles, sorted by key
  int64_t n = 0;
  DevBuf pos4;    // double4 (x, y, z, m)
  DevBuf keys;    // uint64
  DevBuf perm;    // int32, sorted -> caller
  DevBuf keys2;   // sort ping-pong
  DevBuf perm2;
  DevBuf bbox;    // 8 doubles: lo[3], hi[3], flags
  DevBuf scratch; // scan / sort temporaries
  DevBuf scratch2;
  DevBuf hist;
  // cells in (level, begin) order
  int32_t ncells = 0, depth = 0, nleaves = 0;
  std::vector<int32_t> level_start;  // host copy, size depth+2
  DevBuf c_begin, c_count, c_parent, c_child0, c_nchild;  // int32
  DevBuf c_level;  // int8 level per cell
  DevBuf leaves;   // int32 ids of leaf cells
  DevBuf leafof;   // int32 leaf cell of every (sorted) particle
  DevBuf geo;      // double4 per cell
  DevBuf mom;      // kMom doubles per cell
  DevBuf msum;     // double4 per cell: sum m*X (x,y,z), unused
  DevBuf loc;      // kLoc doubles per cell
  DevBuf mono;     // expansion order 4: 35 moments per cell (sum mu x^alpha, |alpha| <= 4)
  DevBuf locg;     // expansion order 4: kLocGen doubles per cell
  // directed interaction lists grouped by target cell
  int64_t n_far = 0, n_near = 0;
  DevBuf far_start, far_count, far_src;     // int32 (start as int64)
  DevBuf near_start, near_count, near_src;
  DevBuf near_parts;  // int64 per cell: particles behind its near list
  DevBuf near_plan;   // near field: segments of the cut lists and their partial sums
  // walk frontier
  // (fx, fx2: the cell of every chunk; fy, fy2: the frontier's source cells;
  // gsave: chunk counts of a level and their offsets)
  DevBuf fx, fy, fx2, fy2, grp, walkrec, fsave, gsave, counters, gqueue;
  bool frontier_mapped = false;  // fx holds the cell of every frontier entry
  DevBuf stage;  // walk: per-chunk staging windows of one level's terminal pairs
  // far field, UC/TC: source record per cell (128 bytes, order 4: 288); empty
  // where it found no room or was given back
  DevBuf farrec;
  // walk: terminal pairs per frontier entry of every level (far, near, split-X
  // bases; -1 = unknown) from the last walk under the rule walk_ratio_key
  std::vector<double> walk_ratio;
  double walk_ratio_key[4] = {-1.0, -1.0, -1.0, -1.0};
  int64_t grp_width = 0, frontier = 0;
  double walk_abs_tol = 0.0;
  int walk_mode = 0;              // 0 geometric, 1 error estimate, 2 learned
  DevBuf model;                   // learned criterion: network with BF16-rounded weights
  DevBuf mlp_tmp, mlp_part, mlp_grad;  // inference and training scratch
  // caller's per-particle field estimate (device): magnitudes in `field`, or
  // components in field, field_y, field_z
  const double* field = nullptr;
  const double* field_y = nullptr;
  const double* field_z = nullptr;
  DevBuf gmin;
  // unordered near-field leaf pairs of the kept lists (built on request)
  std::vector<std::pair<int32_t, int32_t>> near_pairs_host;
  bool near_pairs_valid = false;
  int grp_cur = 0;
  int64_t* pinned = nullptr;  // kPinWords pinned host words for read-backs (kernels write them)
  double box[6] = {};         // bounding box of the tree's particles: lo, hi
  int64_t far_evals = 0;      // directed far-field evaluations of the last solve
  int64_t far_launches = 0, near_launches = 0;  // kernel launches of the last evaluation
  int64_t pass_launches = 0;    // launches of the walk's pass kernel in the last walk
  int64_t walk_candidates = 0;  // pairs the last walk decided on (batches over budget excluded)
  bool batched = false;       // last solve ran batch by batch (lists not kept)
  size_t walk_budget = 0;     // bytes of lists + frontier a walk may take (0 = unlimited)
  // batch size that worked for the last solve of the same size and criterion
  int64_t batch_hint = 0, hint_n = 0;
  int64_t batch_fail = 0;  // smallest batch (particles) that exceeded the budget, same problem
  double hint_theta = 0.0, hint_tol = 0.0;
  int hint_mode = -1;
  double theta = 0.5;
  bool have_tree = false, have_moments = false, have_lists = false;
  // timing: device clock values taken by the first kernel of each phase; the
  // time between two belongs to the phase of the first
  unsigned long long* stamps = nullptr;  // kMaxStamps device words
  std::vector<int> st_phase;             // phase of every word taken so far
  bool st_pending = false;               // the last word waits for its kernel
  double folded_ms[kPhEnd] = {};         // times of the timeline's earlier words, where it outgrew them
  int clock_khz = 100000;
  // allocation-free solve: while arena is set, every device buffer is carved
  // from [arena, arena + arena_cap) (a static device array) instead of being
  // allocated (first fit over the free blocks, released blocks merged with
  // their neighbours), and no phase times are taken
  char* arena = nullptr;
  size_t arena_cap = 0;
  bool arena_tight = false;  // second attempt of a solve that did not fit
  std::map<size_t, size_t> arena_free;  // offset -> bytes of each free block
};

// device bytes a solve may still take in one buffer: the free device memory,
// or the largest free block of the arena in an allocation-free solve
size_t free_device_bytes(Ctx& c);

// allocate (grow-only) a device buffer of at least `bytes`; contents are lost on growth
void* ensure(Ctx& c, DevBuf& b, size_t bytes);
// ensure, in an arena from its top end: the walk's transient buffers stay out
// of the way of the lists that grow beside them
void* ensure_top(Ctx& c, DevBuf& b, size_t bytes);
// ensure for a buffer that a solve can do without: nullptr (and an empty buffer)
// where there is no room
void* ensure_if_room(Ctx& c, DevBuf& b, size_t bytes);
// grow keeping the first `keep` bytes
void* ensure_keep(Ctx& c, DevBuf& b, size_t bytes, size_t keep);
template <typename T>
T* as(DevBuf& b) {
  return static_cast<T*>(b.p);
}
void sync(Ctx& c);

// ---- scan.hip ----
// exclusive prefix sum of n int32 values into out[0..n], out[n] = total
void scan_i32(Ctx& c, const int32_t* in, int32_t* out, int64_t n);
// the same for `count` int64 arrays of length n at once
constexpr int kScanMax = 6;
template <typename T>
struct ScanSet {
  const T* in[kScanMax];
  T* out[kScanMax];
};
void scan_i64(Ctx& c, const ScanSet<int64_t>& set, int count, int64_t n, unsigned long long* clock = nullptr);

// ---- sort.hip ----
// stable LSD radix sort of (key, value) pairs by the low `bits` bits of key;
// results end in keys/vals (the alt buffers are scratch)
void radix_sort(Ctx& c, uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt,
                int64_t n, int bits);

// ---- tree.hip ----
// bounding box and input checks (enqueued: build_levels reads the result)
void bbox_start(Ctx& c, const double* x, const double* y, const double* z, const double* m, int64_t n);
// after bbox_start: synchronises; 0, or the amfmm_status of a non-finite or non-positive input
int input_status(Ctx& c);
void build_keys_sort(Ctx& c, const double* x, const double* y, const double* z, const double* m,
                     int64_t n);
// cells of all levels; synchronises once; returns input_status (the keys of bad
// inputs are arbitrary but valid)
int build_levels(Ctx& c);

// ---- moments.hip ----
void upward_pass(Ctx& c);

// ---- walk.hip ----
void dual_walk(Ctx& c, double theta);  // whole walk, lists kept for every cell
void walk_prepare(Ctx& c, double theta);
void walk_start(Ctx& c);  // frontier = {(root, root)} at level 0
// walks levels [lev_first, lev_last] over the cells [lo[l], hi[l]) of each level,
// starting from the frontier held in c.fy / c.grp; appends lists at the bases;
// returns the size of the frontier left for level lev_last + 1
int64_t walk_levels(Ctx& c, int lev_first, int lev_last, const std::vector<int32_t>& lo,
                    const std::vector<int32_t>& hi, int64_t& far_base, int64_t& near_base);
void group_arrays(Ctx& c, int64_t** gbeg, int32_t** gcnt);  // current level's groups

// ---- eval.hip ----
// UC and TC of the plain -1/R, and order 4: the far field's source records, one
// per cell (after the moments)
void far_prepare(Ctx& c);
int length_exponent(const Ctx& c);  // of the larger of the box's side and the softening (FarUnit)
void far_field(Ctx& c, int32_t c_lo, int32_t c_hi);
// expansion order 4 (order.hip): moments, far field, push-down, evaluation at the particles
void order_upward(Ctx& c);
void order_pack(Ctx& c);
void order_far(Ctx& c, int32_t c_lo, int32_t c_hi, double* loc);
void order_push_down(Ctx& c, int32_t c_lo, int32_t c_hi);
void order_l2p(Ctx& c, const int32_t* leaves, int32_t c_lo, int32_t count, double* ax, double* ay, double* az,
               double* pot);
void push_down(Ctx& c, int32_t c_lo, int32_t c_hi);  // cells of one level
void push_down_all(Ctx& c);                         // every level, downwards
// bytes of Ctx::counters: the counters, then the near field's ranges
constexpr size_t kCounterBytes = 64, kRangeBytes = 8 * (kMaxLevel + 1);
// a range of cells on each of some levels (a batch of subtrees)
struct CellRanges {
  int n = 0;
  int32_t lo[kMaxLevel + 1], hi[kMaxLevel + 1];
  void add(int32_t a, int32_t b) {
    if (b > a) {
      lo[n] = a;
      hi[n++] = b;
    }
  }
};
// all leaves, or the leaves of those ranges
void near_field(Ctx& c, const CellRanges* ranges, double* ax, double* ay, double* az, double* pot);
// fills n (<= 64) device words with zero (a kernel, so it can sit in a graph)
void zero_u64(Ctx& c, unsigned long long* p, int n, unsigned long long* clock = nullptr);

// ---- mlp.hip ----
// features (8 floats) and labels (log2 error factor) of cell pairs (device)
void compute_pair_features(Ctx& c, int64_t np, const int32_t* pairs, float* feats);
void compute_pair_labels(Ctx& c, int variant, int64_t np, const int32_t* pairs, double* labels);
// model with its weights rounded to BF16 (device to device)
void round_model(Ctx& c, const float* in, float* out);
void mlp_predict(Ctx& c, int64_t n, const float* model, const float* feats, float* y);
// gradient into grad (device); returns the loss (synchronises)
double mlp_grad(Ctx& c, int64_t n, const float* model, const float* feats, const float* labels, double tau,
                float* grad);
// Adam steps; returns the loss of the last batch (synchronises)
double mlp_train(Ctx& c, int64_t n, const float* feats, const float* labels, float* model, float* am, float* av,
                 int64_t step0, int32_t steps, int32_t batch, double lr, double tau);

// ---- integrate.hip ----
// v += h a and x += dt v over n particles (device SoA arrays)
void kick(Ctx& c, int64_t n, double h, const double* ax, const double* ay, const double* az, double* vx, double* vy,
          double* vz);
void drift(Ctx& c, int64_t n, double dt, const double* vx, const double* vy, const double* vz, double* x, double* y,
           double* z);

// ---- direct.hip ----
void direct_sum(Ctx& c, int64_t n, const double* x, const double* y, const double* z,
                const double* m, int64_t ntarget, const int64_t* targets, double* ax, double* ay,
                double* az, double* pot, double* gabs);
void balance(Ctx& c, int64_t n, const double* x, const double* y, const double* z,
             const double* m, const double* ax, const double* ay, const double* az, double* out);

// A phase starts: the next kernel given clock_word(c) writes the device clock
// there as it starts (a phase whose kernels are not launched takes no time).
// An event per phase costs 3.7 us on the stream, and a solve of ten levels had
// 28 of them.
void mark(Ctx& c, int phase);
unsigned long long* clock_word(Ctx& c);
void end_timeline(Ctx& c);  // the last phase ends here
#ifdef __HIPCC__
__device__ inline void take_time(unsigned long long* word) {
  if (word && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *word = wall_clock64();
}
#endif

inline unsigned blocks_for(int64_t n, int threads) {
  return (unsigned)((n + threads - 1) / threads);
}

}  // namespace amfmm
