// pasur_internal.hpp -- internals shared by the HIP translation units of
// libpasur (gfx950).  Not part of the public ABI (include/pasur.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cmath>
#include <cstdio>

#include "../../include/pasur.h"

namespace pasur {

void set_error(const char *fmt, ...);

#define PASUR_TRY_HIP(expr)                                                   \
  do {                                                                        \
    hipError_t e_ = (expr);                                                   \
    if (e_ != hipSuccess) {                                                   \
      ::pasur::set_error("%s failed: %s", #expr, hipGetErrorString(e_));      \
      return PASUR_E_HIP;                                                     \
    }                                                                         \
  } while (0)

#define PASUR_TRY(expr)                                                       \
  do {                                                                        \
    int s_ = (expr);                                                          \
    if (s_ != PASUR_OK) return s_;                                            \
  } while (0)

// Gives the cached blocks of the current device back (below); a failed
// allocation of any kind is tried again after it.
void blocks_release();
hipError_t malloc_async(void **p, size_t bytes, hipStream_t s);  // hipMallocAsync

template <class T>
int dev_alloc(T **p, int64_t n) {
  *p = nullptr;
  size_t bytes = (size_t)(n > 0 ? n : 1) * sizeof(T);
  hipError_t e = hipMalloc((void **)p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    blocks_release();
    e = hipMalloc((void **)p, bytes);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    set_error("hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    *p = nullptr;
    return PASUR_E_NOMEM;
  }
  return PASUR_OK;
}

template <class T>
void dev_free(T *&p) {
  if (p) (void)hipFree((void *)p);
  p = nullptr;
}

// Device memory for trees and their construction, from a cache of freed blocks
// (pasur_util.hip): hipMalloc costs up to 40 ms per GB for blocks of 8 to 500 MB,
// and building a game takes and gives back hundreds of them.  A block that goes
// back must be idle: nothing that uses it is pending on any stream.
int block_alloc(void **p, size_t bytes);
void block_free(void *p);
// Scratch of the work that the caller enqueues on s: given back behind that work,
// while it is pending, to be had by later work on s at once and by others when it
// has ended.  Not while s is being captured.
int block_alloc_on(void **p, size_t bytes, hipStream_t s);
void block_free_on(void *p, hipStream_t s);
// The wait of a hipFree, for handles that the caller may free while work that
// uses them is still running: an anchor is a small plain allocation, and freeing
// it waits for the device as freeing the arrays themselves did.
int anchor_alloc(void **a);
// Frees the anchor (NULL: the blocks are idle) and gives the n blocks (at most
// kRetired, NULLs among them) back.  Where the wait is refused, as while another
// thread captures a stream, they are set aside until a later one succeeds.
constexpr int kRetired = 9;
void blocks_retire(void *anchor, void *const *blocks, int n);

// Exclusive scan of n int32 counts into out[0..n] (out[n] = total); the
// total is returned through *total (synchronises `stream`).  Fails with
// PASUR_E_OVERFLOW when the total exceeds INT32_MAX.
int scan_counts(const int32_t *d_counts, int64_t n, int32_t *d_out,
                int64_t *total, hipStream_t stream);

// Bit masks over the 52 card indices.
constexpr uint64_t kNumericMask = (1ull << 40) - 1;       // A..10, 40 cards
constexpr uint64_t kJackMask = 0xFull << 40;
constexpr uint64_t kClubMask = 0x0001111111111111ull;      // every 4th card
constexpr uint64_t kAllCards = (1ull << 52) - 1;

// 16-bit score key ordered by (bonus, ca, cb, d): bonus 2 bits, ca and cb
// 3 bits each (0..6 while the bonus is undecided, else 0), d + 128 8 bits.
__host__ __device__ inline uint32_t score_key(int ca, int cb, int d, int bonus) {
  return ((uint32_t)bonus << 14) | ((uint32_t)ca << 11) | ((uint32_t)cb << 8) |
         (uint32_t)(d + 128);
}
__host__ __device__ inline void score_unkey(uint32_t k, int *ca, int *cb,
                                            int *d, int *bonus) {
  *bonus = (int)((k >> 14) & 3);
  *ca = (int)((k >> 11) & 7);
  *cb = (int)((k >> 8) & 7);
  *d = (int)(k & 0xFF) - 128;
}

// Sampling shared by self-play and external-sampling CFR.
// The i-th output of SplitMix64 started at `seed` (its state after i + 1
// steps, through the generator's finaliser), as a double in [0, 1).
__device__ inline double splitmix_uniform(uint64_t seed, uint64_t i) {
  uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

// Index of the sampled child among k (k >= 2) whose strategy is prob(0..k-1)
// (any accessor returning a child's probability): the first whose running
// sum (FP64, in child order) exceeds u * total; uniform choice when the
// policy is uniform or the total is 0.
template <class Prob>
__device__ __forceinline__ int choose_by(double u, int k, int policy, const Prob &prob) {
  const int uni = min((int)(u * (double)k), k - 1);
  if (policy == PASUR_PLAY_UNIFORM) return uni;
  double total = 0.0;
  for (int c = 0; c < k; ++c) total += prob(c);
  if (!(total > 0.0)) return uni;
  const double x = u * total;
  double acc = 0.0;
  int last = 0;
  for (int c = 0; c < k; ++c) {
    const double pc = prob(c);
    acc += pc;
    if (pc > 0.0) last = c;
    if (acc > x) return c;
  }
  return last;
}

// choose_by over a contiguous array p[0..k-1].
template <class T>
__device__ inline int choose(double u, const T *__restrict__ p, int k, int policy) {
  return choose_by(u, k, policy, [p](int c) { return (double)p[c]; });
}


// ---- DCFR iteration constants (computed on the host so that FP64 results
// stay bit-exact) --------------------------------------------------------------
struct IterConsts {
  double dpos, dneg;  // DCFR discounts for R > 0 and R <= 0
  double avg_w;       // weight of the previous average-strategy sum
  double avg_t;       // multiplier of the new term (t for CFR+, else 1)
  double eps;
  int variant, rm_mode;
  int flags;  // pasur_cfr_flags (DCFR only)
};

struct IterK {
  double dpos, dneg, avg_w, avg_t;
};

inline IterConsts consts_for(const pasur_cfr_params *p, int64_t t) {
  IterConsts ic;
  const double tm1 = (double)(t - 1);
  double pa = std::pow(tm1, p->alpha);
  double pb = std::pow(tm1, p->beta);
  ic.dpos = pa / (pa + 1.0);
  ic.dneg = pb / (pb + 1.0);
  if (p->variant != PASUR_DCFR)
    ic.avg_w = 1.0;
  else if (p->flags & PASUR_CFR_SNIPPET_AVG)
    ic.avg_w = 1.0 - 1.0 / std::pow((double)t, p->gamma);
  else
    ic.avg_w = std::pow(tm1 / (double)t, p->gamma);
  ic.avg_t = (double)t;
  ic.eps = p->eps;
  ic.variant = p->variant;
  ic.rm_mode = p->rm_mode;
  ic.flags = p->flags;
  return ic;
}

inline IterK iter_k(const pasur_cfr_params *p, int64_t t) {
  const IterConsts ic = consts_for(p, t);
  return IterK{ic.dpos, ic.dneg, ic.avg_w, ic.avg_t};
}

// The state's arrays are there and its type is known (pasur_cfr.hip).
int check_state(const pasur_fgt *f, const pasur_cfr_state *st);

// ---- optional per-launch timing (pasur_profile_enable) ------------------------
struct ProfRec {
  int kernel, level;
  int64_t work[5];  // kernel-specific work counts (edges, parents, roots, ..., iterations)
  hipEvent_t a, b;
};
bool prof_on(int kernel);
void prof_push(const ProfRec &r);
void prof_events(hipEvent_t *a, hipEvent_t *b);  // two events from the pool

// Records HIP events around the launches made in its scope when profiling is on.
struct ProfScope {
  ProfRec rec;
  hipStream_t s;
  bool on;
  ProfScope(int kernel, int level, hipStream_t stream, int64_t w0 = 0, int64_t w1 = 0,
            int64_t w2 = 0, int64_t w3 = 0, int64_t w4 = 1)
      : s(stream), on(prof_on(kernel)) {
    if (!on) return;
    rec.kernel = kernel;
    rec.level = level;
    rec.work[0] = w0;
    rec.work[1] = w1;
    rec.work[2] = w2;
    rec.work[3] = w3;
    rec.work[4] = w4;
    prof_events(&rec.a, &rec.b);
    (void)hipEventRecord(rec.a, s);
  }
  ~ProfScope() {
    if (!on) return;
    (void)hipEventRecord(rec.b, s);
    prof_push(rec);
  }
};

// ---- HBM-streaming schedule (pasur_sweep.hip) --------------------------------
struct SweepIndex;
void sweep_index_free(SweepIndex *x);
// Iterations t0 .. t0+n_iters-1 of one round with level-wide streaming
// launches (PASUR_SCHED_STREAM); same arguments as pasur_cfr_iterate.
int sweep_iterate(pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p,
                  int64_t t0, int n_iters, hipStream_t s);
// Rounds of as many nodes, whose calls PASUR_SCHED_AUTO only enqueues, and whether
// the streaming schedule is expected to beat the persistent segment schedule on
// n_iters iterations of one.
bool large_round(const pasur_fgt *f);
bool sweep_pays(const pasur_fgt *f, int dtype, int n_iters);

// Iterations t0 .. t0+n_iters-1 of one round with the persistent segment
// schedule (pasur_seg.hip); n_iters >= 1.  Waits for the stream.
int seg_iterate(const pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p,
                int64_t t0, int n_iters, hipStream_t s);
// The same without a wait, with a segment index of the tree that its first call
// builds (seg_ready: there is one for this type, as a capture needs).  Sets *done,
// or leaves it false where there is no memory for the segments' far arrays.
struct SegIndex;
constexpr int kSegIndexes = 6;  // of one tree
// The blocks of a tree's indexes, into p[0 .. n-1]; returns how many.
int seg_index_blocks(const SegIndex *x, void **p, int n);
void seg_index_free(SegIndex *x);
bool seg_ready(const pasur_fgt *f, int dtype);
int seg_enqueue(pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p, int64_t t0,
                int n_iters, bool capturing, bool *done, hipStream_t s);

// ---- exact values (pasur_values.hip) -----------------------------------------
// Root values of one round from an array of leaf values (leaf_dtype; FP64
// leaves when dtype is PASUR_F64), as pasur_tree_values.  alloc: a tree with a
// value_stop() takes stream-ordered scratch, else its own.
int tree_values(const pasur_fgt *f, const void *leaf, int leaf_dtype, int dtype,
                void *const *sigma, int mode, double *out, bool alloc, hipStream_t s);
// Where some root is too large for one workgroup, the level (1 to 5) down from
// which the roots' nodes fit one each, those of that level to 6 being evaluated
// before; 0: a workgroup per root from the leaves.  root_off: 9 levels of
// n_roots + 1 offsets.
int value_stop(const int64_t n[9], int64_t n_roots, const int32_t *root_off);
// Nodes of a tree's levels value_stop .. 6, whose values are passed on.
int64_t split_nodes(const pasur_fgt *f);
// The widest of levels 0..7, and the widest that pasur_tree_values_noalloc takes.
inline int64_t widest_level(const int64_t n[9]) {
  int64_t mx = 1;
  for (int l = 0; l <= 7; ++l) mx = n[l] > mx ? n[l] : mx;
  return mx;
}
constexpr int64_t kNoAllocLevel = (int64_t)1 << 21;
// pasur_exploitability on checked arguments.
int composed_values(const pasur_fgt *const *fgts, int n_rounds, void *const *sigma_bar, int dtype,
                    int leaf_flags, double *br_a, double *br_b, double *v, hipStream_t s);

}  // namespace pasur

// Round game tree, device arrays per level.
struct pasur_gt {
  int round;
  int64_t n[9];
  uint64_t *pool[9];
  uint8_t *hands[9];
  uint64_t *rs[9];  // 8 signed bytes per node, see PASUR_GT_RS
  int32_t *parent[9];
  int32_t *child_begin[8];
  uint8_t *act_card[9];
  uint64_t *act_cap[9];
  uint8_t deck[52];
  void *block[9];  // the block that holds a level's arrays
  void *anchor;
};

// Unfolded tree of one round.
struct pasur_fgt {
  int round;
  int64_t n[9];
  int32_t *gt[9];
  int32_t *sid[9];
  int32_t *parent[9];
  int32_t *child_begin[8];
  int64_t n_scores;
  int8_t *score_tab;  // 4 per score: ca, cb, d, bonus
  int64_t n_next;
  pasur_root *next_roots;
  int32_t *link;
  int16_t *leaf_base;
  int8_t *leaf_bonus;  // round 5: the final 7-club bonus state of each leaf
  // root_off[l][j] .. root_off[l][j+1]: level-l nodes of root j's subtree
  // (levels are root-major), on the device and copied to the host
  int64_t n_roots;
  int32_t *root_off[9];
  int32_t *h_root_off;  // 9 * (n_roots + 1), level-major
  // structure index of the streaming schedule, built on first use
  pasur::SweepIndex *sweep;
  // per root, what a segment's LDS layout counts (4 ints: see pasur_seg.hip),
  // on the host; computed on first use
  int32_t *h_root_seg;
  // the largest root's nodes (0: not computed yet) and those below large roots
  // (per state type: see sweep_pays)
  int64_t root_largest, root_tail[2];
  // the segments of the tree by itself, one index after another, built on first use
  pasur::SegIndex *seg_index;
  // split_ws: a double per node of split_nodes(), where pasur_tree_values_noalloc
  // takes the tree
  int value_stop;
  double *split_ws;
  // the blocks behind root_off, the arrays of the levels, and next_roots
  void *off_block, *block, *next_block;
  void *anchor;
};
