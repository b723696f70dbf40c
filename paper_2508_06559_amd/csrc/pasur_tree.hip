// pasur_tree.hip -- round game tree (move generation), the Unfolding
// Process and the Between-Hand linkage, as level-synchronous HIP kernels.
//
// Every level is laid out count -> exclusive scan -> fill, a fixed set of threads
// per parent, so children land parent-major in canonical order without atomics.
//
// Small rounds are bound by what surrounds the kernels: a round's build and
// unfolding wait for the stream 13 times (a level's size has to be known before
// it is allocated) and allocate 14 times, against about 60 and 120 with an
// allocation per array and a wait per scan.  Totals arrive in pinned host words
// that the scans write.
#include "pasur_sort.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

using namespace pasur;

namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n) {
  return (unsigned)((n + kThreads - 1) / kThreads);
}

__device__ inline int card_value(int c) { return (c >> 2) + 1; }

// Scoring table of section "Pasur": each Ace 1, each Jack 1, the 2 of clubs
// 2, the 10 of diamonds 3.
__device__ inline int points_of(uint64_t m) {
  return __popcll(m & 0xFull) + 2 * (int)((m >> 4) & 1) + 3 * (int)((m >> 37) & 1) +
         __popcll(m & kJackMask);
}

// Cards dealt to the two players in this round, per hand bit, and for each
// player the order of his 4 hand bits by ascending card index.
struct DealInfo {
  uint8_t card[8];
  uint8_t order[2][4];
};

// The hand bit of the mover's slot-th held card in ascending order, or -1.
__device__ __forceinline__ int held_bit(const DealInfo &di, uint8_t hands, int mover, int slot) {
  int left = slot, bit = -1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int b = 4 * mover + di.order[mover][j];
    if ((hands >> b) & 1) {
      if (left == 0) bit = b;
      --left;
    }
  }
  return bit;
}

// Legal moves with card c on a pool, in canonical order (capture mask
// ascending), passed to emit(capture mask):
//  - numeric card: every set of pool numerics whose values complete 11,
//    enumerated in colex order (= ascending mask) by a depth-first search over
//    the pool's bits: a set's cards are chosen from the highest down, the
//    candidates of a step are the pool cards below the last chosen one, and
//    values never decrease with the index, which ends a step early.  The
//    chosen cards (at most 9) are a stack of 6-bit fields in one register;
//    no capture -> lay;
//  - Jack: all pool numerics and Jacks, or a lay if there are none;
//  - Queen/King: one capture per same-rank pool card, else a lay.
template <class Emit>
__device__ __forceinline__ void for_each_move(int c, uint64_t pool, Emit &&emit) {
  bool found = false;
  if (c < 40) {
    const uint64_t pn = pool & kNumericMask;
    uint64_t acc = 0, stack = 0, m = pn;
    int rem = 11 - card_value(c), depth = 0;
    while (true) {
      if (m == 0) {
        if (depth == 0) break;
        const int x = (int)(stack & 63);
        stack >>= 6;
        --depth;
        acc &= ~(1ull << x);
        rem += card_value(x);
        const uint64_t below = depth ? (1ull << (stack & 63)) - 1 : ~0ull;
        m = pn & below & ~((2ull << x) - 1);
        continue;
      }
      const int x = __ffsll((long long)m) - 1, v = card_value(x);
      if (v > rem) {  // every later card is at least as large
        m = 0;
      } else if (v == rem) {
        emit(acc | (1ull << x));
        found = true;
        m &= m - 1;
      } else {
        acc |= 1ull << x;
        rem -= v;
        stack = (stack << 6) | (uint64_t)x;
        ++depth;
        m = pn & ((1ull << x) - 1);
      }
    }
  } else if (c < 44) {
    const uint64_t cap = pool & (kNumericMask | kJackMask);
    if (cap) {
      emit(cap);
      found = true;
    }
  } else {
    for (uint64_t cap = pool & (0xFull << (c & ~3)); cap; cap &= cap - 1) {
      emit(cap & (~cap + 1));
      found = true;
    }
  }
  if (!found) emit(0ull);
}

// Moves per held card (16 bits each) of every node of a level; four threads per
// node, one per card: the search is a serial walk, and early levels have few
// nodes (one thread per node with its cards in turn and the search's state in
// indexed arrays took 17 us for the levels of a two-round subgame).
__global__ void __launch_bounds__(kThreads)
    k_gt_count(int64_t n, const uint64_t *__restrict__ pool, const uint8_t *__restrict__ hands,
               DealInfo di, int mover, uint64_t *__restrict__ counts) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = t >> 2;
  const int slot = (int)(t & 3);
  uint64_t cnt = 0;
  if (i < n) {
    const int b = held_bit(di, hands[i], mover, slot);
    if (b >= 0) for_each_move(di.card[b], pool[i], [&](uint64_t) { ++cnt; });
  }
  cnt <<= 16 * slot;
  cnt |= __shfl_xor((unsigned long long)cnt, 1, 64);
  cnt |= __shfl_xor((unsigned long long)cnt, 2, 64);
  if (i < n && slot == 0) counts[i] = cnt;
}

struct MovesIn {
  using Acc = int;
  const uint64_t *counts;
  __device__ __forceinline__ int operator()(int, int64_t i) const {
    const uint64_t c = counts[i];
    return (int)((c & 0xFFFF) + ((c >> 16) & 0xFFFF) + ((c >> 32) & 0xFFFF) + (c >> 48));
  }
};

// ApplyActions (and the capture/Sur/clean-up scoring): children of node i
// written at child_begin[i] + j, by four threads as in k_gt_count.
__global__ void __launch_bounds__(kThreads)
    k_gt_fill(int64_t n, int round, int ply, const uint64_t *__restrict__ pool,
              const uint8_t *__restrict__ hands, const uint64_t *__restrict__ rs,
              const int32_t *__restrict__ cb, const uint64_t *__restrict__ counts, DealInfo di,
              uint64_t *__restrict__ c_pool, uint8_t *__restrict__ c_hands,
              uint64_t *__restrict__ c_rs, int32_t *__restrict__ c_parent,
              uint8_t *__restrict__ c_card, uint64_t *__restrict__ c_cap) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = t >> 2;
  const int slot = (int)(t & 3);
  if (i >= n) return;
  const int mover = ply & 1;
  const uint8_t h0 = hands[i];
  const int bit = held_bit(di, h0, mover, slot);
  if (bit < 0) return;
  const int c = di.card[bit];
  const uint64_t p0 = pool[i], r0 = rs[i], cnt = counts[i];
  int64_t q = cb[i];
  for (int s = 0; s < slot; ++s) q += (int64_t)((cnt >> (16 * s)) & 0xFFFF);
  for_each_move(c, p0, [&](uint64_t cap) {
    uint64_t p = p0;
    int8_t r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) r[k] = (int8_t)((r0 >> (8 * k)) & 0xFF);
    const uint64_t cbit = 1ull << c;
    if (cap == 0) {
      p |= cbit;
    } else {
      const uint64_t taken = cap | cbit;
      const int8_t clubs = (int8_t)__popcll(taken & kClubMask), pts = (int8_t)points_of(taken);
      const int8_t sur = cap == p0 && !(c >= 40 && c < 44) && round != 5 ? 1 : 0;
      if (mover == 0) {
        r[0] += clubs;
        r[3] += pts;
        r[4] += sur;
      } else {
        r[1] += clubs;
        r[5] += pts;
        r[6] += sur;
      }
      r[2] = (int8_t)(mover + 1);
      p &= ~cap;
    }
    if (round == 5 && ply == 7 && r[2] != 0) {
      const int8_t clubs = (int8_t)__popcll(p & kClubMask), pts = (int8_t)points_of(p);
      if (r[2] == 1) {
        r[0] += clubs;
        r[3] += pts;
      } else {
        r[1] += clubs;
        r[5] += pts;
      }
    }
    uint64_t packed = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) packed |= (uint64_t)(uint8_t)r[k] << (8 * k);
    c_pool[q] = p;
    c_hands[q] = (uint8_t)(h0 & ~(1u << bit));
    c_rs[q] = packed;
    c_parent[q] = (int32_t)i;
    c_card[q] = (uint8_t)c;
    c_cap[q] = cap;
    ++q;
  });
}

// Root checks: canonical order (strictly ascending by pool, bonus, ca, cb,
// d), valid scores, pools made of cards dealt before the round, zero pad.
// *bad is a host word; with `keys`, also marks every root's score key in that
// set of 2^16 bits.
__global__ void k_check_roots(int64_t n, const pasur_root *__restrict__ roots,
                              uint64_t dealt_before, int64_t *__restrict__ bad,
                              unsigned long long *__restrict__ keys) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const pasur_root r = roots[j];
  bool ok = (r.pool & ~dealt_before) == 0 && r.pad == 0 && r.bonus >= 0 && r.bonus <= 2;
  ok = ok && (r.bonus == 0 ? (r.ca >= 0 && r.ca <= 6 && r.cb >= 0 && r.cb <= 6)
                           : (r.ca == 0 && r.cb == 0));
  const uint32_t kr = score_key(r.ca, r.cb, r.d, r.bonus);
  if (ok && j > 0) {
    const pasur_root p = roots[j - 1];
    const uint32_t kp = score_key(p.ca, p.cb, p.d, p.bonus);
    ok = r.pool > p.pool || (r.pool == p.pool && kr > kp);
  }
  if (!ok) *bad = 1;
  if (keys) atomicOr(&keys[(kr & 0xFFFF) >> 6], 1ull << (kr & 63));
}

// 1 where a root's pool differs from the root's before it.
struct PoolChange {
  using Acc = int;
  const pasur_root *roots;
  __device__ __forceinline__ int operator()(int, int64_t j) const {
    return j == 0 || roots[j].pool != roots[j - 1].pool ? 1 : 0;
  }
};

// Level 0 of the game tree: the distinct pools, everything held, no points.
__global__ void k_gt_roots(int64_t n, const pasur_root *__restrict__ roots,
                           const int32_t *__restrict__ pos, uint64_t *__restrict__ pools,
                           uint8_t *__restrict__ hands, uint64_t *__restrict__ rs) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n || pos[j + 1] == pos[j]) return;
  pools[pos[j]] = roots[j].pool;
  hands[pos[j]] = 0xFF;
  rs[pos[j]] = 0;
}

int validate_deck(const uint8_t *deck) {
  if (!deck) {
    set_error("deck is NULL");
    return PASUR_E_INVAL;
  }
  uint64_t seen = 0;
  for (int i = 0; i < 52; ++i) {
    if (deck[i] >= 52 || ((seen >> deck[i]) & 1)) {
      set_error("deck is not a permutation of 0..51 (slot %d)", i);
      return PASUR_E_INVAL;
    }
    seen |= 1ull << deck[i];
  }
  return PASUR_OK;
}

int check_root_list(const pasur_root *d_roots, int64_t n_roots) {
  if (!d_roots || n_roots < 1) {
    set_error("need at least one root");
    return PASUR_E_INVAL;
  }
  if (n_roots > INT32_MAX) {
    set_error("too many roots");
    return PASUR_E_OVERFLOW;
  }
  return PASUR_OK;
}

int bad_roots(int round) {
  set_error("roots must be strictly ascending by (pool, bonus, ca, cb, d), hold valid "
            "scores and pools of cards dealt before round %d", round);
  return PASUR_E_INVAL;
}

uint64_t dealt_before(const uint8_t *deck, int round) {
  uint64_t dealt = 0;
  for (int i = 0; i < 4 + 8 * round; ++i) dealt |= 1ull << deck[i];
  return dealt;
}

DealInfo deal_info(const uint8_t *deck, int round) {
  DealInfo di;
  for (int b = 0; b < 8; ++b) di.card[b] = deck[4 + 8 * round + b];
  for (int w = 0; w < 2; ++w) {
    int idx[4] = {0, 1, 2, 3};
    std::sort(idx, idx + 4, [&](int a, int b) { return di.card[4 * w + a] < di.card[4 * w + b]; });
    for (int j = 0; j < 4; ++j) di.order[w][j] = (uint8_t)idx[j];
  }
  return di;
}

}  // namespace

extern "C" void pasur_gt_free(pasur_gt *g) {
  if (!g) return;
  blocks_retire(g->anchor, g->block, 9);
  delete g;
}

namespace {

// The arrays of level l with n nodes, and room for the moves' counts.
int alloc_level(pasur_gt *g, int l, int64_t n, uint64_t **counts) {
  g->n[l] = n;
  Arena a;
  a.want(&g->pool[l], n);
  a.want(&g->rs[l], n);
  a.want(&g->hands[l], n);
  if (l > 0) {
    a.want(&g->act_cap[l], n);
    a.want(&g->parent[l], n);
    a.want(&g->act_card[l], n);
  }
  if (l < 8) {
    a.want(&g->child_begin[l], n + 1);
    a.want(counts, n);
  }
  PASUR_TRY(a.alloc());
  g->block[l] = a.release();
  return PASUR_OK;
}

int build_levels(pasur_gt *g, const pasur_root *d_roots, int64_t n_roots, hipStream_t stream) {
  Arena scratch, level_words;
  HostWords host(stream);  // its end waits for the stream before the arenas'
  if (!host.ok()) return PASUR_E_NOMEM;
  PASUR_TRY(anchor_alloc(&g->anchor));
  int32_t *pos = nullptr;
  int64_t *words = nullptr;
  scratch.want(&pos, n_roots + 1);
  scratch.want(&words, scan_scratch(n_roots));
  PASUR_TRY(scratch.alloc());
  k_check_roots<<<grid_for(n_roots), kThreads, 0, stream>>>(
      n_roots, d_roots, dealt_before(g->deck, g->round), host.dev(0), nullptr);
  scan_enqueue(PoolChange{d_roots}, OffsetsOut{pos, 0}, n_roots, 1, words, host.dev(1), stream);
  PASUR_TRY(host.wait());
  if (host[0]) return bad_roots(g->round);
  // level 0: distinct root pools (ascending because the roots are sorted)
  uint64_t *counts = nullptr;
  PASUR_TRY(alloc_level(g, 0, host[1], &counts));
  k_gt_roots<<<grid_for(n_roots), kThreads, 0, stream>>>(n_roots, d_roots, pos, g->pool[0],
                                                         g->hands[0], g->rs[0]);
  (void)host.dev(0);  // and reads the scratch until it has ended
  const DealInfo di = deal_info(g->deck, g->round);
  // scans of the levels: their scratch grows with them (every scan has ended
  // when the next level's begins)
  int64_t have = 0;
  int64_t *lw = nullptr;
  for (int l = 0; l < 8; ++l) {
    const int64_t n = g->n[l];
    const unsigned grid = (unsigned)((4 * n + kThreads - 1) / kThreads);
    if (n >= kScanTile && scan_scratch(n) > have) {
      block_free(level_words.release());
      level_words = Arena();
      have = 4 * scan_scratch(n);
      level_words.want(&lw, have);
      PASUR_TRY(level_words.alloc());
    }
    k_gt_count<<<grid, kThreads, 0, stream>>>(n, g->pool[l], g->hands[l], di, l & 1, counts);
    scan_enqueue(MovesIn{counts}, OffsetsOut{g->child_begin[l], 0}, n, 1, lw, host.dev(2), stream);
    PASUR_TRY(host.wait());
    PASUR_TRY(total_fits(host[2]));
    uint64_t *next_counts = nullptr;
    PASUR_TRY(alloc_level(g, l + 1, host[2], &next_counts));
    k_gt_fill<<<grid, kThreads, 0, stream>>>(
        n, g->round, l, g->pool[l], g->hands[l], g->rs[l], g->child_begin[l], counts, di,
        g->pool[l + 1], g->hands[l + 1], g->rs[l + 1], g->parent[l + 1], g->act_card[l + 1],
        g->act_cap[l + 1]);
    PASUR_TRY_HIP(hipGetLastError());
    counts = next_counts;
    (void)host.dev(0);  // the fill is pending
  }
  return host.wait();
}

}  // namespace

extern "C" int pasur_build_round_tree(const uint8_t deck[52], int round,
                                      const pasur_root *d_roots, int64_t n_roots,
                                      pasur_gt **out_gt, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!out_gt) {
    set_error("out_gt is NULL");
    return PASUR_E_INVAL;
  }
  *out_gt = nullptr;
  if (round < 0 || round > 5) {
    set_error("round %d outside 0..5", round);
    return PASUR_E_RANGE;
  }
  PASUR_TRY(validate_deck(deck));
  PASUR_TRY(check_root_list(d_roots, n_roots));
  pasur_gt *g = new pasur_gt();
  std::memset(g, 0, sizeof(*g));
  g->round = round;
  std::memcpy(g->deck, deck, 52);
  const int st = build_levels(g, d_roots, n_roots, stream);
  if (st) {
    pasur_gt_free(g);
    return st;
  }
  *out_gt = g;
  return PASUR_OK;
}

extern "C" int pasur_gt_sizes(const pasur_gt *gt, int64_t n[9]) {
  if (!gt || !n) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  for (int l = 0; l < 9; ++l) n[l] = gt->n[l];
  return PASUR_OK;
}

extern "C" int pasur_gt_read(const pasur_gt *gt, int field, int level, void *host_dst) {
  if (!gt || !host_dst) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (level < 0 || level > 8) {
    set_error("level %d outside 0..8", level);
    return PASUR_E_RANGE;
  }
  const int64_t n = gt->n[level];
  const void *src = nullptr;
  size_t bytes = 0;
  switch (field) {
    case PASUR_GT_POOL: src = gt->pool[level]; bytes = n * 8; break;
    case PASUR_GT_HANDS: src = gt->hands[level]; bytes = n; break;
    case PASUR_GT_RS: src = gt->rs[level]; bytes = n * 8; break;
    case PASUR_GT_PARENT: src = gt->parent[level]; bytes = n * 4; break;
    case PASUR_GT_CHILD_BEGIN:
      src = level < 8 ? gt->child_begin[level] : nullptr;
      bytes = (n + 1) * 4;
      break;
    case PASUR_GT_ACT_CARD: src = gt->act_card[level]; bytes = n; break;
    case PASUR_GT_ACT_CAP: src = gt->act_cap[level]; bytes = n * 8; break;
    default:
      set_error("unknown GT field %d", field);
      return PASUR_E_RANGE;
  }
  if (!src) {
    set_error("GT field %d does not exist at level %d", field, level);
    return PASUR_E_INVAL;
  }
  PASUR_TRY_HIP(hipMemcpy(host_dst, src, bytes, hipMemcpyDeviceToHost));
  return PASUR_OK;
}

// --------------------------------------------------------------------------
// Unfolding (section "In-Hand Updates") and Between-Hand linkage
// --------------------------------------------------------------------------
namespace {

constexpr int kKeyWords = 65536 / 64;

__global__ void k_clear_words(unsigned long long *w, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = 0;
}

// The score table from the set of the roots' score keys (one workgroup, a
// thread per 64 keys): ids ascend with the key; before[i] = ids below key 64 i.
__global__ void __launch_bounds__(kKeyWords)
    k_score_table(const unsigned long long *__restrict__ keys, int32_t *__restrict__ before,
                  int8_t *__restrict__ tab, int64_t *__restrict__ total) {
  __shared__ int part[kKeyWords / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  unsigned long long m = keys[t];
  const int n = __popcll(m), incl = wave_inclusive(n, lane);
  if (lane == 63) part[w] = incl;
  __syncthreads();
  int s = incl - n;
  for (int k = 0; k < w; ++k) s += part[k];
  before[t] = s;
  if (t == kKeyWords - 1) *total = s + n;
  for (; m; m &= m - 1, ++s) {
    int ca, cb, d, bonus;
    score_unkey((uint32_t)(64 * t + __ffsll((long long)m) - 1), &ca, &cb, &d, &bonus);
    tab[4 * s + 0] = (int8_t)ca;
    tab[4 * s + 1] = (int8_t)cb;
    tab[4 * s + 2] = (int8_t)d;
    tab[4 * s + 3] = (int8_t)bonus;
  }
}

struct GtChildBegin {
  const int32_t *cb[8];
};

// Per FGT root: its GT root (index of its pool among the distinct pools),
// its score id, and the descendant range [lo, hi) of that GT root on every
// level (a GT subtree is contiguous on each level because levels are
// parent-major).
__global__ void k_root_ranges(int64_t n_roots, const pasur_root *__restrict__ roots,
                              const int32_t *__restrict__ pool_pos, const uint64_t *__restrict__ gt_pool0,
                              int64_t gt_n0, const unsigned long long *__restrict__ keys,
                              const int32_t *__restrict__ before, GtChildBegin gt,
                              int32_t *__restrict__ lo, int32_t *__restrict__ hi,
                              int32_t *__restrict__ root_sid, int64_t *__restrict__ bad) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_roots) return;
  const pasur_root r = roots[j];
  // inclusive scan of pool-change flags; roots that are not the game tree's
  // are reported and kept inside its arrays
  int32_t g = pool_pos[j + 1] - 1;
  if (g >= gt_n0) g = (int32_t)gt_n0 - 1;
  if (gt_pool0[g] != r.pool) *bad = 1;
  const uint32_t k = score_key(r.ca, r.cb, r.d, r.bonus) & 0xFFFF;
  root_sid[j] = before[k >> 6] + __popcll(keys[k >> 6] & ((1ull << (k & 63)) - 1));
  int32_t l0 = g, h0 = g + 1;
  lo[j] = l0;
  hi[j] = h0;
  for (int l = 0; l < 8; ++l) {
    l0 = gt.cb[l][l0];
    h0 = gt.cb[l][h0];
    lo[(int64_t)(l + 1) * n_roots + j] = l0;
    hi[(int64_t)(l + 1) * n_roots + j] = h0;
  }
}

// Nodes of every root's subtree on level `batch`.
struct RangeSizes {
  using Acc = int64_t;
  const int32_t *lo, *hi;
  int64_t n_roots;
  __device__ __forceinline__ int64_t operator()(int batch, int64_t j) const {
    return hi[batch * n_roots + j] - lo[batch * n_roots + j];
  }
};

struct FgtFill {
  int64_t n[9];
  unsigned block[10];  // first workgroup of each level
  int64_t n_roots;
  const int32_t *off;  // [9][n_roots + 1] root offsets
  const int32_t *lo;   // [9][n_roots] first GT node of a root
  const int32_t *root_sid;
  const int32_t *gt_parent[9], *gt_cb[8];
  int32_t *gt[9], *sid[9], *parent[9], *cb[8];
};
constexpr int kFillNodes = 4 * kThreads;  // per workgroup

// FGT nodes of a level, four consecutive ones per thread (16-byte stores): the
// root of the first (binary search in the level's root offsets, between the
// roots of the workgroup's first and last node), then of each its GT node, score
// id, parent and child range.  Bound by the 16 B written per node; one node per
// thread, with a search over all roots or between the workgroup's, wrote 1.8e8
// nodes in 2.1 ms.
__global__ void __launch_bounds__(kThreads) k_fgt_fill(FgtFill a) {
  __shared__ int64_t bound[2];
  int l = 0;
#pragma unroll
  for (int k = 1; k < 9; ++k) l += blockIdx.x >= a.block[k] ? 1 : 0;
  const int64_t n = a.n[l], on = a.n_roots + 1;
  const int64_t i0 = (int64_t)(blockIdx.x - a.block[l]) * kFillNodes;
  const int32_t *const off = a.off + l * on;
  auto root_of = [&](int64_t i, int64_t lo, int64_t hi) {
    while (hi - lo > 1) {  // largest j with off[j] <= i
      const int64_t m = (lo + hi) >> 1;
      if (off[m] <= i) lo = m; else hi = m;
    }
    return lo;
  };
  if ((threadIdx.x & 63) == 0 && threadIdx.x < 128) {
    const int64_t last = i0 + kFillNodes < n ? i0 + kFillNodes - 1 : n - 1;
    bound[threadIdx.x >> 6] = root_of(threadIdx.x == 0 ? i0 : last, 0, a.n_roots);
  }
  __syncthreads();
  const int64_t i = i0 + 4 * threadIdx.x;
  if (i >= n) return;
  int64_t j = root_of(i, bound[0], bound[1] + 1);
  const int32_t *const lo = a.lo + l * a.n_roots;
  int32_t gt[4], sid[4], par[4], cb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t x = i + k < n ? i + k : n - 1;
    while (j + 1 < a.n_roots && off[j + 1] <= x) ++j;
    const int32_t g = lo[j] + (int32_t)(x - off[j]);
    gt[k] = g;
    sid[k] = a.root_sid[j];
    par[k] = l > 0 ? (off - on)[j] + (a.gt_parent[l][g] - (lo - a.n_roots)[j]) : 0;
    cb[k] = l < 8 ? (off + on)[j] + (a.gt_cb[l][g] - (lo + a.n_roots)[j]) : 0;
  }
  auto put = [&](int32_t *p, const int32_t *v) {
    if (i + 4 <= n) {
      *reinterpret_cast<int4 *>(p + i) = make_int4(v[0], v[1], v[2], v[3]);
    } else {
      for (int k = 0; i + k < n; ++k) p[i + k] = v[k];
    }
  };
  put(a.gt[l], gt);
  put(a.sid[l], sid);
  if (l > 0) put(a.parent[l], par);
  if (l < 8) {
    put(a.cb[l], cb);
    if (i + 4 >= n) a.cb[l][n] = (int32_t)a.n[l + 1];
  }
}

__device__ inline void combine_score(const int8_t *s, uint64_t rs, int *ca, int *cb, int *d,
                                     int *bonus, int *pts) {
  const int acl = (int8_t)(rs & 0xFF), bcl = (int8_t)((rs >> 8) & 0xFF);
  const int apt = (int8_t)((rs >> 24) & 0xFF), asr = (int8_t)((rs >> 32) & 0xFF);
  const int bpt = (int8_t)((rs >> 40) & 0xFF), bsr = (int8_t)((rs >> 48) & 0xFF);
  int a = s[0], b = s[1], dd = s[2], bo = s[3];
  const int p = (apt + 5 * asr) - (bpt + 5 * bsr);
  if (bo == 0) {
    a += acl;
    b += bcl;
  }
  dd += p;
  if (bo == 0 && a >= 7) {
    bo = 1; a = 0; b = 0;
  } else if (bo == 0 && b >= 7) {
    bo = 2; a = 0; b = 0;
  }
  *ca = a; *cb = b; *d = dd; *bonus = bo; *pts = p;
}

// Leaf base utility (equations final_util, passuputil) and, for rounds 0..4,
// the sort key of the leaf's next-round root: the pool compressed to the
// cards dealt so far (order preserving), then the 16-bit score key.
__global__ void k_leaf_pass(int64_t n, int round, const int32_t *__restrict__ f_gt,
                            const int32_t *__restrict__ f_sid, const int8_t *__restrict__ tab,
                            const uint64_t *__restrict__ gt_rs, const uint64_t *__restrict__ gt_pool,
                            uint64_t dealt, int16_t *__restrict__ base,
                            int8_t *__restrict__ bonus_out, uint64_t *__restrict__ keys,
                            int32_t *__restrict__ idx) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t t = f_gt[i];
  int ca, cb, d, bonus, pts;
  combine_score(tab + 4 * f_sid[i], gt_rs[t], &ca, &cb, &d, &bonus, &pts);
  if (round == 5) {
    base[i] = (int16_t)((bonus == 1 ? 7 : (bonus == 2 ? -7 : 0)) + pts);
    bonus_out[i] = (int8_t)bonus;
    return;
  }
  base[i] = (int16_t)pts;
  const uint64_t p = gt_pool[t];
  uint64_t cp = 0;
  for (uint64_t m = p; m; m &= m - 1) {
    const int c = __ffsll((long long)m) - 1;
    cp |= 1ull << __popcll(dealt & ((1ull << c) - 1));
  }
  keys[i] = (cp << 16) | score_key(ca, cb, d, bonus);
  idx[i] = (int32_t)i;
}

// 1 where a sorted key differs from the one before it.
struct KeyChange {
  using Acc = int;
  const uint64_t *keys;
  __device__ __forceinline__ int operator()(int, int64_t j) const {
    return j == 0 || keys[j] != keys[j - 1] ? 1 : 0;
  }
};

struct DealtCards {
  uint8_t card[52];  // cards dealt up to the end of the round, ascending
};

__global__ void k_next_roots(int64_t n, const uint64_t *__restrict__ keys,
                             const int32_t *__restrict__ idx, const int32_t *__restrict__ pos,
                             DealtCards dc,
                             pasur_root *__restrict__ next, int32_t *__restrict__ link) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t u = pos[k + 1] - 1;
  link[idx[k]] = u;
  if (pos[k] != u) return;  // not the first of its key
  const uint64_t key = keys[k];
  uint64_t pool = 0;
  for (uint64_t m = key >> 16; m; m &= m - 1) pool |= 1ull << dc.card[__ffsll((long long)m) - 1];
  int ca, cb, d, bonus;
  score_unkey((uint32_t)(key & 0xFFFF), &ca, &cb, &d, &bonus);
  pasur_root r;
  r.pool = pool;
  r.ca = (int8_t)ca;
  r.cb = (int8_t)cb;
  r.d = (int8_t)d;
  r.bonus = (int8_t)bonus;
  r.pad = 0;
  next[u] = r;
}

}  // namespace

extern "C" void pasur_fgt_free(pasur_fgt *f) {
  if (!f) return;
  // (one segment index per state type and per choice of block and seg_nodes)
  void *blocks[kRetired] = {f->off_block, f->block, f->next_block};
  const int n = 3 + seg_index_blocks(f->seg_index, blocks + 3, kRetired - 3);
  blocks_retire(f->anchor, blocks, n);
  std::free(f->h_root_off);
  std::free(f->h_root_seg);
  sweep_index_free(f->sweep);
  seg_index_free(f->seg_index);
  delete f;
}

namespace {

int unfold_impl(const pasur_gt *gt, const pasur_root *d_roots, int64_t n_roots, pasur_fgt *f,
                hipStream_t stream) {
  Arena kept, scratch, levels, leaves;
  HostWords host(stream);  // its end waits for the stream before the arenas'
  if (!host.ok()) return PASUR_E_NOMEM;
  PASUR_TRY(anchor_alloc(&f->anchor));
  enum { H_BAD, H_POOLS, H_SCORES, H_MISMATCH, H_LEVEL, H_SORT = H_LEVEL + 9, H_NEXT = H_SORT + 2 };
  f->n_roots = n_roots;
  // --- roots: score ids, GT roots, descendant ranges, offsets per level
  int32_t *off = nullptr, *pos = nullptr, *before = nullptr, *lo = nullptr, *hi = nullptr;
  int32_t *root_sid = nullptr;
  unsigned long long *keys = nullptr;
  int64_t *words = nullptr;
  kept.want(&off, 9 * (n_roots + 1));
  kept.want(&f->score_tab, 4 * std::min<int64_t>(n_roots, 65536));
  PASUR_TRY(kept.alloc());
  f->off_block = kept.release();
  for (int l = 0; l <= 8; ++l) f->root_off[l] = off + l * (n_roots + 1);
  scratch.want(&pos, n_roots + 1);
  scratch.want(&before, kKeyWords);
  scratch.want(&keys, kKeyWords);
  scratch.want(&lo, 9 * n_roots);
  scratch.want(&hi, 9 * n_roots);
  scratch.want(&root_sid, n_roots);
  scratch.want(&words, scan_scratch(n_roots, 9));
  PASUR_TRY(scratch.alloc());
  f->h_root_off = (int32_t *)std::malloc(sizeof(int32_t) * 9 * (size_t)(n_roots + 1));
  if (!f->h_root_off) {
    set_error("host allocation failed");
    return PASUR_E_NOMEM;
  }
  GtChildBegin gcb;
  for (int l = 0; l < 8; ++l) gcb.cb[l] = gt->child_begin[l];
  const unsigned grid = grid_for(n_roots);
  k_clear_words<<<grid_for(kKeyWords), kThreads, 0, stream>>>(keys, kKeyWords);
  k_check_roots<<<grid, kThreads, 0, stream>>>(n_roots, d_roots, dealt_before(gt->deck, gt->round),
                                               host.dev(H_BAD), keys);
  scan_enqueue(PoolChange{d_roots}, OffsetsOut{pos, 0}, n_roots, 1, words, host.dev(H_POOLS), stream);
  k_score_table<<<1, kKeyWords, 0, stream>>>(keys, before, f->score_tab, host.dev(H_SCORES));
  k_root_ranges<<<grid, kThreads, 0, stream>>>(n_roots, d_roots, pos, gt->pool[0], gt->n[0], keys,
                                               before, gcb, lo, hi, root_sid,
                                               host.dev(H_MISMATCH));
  scan_enqueue(RangeSizes{lo, hi, n_roots}, OffsetsOut{off, n_roots + 1}, n_roots, 9, words,
               host.dev(H_LEVEL), stream);
  PASUR_TRY_HIP(hipGetLastError());
  PASUR_TRY_HIP(hipMemcpyAsync(f->h_root_off, off, sizeof(int32_t) * 9 * (size_t)(n_roots + 1),
                               hipMemcpyDeviceToHost, stream));
  PASUR_TRY(host.wait());
  if (host[H_BAD]) return bad_roots(gt->round);
  if (host[H_POOLS] != gt->n[0]) {
    set_error("roots have %lld distinct pools, the game tree %lld roots",
              (long long)host[H_POOLS], (long long)gt->n[0]);
    return PASUR_E_INVAL;
  }
  if (host[H_MISMATCH]) {
    set_error("root pools do not match the game tree's level 0");
    return PASUR_E_INVAL;
  }
  f->n_scores = host[H_SCORES];
  for (int l = 0; l <= 8; ++l) {
    PASUR_TRY(total_fits(host[H_LEVEL + l]));
    f->n[l] = host[H_LEVEL + l];
  }
  // --- all arrays of the levels and leaves
  const int64_t nl = f->n[8];
  const int r = gt->round;
  for (int l = 0; l <= 8; ++l) {
    levels.want(&f->gt[l], f->n[l]);
    levels.want(&f->sid[l], f->n[l]);
    if (l > 0) levels.want(&f->parent[l], f->n[l]);
    if (l < 8) levels.want(&f->child_begin[l], f->n[l] + 1);
  }
  f->value_stop = value_stop(f->n, n_roots, f->h_root_off);
  if (f->value_stop && widest_level(f->n) <= kNoAllocLevel)
    levels.want(&f->split_ws, split_nodes(f));
  levels.want(&f->leaf_base, nl);
  if (r == 5) levels.want(&f->leaf_bonus, nl);
  else levels.want(&f->link, nl);
  PASUR_TRY(levels.alloc());
  f->block = levels.release();
  FgtFill fa;
  fa.block[0] = 0;
  for (int l = 0; l <= 8; ++l) {
    fa.n[l] = f->n[l];
    fa.block[l + 1] = fa.block[l] + (unsigned)((f->n[l] + kFillNodes - 1) / kFillNodes);
    fa.gt_parent[l] = gt->parent[l];
    fa.gt[l] = f->gt[l];
    fa.sid[l] = f->sid[l];
    fa.parent[l] = f->parent[l];
    if (l < 8) {
      fa.gt_cb[l] = gt->child_begin[l];
      fa.cb[l] = f->child_begin[l];
    }
  }
  fa.n_roots = n_roots;
  fa.off = off;
  fa.lo = lo;
  fa.root_sid = root_sid;
  (void)host.dev(H_BAD);  // work is pending
  k_fgt_fill<<<fa.block[9], kThreads, 0, stream>>>(fa);
  PASUR_TRY_HIP(hipGetLastError());
  // --- leaves: base utilities and next-round linkage
  if (r == 5) {
    k_leaf_pass<<<grid_for(nl), kThreads, 0, stream>>>(nl, r, f->gt[8], f->sid[8], f->score_tab,
                                                       gt->rs[8], gt->pool[8], 0, f->leaf_base,
                                                       f->leaf_bonus, nullptr, nullptr);
    return host.wait();
  }
  const uint64_t dealt = dealt_before(gt->deck, r + 1);
  DealtCards dc;
  std::memset(&dc, 0, sizeof(dc));
  for (int c = 0, k = 0; c < 52; ++c)
    if ((dealt >> c) & 1) dc.card[k++] = (uint8_t)c;
  uint64_t *lkeys[2] = {nullptr, nullptr};
  int32_t *lidx[2] = {nullptr, nullptr}, *ints = nullptr, *lpos = nullptr;
  int64_t *lwords = nullptr;
  leaves.want(&lkeys[0], nl);
  leaves.want(&lkeys[1], nl);
  leaves.want(&lidx[0], nl);
  leaves.want(&lidx[1], nl);
  leaves.want(&ints, sort_scratch_ints(nl));
  leaves.want(&lwords, std::max(sort_scratch_words(nl), scan_scratch(nl)));
  leaves.want(&lpos, nl + 1);
  PASUR_TRY(leaves.alloc());
  k_leaf_pass<<<grid_for(nl), kThreads, 0, stream>>>(nl, r, f->gt[8], f->sid[8], f->score_tab,
                                                     gt->rs[8], gt->pool[8], dealt, f->leaf_base,
                                                     nullptr, lkeys[0], lidx[0]);
  PASUR_TRY_HIP(hipGetLastError());
  int at = 0;
  PASUR_TRY(sort_pairs(lkeys, lidx, nl, ints, lwords, host.dev(H_SORT), &at, stream));
  scan_enqueue(KeyChange{lkeys[at]}, OffsetsOut{lpos, 0}, nl, 1, lwords, host.dev(H_NEXT), stream);
  PASUR_TRY(host.wait());
  f->n_next = host[H_NEXT];
  PASUR_TRY(block_alloc(&f->next_block, (size_t)f->n_next * sizeof(pasur_root)));
  f->next_roots = (pasur_root *)f->next_block;
  (void)host.dev(H_BAD);
  k_next_roots<<<grid_for(nl), kThreads, 0, stream>>>(nl, lkeys[at], lidx[at], lpos, dc,
                                                      f->next_roots, f->link);
  return host.wait();
}

}  // namespace

extern "C" int pasur_unfold_scores(const pasur_gt *gt, const pasur_root *d_roots, int64_t n_roots,
                                   pasur_fgt **out_fgt, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!out_fgt || !gt) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  *out_fgt = nullptr;
  PASUR_TRY(check_root_list(d_roots, n_roots));
  pasur_fgt *f = new pasur_fgt();
  std::memset(f, 0, sizeof(*f));
  f->round = gt->round;
  int st = unfold_impl(gt, d_roots, n_roots, f, stream);
  if (st) {
    pasur_fgt_free(f);
    return st;
  }
  *out_fgt = f;
  return PASUR_OK;
}

extern "C" int pasur_fgt_sizes(const pasur_fgt *f, int64_t n[9], int64_t *n_scores,
                               int64_t *n_next) {
  if (!f) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (n)
    for (int l = 0; l < 9; ++l) n[l] = f->n[l];
  if (n_scores) *n_scores = f->n_scores;
  if (n_next) *n_next = f->n_next;
  return PASUR_OK;
}

extern "C" const pasur_root *pasur_fgt_next_roots(const pasur_fgt *f) {
  return f ? f->next_roots : nullptr;
}

extern "C" int pasur_fgt_read(const pasur_fgt *f, int field, int level, void *host_dst) {
  if (!f || !host_dst) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (level < 0 || level > 8) {
    set_error("level %d outside 0..8", level);
    return PASUR_E_RANGE;
  }
  const int64_t n = f->n[level];
  const void *src = nullptr;
  size_t bytes = 0;
  switch (field) {
    case PASUR_FGT_GT: src = f->gt[level]; bytes = n * 4; break;
    case PASUR_FGT_SID: src = f->sid[level]; bytes = n * 4; break;
    case PASUR_FGT_PARENT: src = f->parent[level]; bytes = n * 4; break;
    case PASUR_FGT_CHILD_BEGIN:
      src = level < 8 ? f->child_begin[level] : nullptr;
      bytes = (n + 1) * 4;
      break;
    case PASUR_FGT_SCORE_TAB: src = f->score_tab; bytes = f->n_scores * 4; break;
    case PASUR_FGT_NEXT_ROOTS: src = f->next_roots; bytes = f->n_next * sizeof(pasur_root); break;
    case PASUR_FGT_LINK: src = f->link; bytes = f->n[8] * 4; break;
    case PASUR_FGT_LEAF_BASE: src = f->leaf_base; bytes = f->n[8] * 2; break;
    default:
      set_error("unknown FGT field %d", field);
      return PASUR_E_RANGE;
  }
  if (!src) {
    set_error("FGT field %d does not exist here", field);
    return PASUR_E_INVAL;
  }
  PASUR_TRY_HIP(hipMemcpy(host_dst, src, bytes, hipMemcpyDeviceToHost));
  return PASUR_OK;
}

extern "C" int pasur_gt_get_view(const pasur_gt *g, pasur_gt_view *out) {
  if (!g || !out) {
    pasur::set_error("null argument");
    return PASUR_E_INVAL;
  }
  std::memset(out, 0, sizeof(*out));
  out->round = g->round;
  for (int l = 0; l < 9; ++l) {
    out->n[l] = g->n[l];
    out->pool[l] = g->pool[l];
    out->hands[l] = g->hands[l];
    out->rs[l] = g->rs[l];
    out->parent[l] = g->parent[l];
    out->act_card[l] = g->act_card[l];
    out->act_cap[l] = g->act_cap[l];
    if (l < 8) out->child_begin[l] = g->child_begin[l];
  }
  return PASUR_OK;
}

extern "C" int pasur_fgt_get_view(const pasur_fgt *f, pasur_fgt_view *out) {
  if (!f || !out) {
    pasur::set_error("null argument");
    return PASUR_E_INVAL;
  }
  std::memset(out, 0, sizeof(*out));
  out->round = f->round;
  for (int l = 0; l < 9; ++l) {
    out->n[l] = f->n[l];
    out->gt[l] = f->gt[l];
    out->sid[l] = f->sid[l];
    out->parent[l] = f->parent[l];
    if (l < 8) out->child_begin[l] = f->child_begin[l];
  }
  out->score_tab = f->score_tab;
  out->n_scores = f->n_scores;
  out->next_roots = f->round < 5 ? f->next_roots : nullptr;
  out->n_next = f->round < 5 ? f->n_next : 0;
  out->link = f->round < 5 ? f->link : nullptr;
  out->leaf_base = f->leaf_base;
  return PASUR_OK;
}
