// pasur_seg.hip -- the persistent segment schedule of full-width DCFR (section
// "CFR Algorithm": CodeSnippets FindReachProbability and FindUtility, equations
// DFCR_REG, RM and DFCR_AVG) and the batched plans that launch it.
//
// The subgames below different roots never interact inside a round, so one
// workgroup owns a segment -- a run of consecutive roots of one tree -- and
// runs all iterations on it.  A launch can cover the trees of many deals.
//
// The segment lives in LDS in a compact form, made when the launch starts and
// dissolved when it ends; no iteration touches memory.  What bounds an
// iteration is then the dependent steps between the workgroup's barriers on
// small launches, and the FP64 instructions on large ones.  Five choices serve
// both; none changes a result:
//
//  * Forced chains are not iterated.  A node of level 6 or 7 whose whole
//    subtree is one line (each player holds one card there, so most nodes of
//    those levels are; called passive) keeps sigma = 1 and zero regret below
//    itself and the utility of its leaf.  Its parent's update carries along
//    the average sums of the at most two edges below it, and nothing else of
//    them exists in LDS: about half of a tree's nodes.
//  * Sibling groups in classes.  The active (non-passive) nodes of a level are
//    ordered by their number of children k, and the j-th children of the n
//    nodes of a class lie side by side: child j of a node is slot + j * n.  The
//    64 parents of a wave then loop over the same k, without divergence, and
//    read consecutive LDS words.
//  * Values first, updates later.  Going up, only utilities pass between the
//    levels; the regret, matching and average updates of all levels run
//    together afterwards in one pass, each parent recomputing its own utility.
//  * One reach per node.  An edge scales its mover's reach only, so a node
//    stores the reach of the player who moved last; the other one's is its
//    parent's.  Two consecutive levels then do not depend on each other, and go
//    down in one step.
//  * A lane per edge where a loop over children would be waited for: at the
//    topmost levels, which one wave runs by itself, and at nodes with more than
//    four children.
//
// An iteration takes one barrier per level above the topmost levels and one
// after the updates.  Every parent's sums run over its children in child order
// in FP64 without contraction, whatever order the nodes are stored in: the
// state ends bit for bit as with the level-synchronous kernels.
//
// Measured (FP32 unless said): seven roots of 3,200 nodes, FP64, 11.3 -> 4.5 us
// per iteration against one phase per level over all nodes; 38,652 roots of 3,900
// nodes, 0.53 ms per iteration (2.8e11 nodes/s, VALU 50 to 64% busy); a batch of
// 64 deals (7.6e7 nodes), 50 iterations, 56 -> 16.2 ms with all that surrounds it.
//
// A segment too large for LDS keeps its far arrays in device memory (roots of
// more than 9,000 to 14,000 nodes, by their shape, F64 half of that), or all of the
// form (32,000, F64 16,000).  One that has no compact form (a node of more than 63
// moves, more than 65,535 edges, discounts that are not numbers) is iterated in
// place in global memory, one phase per level.
#pragma clang fp contract(off)

#include "pasur_internal.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <utility>
#include <vector>

using namespace pasur;

namespace {

// One (tree, state) pair of a launch.
template <class T>
struct ItemDesc {
  const int32_t *off[9];     // per-root level offsets
  const int32_t *parent[9];  // levels 1..8
  const int32_t *cb[9];      // levels 0..7
  T *sigma[9], *R[9], *Sbar[9], *ra[9], *rb[9], *u[9];
  double *vacc;
};

struct Seg {
  int32_t item, j0, j1;  // roots j0 .. j1-1 of item
  int32_t far, far_n;    // place and size of its far arrays in units of kFarUnit
  int32_t form;          // where the compact form's arrays are
};
// LDS; "far" arrays in device memory; all arrays there; no compact form.
enum { F_LDS, F_FAR, F_ALL_FAR, F_NONE };
constexpr int kFarUnit = 256;

// ---- the compact form ----------------------------------------------------------

// What a segment's LDS layout depends on: active nodes (levels 0..7), their
// children (edges), those of levels 6 and 7, roots, and the tree's nodes.
struct SegCounts {
  int na, ne, ne67, roots;
  int c07, c6, c7;  // nodes of levels 0..7, of level 6, of level 7
};

// Byte offsets of a segment's arrays in LDS.  While the form is made, class
// tables and a map from tree nodes to active nodes take the edge arrays'
// place.  A segment too large for this keeps rs, chain, kids, up and pos (its far
// arrays) in device memory: each is read once per iteration or pass, in order,
// while su and x are read at random.  That carries roots of up to 32,000
// nodes (f32) at a fifth of the time of iterating them in place.
struct SegLds {
  uint32_t b6, b7;   // passive bits of levels 6 and 7
  uint32_t tmp;      // = the start of the edge arrays
  uint32_t vacc;     // double per root: running sum of root utilities
  uint32_t su, rs;   // per edge: sigma and utility, regret and average sum (pairs of T);
                     // su also per root, after the edges
  uint32_t chain;    // per edge of levels 6 and 7: the average sums below it (pair of T)
  uint32_t x;        // T per active node, then per root: reaches
  uint32_t kids, up; // words of an active node, see below
  uint32_t pos;      // 16 bits per active node: its index within its level of the segment
  uint32_t list;     // edges that are updated a lane each, see list_build
  uint32_t bytes;
  uint32_t far;      // bytes of the far arrays
};
// Words of active node i:
//   kids.x: slot of its first child | distance to the next child << 16
//   kids.y: its own slot as a child | number of children << 16 | level << 24
//           | its children are in the list << 31
//   up:     its parent | active node two levels up << 16
// A root's slot as a child is its place in su after the edges, and its parent
// is its second entry of x (the reach of the player who moves first).  After
// the roots su has a pair of zeros, what a node reads in place of further children,
// and a spare pair, which it writes in their place; rs and chain have a spare edge.
template <class T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

constexpr int kClasses = 64;  // children per node: 0 .. 63
constexpr uint32_t kTableBytes = 3 * 8 * kClasses * 4;
constexpr int kList = 512;     // capacity of the list
constexpr uint32_t kNoEdge = 0xFFFFFFFFu;
constexpr int kTopEdges = 64;  // one wave updates them
constexpr uint32_t kListed = 1u << 31;

template <class U>
__host__ __device__ inline U align16(U x) {
  return (x + 15u) & ~(U)15u;
}

__host__ __device__ inline SegLds seg_layout(const SegCounts &c, uint32_t t, int form) {
  SegLds L;
  uint32_t p = 0, q = 0;
  auto take = [&p](uint32_t bytes) {
    const uint32_t at = p;
    p = align16(p + bytes);
    return at;
  };
  auto take_far = [&](uint32_t bytes) {
    if (form == F_LDS) return take(bytes);
    const uint32_t at = q;
    q = align16(q + bytes);
    return at;
  };
  L.b6 = take((uint32_t)((c.c6 + 63) / 64) * 8u);
  L.b7 = take((uint32_t)((c.c7 + 63) / 64) * 8u);
  L.tmp = p;
  const uint32_t tmp_end = p + kTableBytes + align16(2u * (uint32_t)c.c07);
  auto take_near = [&](uint32_t bytes) { return form == F_ALL_FAR ? take_far(bytes) : take(bytes); };
  L.su = take_near(2 * t * (uint32_t)(c.ne + c.roots + 2));
  L.rs = take_far(2 * t * (uint32_t)(c.ne + 1));
  L.chain = take_far(2 * t * (uint32_t)(c.ne67 + 1));
  L.x = take_near(t * (uint32_t)(c.na + c.roots));
  L.vacc = take(8u * (uint32_t)c.roots);
  if (p < tmp_end) p = tmp_end;
  L.kids = take_far(8u * (uint32_t)c.na);
  L.up = take_far(4u * (uint32_t)c.na);
  L.pos = take_far(2u * (uint32_t)c.na);
  L.list = take(4u * kList);
  L.bytes = p;
  L.far = q;
  return L;
}
// Indices are held in 16 bits.
__host__ __device__ inline bool seg_indices_fit(const SegCounts &c) {
  return c.ne + c.roots + 2 < 65536 && c.na + c.roots < 65536 && c.c07 < 8 * 65536;
}

extern __shared__ __align__(16) unsigned char g_lds[];
// the segment's active nodes and edges per level (first index; [8], [9]: end)
__shared__ int g_nb[9], g_sb[10];
__shared__ int g_sum[2][8];
__shared__ int g_bad;
__shared__ int g_list_top, g_list_end;  // where the list's two parts end

template <class T>
__device__ __forceinline__ T *lds(uint32_t off) {
  return reinterpret_cast<T *>(g_lds + off);
}

// A far array, and su or x.
template <class T, int FORM>
__device__ __forceinline__ T *arr(unsigned char *far, uint32_t off) {
  return FORM != F_LDS ? reinterpret_cast<T *>(far + off) : lds<T>(off);
}
template <class T, int FORM>
__device__ __forceinline__ T *near(unsigned char *far, uint32_t off) {
  return FORM == F_ALL_FAR ? reinterpret_cast<T *>(far + off) : lds<T>(off);
}

__device__ __forceinline__ bool bit_of(uint32_t off, int i) {
  return (lds<uint32_t>(off)[i >> 5] >> (i & 31)) & 1u;
}

// Between steps that one wave runs by itself: LDS accesses of a wave run in
// order, and only the compiler has to keep them so.
template <int FORM>
__device__ __forceinline__ void wave_order() {
  if (FORM == F_ALL_FAR) __threadfence_block();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// A node's children: slot, distance and number, from its words.
struct Kids {
  int e, step, k;
  __device__ __forceinline__ Kids(uint2 w)
      : e((int)(w.x & 0xFFFFu)), step((int)(w.x >> 16)), k((int)(w.y >> 16) & 0xFF) {}
};

// Levels 0 .. top-1: at most kTopEdges children (and so fewer nodes).
__device__ __forceinline__ int top_levels() {
  int top = 0;
  while (top < 4 && g_sb[top + 2] <= kTopEdges) ++top;
  return top;
}

// The list of edges that are updated a lane each instead of in a loop over a
// node's children: first those of the top levels' nodes, whose updates every
// other wave would wait for, then of nodes with more than four children.  An
// entry is the parent | the child's number << 16.  The children of a node have
// neighbouring places of one wave, so that its lanes can follow each other
// without a barrier; a node that no longer fits in a wave begins the next.  Nodes
// past the list's end stay with update_many.  For one wave; before it, the list
// is kNoEdge.
template <int FORM>
__device__ __forceinline__ void list_build(unsigned char *far, const SegLds &L) {
  const int lane = threadIdx.x & 63;
  uint2 *const w_kids = arr<uint2, FORM>(far, L.kids);
  uint32_t *const list = lds<uint32_t>(L.list);
  const int top = top_levels();
  int at = 0;
  bool room = true;
  for (int l = 0; l < 8 && room; ++l) {
    if (l == top) {
      at = (at + 63) & ~63;
      if (lane == 0) g_list_top = at;
    }
    const int end = g_nb[l + 1];
    for (int id0 = g_nb[l]; id0 < end && room; id0 += 64) {
      const int id = id0 + lane;
      const Kids n(id < end ? w_kids[id] : make_uint2(0, 0));
      const bool in = n.k > (l < top ? 0 : 4);
      unsigned long long todo = __ballot(in);
      if (!todo) break;  // of a level's nodes the widest come first
      int mine = -1;
      while (todo && room) {
        const int i = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int k = __builtin_amdgcn_readlane(n.k, i);
        if ((at & 63) + k > 64) at = (at + 63) & ~63;
        room = at + k <= kList;
        if (room) {
          if (lane == i) mine = at;
          at += k;
        }
      }
      if (mine >= 0) {
        for (int j = 0; j < n.k; ++j) list[mine + j] = (uint32_t)id | ((uint32_t)j << 16);
        w_kids[id].y |= kListed;
      }
    }
  }
  if (lane == 0) g_list_end = at;
}

// The level arrays of the segment's tree, from its first node on each level on:
// a pointer table in LDS, since the 72 pointers don't fit in registers and a
// level may differ from lane to lane.
enum { P_SIGMA, P_R, P_SBAR, P_U, P_RA, P_RB, P_PARENT, P_CB };
__shared__ void *g_ptab[8][9];
__shared__ int g_lo[9], g_cnt[9];  // first node and nodes per level

template <class T>
using GlobalPtr = __attribute__((address_space(1))) T *;

template <class T>
__device__ __forceinline__ GlobalPtr<T> tab(int slot, int l) {
  return (GlobalPtr<T>)g_ptab[slot][l];
}

template <class T>
__device__ __forceinline__ void seg_open(const ItemDesc<T> &D, int j0, int j1) {
  if (threadIdx.x < 9) {
    const int l = threadIdx.x;
    const GlobalPtr<const int32_t> off = (GlobalPtr<const int32_t>)D.off[l];
    const int lo = off[j0];
    g_ptab[P_SIGMA][l] = l >= 1 ? (void *)(D.sigma[l] + lo) : nullptr;
    g_ptab[P_R][l] = l >= 1 ? (void *)(D.R[l] + lo) : nullptr;
    g_ptab[P_SBAR][l] = l >= 1 ? (void *)(D.Sbar[l] + lo) : nullptr;
    g_ptab[P_U][l] = (void *)(D.u[l] + lo);
    g_ptab[P_RA][l] = l <= 7 ? (void *)(D.ra[l] + lo) : nullptr;
    g_ptab[P_RB][l] = l <= 7 ? (void *)(D.rb[l] + lo) : nullptr;
    g_ptab[P_PARENT][l] = l >= 1 ? (void *)(D.parent[l] + lo) : nullptr;
    g_ptab[P_CB][l] = l <= 7 ? (void *)(D.cb[l] + lo) : nullptr;
    g_lo[l] = lo;
    g_cnt[l] = off[j1] - lo;
  }
  __syncthreads();
}

// Makes the compact form of the segment's roots; false (for every thread) if it
// does not fit in lds_bytes.  `L` is the layout, g_nb and g_sb the levels.
// Every pass runs over the nodes of all levels at once: what it waits for is
// memory latency, and level by level it did so eight times (loading and storing
// a segment of 3,900 nodes took as long as 12 iterations).
template <class T, int BLOCK, int FORM>
__device__ __forceinline__ bool seg_load(const ItemDesc<T> &D, uint32_t lds_bytes,
                                         unsigned char *far, int64_t far_bytes, SegLds &L, int &na,
                                         int &ne) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int NW = BLOCK / 64;
  constexpr uint32_t kPassive = 0xFFFF;
  SegCounts c;
  int at[9];  // nodes above each level
  bool fits = true;
  at[0] = 0;
#pragma unroll
  for (int l = 0; l < 8; ++l) {
    const int n = __builtin_amdgcn_readfirstlane(g_cnt[l]);
    fits = fits && n <= 65535;
    at[l + 1] = fits ? at[l] + n : at[l];
  }
  if (!fits) return false;
  c.roots = at[1];
  c.c07 = at[8];
  c.c6 = at[7] - at[6];
  c.c7 = at[8] - at[7];
  // where bits, tables and the map go does not depend on the other counts
  c.na = c.ne = c.ne67 = 0;
  L = seg_layout(c, sizeof(T), FORM);
  if (L.bytes > lds_bytes) return false;
  uint32_t *const count = lds<uint32_t>(L.tmp);  // per level and class: nodes
  uint32_t *const next = count + 8 * kClasses;   // next rank within the level
  uint32_t *const first = next + 8 * kClasses;   // first slot - first rank
  uint16_t *const map = lds<uint16_t>(L.tmp + kTableBytes);
  auto level_of = [&](int i) {
    int l = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) l += i >= at[k] ? 1 : 0;
    return l;
  };
  auto above = [&](int l) {  // at[l]
    int v = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) v = l == k ? at[k] : v;
    return v;
  };
  // passive nodes: one child, along an edge of sigma 1, that is a leaf of
  // finite utility or passive itself
  if (tid == 0) g_bad = 0;
  for (int i = tid; i < 8 * kClasses; i += BLOCK) count[i] = 0;
#pragma unroll
  for (int l = 7; l >= 6; --l) {
    const int n = l == 7 ? c.c7 : c.c6, lo = g_lo[l + 1];
    const GlobalPtr<const int32_t> cb = tab<const int32_t>(P_CB, l);
    const GlobalPtr<const T> sg = tab<const T>(P_SIGMA, l + 1);
    for (int i0 = tid; i0 < ((n + 63) & ~63); i0 += 4 * BLOCK) {
      int q[4];
      T s1[4];
      bool p[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int i = i0 + m * BLOCK < n ? i0 + m * BLOCK : n - 1;
        q[m] = cb[i] - lo;
        p[m] = cb[i + 1] - lo - q[m] == 1;
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {  // (a node without children: any place will do)
        s1[m] = sg[p[m] ? q[m] : 0];
        if (l == 7) p[m] = p[m] && isfinite((double)tab<const T>(P_U, 8)[p[m] ? q[m] : 0]);
        else p[m] = p[m] && bit_of(L.b7, q[m]);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int i = i0 + m * BLOCK;
        const unsigned long long w = __ballot(i < n && p[m] && (double)s1[m] == 1.0);
        if (lane == 0 && i < n) lds<unsigned long long>(l == 7 ? L.b7 : L.b6)[i >> 6] = w;
      }
    }
    __syncthreads();
  }
  // the active nodes' classes; the map holds their numbers of children for now
  for (int i0 = tid; i0 < c.c07; i0 += 4 * BLOCK) {
    int l[4];
    uint32_t k[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = i0 + m * BLOCK < c.c07 ? i0 + m * BLOCK : i0;
      l[m] = level_of(i);
      const int j = i - above(l[m]);
      const GlobalPtr<const int32_t> cb = tab<const int32_t>(P_CB, l[m]);
      k[m] = (uint32_t)(cb[j + 1] - cb[j]);
      if (l[m] >= 6 && bit_of(l[m] == 6 ? L.b6 : L.b7, j)) l[m] = 8;
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int i = i0 + m * BLOCK;
      if (i >= c.c07) break;
      map[i] = (uint16_t)(l[m] < 8 ? k[m] : kPassive);
      if (l[m] == 8) continue;
      if (k[m] < (uint32_t)kClasses) atomicAdd(&count[l[m] * kClasses + k[m]], 1u);
      else g_bad = 1;
    }
  }
  __syncthreads();
  if (g_bad) return false;
  // classes in order of descending k: lane i of a wave takes k = 63 - i
  for (int l = wave; l < 8; l += NW) {
    const int k = kClasses - 1 - lane;
    const int n = (int)count[l * kClasses + k];
    int nodes = n, kids = n * k;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int a = __shfl_up(nodes, d, 64), b = __shfl_up(kids, d, 64);
      if (lane >= d) {
        nodes += a;
        kids += b;
      }
    }
    next[l * kClasses + k] = (uint32_t)(nodes - n);
    first[l * kClasses + k] = (uint32_t)((kids - n * k) - (nodes - n));
    if (lane == 63) {
      g_sum[0][l] = nodes;
      g_sum[1][l] = kids;
    }
  }
  __syncthreads();
  for (int l = 0; l < 8; ++l) {
    c.na += g_sum[0][l];
    c.ne += g_sum[1][l];
    if (l == 5 || l == 6) c.ne67 += g_sum[1][l];
  }
  na = c.na;
  ne = c.ne;
  L = seg_layout(c, sizeof(T), FORM);
  if (L.bytes > lds_bytes || L.far > far_bytes || !seg_indices_fit(c)) return false;
  if (tid == 0) {
    int a = 0, e = 0;
    for (int l = 0; l < 8; ++l) {
      g_nb[l] = a;
      g_sb[l + 1] = e;
      a += g_sum[0][l];
      e += g_sum[1][l];
    }
    g_nb[8] = a;
    g_sb[9] = e;
  }
  __syncthreads();
  uint2 *const w_kids = arr<uint2, FORM>(far, L.kids);
  uint32_t *const w_up = arr<uint32_t, FORM>(far, L.up);
  uint16_t *const w_pos = arr<uint16_t, FORM>(far, L.pos);
  // every active node's place and its children's slots
  for (int i = tid; i < c.c07; i += BLOCK) {
    const uint32_t k = map[i];
    if (k == kPassive) continue;
    const int l = level_of(i);
    const uint32_t rank = atomicAdd(&next[l * kClasses + k], 1u);
    const uint32_t id = (uint32_t)g_nb[l] + rank;
    w_kids[id] = make_uint2(((uint32_t)g_sb[l + 1] + first[l * kClasses + k] + rank) |
                                (count[l * kClasses + k] << 16),
                            (k << 16) | ((uint32_t)l << 24));
    w_pos[id] = (uint16_t)(i - above(l));
    map[i] = (uint16_t)id;
  }
  __syncthreads();
  // own slots and parents, written by the parents: low halves of the words
  for (int id0 = tid; id0 < na; id0 += 2 * BLOCK) {
    uint2 w[2];
    int l[2], q[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int id = id0 + m * BLOCK < na ? id0 + m * BLOCK : id0;
      w[m] = w_kids[id];
      l[m] = (int)(w[m].y >> 24) & 7;
      q[m] = tab<const int32_t>(P_CB, l[m])[w_pos[id]] - g_lo[l[m] + 1] + above(l[m] + 1);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int id = id0 + m * BLOCK, k = (int)(w[m].y >> 16) & 0xFF;
      if (id >= na) break;
      if (l[m] == 0) {
        *reinterpret_cast<uint16_t *>(&w_kids[id].y) = (uint16_t)(c.ne + id);
        w_up[id] = (uint32_t)(c.na + id);
      }
      if (l[m] == 7) continue;
      uint32_t e = w[m].x & 0xFFFFu;
      for (int j = 0; j < k; ++j, e += w[m].x >> 16) {
        const uint32_t child = map[q[m] + j];
        if (child == kPassive) continue;
        *reinterpret_cast<uint16_t *>(&w_kids[child].y) = (uint16_t)e;
        w_up[child] = (uint32_t)id;
      }
    }
  }
  __syncthreads();
  // the nodes two levels up: high halves
  for (int id = g_nb[1] + tid; id < na; id += BLOCK)
    reinterpret_cast<uint16_t *>(w_up + id)[1] =
        *reinterpret_cast<const uint16_t *>(w_up + *reinterpret_cast<const uint16_t *>(w_up + id));
  // the state; from here on the edge arrays take the tables' place
  Pair<T> *const su = near<Pair<T>, FORM>(far, L.su), *const rs = arr<Pair<T>, FORM>(far, L.rs);
  Pair<T> *const chain = arr<Pair<T>, FORM>(far, L.chain);
  const int e6 = g_sb[6], lo8 = g_lo[8], lo7 = g_lo[7];
  for (int id0 = tid; id0 < na; id0 += 2 * BLOCK) {
    // two nodes, and two children of each, at a time
    int lev[2], kids[2], b[2], e0[2], step[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool in = id0 + u * BLOCK < na;
      const int id = in ? id0 + u * BLOCK : id0;
      const uint2 w = w_kids[id];
      lev[u] = (int)(w.y >> 24) & 7;
      kids[u] = in ? (int)(w.y >> 16) & 0xFF : 0;
      e0[u] = (int)(w.x & 0xFFFFu);
      step[u] = (int)(w.x >> 16);
      b[u] = tab<const int32_t>(P_CB, lev[u])[w_pos[id]] - g_lo[lev[u] + 1];
    }
    for (int j = 0; j < kids[0] || j < kids[1]; j += 2) {
      int q[4], q7[4], q8[4];
      T r[4], sb[4], s0[4], v[4], a1[4], a2[4];
      bool in[4], p[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int u = m / 2, l = lev[u];
        in[m] = j + m % 2 < kids[u];
        q[m] = b[u] + (in[m] ? j + m % 2 : 0);
        r[m] = tab<const T>(P_R, l + 1)[q[m]];
        sb[m] = tab<const T>(P_SBAR, l + 1)[q[m]];
        s0[m] = tab<const T>(P_SIGMA, l + 1)[q[m]];
        v[m] = a1[m] = a2[m] = (T)0;
        if (l == 7) v[m] = tab<const T>(P_U, 8)[q[m]];
        p[m] = in[m] && (l == 5 ? bit_of(L.b6, q[m]) : l == 6 && bit_of(L.b7, q[m]));
        q7[m] = q8[m] = q[m];
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m] && lev[m / 2] == 5) q7[m] = tab<const int32_t>(P_CB, 6)[q[m]] - lo7;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m]) q8[m] = tab<const int32_t>(P_CB, 7)[q7[m]] - lo8;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m]) {
          v[m] = (T)(0.0 + (double)tab<const T>(P_U, 8)[q8[m]]);
          a2[m] = tab<const T>(P_SBAR, 8)[q8[m]];
          if (lev[m / 2] == 5) a1[m] = tab<const T>(P_SBAR, 7)[q7[m]];
        }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int u = m / 2, l = lev[u], e = e0[u] + (j + m % 2) * step[u];
        if (!in[m]) continue;
        rs[e] = Pair<T>{r[m], sb[m]};
        su[e] = Pair<T>{s0[m], v[m]};
        if (l == 5) chain[e - e6] = Pair<T>{a1[m], a2[m]};
        if (l == 6) chain[e - e6] = Pair<T>{a2[m], (T)0};
      }
    }
  }
  if (tid == 0) su[c.ne + c.roots] = Pair<T>{(T)0, (T)0};
  for (int i = tid; i < kList; i += BLOCK) lds<uint32_t>(L.list)[i] = kNoEdge;
  __syncthreads();
  if (wave == 0) list_build<FORM>(far, L);
  for (int id = tid; id < c.roots; id += BLOCK) {
    const int j = w_pos[id];
    near<T, FORM>(far, L.x)[id] = tab<const T>(P_RB, 0)[j];
    near<T, FORM>(far, L.x)[c.na + id] = tab<const T>(P_RA, 0)[j];
    lds<double>(L.vacc)[id] = D.vacc[g_lo[0] + j];
  }
  __syncthreads();
  return true;
}

// uh + the sum of sigma * u over K children (ALL), or at most K, from slot e, in
// child order.  All K are read at once, so that LDS latency is paid once; past
// the last child the pair of zeros is read (adding zero leaves the sum's bits
// alone: it is never -0).
template <class T, int K, bool ALL>
__device__ __forceinline__ double value_few(const Pair<T> *su, int zero, int e, int step, int k,
                                            double uh) {
  Pair<T> p[K];
#pragma unroll
  for (int i = 0; i < K; ++i) p[i] = su[ALL || i < k ? e + i * step : zero];
#pragma unroll
  for (int i = 0; i < K; ++i) uh += (double)p[i].a * (double)p[i].b;
  return uh;
}

// u of an active node.  The form is the wave's: a class's nodes are
// neighbours, so its lanes mostly agree.
template <class T>
__device__ __forceinline__ double node_value(const Pair<T> *su, int zero, const Kids &n) {
  if (!__ballot(n.k != 2)) return value_few<T, 2, true>(su, zero, n.e, n.step, n.k, 0.0);
  if (!__ballot(n.k > 4)) return value_few<T, 4, false>(su, zero, n.e, n.step, n.k, 0.0);
  double uh = 0.0;
  for (int left = n.k, e = n.e; left > 0; left -= 8, e += 8 * n.step)
    uh = value_few<T, 8, false>(su, zero, e, n.step, left, uh);
  return uh;
}

// (as one instruction: fmax would quiet its second operand each time)
__device__ __forceinline__ double matched(double R, int rm_mode, double eps) {
  const double low = rm_mode == PASUR_RM_FLOOR ? eps : 0.0;
  double x;
  asm("v_max_f64 %0, %1, %2" : "=v"(x) : "v"(R), "s"(low));
  return x;
}

// Quotients by one divisor.  The reciprocal is refined once, as a division does
// it, and each quotient takes the division's last three steps (multiply,
// remainder, correction): the same operations, so the same bits, where a division
// would not scale its operands.  That is so for divisors and numerators of
// magnitude 2^-200 .. 2^200 and numerators of zero; `exact` says that a launch's
// numerators are among these, and other divisors take the division itself.
struct Quotient {
  double den, inv;
  bool plain;
  __device__ __forceinline__ Quotient(double d, bool exact) : den(d) {
    // (the exponent's bits: 1023 - 200 .. 1023 + 200)
    plain = !(exact && (uint32_t)__double2hiint(d) - (823u << 20) < (400u << 20));
    inv = __builtin_amdgcn_rcp(d);
    inv = __builtin_fma(inv, __builtin_fma(-d, inv, 1.0), inv);
    inv = __builtin_fma(inv, __builtin_fma(-d, inv, 1.0), inv);
  }
  __device__ __forceinline__ double of(double x) const {
    const double q = x * inv;
    return __builtin_fma(__builtin_fma(-den, q, x), inv, q);
  }
  // x over the sum, or 1 / k where the sum is not positive, by the division
  __device__ __forceinline__ double plainly(double x, int k) const {
    return den > 0.0 ? x / den : 1.0 / (double)k;
  }
};

// Numerators are regrets of type T above the floor.
template <class T>
__device__ __forceinline__ bool exact_quotients(int rm_mode, double eps) {
  const bool floor = rm_mode == PASUR_RM_FLOOR;
  if (floor && eps >= 0x1p-200 && eps <= 0x1p200) return true;
  return sizeof(T) == 4 && (!floor || eps == 0.0);
}

__device__ __forceinline__ double next_regret(double Rq, double r, const IterK &ik, int variant) {
  if (variant == PASUR_DCFR) {
    const double d = Rq > 0.0 ? ik.dpos : ik.dneg;
    return d * Rq + r;
  }
  if (variant == PASUR_CFR_PLUS) {
    const double x = Rq + r;
    return x < 0.0 ? 0.0 : x;
  }
  return Rq + r;
}

// Average sum of a child: w * Sbar + own reach * sigma^t.
template <class T>
__device__ __forceinline__ T average_update(double own, T sg, T sb, const IterK &ik, int variant) {
  const double add = own * (double)sg;
  return (T)(ik.avg_w * (double)sb + (variant == PASUR_CFR_PLUS ? add * ik.avg_t : add));
}

// Average sums of the chain below a child: there first the other player moves
// (reach opp, as inherited), then the mover of the child's parent (the child's
// own reach).
template <class T>
__device__ __forceinline__ void chain_update(Pair<T> *chain, double opp, double own, T sg,
                                             const IterK &ik, int variant) {
  double a1 = opp, a2 = (double)(T)(own * (double)sg);
  if (variant == PASUR_CFR_PLUS) {
    a1 *= ik.avg_t;
    a2 *= ik.avg_t;
  }
  const Pair<T> c = *chain;
  *chain = Pair<T>{(T)(ik.avg_w * (double)c.a + a1), (T)(ik.avg_w * (double)c.b + a2)};
}

// The update of one active node: reaches, regret sign and arrays.
template <class T>
struct Update {
  Pair<T> *su, *rs, *chain;  // chain: of edge 0 (only edges of levels 6 and 7 exist)
  int zero, spare;           // the pair of zeros in su (a spare one follows), rs's spare edge
  int chain_spare;           // and chain's
  double sopp, opp, own;     // signed opponent's, opponent's and own reach
  bool chains, exact;
  IterK ik;
  int variant, rm_mode;
  double eps;
};

// Regret, matching and average updates of the K children of a node (ALL), or at
// most K, without a branch: every child is read once and held in registers, and
// past the last one the work is done on the spare edge.
template <class T, int K, bool ALL>
__device__ __forceinline__ void update_few(const Update<T> &c, const Kids &n) {
  Pair<T> p[K], r[K];
  int e[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const bool in = ALL || i < n.k;
    e[i] = in ? n.e + i * n.step : c.spare;
    p[i] = c.su[in ? e[i] : c.zero];
    r[i] = c.rs[e[i]];
  }
  double uh = 0.0;
#pragma unroll
  for (int i = 0; i < K; ++i) uh += (double)p[i].a * (double)p[i].b;
  double sum = 0.0, m[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    r[i].a = (T)next_regret((double)r[i].a, c.sopp * ((double)p[i].b - uh), c.ik, c.variant);
    m[i] = matched((double)r[i].a, c.rm_mode, c.eps);
    sum += ALL || i < n.k ? m[i] : 0.0;
  }
  const Quotient quo(sum, c.exact);
  T s_new[K];
#pragma unroll
  for (int i = 0; i < K; ++i) s_new[i] = (T)quo.of(m[i]);
  if (__ballot(quo.plain)) {  // (a branch: rare)
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (quo.plain) s_new[i] = (T)quo.plainly(m[i], n.k);
  }
#pragma unroll
  for (int i = 0; i < K; ++i) {
    r[i].b = average_update<T>(c.own, p[i].a, r[i].b, c.ik, c.variant);
    c.su[ALL || i < n.k ? e[i] : c.zero + 1].a = s_new[i];
    c.rs[e[i]] = r[i];
  }
  if (c.chains) {
#pragma unroll
    for (int i = 0; i < K; ++i)
      chain_update<T>(c.chain + (ALL || i < n.k ? e[i] : c.chain_spare), c.opp, c.own, p[i].a, c.ik,
                      c.variant);
  }
}

// The sum of v over the node's children in child order, for lanes that hold one
// child each: first is the lane of the first, k their number.
__device__ __forceinline__ double sum_lanes(double v, int first, int k) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  double sum = 0.0;
  for (int i = 0; __ballot(i < k); i += 8) {
    int xl[8], xh[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      xl[m] = __builtin_amdgcn_ds_bpermute(4 * (first + i + m), lo);
      xh[m] = __builtin_amdgcn_ds_bpermute(4 * (first + i + m), hi);
    }
    __builtin_amdgcn_sched_barrier(0);  // all on their way before the first is used
#pragma unroll
    for (int m = 0; m < 8; ++m) sum += i + m < k ? __hiloint2double(xh[m], xl[m]) : 0.0;
  }
  return sum;
}

// The update of child j of a node, one lane per edge of a wave that holds all of
// the node's edges side by side.
template <class T>
__device__ __forceinline__ void update_edge(const Update<T> &c, const Kids &n, int j) {
  const int e = n.e + j * n.step, first = (int)(threadIdx.x & 63) - j;
  const Pair<T> p = c.su[e], r = c.rs[e];
  const double uh = sum_lanes((double)p.a * (double)p.b, first, n.k);
  const T Rs = (T)next_regret((double)r.a, c.sopp * ((double)p.b - uh), c.ik, c.variant);
  const double m = matched((double)Rs, c.rm_mode, c.eps);
  const double sum = sum_lanes(m, first, n.k);
  const Quotient quo(sum, c.exact);
  T s_new = (T)quo.of(m);
  if (__ballot(quo.plain))  // (a branch: rare)
    if (quo.plain) s_new = (T)quo.plainly(m, n.k);
  c.rs[e] = Pair<T>{Rs, average_update<T>(c.own, p.a, r.b, c.ik, c.variant)};
  c.su[e].a = s_new;
  if (c.chains) chain_update<T>(c.chain + e, c.opp, c.own, p.a, c.ik, c.variant);
}

// The same for any number of children, four at a time.
template <class T>
__device__ __forceinline__ void update_many(const Update<T> &c, const Kids &n, double uh) {
  double sum = 0.0;
  for (int left = n.k, e0 = n.e; left > 0; left -= 4, e0 += 4 * n.step) {
    T v[4], r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = i < left ? e0 + i * n.step : e0;
      v[i] = c.su[e].b;
      r[i] = c.rs[e].a;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T Rs = (T)next_regret((double)r[i], c.sopp * ((double)v[i] - uh), c.ik, c.variant);
      if (i < left) c.rs[e0 + i * n.step].a = Rs;
      sum += i < left ? matched((double)Rs, c.rm_mode, c.eps) : 0.0;
    }
  }
  const double inv_k = sum > 0.0 ? 0.0 : 1.0 / (double)n.k;
  for (int left = n.k, e0 = n.e; left > 0; left -= 4, e0 += 4 * n.step) {
    T s[4];
    Pair<T> r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = i < left ? e0 + i * n.step : e0;
      s[i] = c.su[e].a;
      r[i] = c.rs[e];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i % 2 == 0) __builtin_amdgcn_sched_barrier(0);
      const T s_new = (T)(sum > 0.0 ? matched((double)r[i].a, c.rm_mode, c.eps) / sum : inv_k);
      if (i < left) {
        const int e = e0 + i * n.step;
        c.rs[e].b = average_update<T>(c.own, s[i], r[i].b, c.ik, c.variant);
        c.su[e].a = s_new;
        if (c.chains) chain_update<T>(c.chain + e, c.opp, c.own, s[i], c.ik, c.variant);
      }
    }
  }
}

// Reach arrays of the segment's nodes below the roots, as the last iteration's
// way down leaves them (before its updates).
template <class T, int BLOCK, int FORM>
__device__ __forceinline__ void seg_store_reach(unsigned char *far, const SegLds &L) {
  const Pair<T> *const su = near<Pair<T>, FORM>(far, L.su);
  const T *const x = near<T, FORM>(far, L.x);
  for (int id = threadIdx.x, end = g_nb[7]; id < end; id += BLOCK) {
    const uint2 w = arr<uint2, FORM>(far, L.kids)[id];
    const int l = (int)(w.y >> 24) & 7;
    const Kids n(w);
    const int b =
        tab<const int32_t>(P_CB, l)[arr<uint16_t, FORM>(far, L.pos)[id]] - g_lo[l + 1];
    const GlobalPtr<T> moved = tab<T>((l & 1) == 0 ? P_RA : P_RB, l + 1);
    const GlobalPtr<T> kept = tab<T>((l & 1) == 0 ? P_RB : P_RA, l + 1);
    const T opp = x[id];
    const double own = (double)x[arr<uint32_t, FORM>(far, L.up)[id] & 0xFFFFu];
    for (int j = 0, e = n.e; j < n.k; ++j, e += n.step) {
      const int q = b + j;
      const T v = (T)(own * (double)su[e].a);
      moved[q] = v;
      kept[q] = opp;
      if (l == 5 && bit_of(L.b6, q)) {
        // level 6's mover moves on with probability 1
        const int q7 = tab<const int32_t>(P_CB, 6)[q] - g_lo[7];
        tab<T>(P_RB, 7)[q7] = v;
        tab<T>(P_RA, 7)[q7] = opp;
      }
    }
  }
}

// A chain edge's regret after the call's iterations: each adds a regret of
// zero (the edge is forced) times the opponent's reach to the discounted one.
// `reaches` is a running sum of these reaches: not a number once one was (as
// infinite utilities above make them).  False: it stays.
template <class T>
__device__ __forceinline__ bool chain_regret(T &v, double sgn, T reaches, const IterK *ks,
                                             int n_iters, int variant) {
  if (isnan(reaches)) {
    v = reaches;
    return true;
  }
  if (v == (T)0 && !signbit((double)v)) return false;
  for (int it = 0; it < n_iters; ++it)
    v = (T)next_regret((double)v, sgn * 0.0, ks[it], variant);
  return true;
}

// The state back into the level arrays.
template <class T, int BLOCK, int FORM>
__device__ __forceinline__ void seg_store(const ItemDesc<T> &D, int roots, unsigned char *far,
                                          const SegLds &L, int na, int ne, const IterK *ks,
                                          int n_iters, int variant) {
  const Pair<T> *const su = near<Pair<T>, FORM>(far, L.su), *const rs = arr<Pair<T>, FORM>(far, L.rs);
  const Pair<T> *const chain = arr<Pair<T>, FORM>(far, L.chain);
  const int e6 = g_sb[6], lo8 = g_lo[8], lo7 = g_lo[7];
  for (int id0 = threadIdx.x; id0 < na; id0 += 2 * BLOCK) {
    // two nodes, and two children of each, at a time
    int lev[2], kids[2], b[2], e0[2], step[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bool in = id0 + u * BLOCK < na;
      const int id = in ? id0 + u * BLOCK : id0;
      const uint2 w = arr<uint2, FORM>(far, L.kids)[id];
      const Kids n(w);
      lev[u] = (int)(w.y >> 24) & 7;
      kids[u] = in ? n.k : 0;
      e0[u] = n.e;
      step[u] = n.step;
      b[u] = tab<const int32_t>(P_CB, lev[u])[arr<uint16_t, FORM>(far, L.pos)[id]] - g_lo[lev[u] + 1];
    }
    for (int j = 0; j < kids[0] || j < kids[1]; j += 2) {
      int q[4], q7[4], q8[4];
      T r7[4], r8[4];
      bool in[4], p[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int u = m / 2, l = lev[u];
        in[m] = j + m % 2 < kids[u];
        q[m] = q7[m] = q8[m] = b[u] + (in[m] ? j + m % 2 : 0);
        p[m] = in[m] && (l == 5 ? bit_of(L.b6, q[m]) : l == 6 && bit_of(L.b7, q[m]));
        r7[m] = r8[m] = (T)0;
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m] && lev[m / 2] == 5) q7[m] = tab<const int32_t>(P_CB, 6)[q[m]] - lo7;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m]) q8[m] = tab<const int32_t>(P_CB, 7)[q7[m]] - lo8;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (p[m]) {
          r8[m] = tab<T>(P_R, 8)[q8[m]];
          if (lev[m / 2] == 5) r7[m] = tab<T>(P_R, 7)[q7[m]];
        }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int u = m / 2, l = lev[u], e = e0[u] + (j + m % 2) * step[u];
        if (!in[m]) continue;
        const Pair<T> s2 = su[e], r = rs[e];
        tab<T>(P_SIGMA, l + 1)[q[m]] = s2.a;
        tab<T>(P_R, l + 1)[q[m]] = r.a;
        tab<T>(P_SBAR, l + 1)[q[m]] = r.b;
        if (l < 7) tab<T>(P_U, l + 1)[q[m]] = s2.b;
        if (!p[m]) continue;
        const Pair<T> ch = chain[e - e6];
        if (l == 5) {
          tab<T>(P_U, 7)[q7[m]] = s2.b;
          tab<T>(P_SBAR, 7)[q7[m]] = ch.a;
          if (chain_regret<T>(r7[m], 1.0, ch.b, ks, n_iters, variant)) tab<T>(P_R, 7)[q7[m]] = r7[m];
        }
        tab<T>(P_SBAR, 8)[q8[m]] = l == 5 ? ch.b : ch.a;
        if (chain_regret<T>(r8[m], -1.0, l == 5 ? ch.a : ch.b, ks, n_iters, variant))
          tab<T>(P_R, 8)[q8[m]] = r8[m];
      }
    }
  }
  for (int id = threadIdx.x; id < roots; id += BLOCK) {
    const int j = arr<uint16_t, FORM>(far, L.pos)[id];
    tab<T>(P_U, 0)[j] = su[ne + id].b;
    D.vacc[g_lo[0] + j] = lds<double>(L.vacc)[id];
  }
}

// All iterations of one segment in its compact form.  PAPER fixes the paper's
// variant (DCFR with the regret floor) at compile time.
template <class T, int BLOCK, bool PAPER, int FORM>
__device__ __forceinline__ void seg_iterations(const ItemDesc<T> &D, int roots, unsigned char *far, const SegLds &L, int na, int ne,
                                           const IterK *__restrict__ ks, int n_iters, int variant,
                                           int rm_mode, double eps) {
  if (PAPER) {
    variant = PASUR_DCFR;
    rm_mode = PASUR_RM_FLOOR;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  Pair<T> *const su = near<Pair<T>, FORM>(far, L.su);
  T *const x = near<T, FORM>(far, L.x);
  double *const vacc = lds<double>(L.vacc);
  const uint2 *const w_kids = arr<uint2, FORM>(far, L.kids);
  const uint32_t *const w_up = arr<uint32_t, FORM>(far, L.up);
  const uint32_t *const list = lds<uint32_t>(L.list);
  const int n_list_top = __builtin_amdgcn_readfirstlane(g_list_top);
  const int n_list = __builtin_amdgcn_readfirstlane(g_list_end);
  // the levels' first nodes, one per lane, read as wave-uniform scalars
  const int nb_lane = lane <= 8 ? g_nb[lane] : na;
  auto nb = [&](int l) { return __builtin_amdgcn_readlane(nb_lane, l); };
  int bottom = 7;  // deepest level with active nodes (5 at least)
  while (bottom > 0 && nb(bottom + 1) == nb(bottom)) --bottom;
  // the utilities and reaches of levels 0 .. top-1 belong to wave 0, a lane each
  const int top = __builtin_amdgcn_readfirstlane(top_levels());
  const int n_top = nb(top);
  const int down0 = top > 0 ? 1 : 0;         // first interval with a step down
  const int first_down = top > 0 ? top : 1;  // its first level
  const int n_up = bottom - top + 1, n_down = (bottom - first_down + 2) / 2;
  const int n_int = n_up > down0 + n_down ? n_up : down0 + n_down;
  const bool top_wave = top > 0 && wave == 0;
  // the way up begins with the first waves, which the hardware prefers, the way
  // down and the list's second part with the last
  const int last_tid = (BLOCK / 64 - 1 - wave) * 64 + lane;

  auto value = [&](uint2 w) {
    const double uh = node_value<T>(su, ne + roots, Kids(w));
    su[w.y & 0xFFFFu].b = (T)uh;
    return uh;
  };
  auto down = [&](int id, uint32_t slot, uint32_t up) {
    x[id] = (T)((double)x[up >> 16] * (double)su[slot & 0xFFFFu].a);
  };
  Update<T> c;
  c.su = su;
  c.rs = arr<Pair<T>, FORM>(far, L.rs);
  c.chain = arr<Pair<T>, FORM>(far, L.chain) - g_sb[6];
  c.variant = variant;
  c.rm_mode = rm_mode;
  c.eps = eps;
  c.zero = ne + roots;
  c.spare = ne;
  c.chain_spare = __builtin_amdgcn_readfirstlane(g_sb[8]);
  c.exact = exact_quotients<T>(rm_mode, eps);
  auto node = [&](int id, uint2 w, uint32_t up) {
    const int level = (int)(w.y >> 24) & 7;
    c.opp = (double)x[id];
    c.own = (double)x[up & 0xFFFFu];
    c.sopp = (level & 1) == 0 ? c.opp : -c.opp;
    c.chains = level == 5 || level == 6;
  };
  auto update = [&](int id, uint2 w, uint32_t up) {
    node(id, w, up);
    const Kids n(w);
    if (!__ballot(n.k != 2)) update_few<T, 2, true>(c, n);
    else if (!__ballot(n.k != 3)) update_few<T, 3, true>(c, n);
    else if (!__ballot(n.k > 4)) update_few<T, 4, false>(c, n);
    else update_many<T>(c, n, node_value<T>(su, c.zero, n));
  };
  // This thread's first node in the updates, and in interval iv on the way up
  // and down (possibly past the level's end); their words never change and are
  // fetched one interval ahead.  Wave 0 joins the updates in their second round.
  const int first_update = top_wave ? n_top + BLOCK - 64 + tid : top > 0 ? n_top + tid - 64 : tid;
  auto up_id = [&](int iv) {
    return iv >= n_int ? first_update : nb(bottom - iv) + (iv == 0 && top > 0 ? last_tid : tid);
  };
  auto down_id = [&](int iv) { return nb(first_down + 2 * (iv - down0)) + last_tid; };
  auto clamp = [&](int id) { return id < na ? id : na - 1; };
  const uint2 top_kids = w_kids[clamp(lane)];
  const uint32_t top_up = w_up[clamp(lane)];
  // the updates of the list's places i0, i0 + BLOCK, ... below end
  struct Place {
    uint32_t edge, up;
    uint2 w;
  };
  auto place = [&](int i) {
    Place p;
    p.edge = list[i < kList ? i : kList - 1];
    p.w = w_kids[clamp((int)(p.edge & 0xFFFFu))];
    p.up = w_up[clamp((int)(p.edge & 0xFFFFu))];
    return p;
  };
  auto update_list = [&](Place p, int i0, int end) {
    if (i0 >= end) return;
    __builtin_amdgcn_s_setprio(3);  // the other waves wait for these few
    for (int i = i0; i < end;) {
      if (p.edge != kNoEdge) {
        node((int)(p.edge & 0xFFFFu), p.w, p.up);
        update_edge<T>(c, Kids(p.w), (int)(p.edge >> 16));
      }
      i += BLOCK;
      if (i < end) p = place(i);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  const Place top_place = place(lane);
  uint2 up_w = w_kids[clamp(up_id(0))];
  uint2 down_w = make_uint2(0, 0);
  if (down0 == 0) down_w = make_uint2(w_kids[clamp(down_id(0))].y, w_up[clamp(down_id(0))]);

  IterK next = ks[0];
  for (int it = 0; it < n_iters; ++it) {
    c.ik = next;
    next = ks[it + 1 < n_iters ? it + 1 : it];
    // utilities go up from the bottom level to `top`, one level per interval,
    // while reaches go down, wave 0's in the first interval, then two levels per
    // interval
    for (int iv = 0; iv < n_int; ++iv) {
      const int ul = bottom - iv, dl = first_down + 2 * (iv - down0);
      uint2 next_up = up_w, next_down = down_w;
      if (iv + 1 >= n_int || ul - 1 >= top) next_up = w_kids[clamp(up_id(iv + 1))];
      if (iv + 1 >= down0 && dl + 2 <= bottom) {
        const int id = clamp(down_id(iv + 1));
        next_down = make_uint2(w_kids[id].y, w_up[id]);
      }
      if (iv == 0 && top_wave) {
        for (int l = 1; l < top; l += 2) {
          if (lane >= nb(l) && lane < nb(l + 2 < top ? l + 2 : top))
            down(lane, top_kids.y, top_up);
          wave_order<FORM>();
        }
      }
      if (ul >= top) {
        const int end = nb(ul + 1);
        int id = up_id(iv);
        for (uint2 w = up_w; id < end; id += BLOCK, w = w_kids[clamp(id)]) {
          const double uh = value(w);
          if (ul == 0) vacc[id] += uh;
        }
      }
      if (iv >= down0 && dl <= bottom) {
        const int end = nb(dl + 2 < 8 ? dl + 2 : 8);
        int id = down_id(iv);
        for (uint2 w = down_w; id < end;
             id += BLOCK, w = make_uint2(w_kids[clamp(id)].y, w_up[clamp(id)]))
          down(id, w.x, w.y);
      }
      up_w = next_up;
      down_w = next_down;
      __syncthreads();
    }
    if (it == n_iters - 1) {
      seg_store_reach<T, BLOCK, FORM>(far, L);
      __syncthreads();
    }
    // the updates; wave 0 finishes the top levels' utilities first, whose
    // strategies no other wave changes, and then updates these levels
    uint2 w = up_w;
    up_w = w_kids[clamp(up_id(0))];
    if (down0 == 0) down_w = make_uint2(w_kids[clamp(down_id(0))].y, w_up[clamp(down_id(0))]);
    if (top_wave) {
      for (int l = top - 1; l >= 0; --l) {
        if (lane >= nb(l) && lane < nb(l + 1)) {
          const double uh = value(top_kids);
          if (l == 0) vacc[lane] += uh;
        }
        wave_order<FORM>();
      }
      update_list(top_place, lane, n_list_top);
    }
    update_list(place(n_list_top + last_tid), n_list_top + last_tid, n_list);
    for (int id = first_update; id < na; id += BLOCK) {
      if (!(w.y & kListed)) update(id, w, w_up[id]);
      w = w_kids[clamp(id + BLOCK)];
    }
    __syncthreads();
  }
  seg_store<T, BLOCK, FORM>(D, roots, far, L, na, ne, ks, n_iters, variant);
}

// ---- in global memory ------------------------------------------------------------
template <class T, int SLOT>
struct TabArr {
  int l;
  __device__ __forceinline__ T &operator[](int i) const {
    return reinterpret_cast<T *>(g_ptab[SLOT][l])[i];
  }
};

// FindUtility for the parents of level L-1, one thread each, over their
// children in child order.  Through flat pointers and with a plain fmax the
// compiler keeps more of the loops' loads in flight (one root of 2.5e6 nodes, 20
// iterations: 147 ms; with global pointers 155, with `matched` as well 166).
__device__ __forceinline__ double low_max(double R, int rm_mode, double eps) {
  return rm_mode == PASUR_RM_FLOOR ? fmax(R, eps) : fmax(R, 0.0);
}
template <class T, int L>
__device__ __forceinline__ void up_global(double *vacc, const IterK &ik, int variant, int rm_mode,
                                          double eps) {
  constexpr int mover = (L - 1) & 1;
  const TabArr<T, 0> sg{L};
  const TabArr<T, 1> Rr{L};
  const TabArr<T, 2> Sb{L};
  const TabArr<T, 3> uu{L};
  const double sgn = mover == 0 ? 1.0 : -1.0;
  int t0 = threadIdx.x;
  asm volatile("" : "+v"(t0));  // per-lane start stays inside the phase
  for (int h = t0; h < g_cnt[L - 1]; h += blockDim.x) {
    const int b = TabArr<const int32_t, 7>{L - 1}[h] - g_lo[L];
    const int e = TabArr<const int32_t, 7>{L - 1}[h + 1] - g_lo[L];
    const double ra = (double)TabArr<T, 4>{L - 1}[h], rb = (double)TabArr<T, 5>{L - 1}[h];
    const double opp = mover == 0 ? rb : ra, own = mover == 0 ? ra : rb;
    double uh = 0.0, sum = 0.0;
    for (int q = b; q < e; ++q) uh += (double)sg[q] * (double)uu[q];
    for (int q = b; q < e; ++q) {
      const double r = sgn * opp * ((double)uu[q] - uh);
      const T Rs = (T)next_regret((double)Rr[q], r, ik, variant);
      Rr[q] = Rs;
      sum += low_max((double)Rs, rm_mode, eps);
    }
    const double inv_k = sum > 0.0 ? 0.0 : 1.0 / (double)(e - b);
    for (int q = b; q < e; ++q) {
      const double m = low_max((double)Rr[q], rm_mode, eps);
      Sb[q] = average_update<T>(own, sg[q], Sb[q], ik, variant);
      sg[q] = (T)(sum > 0.0 ? m / sum : inv_k);
    }
    TabArr<T, 3>{L - 1}[h] = (T)uh;
    if (L == 1) vacc[h] += uh;
  }
  __syncthreads();
}

template <class T, int BLOCK, bool PAPER>
__device__ __forceinline__ void seg_in_global(const ItemDesc<T> &D, int j0, int j1,
                                              const IterK *__restrict__ ks, int n_iters,
                                              int variant, int rm_mode, double eps) {
  if (PAPER) {
    variant = PASUR_DCFR;
    rm_mode = PASUR_RM_FLOOR;
  }
  double *const vacc = D.vacc + j0;
  for (int it = 0; it < n_iters; ++it) {
    const IterK k = ks[it];
    // FindReachProbability, two levels per phase: a node of the second level
    // starts from its grandparent's reaches and applies its parent's and its
    // own action probability, rounding to T after each level
#pragma unroll
    for (int l = 1; l <= 7; l += 2) {
      const int l2 = l < 7 ? l + 1 : 0;  // second level of the phase (0: none)
      const int n1 = g_cnt[l], n2 = l2 ? g_cnt[l2] : 0;
      int t0 = threadIdx.x;
      asm volatile("" : "+v"(t0));
      for (int i = t0; i < n1 + n2; i += BLOCK) {
        const bool second = i >= n1;
        const int q = second ? i - n1 : i;
        const int h1 = second ? TabArr<const int32_t, 6>{l2}[q] - g_lo[l] : q;
        const int g = TabArr<const int32_t, 6>{l}[h1] - g_lo[l - 1];
        double a = (double)TabArr<T, 4>{l - 1}[g], b = (double)TabArr<T, 5>{l - 1}[g];
        const double s1 = (double)TabArr<T, 0>{l}[h1];
        if (((l - 1) & 1) == 0) a *= s1;
        else b *= s1;
        a = (double)(T)a;
        b = (double)(T)b;
        if (second) {
          const double s2 = (double)TabArr<T, 0>{l2}[q];
          if ((l & 1) == 0) a *= s2;
          else b *= s2;
        }
        TabArr<T, 4>{second ? l2 : l}[q] = (T)a;
        TabArr<T, 5>{second ? l2 : l}[q] = (T)b;
      }
      __syncthreads();
    }
    up_global<T, 8>(vacc, k, variant, rm_mode, eps);
    up_global<T, 7>(vacc, k, variant, rm_mode, eps);
    up_global<T, 6>(vacc, k, variant, rm_mode, eps);
    up_global<T, 5>(vacc, k, variant, rm_mode, eps);
    up_global<T, 4>(vacc, k, variant, rm_mode, eps);
    up_global<T, 3>(vacc, k, variant, rm_mode, eps);
    up_global<T, 2>(vacc, k, variant, rm_mode, eps);
    up_global<T, 1>(vacc, k, variant, rm_mode, eps);
  }
}

// One workgroup per segment; the segment runs in its compact form when that fits
// in the launch's dynamic LDS (lds_bytes), otherwise in global memory.  FAR: some
// segments have far arrays.  unplanned (may be NULL): counts segments in global
// memory for which that was not planned (their state has more active nodes than
// the tree's structure says).
template <class T, int BLOCK, bool PAPER, bool FAR>
__global__ void __launch_bounds__(BLOCK)
    k_cfr_seg(const ItemDesc<T> *__restrict__ items, const Seg *__restrict__ segs,
              const IterK *__restrict__ ks, unsigned char *far, int n_iters, int variant,
              int rm_mode, double eps, uint32_t lds_bytes, unsigned *unplanned) {
  const Seg sg = segs[blockIdx.x];
  const ItemDesc<T> &D = items[sg.item];
  seg_open(D, sg.j0, sg.j1);
  SegLds L;
  int na = 0, ne = 0;
  const int roots = sg.j1 - sg.j0;
  if (sg.form == F_LDS) {
    if (seg_load<T, BLOCK, F_LDS>(D, lds_bytes, nullptr, 0, L, na, ne)) {
      seg_iterations<T, BLOCK, PAPER, F_LDS>(D, roots, nullptr, L, na, ne, ks, n_iters, variant,
                                             rm_mode, eps);
      return;
    }
  } else if (FAR && sg.form != F_NONE) {
    far += (int64_t)sg.far * kFarUnit;
    const int64_t far_bytes = (int64_t)sg.far_n * kFarUnit;
    if (sg.form == F_FAR) {
      if (seg_load<T, BLOCK, F_FAR>(D, lds_bytes, far, far_bytes, L, na, ne)) {
        seg_iterations<T, BLOCK, PAPER, F_FAR>(D, roots, far, L, na, ne, ks, n_iters, variant,
                                               rm_mode, eps);
        return;
      }
    } else if (seg_load<T, BLOCK, F_ALL_FAR>(D, lds_bytes, far, far_bytes, L, na, ne)) {
      seg_iterations<T, BLOCK, PAPER, F_ALL_FAR>(D, roots, far, L, na, ne, ks, n_iters, variant,
                                                 rm_mode, eps);
      return;
    }
  }
  if (unplanned && sg.form != F_NONE && threadIdx.x == 0) atomicAdd(unplanned, 1u);
  seg_in_global<T, BLOCK, PAPER>(D, sg.j0, sg.j1, ks, n_iters, variant, rm_mode, eps);
}

// Per root, what the tree's structure says of its compact form on levels 6 and
// 7: active nodes of level 6 and of level 7, and the children of either.
__global__ void __launch_bounds__(64) k_seg_counts(const int32_t *__restrict__ off6,
                                                   const int32_t *__restrict__ off7,
                                                   const int32_t *__restrict__ cb6,
                                                   const int32_t *__restrict__ cb7,
                                                   int32_t *__restrict__ out) {
  const int64_t j = blockIdx.x;
  int v[4] = {0, 0, 0, 0};
  for (int i = off6[j] + (int)threadIdx.x; i < off6[j + 1]; i += 64) {
    const int32_t b = cb6[i], k = cb6[i + 1] - b;
    if (k != 1 || cb7[b + 1] - cb7[b] != 1) {
      v[0] += 1;
      v[2] += k;
    }
  }
  for (int i = off7[j] + (int)threadIdx.x; i < off7[j + 1]; i += 64) {
    const int32_t k = cb7[i + 1] - cb7[i];
    if (k != 1) {
      v[1] += 1;
      v[3] += k;
    }
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v[m] += __shfl_xor(v[m], d, 64);
    if (threadIdx.x == 0) out[4 * j + m] = v[m];
  }
}

constexpr uint32_t kLdsPerWorkgroup = 160 * 1024;
// static LDS: the global-memory path's pointer table, the levels' bounds
constexpr uint32_t kStaticLds = 1024;

inline bool paper_variant(int variant, int rm_mode) {
  return variant == PASUR_DCFR && rm_mode == PASUR_RM_FLOOR;
}

template <class T>
using SegKernel = void (*)(const ItemDesc<T> *, const Seg *, const IterK *, unsigned char *, int,
                           int, int, double, uint32_t, unsigned *);

template <class T>
SegKernel<T> seg_kernel(int block, bool paper, bool far) {
  if (far) return paper ? k_cfr_seg<T, 1024, true, true> : k_cfr_seg<T, 1024, false, true>;
  if (block == 256) return paper ? k_cfr_seg<T, 256, true, false> : k_cfr_seg<T, 256, false, false>;
  if (block == 512) return paper ? k_cfr_seg<T, 512, true, false> : k_cfr_seg<T, 512, false, false>;
  return paper ? k_cfr_seg<T, 1024, true, false> : k_cfr_seg<T, 1024, false, false>;
}

std::mutex g_counts_mu;

int root_counts(pasur_fgt *f, hipStream_t s) {
  std::lock_guard<std::mutex> lock(g_counts_mu);
  if (f->h_root_seg) return PASUR_OK;
  const size_t n = 4 * (size_t)f->n_roots;
  void *d = nullptr;
  PASUR_TRY(block_alloc(&d, n * sizeof(int32_t)));
  int32_t *h = (int32_t *)std::malloc(n * sizeof(int32_t));
  if (!h) {
    block_free(d);
    set_error("host allocation failed");
    return PASUR_E_NOMEM;
  }
  k_seg_counts<<<(unsigned)f->n_roots, 64, 0, s>>>(f->root_off[6], f->root_off[7],
                                                   f->child_begin[6], f->child_begin[7], (int32_t *)d);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(h, d, n * sizeof(int32_t), hipMemcpyDeviceToHost, s);
  const hipError_t e2 = hipStreamSynchronize(s);
  if (e == hipSuccess) e = e2;
  if (e2 == hipSuccess) block_free(d);  // (else it may be in use)
  if (e != hipSuccess) {
    std::free(h);
    set_error("segment counts: %s", hipGetErrorString(e));
    return PASUR_E_HIP;
  }
  f->h_root_seg = h;
  return PASUR_OK;
}

// One kernel launch of a plan: consecutive segments with the same LDS size.
struct SegLaunch {
  int first, count, block;
  uint32_t lds_bytes;
  bool far;  // some segments have far arrays (1024 threads)
};

}  // namespace

struct pasur_plan {
  int dtype, block, variant, rm_mode;
  double eps;
  int64_t t_first, t_last;
  int n_items, n_segs;
  void *mem, *anchor;  // the arrays below in one block; see anchor_alloc
  void *far;           // far arrays of the launch that needs most (launches follow each other)
  void *d_items;
  Seg *d_segs;
  IterK *d_ks;
  uint32_t lds_bytes;
  unsigned *d_unplanned;
  int64_t work[4];   // edges, internal nodes, roots, level-7 nodes
  int64_t forms[4];  // segments of each form
  std::vector<SegLaunch> launches;
};

namespace {

struct SegPlan {
  Seg seg;
  int64_t nodes;
  uint32_t bytes;  // of its compact form in LDS, 0: in global memory
};

// How many workgroups of such a segment a CU takes, up to 4.
int per_cu(const SegPlan &sp) {
  const int n = (int)(kLdsPerWorkgroup / (sp.bytes + kStaticLds));
  return sp.seg.form != F_LDS || n < 1 ? 1 : n > 4 ? 4 : n;
}

// Far arrays of one launch: at most this much (a launch's segments beyond it go
// to the next launch, which uses the same memory).
constexpr int64_t kFarBytes = (int64_t)1 << 30;

// Launches of segments ordered by descending size, those in global memory
// first, then those with far arrays.  A launch's workgroups all hold the LDS of
// its largest segment, so segments of which more fit on a CU get a launch of
// their own, unless there are too few of them to fill the chip; the segments of
// the first two kinds, the longest of all, run beside the largest ones in LDS.
// Gives far arrays their places; returns the bytes these take.
int64_t plan_launches(std::vector<SegLaunch> &launches, std::vector<SegPlan> &segs, int user_block) {
  constexpr int kCus = 256;
  int64_t far_max = 0;
  const int n = (int)segs.size();
  launches.clear();
  for (int i = 0; i < n;) {
    SegLaunch la;
    const int c = per_cu(segs[(size_t)i]);
    int j = i;
    int64_t far = 0;
    la.lds_bytes = 0;
    for (bool rest = false; j < n; ++j) {
      SegPlan &sp = segs[(size_t)j];
      if (!rest && per_cu(sp) != c) {
        if (n - j >= kCus) break;
        rest = true;
      }
      if (sp.seg.far_n > 0) {
        const int64_t need = (int64_t)sp.seg.far_n * kFarUnit;
        if (far > 0 && far + need > kFarBytes) break;
        sp.seg.far = (int32_t)(far / kFarUnit);
        far += need;
      }
      la.lds_bytes = std::max(la.lds_bytes, sp.bytes);
    }
    far_max = std::max(far_max, far);
    la.first = i;
    la.count = j - i;
    la.far = far > 0;
    la.block = la.far       ? 1024
               : user_block ? user_block
               : la.count <= kCus || c == 1 ? 1024
               : c == 2     ? 512
                            : 256;
    launches.push_back(la);
    i = j;
  }
  return far_max;
}

// Orders segments for their launches: those in global memory first, then those
// with far arrays, then the largest, these by how many a CU takes, and in buckets
// of 512 bytes (a comparison sort of 1e5 segments takes milliseconds).  Returns the
// bytes of far arrays.
int64_t order_segments(std::vector<SegLaunch> &launches, std::vector<SegPlan> &segs,
                       int user_block) {
  std::vector<SegPlan> large, by_bytes(segs.size());
  constexpr size_t kBuckets = kLdsPerWorkgroup / 512 + 1;
  auto bucket = [](const SegPlan &sp) {
    return (size_t)(per_cu(sp) - 1) * kBuckets + (kLdsPerWorkgroup - sp.bytes) / 512;
  };
  std::vector<size_t> at(4 * kBuckets + 1, 0);
  for (const SegPlan &sp : segs) {
    if (sp.seg.form != F_LDS) large.push_back(sp);
    else at[bucket(sp) + 1] += 1;
  }
  std::stable_sort(large.begin(), large.end(), [](const SegPlan &a, const SegPlan &b) {
    return a.seg.form != b.seg.form ? a.seg.form > b.seg.form : a.nodes > b.nodes;
  });
  at[0] = large.size();
  for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
  std::copy(large.begin(), large.end(), by_bytes.begin());
  for (const SegPlan &sp : segs)
    if (sp.seg.form == F_LDS) by_bytes[at[bucket(sp)]++] = sp;
  segs.swap(by_bytes);
  return plan_launches(launches, segs, user_block);
}

template <class T>
ItemDesc<T> item_desc(const pasur_fgt *f, const pasur_cfr_state *st) {
  ItemDesc<T> D;
  for (int l = 0; l <= 8; ++l) {
    D.off[l] = f->root_off[l];
    D.parent[l] = f->parent[l];
    D.cb[l] = l <= 7 ? f->child_begin[l] : nullptr;
    D.sigma[l] = l >= 1 ? (T *)st->sigma[l] : nullptr;
    D.R[l] = l >= 1 ? (T *)st->R[l] : nullptr;
    D.Sbar[l] = l >= 1 ? (T *)st->Sbar[l] : nullptr;
    D.ra[l] = l <= 7 ? (T *)st->reachA[l] : nullptr;
    D.rb[l] = l <= 7 ? (T *)st->reachB[l] : nullptr;
    D.u[l] = (T *)st->u[l];
  }
  D.vacc = st->vacc;
  return D;
}

// The segments of one tree (item `it` of its plan), whose root counts are there,
// appended: runs of consecutive roots, closed when the next root would exceed
// seg_nodes nodes, `block` roots, or LDS.  t: bytes of the state's type.
void tree_segments(const pasur_fgt *f, int it, uint32_t t, int seg_nodes, int block,
                   bool force_global, std::vector<SegPlan> &segs) {
  const uint32_t budget = force_global ? 0u : kLdsPerWorkgroup - kStaticLds;
  const int64_t nr = f->n_roots;
  auto level_nodes = [&](int l, int64_t j) {
    const int32_t *o = f->h_root_off + (size_t)l * (nr + 1);
    return o[j + 1] - o[j];
  };
  auto add_root = [&](SegCounts &c, int64_t &tot, int64_t j) {
    int n[9], c07 = 0, ne = 0;
    for (int l = 0; l <= 8; ++l) n[l] = level_nodes(l, j);
    for (int l = 0; l <= 7; ++l) c07 += n[l];
    for (int l = 1; l <= 6; ++l) ne += n[l];
    const int32_t *x = f->h_root_seg + 4 * j;
    c.na += c07 - n[6] - n[7] + x[0] + x[1];
    c.ne += ne + x[2] + x[3];
    c.ne67 += n[6] + x[2];
    c.roots += 1;
    c.c07 += c07;
    c.c6 += n[6];
    c.c7 += n[7];
    tot += c07 + n[8];
  };
  auto bytes_of = [&](const SegCounts &c, int form) -> uint32_t {
    if (c.c6 > 65535 || c.c7 > 65535 || !seg_indices_fit(c)) return 0u;
    const uint32_t b = seg_layout(c, t, form).bytes;
    return b <= budget ? b : 0u;
  };
  int64_t j0 = 0;
  while (j0 < nr) {
    int64_t j1 = j0 + 1, tot = 0;
    SegCounts c = {};
    add_root(c, tot, j0);
    uint32_t bytes = bytes_of(c, F_LDS);
    while (seg_nodes > 0 && bytes && j1 < nr && j1 - j0 < block) {
      SegCounts c2 = c;
      int64_t t2 = tot;
      add_root(c2, t2, j1);
      const uint32_t b2 = bytes_of(c2, F_LDS);
      if (t2 > seg_nodes || !b2) break;
      ++j1;
      c = c2;
      tot = t2;
      bytes = b2;
    }
    SegPlan sp;
    sp.seg.item = it;
    sp.seg.j0 = (int32_t)j0;
    sp.seg.j1 = (int32_t)j1;
    sp.seg.far = sp.seg.far_n = 0;
    sp.seg.form = F_LDS;
    while (!bytes && sp.seg.form != F_NONE && !force_global)  // (a single root)
      if (++sp.seg.form != F_NONE) bytes = bytes_of(c, sp.seg.form);
    if (!bytes) sp.seg.form = F_NONE;
    else if (sp.seg.form != F_LDS)
      sp.seg.far_n = (int32_t)((seg_layout(c, t, sp.seg.form).far + kFarUnit - 1) / kFarUnit);
    sp.nodes = tot;
    sp.bytes = bytes;
    segs.push_back(sp);
    j0 = j1;
  }
}

void count_forms(int64_t forms[4], const std::vector<SegPlan> &segs) {
  for (int k = 0; k < 4; ++k) forms[k] = 0;
  for (const SegPlan &sp : segs) forms[sp.seg.form] += 1;
}

// The compact form leaves a forced chain's regrets of zero alone.  They don't stay
// zero where a discount is not a number: after an infinite power of t - 1 (an
// exponent below zero at t = 1, or one so large that the power overflows).
bool zeros_stay(const IterK *ks, int64_t n, int variant) {
  if (variant != PASUR_DCFR) return true;
  for (int64_t i = 0; i < n; ++i)
    if (!std::isfinite(ks[i].dneg)) return false;
  return true;
}

bool all_lds(const int64_t forms[4]) {
  return forms[F_FAR] + forms[F_ALL_FAR] + forms[F_NONE] == 0;
}

void add_work(int64_t work[4], const pasur_fgt *f) {
  for (int l = 1; l <= 8; ++l) work[0] += f->n[l];
  for (int l = 0; l <= 7; ++l) work[1] += f->n[l];
  work[2] += f->n[0];
  work[3] += f->n[7];
}

// The attribute is a ceiling shared by every launch of this instance, so it is
// raised to the whole budget (plans may be launched in any order); each launch
// still asks for its own lds_bytes.
template <class T>
int allow_lds(const std::vector<SegLaunch> &launches, bool paper) {
  for (const SegLaunch &la : launches)
    PASUR_TRY_HIP(hipFuncSetAttribute((const void *)seg_kernel<T>(la.block, paper, la.far),
                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)(kLdsPerWorkgroup - kStaticLds)));
  return PASUR_OK;
}

template <class T>
void launch_segments(const std::vector<SegLaunch> &launches, const void *items, const Seg *segs,
                     const IterK *ks, void *far, int n_iters, int variant, int rm_mode, double eps,
                     unsigned *unplanned, hipStream_t s) {
  const bool paper = paper_variant(variant, rm_mode);
  for (const SegLaunch &la : launches)
    seg_kernel<T>(la.block, paper, la.far)<<<(unsigned)la.count, la.block, la.lds_bytes, s>>>(
        (const ItemDesc<T> *)items, segs + la.first, ks, (unsigned char *)far, n_iters, variant,
        rm_mode, eps, la.lds_bytes, unplanned);
}

template <class T>
int plan_build(pasur_plan *pl, const pasur_fgt *const *fgts, const pasur_cfr_state *const *states,
               const pasur_cfr_params *p, int force_global, hipStream_t s) {
  const int n_items = pl->n_items;
  // iteration constants for t_first .. t_last, computed on the host
  const int64_t nt = pl->t_last - pl->t_first + 1;
  std::vector<IterK> ks((size_t)nt);
  for (int64_t i = 0; i < nt; ++i) ks[(size_t)i] = iter_k(p, pl->t_first + i);
  if (!zeros_stay(ks.data(), nt, p->variant)) force_global = 1;
  std::vector<ItemDesc<T>> items((size_t)n_items);
  std::vector<SegPlan> segs;
  for (int64_t k = 0; k < 4; ++k) pl->work[k] = 0;
  for (int it = 0; it < n_items; ++it) {
    PASUR_TRY(root_counts(const_cast<pasur_fgt *>(fgts[it]), s));
    items[(size_t)it] = item_desc<T>(fgts[it], states[it]);
    tree_segments(fgts[it], it, sizeof(T), p->seg_nodes, pl->block, force_global, segs);
    add_work(pl->work, fgts[it]);
  }
  const int64_t far_bytes = order_segments(pl->launches, segs, p->block);
  if (far_bytes > 0 && block_alloc(&pl->far, (size_t)far_bytes) != PASUR_OK) {
    // no memory for far arrays: in global memory
    pl->far = nullptr;
    for (SegPlan &sp : segs)
      if (sp.seg.far_n > 0) {
        sp.seg.far_n = 0;
        sp.seg.form = F_NONE;
        sp.bytes = 0;
      }
    (void)order_segments(pl->launches, segs, p->block);
  }
  count_forms(pl->forms, segs);
  std::vector<Seg> sorted(segs.size());
  uint32_t max_bytes = 0;
  for (size_t i = 0; i < segs.size(); ++i) {
    sorted[i] = segs[i].seg;
    max_bytes = std::max(max_bytes, segs[i].bytes);
  }
  pl->n_segs = (int)sorted.size();
  pl->lds_bytes = max_bytes;
  // one upload
  const size_t at_segs = align16(sizeof(ItemDesc<T>) * items.size());
  const size_t at_ks = at_segs + align16(sizeof(Seg) * sorted.size());
  const size_t at_unplanned = at_ks + sizeof(IterK) * ks.size();
  std::vector<unsigned char> stage(at_unplanned + sizeof(unsigned), 0);
  std::memcpy(stage.data(), items.data(), sizeof(ItemDesc<T>) * items.size());
  std::memcpy(stage.data() + at_segs, sorted.data(), sizeof(Seg) * sorted.size());
  std::memcpy(stage.data() + at_ks, ks.data(), sizeof(IterK) * ks.size());
  PASUR_TRY(block_alloc(&pl->mem, stage.size()));
  pl->d_items = pl->mem;
  pl->d_segs = (Seg *)((unsigned char *)pl->mem + at_segs);
  pl->d_ks = (IterK *)((unsigned char *)pl->mem + at_ks);
  pl->d_unplanned = (unsigned *)((unsigned char *)pl->mem + at_unplanned);
  PASUR_TRY_HIP(hipMemcpyAsync(pl->mem, stage.data(), stage.size(), hipMemcpyHostToDevice, s));
  const hipError_t e = hipStreamSynchronize(s);  // the staging vector goes out of scope
  if (e != hipSuccess) {
    pl->mem = nullptr;  // may be in use: not handed out again
    set_error("plan upload: %s", hipGetErrorString(e));
    return PASUR_E_HIP;
  }
  return allow_lds<T>(pl->launches, paper_variant(p->variant, p->rm_mode));
}

}  // namespace

extern "C" void pasur_plan_free(pasur_plan *pl) {
  if (!pl) return;
  void *const blocks[] = {pl->mem, pl->far};
  blocks_retire(pl->anchor, blocks, 2);
  delete pl;
}

namespace {

// anchored: the plan may be freed while launches of it are pending.
int plan_create(const pasur_fgt *const *fgts,
                const pasur_cfr_state *const *states, int n_items, const pasur_cfr_params *p,
                int64_t t_first, int64_t t_last, pasur_plan **out, void *stream, bool anchored) {
  if (!out || !fgts || !states || !p || n_items < 1) {
    set_error("null argument or empty batch");
    return PASUR_E_INVAL;
  }
  *out = nullptr;
  if (t_first < 1 || t_last < t_first) {
    set_error("need 1 <= t_first <= t_last");
    return PASUR_E_RANGE;
  }
  if (p->variant < 0 || p->variant > 2 || p->rm_mode < 0 || p->rm_mode > 1 ||
      p->schedule < 0 || p->schedule > PASUR_SCHED_AUTO || p->seg_nodes < 0 ||
      (p->block != 0 && p->block != 256 && p->block != 512 && p->block != 1024)) {
    set_error("unknown variant, regret-matching mode, schedule, block or segment size");
    return PASUR_E_RANGE;
  }
  if (p->schedule == PASUR_SCHED_LEVEL_SYNC || p->schedule == PASUR_SCHED_STREAM) {
    set_error("plans use the persistent segment schedule");
    return PASUR_E_RANGE;
  }
  if (p->flags) {
    set_error("the snippet flags run on PASUR_SCHED_LEVEL_SYNC only, not in plans");
    return PASUR_E_RANGE;
  }
  if (!states[0]) {
    set_error("item 0 is NULL");
    return PASUR_E_INVAL;
  }
  const int dtype = states[0]->dtype;
  for (int i = 0; i < n_items; ++i) {
    if (!fgts[i] || !states[i]) {
      set_error("item %d is NULL", i);
      return PASUR_E_INVAL;
    }
    PASUR_TRY(check_state(fgts[i], states[i]));
    if (states[i]->dtype != dtype) {
      set_error("all items of a plan need the same dtype");
      return PASUR_E_INVAL;
    }
  }
  pasur_plan *pl = new pasur_plan();
  pl->dtype = dtype;
  pl->block = p->block ? p->block : 1024;
  pl->variant = p->variant;
  pl->rm_mode = p->rm_mode;
  pl->eps = p->eps;
  pl->t_first = t_first;
  pl->t_last = t_last;
  pl->n_items = n_items;
  hipStream_t s = (hipStream_t)stream;
  const int fg = p->schedule == PASUR_SCHED_ROOT_GLOBAL;
  int st = anchored ? anchor_alloc(&pl->anchor) : PASUR_OK;
  if (!st)
    st = dtype == PASUR_F32 ? plan_build<float>(pl, fgts, states, p, fg, s)
                            : plan_build<double>(pl, fgts, states, p, fg, s);
  if (st) {
    pasur_plan_free(pl);
    return st;
  }
  *out = pl;
  return PASUR_OK;
}

}  // namespace

extern "C" int pasur_plan_create(const pasur_fgt *const *fgts,
                                 const pasur_cfr_state *const *states, int n_items,
                                 const pasur_cfr_params *p, int64_t t_first, int64_t t_last,
                                 pasur_plan **out, void *stream) {
  return plan_create(fgts, states, n_items, p, t_first, t_last, out, stream, true);
}

namespace pasur {
int seg_iterate(const pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p,
                int64_t t0, int n_iters, hipStream_t s) {
  pasur_plan *pl = nullptr;
  PASUR_TRY(plan_create(&f, &st, 1, p, t0, t0 + n_iters - 1, &pl, s, false));
  const int rc = pasur_plan_iterate(pl, t0, n_iters, s);
  const hipError_t e = hipStreamSynchronize(s);  // the plan's blocks are idle below
  if (e != hipSuccess) pl->mem = pl->far = nullptr;  // or may be in use: not handed out again
  pasur_plan_free(pl);
  if (rc) return rc;
  if (e != hipSuccess) {
    set_error("iterate: %s", hipGetErrorString(e));
    return PASUR_E_HIP;
  }
  return PASUR_OK;
}
}  // namespace pasur

// ---- one tree, without waiting ---------------------------------------------------
namespace {
// Bytes from the host behind the arguments of a kernel, which copies them (no
// pinned memory to keep until a copy has ended, and a graph keeps them).
struct PutBytes {
  uint4 b[224];
};
__global__ void __launch_bounds__(256) k_put(PutBytes a, int n, uint4 *__restrict__ out) {
  if ((int)threadIdx.x < n) out[threadIdx.x] = a.b[threadIdx.x];
}

// (their constants pass through the host's memory and kernel arguments)
constexpr int kSegIters = 1 << 20;

void put(unsigned char *to, const unsigned char *from, size_t bytes, hipStream_t s) {
  for (size_t at = 0; at < bytes; at += sizeof(PutBytes)) {
    PutBytes a;
    const size_t n = std::min(bytes - at, sizeof(a));
    std::memcpy(&a, from + at, n);
    k_put<<<1, 256, 0, s>>>(a, (int)((n + 15) / 16), (uint4 *)(to + at));
  }
}

}  // namespace

namespace pasur {
// The segments of a tree by itself, for one state type and one choice of
// workgroup and segment size.  Never changed once it is on the tree's list.
struct SegIndex {
  int dtype, block, seg_nodes;
  std::vector<SegLaunch> launches;
  void *mem;  // the segments, on the device
  int64_t far_bytes, forms[4];
  SegIndex *next;
};

int seg_index_blocks(const SegIndex *x, void **p, int n) {
  int k = 0;
  for (; x && k < n; x = x->next) p[k++] = x->mem;
  return k;
}

void seg_index_free(SegIndex *x) {
  while (x) {
    SegIndex *const next = x->next;
    delete x;
    x = next;
  }
}
}  // namespace pasur

namespace {
// The tree's index for these, or else (any) for this type; g_counts_mu is held.
const SegIndex *find_index(const pasur_fgt *f, int dtype, int block, int seg_nodes, bool any) {
  for (const SegIndex *x = f->seg_index; x; x = x->next)
    if (x->dtype == dtype && (any || (x->block == block && x->seg_nodes == seg_nodes))) return x;
  return nullptr;
}

int build_index(pasur_fgt *f, int dtype, int block, int seg_nodes, hipStream_t s) {
  std::vector<SegPlan> segs;
  tree_segments(f, 0, dtype == PASUR_F32 ? 4 : 8, seg_nodes, block ? block : 1024, false, segs);
  SegIndex *const x = new SegIndex();
  x->dtype = dtype;
  x->block = block;
  x->seg_nodes = seg_nodes;
  count_forms(x->forms, segs);
  x->far_bytes = order_segments(x->launches, segs, block);
  std::vector<Seg> sorted(segs.size());
  for (size_t i = 0; i < segs.size(); ++i) sorted[i] = segs[i].seg;
  x->mem = nullptr;
  int st = block_alloc(&x->mem, sizeof(Seg) * sorted.size());
  if (!st) {
    hipError_t e = hipMemcpyAsync(x->mem, sorted.data(), sizeof(Seg) * sorted.size(),
                                  hipMemcpyHostToDevice, s);
    const hipError_t e2 = hipStreamSynchronize(s);  // `sorted` goes out of scope
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) {
      set_error("segment index: %s", hipGetErrorString(e));
      st = PASUR_E_HIP;
      if (e2 == hipSuccess) block_free(x->mem);  // (else it may be in use)
    }
  }
  if (st) {
    delete x;
    return st;
  }
  std::lock_guard<std::mutex> lock(g_counts_mu);
  // another thread may have been faster: what it put there stays
  const SegIndex *const there = find_index(f, dtype, block, seg_nodes, false);
  int n = 0;
  for (const SegIndex *y = f->seg_index; y; y = y->next) ++n;
  if (there || n == kSegIndexes) {
    block_free(x->mem);
    delete x;
    return PASUR_OK;
  }
  x->next = f->seg_index;
  f->seg_index = x;
  return PASUR_OK;
}

template <class T>
int enqueue(const pasur_fgt *f, const SegIndex &x, const pasur_cfr_state *st,
            const pasur_cfr_params *p, int64_t t0, int n_iters, bool capturing, bool *done,
            hipStream_t s) {
  const bool paper = paper_variant(p->variant, p->rm_mode);
  // far arrays, the item, the iterations' constants
  const ItemDesc<T> D = item_desc<T>(f, st);
  std::vector<unsigned char> stage(align16(sizeof(D)) + sizeof(IterK) * (size_t)n_iters);
  std::memcpy(stage.data(), &D, sizeof(D));
  IterK *const ks = (IterK *)(stage.data() + align16(sizeof(D)));
  for (int i = 0; i < n_iters; ++i) ks[i] = iter_k(p, t0 + i);
  if (!zeros_stay(ks, n_iters, p->variant)) return PASUR_OK;
  PASUR_TRY(allow_lds<T>(x.launches, paper));
  const size_t far_bytes = align16((size_t)x.far_bytes), bytes = far_bytes + stage.size() + 16;
  void *mem = nullptr;
  if (capturing) {
    if (hipMallocAsync(&mem, bytes, s) != hipSuccess) {
      (void)hipGetLastError();
      return PASUR_OK;
    }
  } else if (block_alloc_on(&mem, bytes, s) != PASUR_OK) {
    return PASUR_OK;
  }
  unsigned char *const at = (unsigned char *)mem + far_bytes;
  put(at, stage.data(), stage.size(), s);
  int64_t work[4] = {0, 0, 0, 0};
  add_work(work, f);
  {
    ProfScope ps(all_lds(x.forms) ? 2 : 3, -1, s, work[0], work[1], work[2], work[3], n_iters);
    launch_segments<T>(x.launches, at, (const Seg *)x.mem, (const IterK *)(at + align16(sizeof(D))),
                       mem, n_iters, p->variant, p->rm_mode, p->eps, nullptr, s);
  }
  const hipError_t e = hipGetLastError();
  if (capturing) (void)hipFreeAsync(mem, s);
  else block_free_on(mem, s);
  *done = true;
  PASUR_TRY_HIP(e);
  return PASUR_OK;
}
}  // namespace

namespace pasur {
bool seg_ready(const pasur_fgt *f, int dtype) {
  std::lock_guard<std::mutex> lock(g_counts_mu);
  return find_index(f, dtype, 0, 0, true) != nullptr;
}

int seg_enqueue(pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p, int64_t t0,
                int n_iters, bool capturing, bool *done, hipStream_t s) {
  if (n_iters > kSegIters) return PASUR_OK;
  const SegIndex *x;
  {
    std::lock_guard<std::mutex> lock(g_counts_mu);
    x = find_index(f, st->dtype, p->block, p->seg_nodes, false);
    if (!x && capturing) x = find_index(f, st->dtype, 0, 0, true);
  }
  if (!x && !capturing) {
    PASUR_TRY(root_counts(f, s));
    // for both types, so that a later call may be captured whatever its state's
    for (int dtype : {PASUR_F32, PASUR_F64}) {
      if (dtype != st->dtype && seg_ready(f, dtype)) continue;
      PASUR_TRY(build_index(f, dtype, p->block, p->seg_nodes, s));
    }
    std::lock_guard<std::mutex> lock(g_counts_mu);
    // (a tree's list has room for kSegIndexes: any has the same results)
    x = find_index(f, st->dtype, p->block, p->seg_nodes, false);
    if (!x) x = find_index(f, st->dtype, 0, 0, true);
  }
  if (!x) return PASUR_OK;
  return st->dtype == PASUR_F32 ? enqueue<float>(f, *x, st, p, t0, n_iters, capturing, done, s)
                                : enqueue<double>(f, *x, st, p, t0, n_iters, capturing, done, s);
}
}  // namespace pasur

extern "C" int pasur_plan_iterate(const pasur_plan *pl, int64_t t0, int n_iters, void *stream) {
  if (!pl) {
    set_error("plan is NULL");
    return PASUR_E_INVAL;
  }
  if (n_iters < 0 || t0 < pl->t_first || t0 + n_iters - 1 > pl->t_last) {
    set_error("iterations %lld..%lld outside the plan's %lld..%lld", (long long)t0,
              (long long)(t0 + n_iters - 1), (long long)pl->t_first, (long long)pl->t_last);
    return PASUR_E_RANGE;
  }
  if (n_iters == 0) return PASUR_OK;
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps(all_lds(pl->forms) ? 2 : 3, -1, s, pl->work[0], pl->work[1], pl->work[2],
                 pl->work[3], n_iters);
    const IterK *const ks = pl->d_ks + (t0 - pl->t_first);
    if (pl->dtype == PASUR_F32)
      launch_segments<float>(pl->launches, pl->d_items, pl->d_segs, ks, pl->far, n_iters,
                             pl->variant, pl->rm_mode, pl->eps, pl->d_unplanned, s);
    else
      launch_segments<double>(pl->launches, pl->d_items, pl->d_segs, ks, pl->far, n_iters,
                              pl->variant, pl->rm_mode, pl->eps, pl->d_unplanned, s);
  }
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

namespace {
// The least and most threads per workgroup of a plan's launches.
std::pair<int, int> threads(const pasur_plan *pl) {
  std::pair<int, int> t(1024, 0);
  for (const SegLaunch &la : pl->launches) {
    t.first = std::min(t.first, la.block);
    t.second = std::max(t.second, la.block);
  }
  return t;
}
}  // namespace

extern "C" int pasur_plan_forms(const pasur_plan *pl, int64_t info[8]) {
  if (!pl || !info) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  for (int k = 0; k < 4; ++k) info[k] = pl->forms[k];
  info[4] = (int64_t)pl->launches.size();
  info[5] = threads(pl).first;
  info[6] = threads(pl).second;
  unsigned n = 0;
  PASUR_TRY_HIP(hipMemcpy(&n, pl->d_unplanned, sizeof(n), hipMemcpyDeviceToHost));
  info[7] = n;
  return PASUR_OK;
}

extern "C" int pasur_plan_info(const pasur_plan *pl, int64_t info[8]) {
  if (!pl || !info) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  info[0] = pl->n_segs;
  info[1] = pl->forms[F_LDS];
  info[2] = pl->lds_bytes;
  info[3] = threads(pl).second;
  info[4] = pl->work[0];
  info[5] = pl->work[1];
  info[6] = pl->work[2];
  info[7] = pl->work[3];
  return PASUR_OK;
}
