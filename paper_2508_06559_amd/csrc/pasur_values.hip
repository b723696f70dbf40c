// pasur_values.hip -- exact values of unfolded trees from the leaves to the
// roots: expectation under a strategy, best responses, minimax, and the best
// responses composed over a subgame's rounds (exploitability).
//
// One launch per round.  The subtrees below different roots never meet, so a
// workgroup takes a root and carries its values from the leaves to the root
// without writing a level to memory: a thread evaluates the whole subtree of
// one node of a base level (nested loops over its descendants, which are
// consecutive on every level), the base level's values go to LDS, and the
// levels above are reduced there.  What bounds a large round is then the
// reading of the tree (strategy 4 or 8 bytes per edge, child range 4 bytes per
// node, leaf points and links 6 bytes per leaf), once for all values wanted:
// best responses of both players and the expectation share every load.
// One level per launch through level buffers in memory, three times over, was
// 3.3 ms of kernels on a game of 1.8e8 nodes, and 97 ms with the allocation
// and release of those buffers.
//
// A root too large for one workgroup beside the others is split: every node of
// level 6 is evaluated by a thread of its own, then the nodes of the levels above
// one level a launch, until the roots' nodes fit a workgroup each (one root of
// 6.2e6 nodes: 88 ms in one workgroup, 0.14 split; from level 5 or 7 on 0.20 and
// 0.15).
//
// Sums run in child order from 0.0 in FP64, one node at a time, whatever the
// base level is.  Contraction of a*b+c into fma is switched off.
#pragma clang fp contract(off)

#include "pasur_internal.hpp"

#include <algorithm>

namespace pasur {
namespace {

// Leaves given as an array, one value for every mode.
template <class L>
struct LeafArray {
  const L *leaf;
  __device__ __forceinline__ void get(int32_t i, double *v, int nm) const {
    const double x = (double)leaf[i];
    for (int m = 0; m < nm; ++m) v[m] = x;
  }
};

// Leaves of a round within a subgame: the round's points plus the next
// round's value of the same mode at the linked root (V[nm * root + mode];
// NULL in round 5).  bonus: with the literal bonus rule, the leaves' final
// bonus states (0 costs 7 points), else NULL.
struct LeafRound {
  const int16_t *base;
  const int32_t *link;
  const int8_t *bonus;
  const double *V;
  __device__ __forceinline__ void get(int32_t i, double *v, int nm) const {
    double pts = (double)base[i];
    if (bonus && bonus[i] == 0) pts -= 7.0;
    if (V) {
      const double *x = V + (int64_t)nm * link[i];
      for (int m = 0; m < nm; ++m) v[m] = x[m] + pts;
    } else {
      for (int m = 0; m < nm; ++m) v[m] = pts;
    }
  }
};

template <class T, class Leaf, int NM>
struct ValueArgs {
  const int32_t *cb[8];
  const T *sigma[9];       // levels 1..8, may be NULL where no mode reads them
  const int32_t *off[6];   // root offsets per level
  Leaf leaf;
  int mode[NM];
  double *out[NM];         // value of root or node j at out[m][j * stride], NULL: not wanted
  int64_t stride;
  const double *part;      // given values of level `base`, the NM of a node side by
  int base;                // side, or NULL: from the leaves
};

enum { V_SUM, V_MAX, V_MIN };

// What a mode does at the nodes of a level whose mover is given.
__device__ __forceinline__ int value_kind(int mode, int mover) {
  if (mover == 0) return mode == PASUR_TV_MINIMAX || mode == PASUR_TV_BR_A ? V_MAX : V_SUM;
  return mode == PASUR_TV_MINIMAX || mode == PASUR_TV_BR_B ? V_MIN : V_SUM;
}

// Accumulator of one node's NM values.  With three modes they are both best
// responses and the expectation, known at compile time.
template <int NM>
struct Node {
  double v[NM];
  template <class Args>
  static __device__ __forceinline__ int kind(const Args &a, int m, int mover) {
    if (NM == 3)
      return m == 0 && mover == 0 ? V_MAX : m == 1 && mover == 1 ? V_MIN : V_SUM;
    return value_kind(a.mode[m], mover);
  }
  // Some value needs the strategy at these nodes.
  template <class Args>
  static __device__ __forceinline__ bool weighs(const Args &a, int mover) {
    return NM > 1 || kind(a, 0, mover) == V_SUM;
  }
  template <class Args>
  __device__ __forceinline__ void start(const Args &a, int mover) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int k = kind(a, m, mover);
      v[m] = k == V_MAX ? -INFINITY : k == V_MIN ? INFINITY : 0.0;
    }
  }
  template <class Args>
  __device__ __forceinline__ void add(const Args &a, int mover, double s, const double *c) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int k = kind(a, m, mover);
      if (k == V_MAX) v[m] = fmax(v[m], c[m]);
      else if (k == V_MIN) v[m] = fmin(v[m], c[m]);
      else v[m] += s * c[m];
    }
  }
};

// Values of node h of level L from its subtree.
template <int L, class T, class Leaf, int NM>
__device__ __forceinline__ void value_of(const ValueArgs<T, Leaf, NM> &a, int32_t h, double *out) {
  if constexpr (L == 8) {
    a.leaf.get(h, out, NM);
  } else {
    const int32_t b = a.cb[L][h], e = a.cb[L][h + 1];
    const T *sg = Node<NM>::weighs(a, L & 1) ? a.sigma[L + 1] : nullptr;
    Node<NM> n;
    n.start(a, L & 1);
    for (int32_t q = b; q < e; ++q) {
      double c[NM];
      const double s = sg ? (double)sg[q] : 0.0;
      value_of<L + 1>(a, q, c);
      n.add(a, L & 1, s, c);
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) out[m] = n.v[m];
  }
}

template <int L, int BLOCK, class T, class Leaf, int NM>
__device__ __forceinline__ void base_level(const ValueArgs<T, Leaf, NM> &a, int32_t h0, int n,
                                           double *lds) {
  for (int i = threadIdx.x; i < n; i += BLOCK) {
    double v[NM];
    value_of<L>(a, h0 + i, v);
#pragma unroll
    for (int m = 0; m < NM; ++m) lds[NM * i + m] = v[m];
  }
}

// A thread per node of level L, from the leaves.
template <int L, class T, class Leaf, int NM>
__global__ void __launch_bounds__(256) k_values_leaves(ValueArgs<T, Leaf, NM> a, int64_t n) {
  const int64_t h = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (h >= n) return;
  double v[NM];
  value_of<L>(a, (int32_t)h, v);
#pragma unroll
  for (int m = 0; m < NM; ++m) a.out[m][h * a.stride] = v[m];
}

// A thread per node of level a.base - 1, from the given values of its children.
template <class T, class Leaf, int NM>
__global__ void __launch_bounds__(256) k_values_level(ValueArgs<T, Leaf, NM> a, int64_t n) {
  const int64_t h = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (h >= n) return;
  const int l = a.base - 1;
  const int32_t b = a.cb[l][h], e = a.cb[l][h + 1];
  const T *sg = Node<NM>::weighs(a, l & 1) ? a.sigma[l + 1] : nullptr;
  Node<NM> v;
  v.start(a, l & 1);
  for (int32_t q = b; q < e; ++q)
    v.add(a, l & 1, sg ? (double)sg[q] : 0.0, a.part + (int64_t)NM * q);
#pragma unroll
  for (int m = 0; m < NM; ++m) a.out[m][h * a.stride] = v.v[m];
}

// One workgroup per root.  The base level is the deepest of levels 1..5 whose
// nodes below the root fit in CAP entries of LDS (deeper: more threads with
// shorter loops; level 6 and below are mostly single-child chains), or that of the
// given values.  A level is then reduced in place: every thread holds its parents'
// values in registers across the barrier that ends the reading of their children.
template <class T, class Leaf, int NM, int BLOCK, int CAP>
__global__ void __launch_bounds__(BLOCK) k_values_roots(ValueArgs<T, Leaf, NM> a) {
  __shared__ double lds[NM * CAP];
  const int64_t j = blockIdx.x;
  int l = a.part ? a.base : 5;
  int32_t h0 = a.off[l][j];
  int n = a.off[l][j + 1] - h0;
  while (!a.part && l > 1 && n > CAP) {
    --l;
    h0 = a.off[l][j];
    n = a.off[l][j + 1] - h0;
  }
  if (n <= CAP) {
    if (a.part) {
      for (int i = threadIdx.x; i < NM * n; i += BLOCK) lds[i] = a.part[(int64_t)NM * h0 + i];
    } else switch (l) {
      case 5: base_level<5, BLOCK>(a, h0, n, lds); break;
      case 4: base_level<4, BLOCK>(a, h0, n, lds); break;
      case 3: base_level<3, BLOCK>(a, h0, n, lds); break;
      case 2: base_level<2, BLOCK>(a, h0, n, lds); break;
      default: base_level<1, BLOCK>(a, h0, n, lds); break;
    }
    constexpr int PER = CAP / BLOCK;  // parents per thread (no level has more than the one below)
    for (--l; l >= 0; --l) {
      __syncthreads();
      const int32_t c0 = h0;
      h0 = a.off[l][j];
      n = a.off[l][j + 1] - h0;
      const T *sg = Node<NM>::weighs(a, l & 1) ? a.sigma[l + 1] : nullptr;
      Node<NM> v[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int i = threadIdx.x + k * BLOCK;
        if (i < n) {
          const int32_t b = a.cb[l][h0 + i], e = a.cb[l][h0 + i + 1];
          v[k].start(a, l & 1);
          for (int32_t q = b; q < e; ++q)
            v[k].add(a, l & 1, sg ? (double)sg[q] : 0.0, lds + NM * (q - c0));
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int i = threadIdx.x + k * BLOCK;
        if (i < n) {
#pragma unroll
          for (int m = 0; m < NM; ++m) lds[NM * i + m] = v[k].v[m];
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < NM && a.out[threadIdx.x])
      a.out[threadIdx.x][j * a.stride] = lds[threadIdx.x];
  } else if (threadIdx.x == 0) {  // more than CAP moves at the root: not in Pasur
    double v[NM];
    value_of<0>(a, (int32_t)j, v);
    for (int m = 0; m < NM; ++m)
      if (a.out[m]) a.out[m][j * a.stride] = v[m];
  }
}

constexpr int kWide = 4096;
constexpr int kFlat = 6;  // the level whose nodes a split round evaluates from the leaves

// Few roots leave most CUs without a workgroup: there a root gets 1024 threads
// and room for a wide base level.  With many, small workgroups of 24 KB of LDS
// (three modes) keep six of them on a CU.
constexpr int64_t kFewRoots = 1024;

// split: room for split_nodes(f) * NM values.
template <class T, class Leaf, int NM>
int launch(const pasur_fgt *f, const Leaf &leaf, void *const *sigma, const int *mode,
           double *const *out, int64_t stride, double *split, hipStream_t s) {
  ValueArgs<T, Leaf, NM> a;
  for (int l = 0; l < 8; ++l) a.cb[l] = f->child_begin[l];
  a.sigma[0] = nullptr;
  for (int l = 1; l < 9; ++l) a.sigma[l] = sigma ? (const T *)sigma[l] : nullptr;
  for (int l = 0; l < 6; ++l) a.off[l] = f->root_off[l];
  a.leaf = leaf;
  for (int m = 0; m < NM; ++m) a.mode[m] = mode[m];
  a.part = nullptr;
  a.base = 0;
  if (f->value_stop) {
    a.stride = NM;
    for (int l = kFlat; l >= f->value_stop; --l) {
      const unsigned grid = (unsigned)((f->n[l] + 255) / 256);
      for (int m = 0; m < NM; ++m) a.out[m] = split + m;
      if (l == kFlat) k_values_leaves<kFlat, T, Leaf, NM><<<grid, 256, 0, s>>>(a, f->n[l]);
      else k_values_level<T, Leaf, NM><<<grid, 256, 0, s>>>(a, f->n[l]);
      a.part = split;
      a.base = l;
      split += NM * f->n[l];
    }
  }
  a.stride = stride;
  for (int m = 0; m < NM; ++m) a.out[m] = out[m];
  const unsigned grid = (unsigned)f->n[0];
  if (a.part || f->n[0] <= kFewRoots)
    k_values_roots<T, Leaf, NM, 1024, kWide><<<grid, 1024, 0, s>>>(a);
  else
    k_values_roots<T, Leaf, NM, 256, 1024><<<grid, 256, 0, s>>>(a);
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

template <class T, int NM>
int composed(const pasur_fgt *const *fgts, int n_rounds, void *const *sigma_bar, int leaf_flags,
             const int *mode, double *const *outs, hipStream_t s) {
  // the root values of rounds 1.., the NM values of a root side by side, and
  // those of split rounds
  int64_t most = 0, split = 0;
  for (int r = 0; r < n_rounds; ++r) {
    if (r > 0) most = std::max(most, fgts[r]->n[0]);
    split = std::max(split, split_nodes(fgts[r]));
  }
  double *buf = nullptr;
  if (most + split > 0) {
    const hipError_t e = malloc_async((void **)&buf, NM * (2 * most + split) * sizeof(double), s);
    if (e != hipSuccess) {
      set_error("hipMallocAsync: %s", hipGetErrorString(e));
      return PASUR_E_NOMEM;
    }
  }
  int st = PASUR_OK;
  const double *V = nullptr;  // the later round's root values
  for (int r = n_rounds - 1; r >= 0 && !st; --r) {
    const pasur_fgt *f = fgts[r];
    LeafRound leaf;
    leaf.base = f->leaf_base;
    leaf.link = f->link;
    leaf.bonus =
        f->round == 5 && (leaf_flags & PASUR_LEAF_LITERAL_BONUS0) ? f->leaf_bonus : nullptr;
    leaf.V = V;
    double *res = buf + (r & 1) * NM * most;
    double *out[NM];
    for (int m = 0; m < NM; ++m) out[m] = r > 0 ? res + m : outs[m];
    st = launch<T, LeafRound, NM>(f, leaf, sigma_bar + r * 9, mode, out, r > 0 ? NM : 1,
                                  buf + 2 * NM * most, s);
    V = res;
  }
  if (buf) (void)hipFreeAsync(buf, s);
  return st;
}

int values_of_leaves(const pasur_fgt *f, const void *leaf, int leaf_dtype, int dtype,
                     void *const *sigma, int mode, double *out, double *split, hipStream_t s) {
  const LeafArray<double> ld{(const double *)leaf};
  if (dtype == PASUR_F64)
    return launch<double, LeafArray<double>, 1>(f, ld, sigma, &mode, &out, 1, split, s);
  if (leaf_dtype == PASUR_F64)
    return launch<float, LeafArray<double>, 1>(f, ld, sigma, &mode, &out, 1, split, s);
  return launch<float, LeafArray<float>, 1>(f, LeafArray<float>{(const float *)leaf}, sigma, &mode,
                                            &out, 1, split, s);
}

}  // namespace

int64_t split_nodes(const pasur_fgt *f) {
  int64_t n = 0;
  if (f->value_stop)
    for (int l = f->value_stop; l <= kFlat; ++l) n += f->n[l];
  return n;
}

int value_stop(const int64_t n[9], int64_t n_roots, const int32_t *root_off) {
  // Leaves of the largest root, a third of its nodes: a workgroup takes 24 us for
  // 6,000 nodes, 100 us for 60,000 and 5.8 ms for 700,000; the chip takes 1e11
  // nodes a second.  A root of more is worth some launches of 5 us if the round's
  // other roots don't take as long.
  auto widest = [&](int l) {
    const int32_t *const o = root_off + l * (n_roots + 1);
    int32_t w = 0;
    for (int64_t j = 0; j < n_roots; ++j) w = std::max(w, o[j + 1] - o[j]);
    return w;
  };
  const int32_t most = widest(8);
  if (most <= 3500 + n[8] / (most > 60000 ? 800 : 160)) return 0;
  int l = 5;
  while (l > 1 && widest(l) > kWide) --l;
  return l;
}

int tree_values(const pasur_fgt *f, const void *leaf, int leaf_dtype, int dtype,
                void *const *sigma, int mode, double *out, bool alloc, hipStream_t s) {
  if (f->n[0] == 0) return PASUR_OK;
  double *split = f->split_ws;
  if (f->value_stop && alloc) {
    const hipError_t e = malloc_async((void **)&split, (size_t)split_nodes(f) * sizeof(double), s);
    if (e != hipSuccess) {
      set_error("hipMallocAsync: %s", hipGetErrorString(e));
      return PASUR_E_NOMEM;
    }
  }
  const int st = values_of_leaves(f, leaf, leaf_dtype, dtype, sigma, mode, out, split, s);
  if (f->value_stop && alloc) (void)hipFreeAsync(split, s);
  return st;
}

int composed_values(const pasur_fgt *const *fgts, int n_rounds, void *const *sigma_bar, int dtype,
                    int leaf_flags, double *br_a, double *br_b, double *v, hipStream_t s) {
  double *outs[3] = {br_a, br_b, v};
  const int modes[3] = {PASUR_TV_BR_A, PASUR_TV_BR_B, PASUR_TV_EXPECT};
  const int wanted = (br_a != nullptr) + (br_b != nullptr) + (v != nullptr);
  if (wanted > 1)
    return dtype == PASUR_F32
               ? composed<float, 3>(fgts, n_rounds, sigma_bar, leaf_flags, modes, outs, s)
               : composed<double, 3>(fgts, n_rounds, sigma_bar, leaf_flags, modes, outs, s);
  const int m = br_a ? 0 : br_b ? 1 : 2;
  return dtype == PASUR_F32
             ? composed<float, 1>(fgts, n_rounds, sigma_bar, leaf_flags, modes + m, outs + m, s)
             : composed<double, 1>(fgts, n_rounds, sigma_bar, leaf_flags, modes + m, outs + m, s);
}

}  // namespace pasur
