// pasur_parents.hpp -- one pass over the nodes of levels 0..7 of a tree and
// their children, all levels in one launch (a launch per level cost the small
// rounds eight times a launch's 2 to 4 us).
#pragma once

#include "pasur_internal.hpp"

namespace pasur {

constexpr int kParentThreads = 256;
// Parents per thread, a workgroup's width apart: what bounds these passes is
// the bytes, but with one parent per thread the chain of dependent loads in
// each of millions of short waves did (set-up of a round of 6.8e8 nodes: 4.2 ms
// at 1.9 TB/s).
constexpr int kParentsPer = 4;

struct AllParents {
  const int32_t *cb[8];
  int64_t n[8];
  unsigned block[9];  // first workgroup of each level
};

inline AllParents all_parents(const pasur_fgt *f) {
  constexpr int64_t per = kParentThreads * kParentsPer;
  AllParents P;
  P.block[0] = 0;
  for (int l = 0; l < 8; ++l) {
    P.cb[l] = f->child_begin[l];
    P.n[l] = f->n[l];
    P.block[l + 1] = P.block[l] + (unsigned)((f->n[l] + per - 1) / per);
  }
  return P;
}

// A workgroup's level, and a thread's parents with their child ranges (empty
// past the level's end).
struct MyParents {
  int level;
  int64_t h[kParentsPer];
  int32_t b[kParentsPer], e[kParentsPer];

  __device__ __forceinline__ MyParents(const AllParents &P, unsigned block) {
    level = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) level += block >= P.block[k] ? 1 : 0;
    const int64_t h0 = (int64_t)(block - P.block[level]) * (kParentThreads * kParentsPer);
    const int32_t *const cb = P.cb[level];
#pragma unroll
    for (int k = 0; k < kParentsPer; ++k) {
      h[k] = h0 + k * kParentThreads + (int)threadIdx.x;
      const bool in = h[k] < P.n[level];
      b[k] = in ? cb[h[k]] : 0;
      e[k] = in ? cb[h[k] + 1] : 0;
    }
  }
};

template <class T>
struct EdgeArrays {
  T *a[9], *b[9], *c[9];  // levels 1..8
};

template <class T>
EdgeArrays<T> edge_arrays(void *const a[9], void *const b[9], void *const c[9]) {
  EdgeArrays<T> E;
  for (int l = 0; l < 9; ++l) {
    E.a[l] = l && a ? (T *)a[l] : nullptr;
    E.b[l] = l && b ? (T *)b[l] : nullptr;
    E.c[l] = l && c ? (T *)c[l] : nullptr;
  }
  return E;
}

// b = w(a) over its sum among the children of the same node, in child order;
// 1 / children where the sum is not positive.  The first kAhead children of all
// of a thread's parents are read before any is used.
template <class T, class Weight>
__device__ __forceinline__ void normalise(const MyParents &m, const T *in, T *out, Weight w) {
  constexpr int kAhead = 2;
  T v[kParentsPer][kAhead];
#pragma unroll
  for (int k = 0; k < kParentsPer; ++k)
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      v[k][j] = m.b[k] + j < m.e[k] ? in[m.b[k] + j] : (T)0;
#pragma unroll
  for (int k = 0; k < kParentsPer; ++k) {
    const int32_t b = m.b[k], e = m.e[k];
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      if (b + j < e) s += w((double)v[k][j]);
    for (int32_t q = b + kAhead; q < e; ++q) s += w((double)in[q]);
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      if (b + j < e) out[b + j] = (T)(s > 0.0 ? w((double)v[k][j]) / s : 1.0 / (double)(e - b));
    for (int32_t q = b + kAhead; q < e; ++q)
      out[q] = (T)(s > 0.0 ? w((double)in[q]) / s : 1.0 / (double)(e - b));
  }
}

template <class T, class Weight>
__global__ void __launch_bounds__(kParentThreads)
    k_normalise(AllParents P, EdgeArrays<T> E, Weight w) {
  const MyParents m(P, blockIdx.x);
  normalise<T>(m, E.a[m.level + 1], E.b[m.level + 1], w);
}

}  // namespace pasur
