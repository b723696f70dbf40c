// pasur_cfr.hip -- full-width DCFR on one round's unfolded tree, leaf
// utilities, average strategy and round values.
//
// State is stored as T (float or double); every arithmetic step runs in
// double registers, with the operations of each parent's update done in the
// order of the paper's FindUtility (sum, regret, discount, matching,
// average).  Contraction of a*b+c into fma is switched off so that the
// double-state path rounds exactly like a plain sequential implementation.
#pragma clang fp contract(off)

#include "pasur_internal.hpp"
#include "pasur_parents.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

using namespace pasur;

namespace {

// Optional per-launch timing of the sweep kernels (HIP events on the launch
// stream), off unless pasur_profile_enable(1) was called.
std::mutex g_prof_mu;
std::vector<ProfRec> g_prof;
std::vector<hipEvent_t> g_event_pool;  // events of cleared records, reused
bool g_prof_on = false;
uint64_t g_prof_mask = ~0ull;  // kernel ids recorded (bit k)

void prof_clear() {
  for (auto &r : g_prof) {
    g_event_pool.push_back(r.a);
    g_event_pool.push_back(r.b);
  }
  g_prof.clear();
}

constexpr int kThreads = 256;
inline unsigned grid_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// Zeros in p[b] .. p[e-1] by a workgroup, 16 bytes per thread and store.
template <class T>
__device__ __forceinline__ void zero_range(T *p, int64_t b, int64_t e) {
  constexpr int kPer = 16 / (int)sizeof(T);
  const int64_t lead = ((16 - (int64_t)(reinterpret_cast<uintptr_t>(p + b) & 15)) & 15) / (int)sizeof(T);
  const int64_t b16 = b + lead < e ? b + lead : e, n16 = (e - b16) / kPer;
  int4 *const q = reinterpret_cast<int4 *>(p + b16);
  for (int64_t i = threadIdx.x; i < n16; i += kParentThreads) q[i] = make_int4(0, 0, 0, 0);
  const int64_t tail = b16 + n16 * kPer;
  if ((int64_t)threadIdx.x < b16 - b) p[b + threadIdx.x] = (T)0;
  if ((int64_t)threadIdx.x < e - tail) p[tail + threadIdx.x] = (T)0;
}

// sigma uniform, R and Sbar zero for the children of a workgroup's parents (their
// children are neighbours); the roots' reaches and utility sums.  Bound by the
// 12 B written per edge (6.8e8 nodes: 3.0 ms with R and Sbar written child by
// child beside sigma).
template <class T>
__device__ __forceinline__ void init_children(const AllParents &P, const MyParents &m,
                                              const EdgeArrays<T> &E, T *ra, T *rb, double *vacc) {
  T *const sg = E.a[m.level + 1];
#pragma unroll
  for (int k = 0; k < kParentsPer; ++k) {
    const int32_t b = m.b[k], e = m.e[k];
    const T s = (T)(1.0 / (double)(e - b));
    for (int32_t q = b; q < e; ++q) sg[q] = s;
    if (m.level == 0 && m.h[k] < P.n[0]) {
      ra[m.h[k]] = (T)1;
      rb[m.h[k]] = (T)1;
      vacc[m.h[k]] = 0.0;
    }
  }
  const int64_t h0 = m.h[0] - (int)threadIdx.x;
  int64_t h1 = h0 + kParentThreads * kParentsPer;
  if (h1 > P.n[m.level]) h1 = P.n[m.level];
  const int64_t b = P.cb[m.level][h0], e = P.cb[m.level][h1];
  zero_range(E.b[m.level + 1], b, e);
  zero_range(E.c[m.level + 1], b, e);
}

template <class T>
__global__ void __launch_bounds__(kParentThreads)
    k_init(AllParents P, EdgeArrays<T> E, T *ra, T *rb, double *vacc) {
  const MyParents m(P, blockIdx.x);
  init_children<T>(P, m, E, ra, rb, vacc);
}

// FindReachProbability, one level: the mover's reach picks up sigma of the
// edge taken, the other player's reach is inherited.
template <class T>
__global__ void k_down(int64_t n, int mover, const int32_t *__restrict__ parent,
                       const T *__restrict__ sigma, const T *__restrict__ ra_up,
                       const T *__restrict__ rb_up, T *__restrict__ ra, T *__restrict__ rb) {
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int32_t h = parent[q];
  double a = (double)ra_up[h];
  double b = (double)rb_up[h];
  if (mover == 0) a *= (double)sigma[q];
  else b *= (double)sigma[q];
  ra[q] = (T)a;
  rb[q] = (T)b;
}

// FindUtility, one level, one thread per parent h (children cb[h]..cb[h+1]):
//   u(h) = sum sigma^t u;  r = s_p pi_{-p}(h) (u(q) - u(h));
//   R <- d R + r;  sigma^{t+1} = max(R, eps) / sum;  Sbar <- w Sbar + pi_p(h) sigma^t
// (with PASUR_CFR_SNIPPET_AVG the term also carries sigma^{t+1}, as stored).
constexpr double kSnippetTol = 1e-5;
template <class T>
__global__ void k_up(int64_t np, int mover, const int32_t *__restrict__ cb,
                     T *__restrict__ sigma, T *__restrict__ R, T *__restrict__ Sbar,
                     const T *__restrict__ u_child, T *__restrict__ u_par,
                     const T *__restrict__ ra, const T *__restrict__ rb, IterConsts ic,
                     double *__restrict__ vacc) {
  int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= np) return;
  const int32_t b = cb[h], e = cb[h + 1];
  double uh = 0.0;
  for (int32_t q = b; q < e; ++q) uh += (double)sigma[q] * (double)u_child[q];
  u_par[h] = (T)uh;
  const double opp = mover == 0 ? (double)rb[h] : (double)ra[h];
  const double own = mover == 0 ? (double)ra[h] : (double)rb[h];
  const double sgn = mover == 0 ? 1.0 : -1.0;
  for (int32_t q = b; q < e; ++q) {
    const double r = sgn * opp * ((double)u_child[q] - uh);
    double Rq = (double)R[q];
    if (ic.variant == PASUR_DCFR) {
      const bool pos = (ic.flags & PASUR_CFR_SNIPPET_TOL) ? Rq >= kSnippetTol : Rq > 0.0;
      const double d = pos ? ic.dpos : ic.dneg;
      Rq = d * Rq + r;
    } else if (ic.variant == PASUR_CFR_PLUS) {
      Rq = Rq + r;
      if (Rq < 0.0) Rq = 0.0;
    } else {
      Rq = Rq + r;
    }
    R[q] = (T)Rq;
  }
  double sum = 0.0;
  for (int32_t q = b; q < e; ++q) {
    const double x = ic.rm_mode == PASUR_RM_FLOOR ? fmax((double)R[q], ic.eps)
                                                  : fmax((double)R[q], 0.0);
    sum += x;
  }
  const double inv_k = 1.0 / (double)(e - b);
  for (int32_t q = b; q < e; ++q) {
    const double x = ic.rm_mode == PASUR_RM_FLOOR ? fmax((double)R[q], ic.eps)
                                                  : fmax((double)R[q], 0.0);
    const double s_new = sum > 0.0 ? x / sum : inv_k;
    double add = own * (double)sigma[q];
    if (ic.variant == PASUR_CFR_PLUS) add *= ic.avg_t;
    if (ic.flags & PASUR_CFR_SNIPPET_AVG) add *= (double)(T)s_new;
    Sbar[q] = (T)(ic.avg_w * (double)Sbar[q] + add);
    sigma[q] = (T)s_new;
  }
  if (vacc) vacc[h] += uh;
}

// the average strategy: sums normalised as they are
struct AsIs {
  __device__ __forceinline__ double operator()(double x) const { return x; }
};

template <class T>
__device__ __forceinline__ void leaf_util(int64_t i, const int16_t *base, const int32_t *link,
                                          const double *V, const int8_t *bonus0_literal, T *out) {
  double pts = (double)base[i];
  if (bonus0_literal && bonus0_literal[i] == 0) pts -= 7.0;
  out[i] = (T)(V ? V[link[i]] + pts : pts);
}

template <class T>
__global__ void k_leaf_util(int64_t n, const int16_t *__restrict__ base,
                            const int32_t *__restrict__ link, const double *__restrict__ V,
                            const int8_t *__restrict__ bonus0_literal, T *__restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) leaf_util<T>(i, base, link, V, bonus0_literal, out);
}

__global__ void k_div(int64_t n, const double *__restrict__ a, double T, double *__restrict__ out) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) out[j] = a[j] / T;
}

// ---- several trees at once ----------------------------------------------------
// What surrounds the iterations of a batch, for kItems trees a launch, as kernel
// arguments: with four launches a tree, of 3 to 9 us each, they took a fifth of
// the solve of a batch of 64 deals.
constexpr int kItems = 8;

template <class T>
struct BeginItem {
  AllParents P;
  EdgeArrays<T> E;  // sigma, R, Sbar
  T *ra, *rb, *leaf;
  double *vacc;
  int64_t n_leaf;
  const int16_t *base;
  const int32_t *link;
  const double *V;
};
template <class T>
struct EndItem {
  AllParents P;
  EdgeArrays<T> E;  // Sbar, average strategy
  const double *vacc;
  double *V;
};
template <class Item>
struct Items {
  unsigned first[kItems + 1];  // first workgroup of each; past the last: the grid
  Item item[kItems];

  __device__ __forceinline__ int mine() const {
    int k = 0;
#pragma unroll
    for (int j = 1; j < kItems; ++j) k += blockIdx.x >= first[j] ? 1 : 0;
    return __builtin_amdgcn_readfirstlane(k);
  }
};

// Leaf utilities and the initial state.
template <class T>
__global__ void __launch_bounds__(kParentThreads) k_begin(Items<BeginItem<T>> a) {
  const int k = a.mine();
  const BeginItem<T> &x = a.item[k];
  const unsigned block = blockIdx.x - a.first[k];
  if (block < x.P.block[8]) {
    const MyParents m(x.P, block);
    init_children<T>(x.P, m, x.E, x.ra, x.rb, x.vacc);
    return;
  }
  const int64_t i0 = (int64_t)(block - x.P.block[8]) * (kParentThreads * kParentsPer) + threadIdx.x;
#pragma unroll
  for (int j = 0; j < kParentsPer; ++j) {
    const int64_t i = i0 + j * kParentThreads;
    if (i < x.n_leaf) leaf_util<T>(i, x.base, x.link, x.V, nullptr, x.leaf);
  }
}

// The average strategy and the roots' mean utility over T iterations.
template <class T>
__global__ void __launch_bounds__(kParentThreads) k_end(Items<EndItem<T>> a, double iters) {
  const int k = a.mine();
  const EndItem<T> &x = a.item[k];
  const MyParents m(x.P, blockIdx.x - a.first[k]);
  normalise<T>(m, x.E.a[m.level + 1], x.E.b[m.level + 1], AsIs());
  if (m.level == 0) {
#pragma unroll
    for (int j = 0; j < kParentsPer; ++j)
      if (m.h[j] < x.P.n[0]) x.V[m.h[j]] = x.vacc[m.h[j]] / iters;
  }
}

// Launches over `n` items, kItems at a time; make(i, &item) fills one and
// returns its workgroups.
template <class Item, class Make, class Launch>
void launch_items(int n, const Make &make, const Launch &launch) {
  for (int i0 = 0; i0 < n; i0 += kItems) {
    Items<Item> a = {};
    unsigned at = 0;
    for (int k = 0; k < kItems; ++k) {
      a.first[k] = at;
      if (i0 + k < n) at += make(i0 + k, a.item[k]);
    }
    a.first[kItems] = at;
    if (at > 0) launch(a, at);
  }
}

template <class T>
int begin_t(const pasur_fgt *const *f, const pasur_cfr_state *const *st, const double *const *V,
            int n, hipStream_t s) {
  launch_items<BeginItem<T>>(
      n,
      [&](int i, BeginItem<T> &x) {
        x.P = all_parents(f[i]);
        x.E = edge_arrays<T>(st[i]->sigma, st[i]->R, st[i]->Sbar);
        x.ra = (T *)st[i]->reachA[0];
        x.rb = (T *)st[i]->reachB[0];
        x.leaf = (T *)st[i]->u[8];
        x.vacc = st[i]->vacc;
        x.n_leaf = f[i]->n[8];
        x.base = f[i]->leaf_base;
        x.link = f[i]->link;
        x.V = f[i]->round < 5 ? V[i] : nullptr;
        constexpr int64_t per = kParentThreads * kParentsPer;
        return x.P.block[8] + (unsigned)((x.n_leaf + per - 1) / per);
      },
      [&](const Items<BeginItem<T>> &a, unsigned grid) {
        k_begin<T><<<grid, kParentThreads, 0, s>>>(a);
      });
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

template <class T>
int end_t(const pasur_fgt *const *f, const pasur_cfr_state *const *st, void *const *sigma_bar,
          double iters, double *const *V, int n, hipStream_t s) {
  launch_items<EndItem<T>>(
      n,
      [&](int i, EndItem<T> &x) {
        x.P = all_parents(f[i]);
        x.E = edge_arrays<T>(st[i]->Sbar, sigma_bar + 9 * i, nullptr);
        x.vacc = st[i]->vacc;
        x.V = V[i];
        return x.P.block[8];
      },
      [&](const Items<EndItem<T>> &a, unsigned grid) {
        k_end<T><<<grid, kParentThreads, 0, s>>>(a, iters);
      });
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

int check_items(const pasur_fgt *const *fgts, const pasur_cfr_state *const *states, int n_items) {
  if (!fgts || !states || n_items < 1) {
    set_error("null argument or empty batch");
    return PASUR_E_INVAL;
  }
  for (int i = 0; i < n_items; ++i) {
    if (!fgts[i] || !states[i]) {
      set_error("item %d is NULL", i);
      return PASUR_E_INVAL;
    }
    PASUR_TRY(check_state(fgts[i], states[i]));
    if (states[i]->dtype != states[0]->dtype) {
      set_error("all items need the same dtype");
      return PASUR_E_INVAL;
    }
  }
  return PASUR_OK;
}

template <class T>
int init_t(const pasur_fgt *f, const pasur_cfr_state *st, hipStream_t s) {
  const AllParents P = all_parents(f);
  k_init<T><<<P.block[8], kParentThreads, 0, s>>>(
      P, edge_arrays<T>(st->sigma, st->R, st->Sbar), (T *)st->reachA[0], (T *)st->reachB[0],
      st->vacc);
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

template <class T>
int iterate_t(const pasur_fgt *f, const pasur_cfr_state *st, const pasur_cfr_params *p,
              int64_t t0, int n_iters, hipStream_t s) {
  for (int64_t t = t0; t < t0 + n_iters; ++t) {
    const IterConsts ic = consts_for(p, t);
    for (int l = 1; l <= 7; ++l) {
      ProfScope ps(0, l, s, f->n[l], f->n[l - 1]);
      k_down<T><<<grid_for(f->n[l]), kThreads, 0, s>>>(
          f->n[l], (l - 1) & 1, f->parent[l], (const T *)st->sigma[l],
          (const T *)st->reachA[l - 1], (const T *)st->reachB[l - 1], (T *)st->reachA[l],
          (T *)st->reachB[l]);
    }
    for (int l = 8; l >= 1; --l) {
      ProfScope ps(1, l, s, f->n[l], f->n[l - 1]);
      k_up<T><<<grid_for(f->n[l - 1]), kThreads, 0, s>>>(
          f->n[l - 1], (l - 1) & 1, f->child_begin[l - 1], (T *)st->sigma[l], (T *)st->R[l],
          (T *)st->Sbar[l], (const T *)st->u[l], (T *)st->u[l - 1],
          (const T *)st->reachA[l - 1], (const T *)st->reachB[l - 1], ic,
          l == 1 ? st->vacc : nullptr);
    }
  }
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

}  // namespace

namespace pasur {
int check_state(const pasur_fgt *f, const pasur_cfr_state *st) {
  if (!f || !st) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (st->dtype != PASUR_F32 && st->dtype != PASUR_F64) {
    set_error("unknown dtype %d", st->dtype);
    return PASUR_E_RANGE;
  }
  for (int l = 0; l <= 8; ++l) {
    if (!st->u[l]) { set_error("u[%d] is NULL", l); return PASUR_E_INVAL; }
    if (l >= 1 && (!st->sigma[l] || !st->R[l] || !st->Sbar[l])) {
      set_error("sigma/R/Sbar[%d] is NULL", l);
      return PASUR_E_INVAL;
    }
    if (l <= 7 && (!st->reachA[l] || !st->reachB[l])) {
      set_error("reach[%d] is NULL", l);
      return PASUR_E_INVAL;
    }
  }
  if (!st->vacc) { set_error("vacc is NULL"); return PASUR_E_INVAL; }
  return PASUR_OK;
}

bool prof_on(int kernel) { return g_prof_on && ((g_prof_mask >> (kernel & 63)) & 1ull); }
void prof_push(const ProfRec &r) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  g_prof.push_back(r);
}
void prof_events(hipEvent_t *a, hipEvent_t *b) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  for (hipEvent_t *e : {a, b}) {
    if (!g_event_pool.empty()) {
      *e = g_event_pool.back();
      g_event_pool.pop_back();
    } else {
      (void)hipEventCreate(e);
    }
  }
}
}  // namespace pasur

namespace {

int check_tree_values(const pasur_fgt *f, const double *d_leaf, int dtype, void *const sigma[9],
                      int mode, double *d_out) {
  if (!f || !d_leaf || !d_out) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (mode < 0 || mode > 3 || (dtype != PASUR_F32 && dtype != PASUR_F64)) {
    set_error("unknown mode or dtype");
    return PASUR_E_RANGE;
  }
  if (mode != PASUR_TV_MINIMAX) {
    if (!sigma) {
      set_error("sigma is NULL");
      return PASUR_E_INVAL;
    }
    for (int l = 1; l <= 8; ++l)
      if (!sigma[l]) {
        set_error("sigma[%d] is NULL", l);
        return PASUR_E_INVAL;
      }
  }
  return PASUR_OK;
}

}  // namespace

extern "C" int pasur_cfr_init(const pasur_fgt *f, const pasur_cfr_state *st, void *stream) {
  PASUR_TRY(check_state(f, st));
  hipStream_t s = (hipStream_t)stream;
  return st->dtype == PASUR_F32 ? init_t<float>(f, st, s) : init_t<double>(f, st, s);
}

extern "C" int pasur_cfr_iterate(const pasur_fgt *f, const pasur_cfr_state *st,
                                 const pasur_cfr_params *p, int64_t t0, int n_iters,
                                 void *stream) {
  PASUR_TRY(check_state(f, st));
  if (!p) {
    set_error("params is NULL");
    return PASUR_E_INVAL;
  }
  if (t0 < 1 || n_iters < 0) {
    set_error("need t0 >= 1 and n_iters >= 0");
    return PASUR_E_RANGE;
  }
  if (p->variant < 0 || p->variant > 2 || p->rm_mode < 0 || p->rm_mode > 1) {
    set_error("unknown variant or regret-matching mode");
    return PASUR_E_RANGE;
  }
  if (p->schedule < 0 || p->schedule > PASUR_SCHED_AUTO ||
      (p->block != 0 && p->block != 256 && p->block != 512 && p->block != 1024)) {
    set_error("unknown schedule or block size");
    return PASUR_E_RANGE;
  }
  if (p->flags & ~(PASUR_CFR_SNIPPET_TOL | PASUR_CFR_SNIPPET_AVG)) {
    set_error("unknown CFR flags %d", p->flags);
    return PASUR_E_RANGE;
  }
  hipStream_t s = (hipStream_t)stream;
  if (p->flags) {
    if (p->variant != PASUR_DCFR) {
      set_error("the snippet flags apply to DCFR only");
      return PASUR_E_RANGE;
    }
    if (p->schedule != PASUR_SCHED_LEVEL_SYNC && p->schedule != PASUR_SCHED_AUTO) {
      set_error("the snippet flags run on PASUR_SCHED_LEVEL_SYNC (or AUTO) only");
      return PASUR_E_RANGE;
    }
    return st->dtype == PASUR_F32 ? iterate_t<float>(f, st, p, t0, n_iters, s)
                                  : iterate_t<double>(f, st, p, t0, n_iters, s);
  }
  if (p->schedule == PASUR_SCHED_STREAM || (p->schedule == PASUR_SCHED_AUTO && large_round(f))) {
    pasur_fgt *const tree = const_cast<pasur_fgt *>(f);
    if (p->schedule == PASUR_SCHED_AUTO && n_iters > 0) {
      hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
      bool capturing = true;
      if (hipStreamIsCapturing(s, &status) == hipSuccess)
        capturing = status != hipStreamCaptureStatusNone;
      else
        (void)hipGetLastError();  // another capture forbids to ask
      // a capture takes the schedule whose index an earlier call has built
      bool segs = !sweep_pays(f, st->dtype, n_iters), done = false;
      if (capturing) segs = seg_ready(f, st->dtype) && (segs || !f->sweep);
      if (segs) PASUR_TRY(seg_enqueue(tree, st, p, t0, n_iters, capturing, &done, s));
      if (done) return PASUR_OK;
    }
    return sweep_iterate(tree, st, p, t0, n_iters, s);
  }
  if (p->schedule == PASUR_SCHED_LEVEL_SYNC)
    return st->dtype == PASUR_F32 ? iterate_t<float>(f, st, p, t0, n_iters, s)
                                  : iterate_t<double>(f, st, p, t0, n_iters, s);
  if (n_iters == 0) return PASUR_OK;
  return seg_iterate(f, st, p, t0, n_iters, s);
}

extern "C" int pasur_average_strategy(const pasur_fgt *f, const pasur_cfr_state *st,
                                      void *const sigma_bar[9], void *stream) {
  PASUR_TRY(check_state(f, st));
  if (!sigma_bar) {
    set_error("sigma_bar is NULL");
    return PASUR_E_INVAL;
  }
  hipStream_t s = (hipStream_t)stream;
  for (int l = 1; l <= 8; ++l) {
    if (!sigma_bar[l]) {
      set_error("sigma_bar[%d] is NULL", l);
      return PASUR_E_INVAL;
    }
  }
  const AllParents P = all_parents(f);
  if (st->dtype == PASUR_F32)
    k_normalise<float><<<P.block[8], kParentThreads, 0, s>>>(
        P, edge_arrays<float>(st->Sbar, sigma_bar, nullptr), AsIs());
  else
    k_normalise<double><<<P.block[8], kParentThreads, 0, s>>>(
        P, edge_arrays<double>(st->Sbar, sigma_bar, nullptr), AsIs());
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

extern "C" int pasur_batch_begin(const pasur_fgt *const *fgts,
                                 const pasur_cfr_state *const *states,
                                 const double *const *d_V_next, int n_items, void *stream) {
  PASUR_TRY(check_items(fgts, states, n_items));
  for (int i = 0; i < n_items; ++i)
    if (fgts[i]->round < 5 && (!d_V_next || !d_V_next[i])) {
      set_error("rounds 0..4 need the next round's root values (item %d)", i);
      return PASUR_E_INVAL;
    }
  hipStream_t s = (hipStream_t)stream;
  return states[0]->dtype == PASUR_F32 ? begin_t<float>(fgts, states, d_V_next, n_items, s)
                                       : begin_t<double>(fgts, states, d_V_next, n_items, s);
}

extern "C" int pasur_batch_end(const pasur_fgt *const *fgts, const pasur_cfr_state *const *states,
                               void *const *sigma_bar, int64_t T, double *const *d_V, int n_items,
                               void *stream) {
  PASUR_TRY(check_items(fgts, states, n_items));
  if (!sigma_bar || !d_V) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (T < 1) {
    set_error("T must be >= 1");
    return PASUR_E_RANGE;
  }
  for (int i = 0; i < n_items; ++i) {
    if (!d_V[i]) {
      set_error("d_V of item %d is NULL", i);
      return PASUR_E_INVAL;
    }
    for (int l = 1; l <= 8; ++l)
      if (!sigma_bar[9 * i + l]) {
        set_error("sigma_bar[%d] of item %d is NULL", l, i);
        return PASUR_E_INVAL;
      }
  }
  hipStream_t s = (hipStream_t)stream;
  return states[0]->dtype == PASUR_F32
             ? end_t<float>(fgts, states, sigma_bar, (double)T, d_V, n_items, s)
             : end_t<double>(fgts, states, sigma_bar, (double)T, d_V, n_items, s);
}

extern "C" int pasur_leaf_utilities(const pasur_fgt *f, const double *d_V_next, int dtype,
                                    int flags, void *d_leaf, void *stream) {
  if (!f || !d_leaf) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (dtype != PASUR_F32 && dtype != PASUR_F64) {
    set_error("unknown dtype %d", dtype);
    return PASUR_E_RANGE;
  }
  if (flags & ~PASUR_LEAF_LITERAL_BONUS0) {
    set_error("unknown leaf-utility flags %d", flags);
    return PASUR_E_RANGE;
  }
  if (f->round < 5 && !d_V_next) {
    set_error("rounds 0..4 need the next round's root values");
    return PASUR_E_INVAL;
  }
  const double *V = f->round < 5 ? d_V_next : nullptr;
  const int8_t *b0 = f->round == 5 && (flags & PASUR_LEAF_LITERAL_BONUS0) ? f->leaf_bonus : nullptr;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == PASUR_F32)
    k_leaf_util<float><<<grid_for(f->n[8]), kThreads, 0, s>>>(f->n[8], f->leaf_base, f->link, V,
                                                              b0, (float *)d_leaf);
  else
    k_leaf_util<double><<<grid_for(f->n[8]), kThreads, 0, s>>>(f->n[8], f->leaf_base, f->link, V,
                                                               b0, (double *)d_leaf);
  PASUR_TRY_HIP(hipGetLastError());
  return PASUR_OK;
}

extern "C" int pasur_round_values(const pasur_fgt *f, const pasur_cfr_state *st, int value_mode,
                                  int64_t T, void *const sigma_bar[9], double *d_V, void *stream) {
  PASUR_TRY(check_state(f, st));
  if (!d_V) {
    set_error("d_V is NULL");
    return PASUR_E_INVAL;
  }
  hipStream_t s = (hipStream_t)stream;
  if (value_mode == PASUR_V_ITERATE_MEAN) {
    if (T < 1) {
      set_error("T must be >= 1");
      return PASUR_E_RANGE;
    }
    k_div<<<grid_for(f->n[0]), kThreads, 0, s>>>(f->n[0], st->vacc, (double)T, d_V);
    PASUR_TRY_HIP(hipGetLastError());
    return PASUR_OK;
  }
  if (value_mode != PASUR_V_SIGMA_BAR) {
    set_error("unknown value mode %d", value_mode);
    return PASUR_E_RANGE;
  }
  if (!sigma_bar) {
    set_error("sigma_bar is NULL");
    return PASUR_E_INVAL;
  }
  return tree_values(f, st->u[8], st->dtype, st->dtype, sigma_bar, PASUR_TV_EXPECT, d_V, true, s);
}

extern "C" int pasur_tree_values(const pasur_fgt *f, const double *d_leaf, int dtype,
                                 void *const sigma[9], int mode, double *d_out, void *stream) {
  PASUR_TRY(check_tree_values(f, d_leaf, dtype, sigma, mode, d_out));
  return tree_values(f, d_leaf, PASUR_F64, dtype, sigma, mode, d_out, true, (hipStream_t)stream);
}

namespace {

int check_exploitability(const pasur_fgt *const *fgts, int n_rounds, void *const *sigma_bar,
                         int dtype, int leaf_flags, const double *d_br_a, const double *d_br_b,
                         const double *d_v) {
  if (!fgts || !sigma_bar) {
    set_error("null argument");
    return PASUR_E_INVAL;
  }
  if (!d_br_a && !d_br_b && !d_v) {
    set_error("no output requested");
    return PASUR_E_INVAL;
  }
  if (n_rounds < 1 || n_rounds > 6) {
    set_error("n_rounds %d outside 1..6", n_rounds);
    return PASUR_E_RANGE;
  }
  if (dtype != PASUR_F32 && dtype != PASUR_F64) {
    set_error("unknown dtype %d", dtype);
    return PASUR_E_RANGE;
  }
  if (leaf_flags & ~PASUR_LEAF_LITERAL_BONUS0) {
    set_error("unknown leaf-utility flags %d", leaf_flags);
    return PASUR_E_RANGE;
  }
  for (int r = 0; r < n_rounds; ++r) {
    const pasur_fgt *f = fgts[r];
    if (!f) {
      set_error("fgts[%d] is NULL", r);
      return PASUR_E_INVAL;
    }
    if (f->n[0] < 1) {
      set_error("fgts[%d] has no roots", r);
      return PASUR_E_INVAL;
    }
    if (r > 0 && (f->round != fgts[r - 1]->round + 1 || f->n[0] != fgts[r - 1]->n_next)) {
      set_error("fgts[%d] is not the unfolding of fgts[%d]'s next-round roots", r, r - 1);
      return PASUR_E_INVAL;
    }
    for (int l = 1; l <= 8; ++l)
      if (!sigma_bar[r * 9 + l]) {
        set_error("sigma_bar[%d*9+%d] is NULL", r, l);
        return PASUR_E_INVAL;
      }
  }
  if (fgts[n_rounds - 1]->round != 5) {
    set_error("the last tree must be round 5 (the hand's last round)");
    return PASUR_E_INVAL;
  }
  return PASUR_OK;
}

}  // namespace

extern "C" int pasur_exploitability(const pasur_fgt *const *fgts, int n_rounds,
                                    void *const *sigma_bar, int dtype, int leaf_flags,
                                    double *d_br_a, double *d_br_b, double *d_v, void *stream) {
  PASUR_TRY(check_exploitability(fgts, n_rounds, sigma_bar, dtype, leaf_flags, d_br_a, d_br_b,
                                 d_v));
  return composed_values(fgts, n_rounds, sigma_bar, dtype, leaf_flags, d_br_a, d_br_b, d_v,
                         (hipStream_t)stream);
}

extern "C" int pasur_tree_values_noalloc(const pasur_fgt *f, const double *d_leaf, int dtype,
                                         void *const sigma[9], int mode, double *d_out,
                                         void *stream) {
  PASUR_TRY(check_tree_values(f, d_leaf, dtype, sigma, mode, d_out));
  const int64_t mx = widest_level(f->n);
  if (mx > kNoAllocLevel) {
    set_error("a tree level of %lld nodes exceeds the %lld nodes that "
              "pasur_tree_values_noalloc takes (use pasur_tree_values)",
              (long long)mx, (long long)kNoAllocLevel);
    return PASUR_E_CAPACITY;
  }
  return tree_values(f, d_leaf, PASUR_F64, dtype, sigma, mode, d_out, false, (hipStream_t)stream);
}

extern "C" int pasur_profile_enable(int on) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  prof_clear();
  g_prof_on = on != 0;
  g_prof_mask = ~0ull;
  return PASUR_OK;
}

extern "C" int pasur_profile_select(uint64_t kernel_mask) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  g_prof_mask = kernel_mask;
  return PASUR_OK;
}

extern "C" int pasur_profile_read(int64_t cap, int32_t *kernel, int32_t *level, float *ms,
                                  int64_t *work, int64_t *n_out) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  if (!n_out) {
    set_error("n_out is NULL");
    return PASUR_E_INVAL;
  }
  *n_out = (int64_t)g_prof.size();
  const int64_t n = cap < *n_out ? cap : *n_out;
  for (int64_t i = 0; i < n; ++i) {
    PASUR_TRY_HIP(hipEventSynchronize(g_prof[i].b));
    float t = 0.f;
    PASUR_TRY_HIP(hipEventElapsedTime(&t, g_prof[i].a, g_prof[i].b));
    if (kernel) kernel[i] = g_prof[i].kernel;
    if (level) level[i] = g_prof[i].level;
    if (ms) ms[i] = t;
    if (work)
      for (int k = 0; k < 5; ++k) work[5 * i + k] = g_prof[i].work[k];
  }
  return PASUR_OK;
}
