// pasur_play.hip -- self-play with average strategies: the paper's way of
// estimating a deal's fair value (section "Experimental Evaluation").  A
// thread walks the unfolded trees of a solved subgame from a root, for one game
// or several: at each decision the player to move samples one child (inverse CDF
// of the average strategy, or uniformly at random); at a round's last level the
// game adds the leaf's round points and continues at the linked next-round
// root.  Random numbers come from a counter-based SplitMix64 stream, so any
// game can be replayed on its own.
#include "pasur_internal.hpp"

#include <algorithm>
#include <cstring>
#include <type_traits>

using namespace pasur;

namespace {

constexpr int kMaxRounds = 6;

struct PlayRound {
  const int32_t *cb[8];
  const void *sbar[9];
  const int32_t *link;
  const int16_t *base;
  int32_t n[9];  // nodes per level
};

struct PlayArgs {
  PlayRound r[kMaxRounds];
  int n_rounds, dtype, policy[2], root;
  uint64_t seed;
  int64_t first, n_games;  // games first .. n_games - 1
};

// The strategy at a node's first four children, in one load where the level does
// not end before.
template <class T>
struct First {
  T p[4];
  __device__ __forceinline__ void load(const T *sb, int32_t b, int k, int32_t n) {
    if (b + 4 <= n) {
      __builtin_memcpy(p, sb + b, sizeof(p));
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) p[c] = c < k ? sb[b + c] : (T)0;
    }
  }
};

// choose_by with the first four probabilities in registers, the others at rest[c].
template <class T>
__device__ __forceinline__ int choose_first(double u, const First<T> &f, const T *rest, int k) {
  const int uni = min((int)(u * (double)k), k - 1);
  double total = 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c < k) total += (double)f.p[c];
  for (int c = 4; c < k; ++c) total += (double)rest[c];
  if (!(total > 0.0)) return uni;
  const double x = u * total;
  double acc = 0.0;
  int last = 0, pick = -1;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c < k && pick < 0) {
      const double pc = (double)f.p[c];
      acc += pc;
      if (pc > 0.0) last = c;
      if (acc > x) pick = c;
    }
  for (int c = 4; c < k && pick < 0; ++c) {
    const double pc = (double)rest[c];
    acc += pc;
    if (pc > 0.0) last = c;
    if (acc > x) pick = c;
  }
  return pick < 0 ? last : pick;
}

// G games per thread, g, g + stride, ... (stride = threads in the grid), stepped
// together so that their dependent gathers overlap; T = void where both players
// are uniform.  A thread's games past the last one are played (indices stay
// valid) and their margins dropped.  Bound by the chain of two dependent gathers
// per decision: 2^20 games of a game of 3.4e7 nodes with one average strategy, 286
// us with eight games per thread and a load per child and per end of the range,
// 195 with four and the wide loads; 2700 games of three rounds 110 us, 18 with one.
template <class T, int G>
__global__ void k_selfplay(PlayArgs a, int32_t *__restrict__ margin) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g0 >= a.n_games - a.first) return;
  int64_t g[G];
  int32_t q[G], m[G];
#pragma unroll
  for (int i = 0; i < G; ++i) {
    g[i] = a.first + g0 + i * stride;
    q[i] = a.root;
    m[i] = 0;
  }
  for (int r = 0; r < a.n_rounds; ++r) {
    const PlayRound &R = a.r[r];
    for (int l = 0; l < 8; ++l) {
      int32_t b[G], e[G];
#pragma unroll
      for (int i = 0; i < G; ++i) {
        int32_t be[2];
        __builtin_memcpy(be, R.cb[l] + q[i], sizeof(be));
        b[i] = be[0];
        e[i] = be[1];
      }
      if constexpr (std::is_void<T>::value) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
          const int k = e[i] - b[i];
          q[i] = b[i];
          if (k > 1) {
            const double u =
                splitmix_uniform(a.seed, (uint64_t)g[i] * 64u + (uint64_t)(r * 8 + l));
            q[i] += min((int)(u * (double)k), k - 1);
          }
        }
      } else {
        const T *const sb = reinterpret_cast<const T *>(R.sbar[l + 1]);
        const bool uniform = a.policy[l & 1] == PASUR_PLAY_UNIFORM;
        First<T> f[G];
        if (!uniform) {
#pragma unroll
          for (int i = 0; i < G; ++i)
            if (e[i] - b[i] > 1) f[i].load(sb, b[i], e[i] - b[i], R.n[l + 1]);
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
          const int k = e[i] - b[i];
          int c = 0;
          if (k > 1) {
            const double u =
                splitmix_uniform(a.seed, (uint64_t)g[i] * 64u + (uint64_t)(r * 8 + l));
            c = uniform ? min((int)(u * (double)k), k - 1) : choose_first(u, f[i], sb + b[i], k);
          }
          q[i] = b[i] + c;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
      m[i] += R.base[q[i]];
      if (r + 1 < a.n_rounds) q[i] = R.link[q[i]];
    }
  }
#pragma unroll
  for (int i = 0; i < G; ++i)
    if (g[i] < a.n_games) margin[g[i]] = m[i];
}

// A launch's threads stay below 2^32.
template <class T, int G>
int play(PlayArgs a, int32_t *d_margin, hipStream_t s) {
  constexpr int64_t kGames = (int64_t)1 << 31;
  const int64_t n_games = a.n_games;
  for (a.first = 0; a.first < n_games; a.first += kGames) {
    a.n_games = std::min(n_games, a.first + kGames);
    const int64_t threads = (a.n_games - a.first + G - 1) / G;
    k_selfplay<T, G><<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(a, d_margin);
    PASUR_TRY_HIP(hipGetLastError());
  }
  return PASUR_OK;
}

}  // namespace

extern "C" int pasur_selfplay(const pasur_fgt *const *fgts, int n_rounds,
                              const void *const *sigma_bar, int dtype, int root,
                              int64_t n_games, uint64_t seed, int policy_a, int policy_b,
                              int32_t *d_margin, void *stream) {
  if (!fgts || !sigma_bar || !d_margin || n_games < 0) {
    set_error("null argument or negative game count");
    return PASUR_E_INVAL;
  }
  if (n_games > (int64_t)INT32_MAX * 256) {
    set_error("n_games %lld beyond one launch (%lld)", (long long)n_games,
              (long long)INT32_MAX * 256);
    return PASUR_E_RANGE;
  }
  if (n_rounds < 1 || n_rounds > kMaxRounds) {
    set_error("n_rounds %d outside 1..%d", n_rounds, kMaxRounds);
    return PASUR_E_RANGE;
  }
  if (dtype != PASUR_F32 && dtype != PASUR_F64) {
    set_error("unknown dtype %d", dtype);
    return PASUR_E_RANGE;
  }
  for (int p : {policy_a, policy_b}) {
    if (p != PASUR_PLAY_SIGMA_BAR && p != PASUR_PLAY_UNIFORM) {
      set_error("unknown policy %d", p);
      return PASUR_E_RANGE;
    }
  }
  PlayArgs a;
  std::memset(&a, 0, sizeof(a));
  for (int r = 0; r < n_rounds; ++r) {
    const pasur_fgt *f = fgts[r];
    if (!f) {
      set_error("fgts[%d] is NULL", r);
      return PASUR_E_INVAL;
    }
    if (r > 0 && f->round != fgts[r - 1]->round + 1) {
      set_error("rounds must be consecutive");
      return PASUR_E_INVAL;
    }
    if (r + 1 < n_rounds && f->round == 5) {
      set_error("round 5 is the last round");
      return PASUR_E_INVAL;
    }
    for (int l = 0; l < 8; ++l) a.r[r].cb[l] = f->child_begin[l];
    for (int l = 1; l <= 8; ++l) {
      a.r[r].sbar[l] = sigma_bar[r * 9 + l];
      if (!a.r[r].sbar[l]) {
        set_error("sigma_bar[%d][%d] is NULL", r, l);
        return PASUR_E_INVAL;
      }
    }
    if ((r + 1 < n_rounds && !f->link) || !f->leaf_base) {
      set_error("tree of round %d has no %s", f->round, f->leaf_base ? "link table" : "leaf scores");
      return PASUR_E_INVAL;
    }
    a.r[r].link = f->link;
    a.r[r].base = f->leaf_base;
    for (int l = 0; l <= 8; ++l) a.r[r].n[l] = (int32_t)f->n[l];
  }
  if (root < 0 || root >= fgts[0]->n[0]) {
    set_error("root %d outside 0..%lld", root, (long long)fgts[0]->n[0] - 1);
    return PASUR_E_RANGE;
  }
  if (n_games == 0) return PASUR_OK;
  a.n_rounds = n_rounds;
  a.dtype = dtype;
  a.policy[0] = policy_a;
  a.policy[1] = policy_b;
  a.root = root;
  a.seed = seed;
  a.n_games = n_games;
  hipStream_t s = (hipStream_t)stream;
  // One game per thread while that leaves no game waiting for another's steps: up
  // to 2^19 games all threads run at once (eight waves per SIMD).  Beyond that more
  // games per thread keep more loads in flight.  2^18, 2^20, 2^24 games of a game of
  // 3.4e7 nodes, one side by its average strategy: 1 game per thread 62, 221, 3450
  // us, 4 games 91, 204, 3160, 8 games 161, 229, 2920 (with FP64 averages 294, 444,
  // 6810: spills).  Uniform players' games spread over the whole tree and need no
  // strategies: 1 game per thread 62, 301, 5900 us, 4 games 71, 260, 5290, 8 games
  // 99, 204, 4910.
  if (policy_a == PASUR_PLAY_UNIFORM && policy_b == PASUR_PLAY_UNIFORM)
    return n_games <= (1 << 18) ? play<void, 1>(a, d_margin, s) : play<void, 8>(a, d_margin, s);
  const bool one = n_games <= (1 << 19);
  if (dtype == PASUR_F32)
    return one ? play<float, 1>(a, d_margin, s) : play<float, 4>(a, d_margin, s);
  return one ? play<double, 1>(a, d_margin, s) : play<double, 4>(a, d_margin, s);
}
