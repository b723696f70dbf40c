// pasur_sort.hip -- stable LSD radix sort of (64-bit key, int32 value) pairs, used
// by the unfolding to group leaves by their next-round root (the canonical
// (compressed pool, score) key of section "Between-Hand Updates").
//
// Only the key bits that vary over the keys are sorted by (an AND/OR reduction
// finds them first), eight of them per pass wherever they lie in the key: the
// leaves of a round differ in 20 to 40 of their 60 bits, and an 8-bit window at
// fixed places took five to eight passes for what three to five do.  A pass is:
//   k_rs_hist     per 4096-key tile, a 256-bucket histogram in LDS, stored
//                 digit-major: hist[d * n_tiles + tile];
//   a scan        of that array: the first output slot of (digit d, tile) in
//                 the sorted order;
//   k_rs_scatter  per tile, the stable rank of every key within its digit
//                 (wavefront ballots over the digit's bits give the rank
//                 among equal digits of one wave; per-wave counts in LDS
//                 order the waves and the tile's 16 rounds), then the tile is
//                 reordered in LDS by digit so that each bucket's run leaves
//                 as consecutive addresses.
#include "pasur_sort.hpp"


namespace pasur {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kItems = 16;
constexpr int kTile = kBlock * kItems;
constexpr int kBuckets = 256;

// The eight key bits of a pass, lowest first (unused places repeat a bit that
// does not vary: its digit bit is the same for all keys).
struct Digit {
  uint8_t bit[8];
  template <class K>
  __device__ __forceinline__ int operator()(K k) const {
    int d = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) d |= (int)((k >> bit[b]) & 1) << b;
    return d;
  }
};

template <class K>
__global__ void __launch_bounds__(kBlock) k_rs_andor(const K *__restrict__ keys, int64_t n,
                                                     unsigned long long *__restrict__ acc) {
  K a = ~K(0), o = K(0);
  const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x;
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + (int64_t)r * kBlock;
    if (i < n) {
      const K k = keys[i];
      a &= k;
      o |= k;
    }
  }
  __shared__ unsigned long long sa[kBlock], so[kBlock];
  sa[threadIdx.x] = (unsigned long long)a;
  so[threadIdx.x] = (unsigned long long)o;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sa[threadIdx.x] &= sa[threadIdx.x + s];
      so[threadIdx.x] |= so[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicAnd(&acc[0], sa[0]);
    atomicOr(&acc[1], so[0]);
  }
}

__global__ void k_rs_andor_init(unsigned long long *acc) {
  if (threadIdx.x == 0) {
    acc[0] = ~0ull;
    acc[1] = 0ull;
  }
}

template <class K>
__global__ void __launch_bounds__(kBlock) k_rs_hist(const K *__restrict__ keys, int64_t n,
                                                    Digit dig, int64_t n_tiles,
                                                    int32_t *__restrict__ hist) {
  __shared__ int32_t h[kBuckets];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x;
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = base + (int64_t)r * kBlock;
    if (i < n) atomicAdd(&h[dig(keys[i])], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

template <class K>
__global__ void __launch_bounds__(kBlock) k_rs_scatter(const K *__restrict__ keys,
                                                       const int32_t *__restrict__ vals, int64_t n,
                                                       Digit dig, int64_t n_tiles,
                                                       const int32_t *__restrict__ off,
                                                       K *__restrict__ okeys,
                                                       int32_t *__restrict__ ovals) {
  __shared__ int32_t cnt[kBuckets];         // keys of each digit in earlier rounds
  __shared__ int32_t wc[kWaves][kBuckets];  // this round's count per wave and digit
  __shared__ int32_t loc[2][kBuckets];      // tile-local exclusive offsets (scan buffers)
  __shared__ int32_t gof[kBuckets];         // this tile's first output slot per digit
  __shared__ K sk[kTile];
  __shared__ int32_t sv[kTile];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  const int count = (int)(n - base < kTile ? n - base : kTile);
  cnt[t] = 0;
  gof[t] = off[(int64_t)t * n_tiles + blockIdx.x];
  K k[kItems];
  int32_t v[kItems];
  int rank[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int i = r * kBlock + t;
    k[r] = i < count ? keys[base + i] : K(0);
    v[r] = i < count ? vals[base + i] : 0;
  }
  const unsigned long long below_mask = (1ull << lane) - 1;
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
#pragma unroll
    for (int q = 0; q < kWaves; ++q) wc[q][t] = 0;
    __syncthreads();
    const bool ok = r * kBlock + t < count;
    const int d = dig(k[r]);
    unsigned long long m = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long bb = __ballot((d >> b) & 1);
      m &= ((d >> b) & 1) ? bb : ~bb;
    }
    const int below = __popcll(m & below_mask);
    if (ok && below == 0) wc[w][d] = __popcll(m);
    __syncthreads();
    int pre = cnt[d];
    for (int q = 0; q < w; ++q) pre += wc[q][d];
    rank[r] = pre + below;
    __syncthreads();
    cnt[t] += wc[0][t] + wc[1][t] + wc[2][t] + wc[3][t];
  }
  // tile-local exclusive offsets of the digits (Hillis-Steele over 256)
  int cur = 0;
  loc[0][t] = cnt[t];
  __syncthreads();
  for (int s = 1; s < kBuckets; s <<= 1) {
    int x = loc[cur][t];
    if (t >= s) x += loc[cur][t - s];
    loc[cur ^ 1][t] = x;
    cur ^= 1;
    __syncthreads();
  }
  const int excl = loc[cur][t] - cnt[t];
  __syncthreads();
  loc[cur ^ 1][t] = excl;
  __syncthreads();
  const int *lo = loc[cur ^ 1];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    if (r * kBlock + t < count) {
      const int d = dig(k[r]);
      const int p = lo[d] + rank[r];
      sk[p] = k[r];
      sv[p] = v[r];
    }
  }
  __syncthreads();
  for (int j = t; j < count; j += kBlock) {
    const K kk = sk[j];
    const int d = dig(kk);
    const int64_t g = (int64_t)gof[d] + (j - lo[d]);
    okeys[g] = kk;
    ovals[g] = sv[j];
  }
}

unsigned grid_tiles(int64_t n) { return (unsigned)((n + kTile - 1) / kTile); }

}  // namespace

int64_t sort_scratch_ints(int64_t n) { return 2 * ((int64_t)grid_tiles(n) * kBuckets + 1); }
int64_t sort_scratch_words(int64_t n) {
  return 2 + scan_scratch((int64_t)grid_tiles(n) * kBuckets) + 1;
}

int sort_pairs(uint64_t *const keys[2], int32_t *const vals[2], int64_t n, int32_t *ints,
               int64_t *words, int64_t *host, int *result, hipStream_t s) {
  *result = 0;
  if (n <= 0) return PASUR_OK;
  const int64_t n_tiles = grid_tiles(n), n_hist = n_tiles * kBuckets;
  unsigned long long *const acc = (unsigned long long *)words;
  k_rs_andor_init<<<1, 64, 0, s>>>(acc);
  k_rs_andor<uint64_t><<<grid_tiles(n), kBlock, 0, s>>>(keys[0], n, acc);
  PASUR_TRY_HIP(hipGetLastError());
  PASUR_TRY_HIP(hipMemcpyAsync(host, acc, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
  PASUR_TRY_HIP(hipStreamSynchronize(s));
  const uint64_t varying = (uint64_t)host[0] ^ (uint64_t)host[1];
  const int fixed = varying == ~0ull ? 0 : __builtin_ctzll(~varying);  // a bit that does not vary
  int32_t *const hist = ints, *const off = ints + n_hist + 1;
  int src = 0;
  for (uint64_t left = varying; left;) {
    Digit dig;
    for (int b = 0; b < 8; ++b) {
      dig.bit[b] = (uint8_t)(left ? __builtin_ctzll(left) : fixed);
      left &= left - 1;
    }
    k_rs_hist<uint64_t><<<grid_tiles(n), kBlock, 0, s>>>(keys[src], n, dig, n_tiles, hist);
    scan_enqueue(CountsIn{hist}, OffsetsOut{off, 0}, n_hist, 1, words + 3, words + 2, s);
    k_rs_scatter<uint64_t><<<grid_tiles(n), kBlock, 0, s>>>(
        keys[src], vals[src], n, dig, n_tiles, off, keys[src ^ 1], vals[src ^ 1]);
    PASUR_TRY_HIP(hipGetLastError());
    src ^= 1;
  }
  *result = src;
  return PASUR_OK;
}

}  // namespace pasur
