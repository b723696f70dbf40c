// pasur_scan.hpp -- device-wide exclusive scans (counts -> CSR offsets) of values
// that a functor computes from an index, and the host's window on device totals.
// Shared by the HIP translation units that lay out trees; not part of the ABI.
#pragma once

#include "pasur_internal.hpp"

namespace pasur {

// A few words of pinned host memory that kernels on `stream` write and the host
// reads after it has waited for them: a total costs no copy and no allocation.
// Taken from a list shared by all threads and devices, which grows by the number
// of calls in flight at once.
constexpr int kHostWords = 31;
class HostWords {
 public:
  explicit HostWords(hipStream_t stream);
  ~HostWords();  // waits if words handed out since the last wait may be written
  HostWords(const HostWords &) = delete;
  HostWords &operator=(const HostWords &) = delete;
  bool ok() const { return w != nullptr; }
  int64_t *dev(int k) {
    pending = true;
    return w + k;
  }
  int64_t operator[](int k) const { return w[k]; }
  int wait();
  // Nothing that writes them is pending: the last wait has succeeded.
  bool idle() const { return !pending; }

 private:
  int64_t *w;  // kHostWords words, zero at first, then a link of the free list
  hipStream_t stream;
  bool pending;
};

constexpr int kScanBlock = 256;
constexpr int kScanWave = 1024;               // consecutive values per wave
constexpr int kScanTile = 4 * kScanWave;      // per workgroup
constexpr int kScanRounds = kScanWave / 64;

template <class Acc>
__device__ __forceinline__ Acc wave_inclusive(Acc v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const Acc x = __shfl_up(v, d, 64);
    if (lane >= d) v += x;
  }
  return v;
}
// 32-bit sums move by DPP, within rows of 16 lanes and then from row to row: 8
// cycles a step instead of an LDS round trip (a small scan 7 -> 3 us).
template <>
__device__ __forceinline__ int wave_inclusive<int>(int v, int) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}
template <class Acc>
__device__ __forceinline__ Acc wave_last(Acc v) {
  return __shfl(v, 63, 64);
}
template <>
__device__ __forceinline__ int wave_last<int>(int v) {
  return __builtin_amdgcn_readlane(v, 63);
}

// Sums of the tiles of n values in(batch, i); batch = blockIdx.y.
template <class In>
__global__ void __launch_bounds__(kScanBlock) k_scan_sums(In in, int64_t n, int64_t nt,
                                                          int64_t *__restrict__ sums) {
  __shared__ int64_t part[kScanBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + w * kScanWave + lane;
  typename In::Acc s = 0;
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    const int64_t i = base + 64 * r;
    if (i < n) s += in(blockIdx.y, i);
  }
  s = wave_inclusive(s, lane);
  if (lane == 63) part[w] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int k = 0; k < kScanBlock / 64; ++k) t += part[k];
    sums[blockIdx.y * nt + blockIdx.x] = t;
  }
}

// sums -> exclusive offsets in place, one workgroup per batch; total[batch].
static __global__ void __launch_bounds__(1024) k_scan_tiles(int64_t nt, int64_t *__restrict__ sums,
                                                            int64_t *__restrict__ total) {
  __shared__ int64_t part[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t *const s = sums + blockIdx.x * nt;
  int64_t carry = 0;
  for (int64_t i0 = 0; i0 < nt; i0 += 1024) {
    const int64_t i = i0 + threadIdx.x;
    const int64_t v = i < nt ? s[i] : 0;
    const int64_t x = wave_inclusive(v, lane);
    if (lane == 63) part[w] = x;
    __syncthreads();
    int64_t before = carry, all = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < w) before += part[k];
      all += part[k];
    }
    if (i < nt) s[i] = before + x - v;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// out(batch, i, sum of in(batch, 0..i-1)) for i = 0..n; offs: the tiles'
// offsets, or NULL for a single tile, which also writes total[batch].
template <class In, class Out>
__global__ void __launch_bounds__(kScanBlock)
    k_scan_apply(In in, Out out, int64_t n, int64_t nt, const int64_t *__restrict__ offs,
                 int64_t *__restrict__ total) {
  __shared__ int64_t part[kScanBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + w * kScanWave + lane;
  typename In::Acc pre[kScanRounds], carry = 0;
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    const int64_t i = base + 64 * r;
    const typename In::Acc v = i < n ? in(blockIdx.y, i) : 0;
    const typename In::Acc x = wave_inclusive(v, lane);
    pre[r] = carry + x - v;
    carry += wave_last(x);
  }
  if (lane == 0) part[w] = carry;
  __syncthreads();
  int64_t off = offs ? offs[blockIdx.y * nt + blockIdx.x] : 0;
  for (int k = 0; k < w; ++k) off += part[k];
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    const int64_t i = base + 64 * r;
    if (i <= n) out((int)blockIdx.y, i, off + pre[r]);
  }
  if (!offs && threadIdx.x == 0)
    total[blockIdx.y] = part[0] + part[1] + part[2] + part[3];
}

// Words of scratch a scan of n values in `batches` batches needs.
inline int64_t scan_scratch(int64_t n, int batches = 1) {
  return (n / kScanTile + 1) * batches;
}

// Enqueues a scan; total: device-visible, one word per batch.  Nothing waits.
template <class In, class Out>
void scan_enqueue(const In &in, const Out &out, int64_t n, int batches, int64_t *scratch,
                  int64_t *total, hipStream_t s) {
  // index n (the total) belongs to a tile as well
  const int64_t nt = n / kScanTile + 1;
  const dim3 grid((unsigned)nt, (unsigned)batches);
  if (nt == 1) {
    k_scan_apply<In, Out><<<grid, kScanBlock, 0, s>>>(in, out, n, nt, nullptr, total);
    return;
  }
  k_scan_sums<In><<<grid, kScanBlock, 0, s>>>(in, n, nt, scratch);
  k_scan_tiles<<<(unsigned)batches, 1024, 0, s>>>(nt, scratch, total);
  k_scan_apply<In, Out><<<grid, kScanBlock, 0, s>>>(in, out, n, nt, scratch, total);
}

// Offsets into an int32 array (batch b at b * stride).
struct OffsetsOut {
  int32_t *p;
  int64_t stride;
  __device__ __forceinline__ void operator()(int b, int64_t i, int64_t v) const {
    p[b * stride + i] = (int32_t)v;
  }
};
// Acc: the type in which a tile's sum is formed (totals are 64 bits wide).
// Counts of a node's children, or of a sort tile's keys: a tile's fit 32 bits.
struct CountsIn {
  using Acc = int;
  const int32_t *p;
  __device__ __forceinline__ int operator()(int, int64_t i) const { return p[i]; }
};

inline int total_fits(int64_t total) {
  if (total <= INT32_MAX) return PASUR_OK;
  set_error("tree level of %lld nodes exceeds INT32_MAX", (long long)total);
  return PASUR_E_OVERFLOW;
}

// One block of device memory carved into arrays (256-byte aligned).  Goes back
// to the cache at the end of its scope, when nothing uses it any more: its owner
// waits for the stream before that, also on errors.
class Arena {
 public:
  ~Arena() { block_free(base); }
  template <class T>
  void want(T **p, int64_t n) {
    slots[count++] = Slot{(void **)p, bytes};
    bytes += ((size_t)(n > 0 ? n : 1) * sizeof(T) + 255) & ~(size_t)255;
  }
  int alloc() {
    PASUR_TRY(block_alloc(&base, bytes));
    for (int i = 0; i < count; ++i) *slots[i].p = (unsigned char *)base + slots[i].at;
    return PASUR_OK;
  }
  // The block's owner from here on is the caller.
  void *release() {
    void *b = base;
    base = nullptr;
    return b;
  }

 private:
  struct Slot {
    void **p;
    size_t at;
  };
  Slot slots[64];
  int count = 0;
  size_t bytes = 0;
  void *base = nullptr;
};

}  // namespace pasur
