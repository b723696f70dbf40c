// pasur_util.hip -- error reporting, the cache of device memory blocks, the pinned
// words that kernels report totals in, and the scan of an array of counts.
#include "pasur_scan.hpp"

#include <cstdlib>
#include <cstring>
#include <mutex>

namespace pasur {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

namespace {
// Freed blocks, oldest first, at most kCacheBytes of them per device (6% of its
// memory: the trees of the largest whole game, 8.5e8 nodes, take 11 GB) in at most
// kCacheBlocks places.  The oldest make room for the newest and are given back to
// the system, as is what comes back when an eighth of the device or less is free,
// and everything when an allocation fails or the caller asks for it.  (With the
// oldest kept, a program that had gone on to a game of another size gave its
// memory back and asked for it anew at each build: 261 ms for 6.4e8 nodes,
// 9.2 ms now.)  Blocks are handed out again only to requests of a similar size.
constexpr size_t kCacheBytes = (size_t)16 << 30;
constexpr int kCacheBlocks = 512;
struct Block {
  void *p;
  size_t bytes;
  int device;
};
// Held for the lists alone: freeing waits for the device, and allocating may.
std::mutex g_block_mu;
Block g_free[kCacheBlocks];
int g_n_free = 0;
// Size and device of the blocks in use, by address.
struct Owned {
  Block b;
  Owned *next;
};
constexpr int kBuckets = 1024;
Owned *g_owned[kBuckets];

Owned **owned_place(void *p) {
  return &g_owned[((uintptr_t)p >> 12) % kBuckets];
}

size_t rounded(size_t bytes) {
  if (bytes <= 4096) return 4096;
  if (bytes <= ((size_t)1 << 20)) {
    size_t r = 4096;
    while (r < bytes) r <<= 1;
    return r;
  }
  const size_t two = (size_t)2 << 20;
  return (bytes + two - 1) / two * two;
}

void remove_cached(int i) {
  for (--g_n_free; i < g_n_free; ++i) g_free[i] = g_free[i + 1];
}

// The smallest cached block of this device that holds `bytes` and is at most a
// quarter larger.
bool take_cached(size_t bytes, int device, Block *out) {
  int best = -1;
  for (int i = 0; i < g_n_free; ++i)
    if (g_free[i].device == device && g_free[i].bytes >= bytes &&
        g_free[i].bytes <= bytes + bytes / 4 &&
        (best < 0 || g_free[i].bytes < g_free[best].bytes))
      best = i;
  if (best < 0) return false;
  *out = g_free[best];
  remove_cached(best);
  return true;
}

// Blocks on their way back to the system: taken off the list under the lock,
// freed at the end, when it is no longer held.
struct Outgoing {
  void *p[kCacheBlocks];
  int n = 0;
  void take(int i) {
    p[n++] = g_free[i].p;
    remove_cached(i);
  }
  ~Outgoing() {
    for (int i = 0; i < n; ++i) (void)hipFree(p[i]);
  }
};

void release_cached(int device) {
  Outgoing out;
  std::lock_guard<std::mutex> lock(g_block_mu);
  for (int i = g_n_free; i-- > 0;)
    if (g_free[i].device == device) out.take(i);
}

// Takes off the device's oldest blocks until one of `bytes` has room; false if it
// cannot have any.
bool make_room(size_t bytes, int device, Outgoing &out) {
  if (bytes > kCacheBytes) return false;
  size_t cached = 0;
  for (int i = 0; i < g_n_free; ++i)
    if (g_free[i].device == device) cached += g_free[i].bytes;
  for (int i = 0; i < g_n_free && (g_n_free == kCacheBlocks || cached + bytes > kCacheBytes);) {
    if (g_free[i].device != device) {
      ++i;
      continue;
    }
    cached -= g_free[i].bytes;
    out.take(i);
  }
  return g_n_free < kCacheBlocks && cached + bytes <= kCacheBytes;
}

// More than an eighth of that device's memory is free.
bool room_on(int device) {
  int current = 0;
  if (hipGetDevice(&current) != hipSuccess) return false;
  if (current != device && hipSetDevice(device) != hipSuccess) return false;
  size_t free_bytes = 0, total = 0;
  const bool room = hipMemGetInfo(&free_bytes, &total) == hipSuccess && free_bytes > total / 8;
  if (current != device) (void)hipSetDevice(current);
  return room;
}

// An idle block goes to the cache or to the system.
void give_back(const Block &b) {
  bool keep = b.bytes < ((size_t)64 << 20) || room_on(b.device);
  if (keep) {
    Outgoing out;
    std::lock_guard<std::mutex> lock(g_block_mu);
    keep = make_room(b.bytes, b.device, out);
    if (keep) g_free[g_n_free++] = b;
  }
  if (!keep) (void)hipFree(b.p);
}

// Blocks whose handles are gone but whose idleness is not known.
struct Retired {
  void *anchor, *blocks[kRetired];
  int n;
  Retired *next;
};
Retired *g_retired = nullptr;

bool anchor_wait(void *a) {
  if (!a || hipFree(a) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// Blocks that go back when the work enqueued before an event has ended.
struct Pending {
  Block b;
  hipStream_t stream;
  hipEvent_t ended;
  Pending *next;
};
Pending *g_pending = nullptr;

// Gives pending blocks back whose work has ended, or all of them (wait).
void pending_again(bool wait) {
  Pending *list;
  {
    std::lock_guard<std::mutex> lock(g_block_mu);
    list = g_pending;
    g_pending = nullptr;
  }
  while (list) {
    Pending *const p = list;
    list = p->next;
    if ((wait ? hipEventSynchronize(p->ended) : hipEventQuery(p->ended)) == hipSuccess) {
      (void)hipEventDestroy(p->ended);
      give_back(p->b);
      std::free(p);
      continue;
    }
    (void)hipGetLastError();
    std::lock_guard<std::mutex> lock(g_block_mu);
    p->next = g_pending;
    g_pending = p;
  }
}

// A pending block of this stream that holds `bytes` and is at most a quarter
// larger: what follows on the stream may have it at once.
bool take_pending(size_t bytes, int device, hipStream_t s, Block *out) {
  Pending *p;
  {
    std::lock_guard<std::mutex> lock(g_block_mu);
    Pending **at = &g_pending;
    while (*at && !((*at)->stream == s && (*at)->b.device == device && (*at)->b.bytes >= bytes &&
                    (*at)->b.bytes <= bytes + bytes / 4))
      at = &(*at)->next;
    p = *at;
    if (!p) return false;
    *at = p->next;
  }
  // (of this stream, or of an earlier one of the same name)
  const bool ok = hipStreamWaitEvent(s, p->ended, 0) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    std::lock_guard<std::mutex> lock(g_block_mu);
    p->next = g_pending;
    g_pending = p;
    return false;
  }
  *out = p->b;
  (void)hipEventDestroy(p->ended);
  std::free(p);
  return true;
}

// Waits once more for the device on behalf of blocks that were set aside.
void retire_again() {
  Retired *r;
  {
    std::lock_guard<std::mutex> lock(g_block_mu);
    r = g_retired;
    g_retired = nullptr;
  }
  while (r) {
    Retired *const next = r->next;
    blocks_retire(r->anchor, r->blocks, r->n);
    std::free(r);
    r = next;
  }
}
}  // namespace

namespace {
int alloc(void **p, size_t bytes, bool on_stream, hipStream_t s) {
  *p = nullptr;
  int device = 0;
  PASUR_TRY_HIP(hipGetDevice(&device));
  retire_again();
  Owned *o = (Owned *)std::malloc(sizeof(Owned));
  if (!o) {
    set_error("host allocation failed");
    return PASUR_E_NOMEM;
  }
  const size_t want = rounded(bytes);
  bool cached;
  {
    std::lock_guard<std::mutex> lock(g_block_mu);
    cached = take_cached(want, device, &o->b);
  }
  if (!cached && on_stream) cached = take_pending(want, device, s, &o->b);
  if (!cached) {
    pending_again(false);
    std::lock_guard<std::mutex> lock(g_block_mu);
    cached = take_cached(want, device, &o->b);
  }
  if (!cached) {
    void *mem = nullptr;
    hipError_t e = hipMalloc(&mem, want);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      pending_again(true);
      release_cached(device);
      e = hipMalloc(&mem, want);
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      std::free(o);
      set_error("hipMalloc of %zu bytes failed: %s", want, hipGetErrorString(e));
      return PASUR_E_NOMEM;
    }
    o->b = Block{mem, want, device};
  }
  std::lock_guard<std::mutex> lock(g_block_mu);
  Owned **at = owned_place(o->b.p);
  o->next = *at;
  *at = o;
  *p = o->b.p;
  return PASUR_OK;
}

// Takes a block off the list of those in use.
bool disown(void *p, Block *b) {
  std::lock_guard<std::mutex> lock(g_block_mu);
  Owned **at = owned_place(p);
  while (*at && (*at)->b.p != p) at = &(*at)->next;
  if (!*at) return false;
  Owned *o = *at;
  *at = o->next;
  *b = o->b;
  std::free(o);
  return true;
}
}  // namespace

int block_alloc(void **p, size_t bytes) { return alloc(p, bytes, false, nullptr); }
int block_alloc_on(void **p, size_t bytes, hipStream_t s) { return alloc(p, bytes, true, s); }

void block_free(void *p) {
  Block b;
  if (p && disown(p, &b)) give_back(b);
}

void block_free_on(void *p, hipStream_t s) {
  Block b;
  if (!p || !disown(p, &b)) return;
  Pending *const n = (Pending *)std::malloc(sizeof(Pending));
  hipEvent_t ended = nullptr;
  if (!n || hipEventCreateWithFlags(&ended, hipEventDisableTiming) != hipSuccess ||
      hipEventRecord(ended, s) != hipSuccess) {
    // when its work ends isn't known: the memory stays unused
    (void)hipGetLastError();
    if (ended) (void)hipEventDestroy(ended);
    std::free(n);
    return;
  }
  n->b = b;
  n->stream = s;
  n->ended = ended;
  std::lock_guard<std::mutex> lock(g_block_mu);
  n->next = g_pending;
  g_pending = n;
}

void blocks_release() {
  retire_again();
  pending_again(false);
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return;
  release_cached(device);
}

hipError_t malloc_async(void **p, size_t bytes, hipStream_t s) {
  const hipError_t e = hipMallocAsync(p, bytes, s);
  if (e == hipSuccess) return e;
  (void)hipGetLastError();
  blocks_release();
  return hipMallocAsync(p, bytes, s);
}

int anchor_alloc(void **a) { return dev_alloc((int64_t **)a, 8); }

void blocks_retire(void *anchor, void *const *blocks, int n) {
  if (anchor_wait(anchor)) {
    for (int i = 0; i < n; ++i) block_free(blocks[i]);
    return;
  }
  Retired *r = (Retired *)std::malloc(sizeof(Retired));
  if (!r) return;  // their memory stays unused
  r->anchor = anchor;
  r->n = n;
  std::memcpy(r->blocks, blocks, (size_t)n * sizeof(void *));
  std::lock_guard<std::mutex> lock(g_block_mu);
  r->next = g_retired;
  g_retired = r;
}

namespace {
// Free sets of words, linked through the word behind them.  A set is allocated
// when a call finds none free, so there are as many as calls have been in flight
// at once (256 bytes each); they stay until the process ends.
std::mutex g_words_mu;
int64_t *g_words = nullptr;
int64_t *&next_of(int64_t *w) { return *reinterpret_cast<int64_t **>(w + kHostWords); }
}  // namespace

HostWords::HostWords(hipStream_t s) : w(nullptr), stream(s), pending(false) {
  {
    std::lock_guard<std::mutex> lock(g_words_mu);
    if (g_words) {
      w = g_words;
      g_words = next_of(w);
    }
  }
  if (!w) {
    const hipError_t e = hipHostMalloc((void **)&w, (kHostWords + 1) * sizeof(int64_t),
                                       hipHostMallocPortable | hipHostMallocMapped);
    if (e != hipSuccess) {
      set_error("pinned host memory: %s", hipGetErrorString(e));
      w = nullptr;
      return;
    }
  }
  std::memset(w, 0, kHostWords * sizeof(int64_t));
}

HostWords::~HostWords() {
  if (!w) return;
  if (pending) (void)hipStreamSynchronize(stream);
  std::lock_guard<std::mutex> lock(g_words_mu);
  next_of(w) = g_words;
  g_words = w;
}

int HostWords::wait() {
  // whatever an earlier call left to report, what is enqueued has to end first
  const hipError_t earlier = hipGetLastError(), e = hipStreamSynchronize(stream);
  PASUR_TRY_HIP(e);
  pending = false;
  PASUR_TRY_HIP(earlier);
  return PASUR_OK;
}

int scan_counts(const int32_t *d_counts, int64_t n, int32_t *d_out,
                int64_t *total, hipStream_t stream) {
  HostWords host(stream);
  if (!host.ok()) return PASUR_E_NOMEM;
  void *scratch = nullptr;
  if (n >= kScanTile)
    PASUR_TRY(block_alloc(&scratch, (size_t)scan_scratch(n) * sizeof(int64_t)));
  scan_enqueue(CountsIn{d_counts}, OffsetsOut{d_out, 0}, n, 1, (int64_t *)scratch,
               host.dev(0), stream);
  const int st = host.wait();
  if (host.idle()) block_free(scratch);  // (else it may be in use)
  PASUR_TRY(st);
  *total = host[0];
  return total_fits(*total);
}

}  // namespace pasur

extern "C" const char *pasur_last_error(void) { return pasur::g_err; }
extern "C" int pasur_version(void) { return 1; }
extern "C" void pasur_release_cache(void) { pasur::blocks_release(); }
