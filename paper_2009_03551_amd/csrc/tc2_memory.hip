// Device memory of the solver's buffers.
//
// A solve grows its large buffers (the iterate's values, the stage of kept
// blocks, the work arrays) over many updates, and a precision switch or a
// new context releases and re-requests tens of gigabytes.  Freeing a large
// allocation and asking for a larger one makes the GPU driver clear memory it has
// just reclaimed, at a few tens of GB/s, which stalls the device for seconds
// at the largest sizes.  Large buffers here therefore live in a virtual
// address range reserved once per buffer; physical memory is mapped into it
// in fixed chunks as the buffer grows, so growing keeps the contents and
// allocates only the increment.  Chunks a buffer gives back go to a pool per
// device and are mapped again by the next buffer that grows, within the same
// solve or in a later context (a later context would otherwise wait for the
// driver to clear the memory again: up to 2.6 s for one chunk at 256 MB after
// a large context was freed).  The pool is returned to the GPU driver when an
// allocation of the library fails for lack of memory (and then retried), and
// by tc2_trim_memory, for callers whose other allocations need the memory.
//
// Buffers below 64 MB are plain allocations, kept after their release in lists
// by size, at most SMALL_HELD bytes per device, and handed out again: a solve
// takes about 100 of them and an orthogonalisation 400, at 10 to 28 us for
// hipMalloc and 12 for hipFree (non-orthogonal solve of 125 atoms: 16 of 85 ms).
// As with hipFree, the device is idle before a released buffer can be another's
// (dev_free waits for it), except where one wait serves many: within a MemScope
// of a stream, buffers pass from one use to the next in the order of that
// stream, and leave the scope once the stream has ended: at its end, when they
// are more than SMALL_HELD, and when an allocation fails for lack of memory.
#include "tc2_context.h"

#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace tc2 {

namespace {

constexpr int MAX_DEVICES = 64;

struct Pool {
  std::mutex m;
  bool init = false;
  bool ok = false;           // the device supports the virtual memory calls
  size_t chunk = 0;          // bytes per physical chunk
  size_t va = 0;             // bytes of virtual range reserved per buffer
  std::vector<hipMemGenericAllocationHandle_t> free;
  // ranges with one chunk mapped, as a buffer left them (mapping again costs
  // 1.5 ms), at most RANGES
  std::vector<std::pair<void*, hipMemGenericAllocationHandle_t>> ranges;
};
constexpr size_t RANGES = 4;

Pool g_pool[MAX_DEVICES];

hipMemAllocationProp chunk_prop(int dev) {
  hipMemAllocationProp prop = {};
  prop.type = hipMemAllocationTypePinned;
  prop.location.type = hipMemLocationTypeDevice;
  prop.location.id = dev;
  return prop;
}

// Pool of the current device, set up on first use; nullptr when the device
// does not support the calls (buffers then fall back to plain allocations).
Pool* pool_of(int* dev_out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  Pool& P = g_pool[dev];
  std::lock_guard<std::mutex> g(P.m);
  if (!P.init) {
    P.init = true;
    P.ranges.reserve(RANGES);
    const hipMemAllocationProp prop = chunk_prop(dev);
    size_t gran = 0;
    size_t total = 0;
    if (hipMemGetAllocationGranularity(&gran, &prop, hipMemAllocationGranularityMinimum) ==
            hipSuccess &&
        gran > 0 && hipDeviceTotalMem(&total, dev) == hipSuccess && total > 0) {
      const size_t want = (size_t)256 << 20;
      P.chunk = (want + gran - 1) / gran * gran;
      P.va = (total / P.chunk + 2) * P.chunk;
      P.ok = true;
    }
    (void)hipGetLastError();
  }
  if (dev_out) *dev_out = dev;
  return P.ok ? &P : nullptr;
}

// The small buffers: sizes of those in use, and the free ones by size.
struct Small {
  std::mutex m;
  std::unordered_map<void*, size_t> used;  // of this device
  SizeLists free;
  size_t held = 0;                         // bytes in free
};
constexpr size_t SMALL_HELD = (size_t)256 << 20;

Small g_small[MAX_DEVICES];
thread_local MemScope* t_scope = nullptr;

// allocated size of a small buffer: four steps per octave
size_t small_size(size_t n) {
  size_t s = 256;
  while (s < n) s *= 2;
  const size_t step = s > 1024 ? s / 8 : s;
  return (n + step - 1) / step * step;
}

void* take(SizeLists& l, size_t n) {
  auto it = l.find(n);
  if (it == l.end() || it->second.empty()) return nullptr;
  void* p = it->second.back();
  it->second.pop_back();
  return p;
}

// false when the host is out of memory
bool put(SizeLists& l, void* p, size_t n) {
  try {
    l[n].push_back(p);
  } catch (const std::bad_alloc&) {
    return false;
  }
  return true;
}

// to the free list, or to the driver when that is full
void give(Small& S, void* p, size_t n) {
  {
    std::lock_guard<std::mutex> g(S.m);
    if (S.held + n <= SMALL_HELD && put(S.free, p, n)) {
      S.held += n;
      return;
    }
    S.used.erase(p);
  }
  (void)hipFree(p);
}

}  // namespace

// Wait for all work of the current device, by the wait that hipFree does.
// hipDeviceSynchronize fails while another thread captures a graph, without
// having waited, and ends that capture; a copy by hipMemcpy does the same (copies
// go through hipMemcpyWithStream therefore).
bool device_wait() {
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, 256);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    pool_trim();
    e = hipMalloc(&p, 256);
  }
  if (e == hipSuccess) e = hipFree(p);
  if (e != hipSuccess) (void)hipGetLastError();
  return e == hipSuccess;
}

namespace {

// Streams not in use by a call, at most IDLE per device: making and destroying
// one takes 25 us, its first use on a hardware queue 1.3 ms.
struct Streams {
  std::mutex m;
  std::vector<hipStream_t> idle;
};
constexpr size_t IDLE = 4;
Streams g_streams[MAX_DEVICES];

}  // namespace

ServiceStream::ServiceStream() {
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return;
  {
    Streams& S = g_streams[dev];
    std::lock_guard<std::mutex> g(S.m);
    if (!S.idle.empty()) {
      st = S.idle.back();
      S.idle.pop_back();
      return;
    }
  }
  if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
    (void)hipGetLastError();
    st = nullptr;
  }
}

ServiceStream::~ServiceStream() {
  if (!st) return;
  if (!broken) {
    Streams& S = g_streams[dev];
    std::lock_guard<std::mutex> g(S.m);
    if (S.idle.capacity() < IDLE) {
      try {
        S.idle.reserve(IDLE);
      } catch (const std::bad_alloc&) {
      }
    }
    if (S.idle.size() < std::min(IDLE, S.idle.capacity())) {
      S.idle.push_back(st);
      return;
    }
  }
  (void)hipStreamDestroy(st);
  (void)hipGetLastError();
}

// Return every pooled chunk and free buffer of the current device to the GPU
// driver, those of this thread's open scopes included, and the idle streams.
void pool_trim() {
  int dev = 0;
  if (hipGetDevice(&dev) == hipSuccess)
    for (MemScope* s = t_scope; s; s = s->outer)
      if (s->dev == dev) (void)s->drain();
  Pool* P = pool_of(&dev);
  if (P) {
    std::lock_guard<std::mutex> g(P->m);
    for (auto& r : P->ranges) {
      (void)hipMemUnmap(r.first, P->chunk);
      (void)hipMemAddressFree(r.first, P->va);
      (void)hipMemRelease(r.second);
    }
    P->ranges.clear();
    for (hipMemGenericAllocationHandle_t h : P->free) (void)hipMemRelease(h);
    P->free.clear();
  }
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return;
  {
    Streams& T = g_streams[dev];
    std::lock_guard<std::mutex> g(T.m);
    for (hipStream_t st : T.idle) (void)hipStreamDestroy(st);
    T.idle.clear();
  }
  Small& S = g_small[dev];
  std::lock_guard<std::mutex> g(S.m);
  for (auto& l : S.free)
    for (void* p : l.second) {
      (void)hipFree(p);
      S.used.erase(p);
    }
  S.free.clear();
  S.held = 0;
}

hipError_t dev_malloc(void** p, size_t n) {
  int dev = 0;
  const bool small = n < VM_MIN && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < MAX_DEVICES;
  size_t want = n;
  if (small) {
    want = small_size(n);
    if (t_scope && t_scope->dev == dev && (*p = take(t_scope->free, want))) {
      t_scope->held -= want;
      return hipSuccess;
    }
    Small& S = g_small[dev];
    std::lock_guard<std::mutex> g(S.m);
    if ((*p = take(S.free, want))) {
      S.held -= want;
      return hipSuccess;
    }
  }
  hipError_t e = hipMalloc(p, want);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    pool_trim();
    e = hipMalloc(p, want);
  }
  if (e == hipSuccess && small) {
    std::lock_guard<std::mutex> g(g_small[dev].m);
    try {
      g_small[dev].used[*p] = want;
    } catch (const std::bad_alloc&) {
      (void)hipFree(*p);
      *p = nullptr;
      return hipErrorOutOfMemory;
    }
  }
  return e;
}

void dev_free(void* p) {
  if (!p) return;
  int cur = 0;
  if (hipGetDevice(&cur) == hipSuccess)
    for (int d = 0; d < MAX_DEVICES; ++d) {
      const int dev = d == 0 ? cur : (d <= cur ? d - 1 : d);  // the current device first
      if (dev < 0 || dev >= MAX_DEVICES) break;
      Small& S = g_small[dev];
      size_t n = 0;
      {
        std::lock_guard<std::mutex> g(S.m);
        auto it = S.used.find(p);
        if (it == S.used.end()) continue;
        n = it->second;
      }
      if (t_scope && t_scope->dev == dev) {
        if (t_scope->idle) {
          give(S, p, n);
          return;
        }
        if (put(t_scope->free, p, n)) {
          if ((t_scope->held += n) > SMALL_HELD) (void)t_scope->drain();
          return;
        }
      }
      if (dev != cur) (void)hipSetDevice(dev);
      const bool done = device_wait();
      if (dev != cur) (void)hipSetDevice(cur);
      if (done) {
        give(S, p, n);
        return;
      }
      std::lock_guard<std::mutex> g(S.m);
      S.used.erase(p);
      break;
    }
  (void)hipFree(p);
}

void MemScope::open(hipStream_t s) {
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return;
  st = s;
  outer = t_scope;
  t_scope = this;
  is_open = true;
}

void MemScope::open_idle() {
  if (!device_wait()) return;
  idle = true;
  open(nullptr);
}

// The free buffers to the pool, once the stream has ended; false when it failed.
bool MemScope::drain() {
  if (held == 0) return true;
  if (hipStreamSynchronize(st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  for (auto& l : free)
    for (void* p : l.second) give(g_small[dev], p, l.first);
  free.clear();
  held = 0;
  return true;
}

MemScope::~MemScope() {
  if (!is_open) return;
  t_scope = outer;
  if (drain()) return;
  for (auto& l : free)
    for (void* p : l.second) dev_free(p);
}

// Grow the virtual range of b to at least n bytes, keeping what is mapped.
hipError_t vm_grow(DBuf& b, size_t n) {
  int dev = 0;
  Pool* P = pool_of(&dev);
  if (!P) return hipErrorNotSupported;
  if (!b.vm) {
    void* base = nullptr;
    {
      std::lock_guard<std::mutex> g(P->m);
      if (!P->ranges.empty()) {
        base = P->ranges.back().first;
        b.chunks.assign(1, P->ranges.back().second);
        P->ranges.pop_back();
      }
    }
    if (!base) {
      hipError_t e = hipMemAddressReserve(&base, P->va, 0, nullptr, 0);
      if (e != hipSuccess) return e;
    }
    b.p = base;
    b.cap = b.chunks.size() * P->chunk;
    b.va = P->va;
    b.vm = true;
    b.dev = dev;
  }
  if (n > b.va) return hipErrorOutOfMemory;
  const size_t need = (n + P->chunk - 1) / P->chunk;
  const hipMemAllocationProp prop = chunk_prop(dev);
  hipMemAccessDesc acc = {};
  acc.location.type = hipMemLocationTypeDevice;
  acc.location.id = dev;
  acc.flags = hipMemAccessFlagsProtReadWrite;
  while (b.chunks.size() < need) {
    hipMemGenericAllocationHandle_t h{};
    bool have = false;
    {
      std::lock_guard<std::mutex> g(P->m);
      if (!P->free.empty()) {
        h = P->free.back();
        P->free.pop_back();
        have = true;
      }
    }
    if (!have) {
      hipError_t e = hipMemCreate(&h, P->chunk, &prop, 0);
      if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        pool_trim();
        e = hipMemCreate(&h, P->chunk, &prop, 0);
      }
      if (e != hipSuccess) return e;
    }
    char* at = (char*)b.p + b.chunks.size() * P->chunk;
    hipError_t e = hipMemMap(at, P->chunk, 0, h, 0);
    if (e == hipSuccess) e = hipMemSetAccess(at, P->chunk, &acc, 1);
    if (e != hipSuccess) {
      (void)hipMemUnmap(at, P->chunk);
      std::lock_guard<std::mutex> g(P->m);
      P->free.push_back(h);
      return e;
    }
    b.chunks.push_back(h);
    b.cap = b.chunks.size() * P->chunk;
  }
  return hipSuccess;
}

// Unmap the chunks of b (once the device is idle) into the pool.  Its range is
// freed, or kept with the first chunk mapped; what stands in the pool may be
// another thread's at once, so the range goes there after its other chunks are
// unmapped.
void vm_release(DBuf& b) {
  if (!b.vm) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != b.dev) (void)hipSetDevice(b.dev);
  (void)device_wait();
  Pool& P = g_pool[b.dev];
  for (size_t k = 1; k < b.chunks.size(); ++k) (void)hipMemUnmap((char*)b.p + k * P.chunk, P.chunk);
  bool kept = false;
  if (!b.chunks.empty()) {
    std::lock_guard<std::mutex> g(P.m);
    P.free.insert(P.free.end(), b.chunks.begin() + 1, b.chunks.end());
    kept = P.ranges.size() < RANGES;
    if (kept) P.ranges.emplace_back(b.p, b.chunks[0]);  // within the capacity reserved in pool_of
  }
  if (!kept) {
    if (!b.chunks.empty()) {
      (void)hipMemUnmap(b.p, P.chunk);
      std::lock_guard<std::mutex> g(P.m);
      P.free.push_back(b.chunks[0]);
    }
    (void)hipMemAddressFree(b.p, b.va);
  }
  b.chunks.clear();
  if (cur != b.dev) (void)hipSetDevice(cur);
  b.p = nullptr;
  b.cap = 0;
  b.va = 0;
  b.vm = false;
}

}  // namespace tc2
