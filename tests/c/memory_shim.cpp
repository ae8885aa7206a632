// The buffer pool of the library (tc2_memory.hip) as a host program over a
// model of the device's memory: which allocations exist, and which chunk is
// mapped at which address of a reserved range.  The model aborts the program
// with a message on a call that the driver would refuse or that would take
// memory away from a buffer in use.  One scenario per run, named by argv[1].
#include "../../paper_2009_03551_amd/csrc/tc2_memory.hip"

#include <stdio.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <functional>
#include <set>
#include <thread>

// host memory that has run out for this thread
static thread_local bool g_no_host_memory = false;
void* operator new(size_t n) {
  void* p = g_no_host_memory ? nullptr : malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

namespace {

constexpr size_t MB = (size_t)1 << 20, GB = (size_t)1 << 30;

[[noreturn]] void fail(const char* what) {
  fprintf(stderr, "FAILED: %s\n", what);
  fflush(stderr);
  _Exit(1);
}
void check(bool ok, const char* what) {
  if (!ok) fail(what);
}

std::mutex g_m;
uintptr_t g_next = GB;                       // next address handed out
size_t g_capacity = 64 * GB, g_in_use = 0;   // device memory
std::map<uintptr_t, size_t> g_alloc;         // plain allocations
std::map<uintptr_t, size_t> g_reserved;      // virtual ranges
std::map<uintptr_t, uint64_t> g_mapped;      // address -> chunk
std::map<uint64_t, size_t> g_chunk;          // chunk -> bytes
uint64_t g_next_chunk = 1;
std::set<hipStream_t> g_streams_made;
uintptr_t g_next_stream = 0;
std::atomic<int> g_stream_waits{0}, g_device_waits{0};
std::function<void(void*)> g_on_unmap;       // before a mapping is taken away
std::atomic<bool> g_busy{false};             // work in flight: no buffer may be handed on
std::atomic<bool> g_capture{false};          // another thread captures a graph

// calls of every kind that the pool makes, in the model
bool chunk_mapped(uint64_t h) {
  for (auto& m : g_mapped)
    if (m.second == h) return true;
  return false;
}

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  check(!g_capture, "a capture of another thread ended by a device-wide wait");
  g_busy = false;
  return ++g_device_waits, hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return ++g_stream_waits, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  std::lock_guard<std::mutex> g(g_m);
  g_streams_made.insert(*s = (hipStream_t)(++g_next_stream * 16));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::lock_guard<std::mutex> g(g_m);
  check(g_streams_made.erase(s) == 1, "a stream destroyed twice");
  return hipSuccess;
}
hipError_t hipDeviceTotalMem(size_t* n, hipDevice_t) { return *n = g_capacity, hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> g(g_m);
  if (g_in_use + n > g_capacity) return hipErrorOutOfMemory;
  g_in_use += n;
  g_alloc[g_next] = n;
  *p = (void*)g_next;
  g_next += (n + MB) / MB * MB;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> g(g_m);
  auto it = g_alloc.find((uintptr_t)p);
  check(it != g_alloc.end(), "hipFree of an address that is not allocated");
  g_in_use -= it->second;
  g_alloc.erase(it);
  g_busy = false;  // hipFree waits for the device
  return hipSuccess;
}
hipError_t hipMemGetAllocationGranularity(size_t* g, const hipMemAllocationProp*,
                                          hipMemAllocationGranularity_flags) {
  return *g = 2 * MB, hipSuccess;
}
hipError_t hipMemAddressReserve(void** p, size_t n, size_t, void*, unsigned long long) {
  std::lock_guard<std::mutex> g(g_m);
  g_reserved[g_next] = n;
  *p = (void*)g_next;
  g_next += n;
  return hipSuccess;
}
hipError_t hipMemAddressFree(void* p, size_t n) {
  std::lock_guard<std::mutex> g(g_m);
  auto it = g_reserved.find((uintptr_t)p);
  check(it != g_reserved.end() && it->second == n, "a range freed that is not reserved");
  for (auto& m : g_mapped)
    check(m.first < it->first || m.first >= it->first + n, "a range freed with a chunk mapped in it");
  g_reserved.erase(it);
  return hipSuccess;
}
hipError_t hipMemCreate(hipMemGenericAllocationHandle_t* h, size_t n, const hipMemAllocationProp*,
                        unsigned long long) {
  std::lock_guard<std::mutex> g(g_m);
  if (g_in_use + n > g_capacity) return hipErrorOutOfMemory;
  g_in_use += n;
  g_chunk[g_next_chunk] = n;
  *h = (hipMemGenericAllocationHandle_t)g_next_chunk++;
  return hipSuccess;
}
hipError_t hipMemRelease(hipMemGenericAllocationHandle_t h) {
  std::lock_guard<std::mutex> g(g_m);
  auto it = g_chunk.find((uint64_t)h);
  check(it != g_chunk.end(), "a chunk released twice");
  check(!chunk_mapped(it->first), "a chunk released while it is mapped");
  g_in_use -= it->second;
  g_chunk.erase(it);
  return hipSuccess;
}
hipError_t hipMemMap(void* p, size_t, size_t, hipMemGenericAllocationHandle_t h, unsigned long long) {
  std::lock_guard<std::mutex> g(g_m);
  check(!g_mapped.count((uintptr_t)p), "a chunk mapped where another one still is");
  check(!chunk_mapped((uint64_t)h), "a chunk mapped twice");
  g_mapped[(uintptr_t)p] = (uint64_t)h;
  return hipSuccess;
}
hipError_t hipMemUnmap(void* p, size_t) {
  check(!g_busy, "a chunk unmapped with work in flight");
  if (g_on_unmap) g_on_unmap(p);
  std::lock_guard<std::mutex> g(g_m);
  check(g_mapped.erase((uintptr_t)p) == 1, "unmapped where nothing is mapped");
  return hipSuccess;
}
hipError_t hipMemSetAccess(void*, size_t, const hipMemAccessDesc*, size_t) { return hipSuccess; }

}  // extern "C"

namespace {

using namespace tc2;

// every chunk of b is mapped where b takes it to be
void whole(const DBuf& b, const char* what) {
  std::lock_guard<std::mutex> g(g_m);
  for (size_t k = 0; k < b.chunks.size(); ++k) {
    auto it = g_mapped.find((uintptr_t)b.p + k * 256 * MB);
    check(it != g_mapped.end() && it->second == (uint64_t)b.chunks[k], what);
  }
}

// One buffer is released, and while its chunks are being unmapped another
// thread grows a buffer of its own.
void release_beside_grow() {
  DBuf first, second;
  check(first.reserve(900 * MB) == hipSuccess, "first buffer");
  std::thread other;
  std::atomic<bool> done{false};
  g_on_unmap = [&](void*) {
    if (other.joinable()) return;
    other = std::thread([&] {
      check(second.reserve(1100 * MB) == hipSuccess, "second buffer");
      whole(second, "a chunk of the second buffer is not where it was mapped");
      done = true;
    });
    // it may have to wait for a lock of the release: no longer than this
    for (int i = 0; i < 200 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  };
  first.release();
  check(other.joinable(), "the release unmapped nothing");
  other.join();
  g_on_unmap = nullptr;
  check(second.chunks.size() == 5, "size of the second buffer");
  whole(second, "a chunk of the second buffer was taken away");
  // what the release gave back serves the next buffers
  DBuf third;
  check(third.reserve(700 * MB) == hipSuccess, "third buffer");
  whole(third, "third buffer");
  second.release();
  third.release();
  pool_trim();
  check(g_in_use == 0 && g_mapped.empty() && g_reserved.empty(), "memory left after the trim");
}

// Several threads growing and releasing buffers of 1 to 5 chunks.
void many_threads() {
  std::vector<std::thread> ts;
  for (int t = 0; t < 6; ++t)
    ts.emplace_back([t] {
      unsigned s = 12345u * (unsigned)(t + 1);
      for (int k = 0; k < 400; ++k) {
        s = s * 1664525u + 1013904223u;
        DBuf b;
        check(b.reserve((100 + (s >> 8) % 1100) * MB) == hipSuccess, "reserve");
        whole(b, "a chunk is not where it was mapped");
        std::this_thread::yield();
        whole(b, "a chunk was taken away");
        if (k % 50 == 49) pool_trim();
      }
    });
  for (std::thread& t : ts) t.join();
  pool_trim();
  check(g_in_use == 0 && g_mapped.empty() && g_reserved.empty(), "memory left after the trim");
}

// Buffers released within a scope: given back when an allocation fails for lack
// of memory, once the scope's stream has ended, and at most 256 MB of them held.
void scope_under_pressure() {
  g_capacity = 2 * GB;
  {
    MemScope scope;
    scope.open((hipStream_t)0x1);
    // released buffers of one size class serve later ones of that class only
    for (size_t n : {40 * MB, 48 * MB, 56 * MB, 63 * MB}) {
      void* p[4];
      for (void*& q : p) check(dev_malloc(&q, n) == hipSuccess, "small buffer");
      for (void* q : p) dev_free(q);
      size_t held = 0;
      for (auto& a : g_alloc) held += a.second;
      check(held <= 2 * 256 * MB, "released buffers held without bound");
    }
    void* p = nullptr;
    const int waits = g_stream_waits;
    check(dev_malloc(&p, 2 * GB) == hipSuccess, "memory that the scope holds was not given back");
    check(g_stream_waits > waits, "buffers given back before the stream had ended");
    dev_free(p);
    // the same for a buffer of mapped chunks
    void* q[4];
    for (void*& v : q) check(dev_malloc(&v, 60 * MB) == hipSuccess, "small buffer");
    for (void* v : q) dev_free(v);
    DBuf b;
    check(b.reserve(2 * GB) == hipSuccess, "memory that the scope holds was not given back");
    b.release();
    // an inner scope's failure reaches the outer one
    for (void*& v : q) check(dev_malloc(&v, 60 * MB) == hipSuccess, "small buffer");
    for (void* v : q) dev_free(v);
    {
      MemScope inner;
      inner.open((hipStream_t)0x2);
      check(dev_malloc(&p, 2 * GB) == hipSuccess, "memory of the outer scope was not given back");
      dev_free(p);
    }
    // and buffers still pass from one use to the next
    check(dev_malloc(&p, 8 * MB) == hipSuccess, "small buffer");
    dev_free(p);
    check(dev_malloc(&q[0], 8 * MB) == hipSuccess && q[0] == p, "a released buffer was not reused");
    dev_free(q[0]);
  }
  pool_trim();
  check(g_in_use == 0, "memory left after the trim");
}

// Buffers of every size released while work is in flight and another thread
// captures a graph: none is handed on before the work has ended.
void release_beside_capture() {
  for (size_t n : {4096 * (size_t)1, 3 * MB, 60 * MB, 300 * MB, 900 * MB}) {
    DBuf b;
    check(b.reserve(n) == hipSuccess, "reserve");
    g_busy = g_capture = true;
    b.release();
    check(!g_busy, "a buffer handed on with work in flight");
    g_capture = false;
  }
  g_busy = g_capture = true;
  {
    MemScope scope;
    scope.open_idle();
    check(!g_busy && scope.is_open, "a context released with work in flight");
  }
  // the same with no memory left for the wait
  DBuf keep, b;
  check(keep.reserve(4096) == hipSuccess && b.reserve(700 * MB) == hipSuccess, "reserve");
  keep.release();
  g_capacity = g_in_use;
  g_busy = true;
  b.release();
  check(!g_busy, "a buffer handed on with work in flight, memory full");
}

// Streams pass from one call to the next, are never two calls' at once, and are
// bounded and given back.
void service_streams() {
  hipStream_t first = nullptr;
  {
    ServiceStream a, b;
    check(a.st && b.st && a.st != b.st, "one stream for two calls");
    first = b.st;  // given back first
  }
  {
    ServiceStream a;
    check(a.st != nullptr, "no stream");
    a.broken = true;
    first = a.st;
  }
  {
    ServiceStream a, b;
    check(a.st != first && b.st != first, "a broken stream was kept");
  }
  std::mutex m;
  std::set<hipStream_t> busy;
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&] {
      for (int k = 0; k < 500; ++k) {
        ServiceStream a;
        {
          std::lock_guard<std::mutex> g(m);
          check(busy.insert(a.st).second, "one stream for two calls");
        }
        std::this_thread::yield();
        std::lock_guard<std::mutex> g(m);
        busy.erase(a.st);
      }
    });
  for (std::thread& t : ts) t.join();
  check(g_streams_made.size() <= 4, "idle streams without bound");
  pool_trim();
  check(g_streams_made.empty(), "streams left after the trim");
}

// tc2_trim_memory has no way to report an exception: without host memory the
// pool still goes back to the driver.
void trim_without_host_memory() {
  {
    DBuf b[6];
    for (DBuf& x : b) check(x.reserve(300 * MB) == hipSuccess && x.chunks.size() == 2, "reserve");
    void* p = nullptr;
    check(dev_malloc(&p, 3 * MB) == hipSuccess, "small buffer");
    dev_free(p);
  }
  // as many free chunks as their list has room for
  DBuf first;
  std::vector<hipMemGenericAllocationHandle_t>& list = g_pool[0].free;
  check(first.reserve(200 * MB) == hipSuccess, "reserve");
  first.release();
  list.shrink_to_fit();
  g_no_host_memory = true;
  pool_trim();
  g_no_host_memory = false;
  check(g_in_use == 0 && g_mapped.empty() && g_reserved.empty(), "memory left after the trim");
}

}  // namespace

int main(int argc, char** argv) {
  const char* name = argc > 1 ? argv[1] : "";
  if (!strcmp(name, "release_beside_grow")) release_beside_grow();
  else if (!strcmp(name, "many_threads")) many_threads();
  else if (!strcmp(name, "trim_without_host_memory")) trim_without_host_memory();
  else if (!strcmp(name, "service_streams")) service_streams();
  else if (!strcmp(name, "scope_under_pressure")) scope_under_pressure();
  else if (!strcmp(name, "release_beside_capture")) release_beside_capture();
  else fail("no such scenario");
  printf("ok\n");
  return 0;
}
