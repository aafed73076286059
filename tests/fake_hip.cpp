#include "fake_hip.h"

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "launch.h"

struct ihipStream_t {
  std::deque<std::function<bool()>> ops;   // an operation returns false while it has to wait
};
struct ihipEvent_t {
  int recorded = 0, reached = 0;
};

namespace {

std::recursive_mutex mu;
std::map<uint8_t*, size_t>& ranges() {
  static std::map<uint8_t*, size_t> r;
  return r;
}
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> k;
  return k;
}
std::vector<hipStream_t> streams;
ihipStream_t null_stream;
std::atomic<bool> closed{false};
std::atomic<size_t> outside{0};
thread_local hipError_t last_error = hipSuccess;

hipError_t result(hipError_t e) {
  if (e != hipSuccess && e != hipErrorNotReady) last_error = e;
  return e;
}

// Work off what can be, one operation of each stream at a time.
bool progress() {
  std::lock_guard<std::recursive_mutex> lk(mu);
  if (closed) return false;
  bool any = false;
  auto turn = [&](ihipStream_t* s) {
    if (!s->ops.empty() && s->ops.front()()) {
      s->ops.pop_front();
      any = true;
    }
  };
  turn(&null_stream);
  for (size_t k = 0; k < streams.size(); ++k) turn(streams[k]);
  return any;
}

void device_thread() {
  for (;;) {
    if (!progress()) std::this_thread::sleep_for(std::chrono::microseconds(20));
  }
}

ihipStream_t* stream(hipStream_t s) {
  static std::once_flag once;
  std::call_once(once, [] { std::thread(device_thread).detach(); });
  return s ? s : &null_stream;
}

void push(hipStream_t s, std::function<bool()> op) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  stream(s)->ops.push_back(std::move(op));
}

// The allocation that holds p, or ranges().end().
std::map<uint8_t*, size_t>::iterator range_of(const void* p) {
  uint8_t* b = const_cast<uint8_t*>(static_cast<const uint8_t*>(p));
  auto it = ranges().upper_bound(b);
  if (it == ranges().begin()) return ranges().end();
  --it;
  return b < it->first + it->second ? it : ranges().end();
}

bool fits(const void* p, size_t bytes) {
  auto it = range_of(p);
  return it == ranges().end() || bytes <= (size_t)(it->first + it->second - static_cast<const uint8_t*>(p));
}

// ----------------------------------------------------------------- kernels
// The queue in host memory, and a serving "grid" of one workgroup that closes
// once it has found nothing for kIdle.
constexpr std::chrono::milliseconds kIdle(500);   // (a busy machine may hold a thread up)
struct HostMemory {
  uint64_t load(const uint64_t* p) { return *p; }
  uint32_t load_agent(const uint32_t* p) { return *p; }
  void load2(const uint64_t* p0, const uint64_t* p1, uint64_t& v0, uint64_t& v1) {
    v0 = *p0;
    v1 = *p1;
  }
  void add_load(uint64_t* claim, const uint64_t* p, uint64_t& w, uint64_t& v) {
    w = (*claim)++;
    v = *p;
  }
  void store(uint64_t* p, uint64_t v) { __atomic_store_n(p, v, __ATOMIC_RELEASE); }
  template <typename T>
  void exchange(T* p, T v) {
    *p = v;
  }
  void settle() {}
  void claimed(const corr::ServeQueue&) {}
  bool idle(const corr::ServeQueue&) { return true; }
};

struct Grid {
  corr::ServeQueue q;
  corr::ServeView v{0, 1, 0, 0, 0, true, false};
  std::chrono::steady_clock::time_point last = std::chrono::steady_clock::now();

  bool run() {
    HostMemory m;
    uint64_t w = 0;
    for (int slot = corr::serve_claim(m, q, v, &w); slot >= 0; slot = corr::serve_claim(m, q, v, &w)) {
      const corr::ServeJob& j = q.slots[slot];
      if (++q.done[(size_t)slot * corr::kServeLine] == (uint32_t)j.x.n_items)
        __atomic_store_n(j.flag, j.flag_value, __ATOMIC_RELEASE);
      last = std::chrono::steady_clock::now();
    }
    if (std::chrono::steady_clock::now() - last < kIdle) return false;
    *q.closing = q.gen;
    __atomic_store_n(q.host_closing, q.gen, __ATOMIC_RELEASE);
    return true;
  }
};

template <typename T>
T arg(void** args, int k) {
  return *static_cast<T*>(args[k]);
}

std::function<bool()> kernel(const std::string& name, void** args) {
  auto has = [&](const char* s) { return name.find(s) != std::string::npos; };
  if (has("xeng_publish_kernel")) {
    const corr::ServeUpdate* u = arg<const corr::ServeUpdate*>(args, 0);
    const int n_jobs = arg<int>(args, 1), n_active = arg<int>(args, 2);
    const uint32_t version = arg<uint32_t>(args, 3);
    const corr::ServeQueue q = arg<corr::ServeQueue>(args, 4);
    return [=] {
      HostMemory m;
      for (int t = 0; t < 256; ++t) corr::serve_publish(m, u, n_jobs, n_active, version, q, t, 256);
      return true;
    };
  }
  if (has("xeng_serve_kernel")) {
    auto g = std::make_shared<Grid>();
    g->q = arg<corr::ServeQueue>(args, 0);
    return [=] { return g->run(); };
  }
  if (has("fill_zero_kernel")) {
    void* p = arg<void*>(args, 0);
    const int64_t n16 = arg<int64_t>(args, 1);
    return [=] {
      std::memset(p, 0, (size_t)n16 * 16);
      return true;
    };
  }
  if (has("dump_kernel")) {   // the check's word, and whether the result fits
    const bool copies = !has("Li0EEE") && !has("Li3EEE");
    const size_t size = has("Li2EEE") || has("Li5EEE") ? 8 : 4;
    void* dst = arg<void*>(args, 2);
    const int64_t n = arg<int64_t>(args, 3);
    const uint8_t* ws = arg<const uint8_t*>(args, 4);
    uint32_t* bad = arg<uint32_t*>(args, 6);
    return [=] {
      if (copies && !fits(dst, (size_t)n * size)) ++outside;
      if (ws) *bad = 0;
      return true;
    };
  }
  return [] { return true; };
}

}  // namespace

namespace fake {

void* device_alloc(size_t bytes) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  uint8_t* p = static_cast<uint8_t*>(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
  std::memset(p, 0, bytes);
  ranges()[p] = bytes;
  return p;
}
void device_free(void* p) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  ranges().erase(static_cast<uint8_t*>(p));
  std::free(p);
}
size_t queued() {
  std::lock_guard<std::recursive_mutex> lk(mu);
  size_t n = null_stream.ops.size();
  for (hipStream_t s : streams) n += s->ops.size();
  return n;
}
size_t stores_outside() { return outside; }
void queue_gate(hipStream_t s, const std::atomic<bool>* open) {
  push(s, [open] { return open->load(); });
}
void close_streams(bool c) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  closed = c;
}
void set_last_error(hipError_t e) { last_error = e; }

}  // namespace fake

extern "C" {

// ------------------------------------------------------------- registration
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
};
static thread_local Config config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  config = Config{grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *s = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s) {
  auto it = kernels().find(f);
  if (it == kernels().end()) return result(hipErrorInvalidDeviceFunction);
  push(s, kernel(it->second, args));
  return hipSuccess;
}

// ------------------------------------------------------------------ runtime
hipError_t hipGetLastError(void) {   // an error stays until it is asked for
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeWallClockRate ? 100000 : 64;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return result(hipErrorInvalidSymbol);
}
hipError_t hipMemcpyToSymbol(const void*, const void*, size_t, size_t, hipMemcpyKind) { return hipSuccess; }

hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = std::aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
  return *p ? hipSuccess : result(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void* p) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  if (range_of(p) == ranges().end()) return result(hipErrorInvalidValue);
  std::memset(at, 0, sizeof(*at));
  at->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  auto it = range_of(p);
  if (it == ranges().end()) return result(hipErrorNotFound);
  *base = it->first;
  *size = it->second;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  if (!fits(dst, bytes) || !fits(src, bytes)) return result(hipErrorInvalidValue);   // as the runtime does
  push(s, [=] {
    std::memcpy(dst, src, bytes);
    return true;
  });
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  *s = new ihipStream_t;
  streams.push_back(*s);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }   // kept: events may name it
hipError_t hipStreamSynchronize(hipStream_t s) {
  for (;;) {
    {
      std::lock_guard<std::recursive_mutex> lk(mu);
      if (stream(s)->ops.empty()) return hipSuccess;
    }
    std::this_thread::sleep_for(std::chrono::microseconds(20));
  }
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  const int n = e->recorded;
  push(s, [=] { return e->reached >= n; });
  return hipSuccess;
}
hipError_t hipLaunchHostFunc(hipStream_t s, hipHostFn_t f, void* user) {
  push(s, [=] {
    f(user);
    return true;
  });
  return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = new ihipEvent_t;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }   // kept: queued operations may name it
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  const int n = ++e->recorded;
  push(s, [=] {
    e->reached = n;
    return true;
  });
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  return e->reached == e->recorded ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  while (hipEventQuery(e) == hipErrorNotReady) std::this_thread::sleep_for(std::chrono::microseconds(20));
  return hipSuccess;
}

}  // extern "C"
