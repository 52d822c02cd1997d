// A stand-in for the HIP runtime calls that libmx's host code makes, preloaded
// into a process of its own (LD_PRELOAD) so that its launches, events and
// staging buffers can be watched, and made to fail, on a machine without a GPU.
// Kernels do not run: a launch is recorded with its name, its stream and the
// staging buffer it would read, which counts as being read from then on until
// an event recorded behind it on its stream has been synchronised.
#include <dlfcn.h>
#include <signal.h>
#include <stdint.h>
#include <string.h>
#include <sys/mman.h>
#include <time.h>

#include <atomic>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

struct Dim3 {
  uint32_t x, y, z;
};
struct Event {
  std::vector<uint64_t> covers;  // launches recorded before it on its stream
};
struct Reader {
  void* stream;
  uintptr_t buf;
};

std::mutex g_mu;
std::map<const void*, std::string> g_names;
std::map<uintptr_t, size_t> g_bufs;       // live staging buffers
std::map<uint64_t, Reader> g_reading;     // launches that may still read theirs
uint64_t g_launches = 0;
std::string g_log;
int g_violations = 0;
std::string g_fail_after;                 // ... or the first one behind a launch of this kernel
bool g_fail_armed = false;

// Page-protected buffers: the first write to one waits until it is let through.
size_t g_guard_bytes = 0;                 // sizes from here on are guarded (0: none)
std::atomic<uintptr_t> g_guard_lo{0}, g_guard_hi{0};
std::atomic<int> g_guard_hit{0}, g_guard_open{0};

thread_local Dim3 t_grid, t_block;
thread_local size_t t_lds;
thread_local void* t_stream;

void on_fault(int sig, siginfo_t* info, void*) {
  const uintptr_t a = (uintptr_t)info->si_addr, lo = g_guard_lo, hi = g_guard_hi;
  if (a < lo || a >= hi) {
    signal(sig, SIG_DFL);
    return;
  }
  g_guard_hit = 1;
  const timespec ms{0, 1000000};
  while (!g_guard_open) nanosleep(&ms, nullptr);
  mprotect((void*)lo, hi - lo, PROT_READ | PROT_WRITE);
}

void check_free(uintptr_t buf) {  // a buffer about to be rewritten or freed
  for (const auto& r : g_reading)
    if (r.second.buf == buf) {
      g_violations++;
      return;
    }
}

}  // namespace

extern "C" {

// ------------------------------------------------------------- for the tests
int fake_violations() { return g_violations; }
void fake_fail_record_behind(const char* kernel) { g_fail_after = kernel; }
void fake_guard(size_t bytes) {
  struct sigaction sa = {};
  sa.sa_sigaction = on_fault;
  sa.sa_flags = SA_SIGINFO;
  sigaction(SIGSEGV, &sa, nullptr);
  g_guard_bytes = bytes;
}
int fake_guard_hit() { return g_guard_hit; }
void fake_guard_release() { g_guard_open = 1; }
// The launches since the last call, one line each: name, grid x, stream.
const char* fake_log() {
  static std::string out;
  std::lock_guard<std::mutex> g(g_mu);
  out.swap(g_log);
  g_log.clear();
  return out.c_str();
}

// ------------------------------------------------------------- the runtime
int hipGetDevice(int* d) { return *d = 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipEventCreate(void** e) { *e = new Event(); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = new Event(); return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }

int hipHostMalloc(void** p, size_t n, unsigned) {
  n = (n + 4095) & ~(size_t)4095;
  const bool guard = g_guard_bytes && n >= g_guard_bytes && !g_guard_lo;
  void* m = mmap(nullptr, n, guard ? PROT_NONE : PROT_READ | PROT_WRITE,
                 MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == MAP_FAILED) return 2;
  if (guard) {
    g_guard_hi = (uintptr_t)m + n;
    g_guard_lo = (uintptr_t)m;
  }
  std::lock_guard<std::mutex> g(g_mu);
  g_bufs[(uintptr_t)m] = n;
  *p = m;
  return 0;
}
int hipHostFree(void* p) {
  std::lock_guard<std::mutex> g(g_mu);
  check_free((uintptr_t)p);
  munmap(p, g_bufs[(uintptr_t)p]);
  g_bufs.erase((uintptr_t)p);
  return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }

int hipEventRecord(void* e, void* stream) {
  std::lock_guard<std::mutex> g(g_mu);
  if (g_fail_armed) {
    g_fail_armed = false;
    return 999;
  }
  Event* ev = (Event*)e;
  ev->covers.clear();
  for (const auto& r : g_reading)
    if (r.second.stream == stream) ev->covers.push_back(r.first);
  return 0;
}
int hipEventSynchronize(void* e) {
  std::lock_guard<std::mutex> g(g_mu);
  for (uint64_t l : ((Event*)e)->covers) g_reading.erase(l);
  return 0;
}

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  t_grid = grid;
  t_block = block;
  t_lds = lds;
  t_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = t_grid;
  *block = t_block;
  *lds = t_lds;
  *stream = t_stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void** args, size_t, void* stream) {
  std::lock_guard<std::mutex> g(g_mu);
  const std::string& name = g_names[f];
  // the staging buffer: argument 0 of the uploads, argument 4 of the KV append
  uintptr_t buf = 0;
  if (name.find("upload_kernel") != std::string::npos ||
      name.find("prologue_kernel") != std::string::npos)
    buf = *(uintptr_t*)args[0];
  else if (name.find("kv_append_kernel") != std::string::npos)
    buf = *(uintptr_t*)args[4];
  if (buf) {
    check_free(buf);
    g_reading[g_launches++] = Reader{stream, buf};
  }
  g_log += name + " " + std::to_string(grid.x) + " " + std::to_string((uintptr_t)stream) + "\n";
  if (!g_fail_after.empty() && name.find(g_fail_after) != std::string::npos) {
    g_fail_armed = true;
    g_fail_after.clear();
  }
  return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }

void __hipRegisterFunction(void** mods, const void* f, char* dev_fn, const char* name, unsigned n,
                           void* a, void* b, void* c, void* d, int* w) {
  {
    std::lock_guard<std::mutex> g(g_mu);
    g_names[f] = name;
  }
  using Fn = void (*)(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*,
                      int*);
  if (Fn real = (Fn)dlsym(RTLD_NEXT, "__hipRegisterFunction"))
    real(mods, f, dev_fn, name, n, a, b, c, d, w);
}

}  // extern "C"
