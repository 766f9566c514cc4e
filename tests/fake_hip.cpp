// A stand-in for the HIP runtime, for tests of the library's host code without a GPU: memory is host memory, kernels do
// nothing (but k_words, which moves flags to the host, runs here), and calls can be made to fail.  The executable defines
// the runtime's functions itself, so the library it loads (argument 1) is bound to these.  Argument 2 names a scenario; each
// prints what it saw, one "name value" per line.
#include <dlfcn.h>

#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <limits>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "dbar.h"

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
constexpr int kOk = 0, kOutOfMemory = 2, kInvalidDevice = 101, kLaunchFailure = 719;

std::mutex mu;
std::map<const void*, std::string> kernels;
std::map<void*, size_t> device;  // live device allocations
size_t device_bytes = 0, device_most = 0, device_limit = std::numeric_limits<size_t>::max();
std::atomic<size_t> pinned_limit{std::numeric_limits<size_t>::max()};
std::atomic<int> captures{0}, stream_waits{0}, launches{0}, reports{0}, lose_report{0};  // lose_report: the ticketed k_words launch that fails (1, 2, ..)
std::string fail_kernel;                                   // launches of kernels whose name holds this fail
thread_local int last_error = kOk;

int set(int e) {
  if (e != kOk) last_error = e;
  return e;
}
// (small buffers hold flags: nonzero, so that every entry is live and active)
void* fresh(size_t bytes) {
  void* p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  if (p && bytes <= (1u << 20)) std::memset(p, 1, bytes);
  return p;
}

// the argument of k_words
struct Words {
  struct {
    const int* src;
    int* dst;
    int n;
  } r[4];
  int* ticket;
  int value;
};
}  // namespace

extern "C" {
#define API __attribute__((visibility("default")))
API int hipGetLastError() {
  const int e = last_error;
  last_error = kOk;
  return e;
}
API int hipPeekAtLastError() { return last_error; }
API const char* hipGetErrorString(int) { return "(test)"; }
API int hipGetDeviceCount(int* n) { return *n = 1, kOk; }
API int hipGetDevice(int* d) { return *d = 0, kOk; }
API int hipSetDevice(int d) { return set(d == 0 ? kOk : kInvalidDevice); }
API int hipDeviceSynchronize() { return kOk; }
API int hipMemGetInfo(size_t* fr, size_t* tot) { return *fr = *tot = size_t(200) << 30, kOk; }
API int hipMalloc(void** p, size_t bytes) {
  std::lock_guard<std::mutex> lock(mu);
  *p = device_bytes + bytes <= device_limit ? fresh(bytes) : nullptr;
  if (!*p) return set(kOutOfMemory);
  device[*p] = bytes;
  device_bytes += bytes;
  device_most = device_most < device_bytes ? device_bytes : device_most;
  return kOk;
}
API int hipFree(void* p) {
  std::lock_guard<std::mutex> lock(mu);
  device_bytes -= device[p];
  device.erase(p);
  std::free(p);
  return kOk;
}
API int hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = bytes <= pinned_limit ? fresh(bytes) : nullptr;
  return set(*p ? kOk : kOutOfMemory);
}
API int hipHostFree(void* p) { return std::free(p), kOk; }
API int hipMemcpy(void* d, const void* s, size_t n, int) { return std::memcpy(d, s, n), kOk; }
API int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { return std::memcpy(d, s, n), kOk; }
API int hipMemsetAsync(void*, int, size_t, void*) { return kOk; }
API int hipStreamCreateWithFlags(void** s, unsigned) { return *s = std::malloc(1), kOk; }
API int hipStreamDestroy(void* s) { return std::free(s), kOk; }
API int hipStreamSynchronize(void*) { return ++stream_waits, kOk; }
API int hipStreamWaitEvent(void*, void*, unsigned) { return kOk; }
API int hipEventCreate(void** e) { return *e = std::malloc(1), kOk; }
API int hipEventCreateWithFlags(void** e, unsigned) { return *e = std::malloc(1), kOk; }
API int hipEventDestroy(void* e) { return std::free(e), kOk; }
API int hipEventRecord(void*, void*) { return kOk; }
API int hipEventSynchronize(void*) { return kOk; }
API int hipEventQuery(void*) { return kOk; }
API int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 1.0f, kOk; }
API int hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, set(kInvalidDevice); }
API int hipStreamBeginCapture(void*, int) { return ++captures, kOk; }
API int hipStreamEndCapture(void*, void** g) { return *g = std::malloc(1), kOk; }
API int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { return *e = std::malloc(1), kOk; }
API int hipGraphLaunch(void*, void*) { return kOk; }
API int hipGraphDestroy(void* g) { return std::free(g), kOk; }
API int hipGraphExecDestroy(void* g) { return std::free(g), kOk; }

API void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
API void __hipUnregisterFatBinary(void**) {}
API void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
API void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels[host] = name;
}
thread_local struct {
  Dim3 grid, block;
  size_t shared;
  void* stream;
} pushed;
API int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void* s) { return pushed = {g, b, shared, s}, kOk; }
API int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shared, void** s) {
  return *g = pushed.grid, *b = pushed.block, *shared = pushed.shared, *s = pushed.stream, kOk;
}
API int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
  const auto it = kernels.find(f);
  const std::string name = it == kernels.end() ? "" : it->second;
  if (!fail_kernel.empty() && name.find(fail_kernel) != std::string::npos) return set(kLaunchFailure);
  launches += name.find("k_count_active") == std::string::npos;  // (the timer's own)
  if (name.find("k_words") == std::string::npos) return kOk;
  const Words& w = *static_cast<const Words*>(args[0]);
  if (w.ticket && ++reports == lose_report) return set(kLaunchFailure);
  for (const auto& r : w.r)
    if (r.n > 0) std::memcpy(r.dst, r.src, r.n * sizeof(int));
  if (w.ticket) __atomic_store_n(w.ticket, w.value, __ATOMIC_RELEASE);
  return kOk;
}
}

namespace {
void* lib;
template <typename F>
F* fn(const char* name) {
  F* f = reinterpret_cast<F*>(dlsym(lib, name));
  if (!f) std::fprintf(stderr, "%s is missing\n", name), std::exit(2);
  return f;
}
#define CALL(name, ...) fn<decltype(name)>(#name)(__VA_ARGS__)

void say(const char* name, long long v) { std::printf("%s %lld\n", name, v), std::fflush(stdout); }

// a solve of nk entries (host arrays), returns its code
int solve(int N, double L, int nk, int max_iter, int lanes, bool nan = false, int precision = DBAR_FP64) {
  const size_t n = (size_t)N * N;
  std::vector<double> Q(2 * n, 0.25), k(2 * nk, 0.5);
  if (nan) Q[2 * n - 1] = std::numeric_limits<double>::quiet_NaN();
  dbar_opts o;
  CALL(dbar_default_opts, &o);
  o.max_iter = max_iter;
  o.lanes = lanes;
  o.batch = nk;
  o.precision = precision;
  const dbar_grid g{N, 11, L};
  return CALL(dbar_solve, &g, Q.data(), nk, k.data(), 1e-12, &o, nullptr, nullptr, nullptr);
}
int transform(int N) {
  const size_t n = (size_t)N * N;
  std::vector<double> in(2 * n, 0.25), out(2 * n);
  const dbar_grid g{N, 11, 3.0};
  return CALL(dbar_transform, &g, 0, in.data(), out.data(), DBAR_FP64);
}
int apply(int N, double L) {
  const size_t n = (size_t)N * N;
  std::vector<double> in(2 * n, 0.25), out(2 * n);
  const double k[2] = {0.5, 0.25};
  const dbar_grid g{N, 11, L};
  return CALL(dbar_apply, &g, in.data(), k, in.data(), out.data(), DBAR_FP64);
}

// one request to a session, its status
int serve(dbar_session* s, int N, bool nan = false) {
  const size_t n = (size_t)N * N;
  std::vector<double> Q(2 * n, 0.25);
  if (nan) Q[2 * n - 1] = std::numeric_limits<double>::quiet_NaN();
  const double k[2] = {0.5, 0.25};
  const dbar_grid g{N, 11, 3.0};
  uint64_t ticket = 0;
  if (const int rc = CALL(dbar_submit, s, &g, Q.data(), k, 1e-12, &ticket)) return rc;
  return CALL(dbar_wait, s, ticket, nullptr, nullptr, nullptr, nullptr);
}

const std::map<std::string, std::function<void()>> scenarios = {
    // an error that the caller's own calls left behind does not refuse a call; a launch that fails does
    {"left_error", [] {
       (void)hipSetDevice(7);
       say("transform", transform(64));
       (void)hipSetDevice(7);
       say("apply", apply(64, 3.0));
       (void)hipSetDevice(7);
       say("solve", solve(64, 3.0, 1, 4, 1));
       say("left", hipGetLastError());
     }},
    {"failed_launch", [] {
       for (const char* k : {"k_stage_copy", "k_lines", "k_tail_table"}) {
         fail_kernel = k;
         say(k, fail_kernel == "k_tail_table" ? apply(64, 4.0) : transform(64));
         fail_kernel.clear();
         say("after", transform(64));
       }
     }},
    // the host's reads of the flags: the n-th of a solve of at most 8 steps is lost, n = 1, 2, .. (0: none)
    {"lost_report", [] {
       for (int N : {64, 128})
         for (int n = 0; n < 4; ++n) {
           lose_report = n ? reports + n : 0;
           say("solve", solve(N, 3.0, 1, 8, 1));
           say("left", hipGetLastError() != kOk);
         }
     }},
    {"lost_report_serving", [] {
       dbar_session* s = nullptr;
       const dbar_session_opts o{size_t(1) << 30, 1, DBAR_MIXED, 20, 0};
       if (CALL(dbar_session_create, &o, &s)) return;
       for (int n = 0; n < 4; ++n) {
         lose_report = n ? reports + n : 0;
         say("lost", serve(s, 128));
         lose_report = 0;
         say("next", serve(s, 128));
       }
       dbar_session_stats st;
       CALL(dbar_session_get_stats, s, &st);
       say("in_flight", st.in_flight + st.queued + st.bytes_in_use);
       CALL(dbar_session_destroy, s);
     }},
    // captures of solves that alternate between two grids of one size, then a larger one between them
    {"captures", [] {
       for (double L : {3.0, 4.0, 3.0, 4.0}) {
         (void)solve(128, L, 1, 8, 1);
         say("captures", captures);
       }
       (void)solve(256, 3.0, 1, 8, 1);
       (void)solve(128, 3.0, 1, 8, 1);
       say("captures", captures);
     }},
    // a potential with NaN where the workspace would not fit; then a solve that replays what an earlier one captured
    {"nan_first", [] {
       device_limit = size_t(64) << 20;
       for (int lanes : {1, 2}) say("nan", solve(1024, 3.0, 4, 8, lanes, true));
       say("most", (long long)device_most);
       say("memory", solve(1024, 3.0, 4, 8, 1));
       device_limit = std::numeric_limits<size_t>::max();
       (void)solve(128, 3.0, 1, 8, 1);
       say("nan", solve(128, 3.0, 1, 8, 1, true));
       say("nan", solve(128, 4.0, 2, 8, 2, true));
       const int before = captures;
       (void)solve(128, 3.0, 1, 8, 1);
       say("captures", captures - before);
       dbar_session* s = nullptr;
       if (CALL(dbar_session_create, nullptr, &s)) return;
       pinned_limit = 0;
       say("nan", serve(s, 64, true));
       say("memory", serve(s, 64));
     }},
    // how transforms of one and of several chunks wait for their results
    {"transform_waits", [] {
       for (int N : {64, 512}) {
         const int before = stream_waits;
         say("transform", transform(N));
         say("stream_waits", stream_waits - before);
       }
     }},
    // launches of a few calls, and those that the timer saw
    {"timer", [] {
       say("on", CALL(dbar_timer_enable, 1));
       launches = 0;
       for (int precision : {DBAR_FP64, DBAR_MIXED})
         for (int N : {8, 64, 128}) (void)solve(N, 3.0, 2, 8, 1, false, precision);
       (void)transform(512);
       (void)apply(128, 4.0);
       const int made = launches;
       say("off", CALL(dbar_timer_enable, 0));
       long long seen = 0;
       for (int i = 0; i < CALL(dbar_timer_num_stages); ++i) {
         int64_t n = 0;
         (void)CALL(dbar_timer_stage, i, nullptr, 0, nullptr, &n, nullptr);
         seen += n;
       }
       say("made", made);
       say("seen", seen);
     }},
};
}  // namespace

int main(int argc, char** argv) {
  if (argc != 3 || !scenarios.count(argv[2])) return 2;
  lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (!lib) return std::fprintf(stderr, "%s\n", dlerror()), 2;
  scenarios.at(argv[2])();
  std::fflush(stdout);
  std::_Exit(0);  // (nothing of the library's own end is under test)
}
