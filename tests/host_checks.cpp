// Checks of the library on the host, without a device: a program that stands in for the HIP runtime.  The library is loaded
// with dlopen, so that its calls of the runtime end here.  Device memory is host memory; of the kernels only moves_kernel does
// its work, the others leave what the memory held (zeros): a build of a cache then goes through all of its stages with
// empty results.  A launch of moves_kernel can be made to fail as the runtime reports it, by hipGetLastError.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <pthread.h>
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <stdexcept>
#include <string>
#include <thread>
#include <vector>

#include "../include/xgm.h"
#include "../paper_2411_15100_amd/csrc/kernels.hpp"

namespace {
std::map<const void*, std::string>& kernel_names() {
  static std::map<const void*, std::string> m;
  return m;
}
int n_launches = 0, n_moves = 0, fail_at = -1;  // fail_at: which launch of moves_kernel fails (-1: none)
int launches_when_it_failed = -1;
xgm::DevTables tables{};  // of the last build
hipError_t last_error = hipSuccess;
struct { dim3 grid, block; size_t shared; hipStream_t stream; } pushed;
}  // namespace

// Threads that the library starts pass through here: how many, and how many at the same time.
std::atomic<int> started{0}, alive{0}, most{0};
thread_local bool own = false;  // this thread starts threads of the checks
struct Start { void* (*run)(void*); void* arg; };
static void* counted(void* p) {
  const Start s = *static_cast<Start*>(p);
  delete static_cast<Start*>(p);
  ++started;
  const int now = ++alive;
  for (int m = most; now > m && !most.compare_exchange_weak(m, now);) {}
  void* const r = s.run(s.arg);
  --alive;
  return r;
}
extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*run)(void*), void* arg) noexcept {
  using Create = int(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
  static Create* const create = reinterpret_cast<Create*>(dlsym(RTLD_NEXT, "pthread_create"));
  return own ? create(t, a, run, arg) : create(t, a, counted, new Start{run, arg});
}

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned int, void*, void*, void*, void*, int*) { kernel_names()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) { pushed = {grid, block, shared, stream}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = pushed.grid; *block = pushed.block; *shared = pushed.shared; *stream = pushed.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
  ++n_launches;
  if (kernel_names()[f].find("first_byte_kernel") != std::string::npos) tables = *static_cast<const xgm::DevTables*>(args[0]);
  if (kernel_names()[f].find("moves_kernel") == std::string::npos) return hipSuccess;
  if (n_moves++ == fail_at) {
    launches_when_it_failed = n_launches;
    return last_error = hipErrorLaunchFailure;
  }
  const xgm::Moves& m = *static_cast<const xgm::Moves*>(args[0]);
  for (int k = 0; k < m.count; ++k) {
    if (m.move[k].src) std::memcpy(m.move[k].dst, m.move[k].src, (size_t)m.move[k].n * 16);
    else std::memset(m.move[k].dst, 0, (size_t)m.move[k].n * 16);
  }
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t s, hipStream_t st, hipEvent_t, hipEvent_t, int) { return hipLaunchKernel(f, g, b, a, s, st); }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "an error of the stand-in"; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(1, n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static void* memory = std::calloc(1, xgm::kStaticScratchBytes); *p = memory; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned int) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}

namespace {
void* library;
template <class F>
F* symbol(const char* name) {
  void* p = dlsym(library, name);
  if (!p) { std::fprintf(stderr, "%s: %s\n", name, dlerror()); std::exit(2); }
  return reinterpret_cast<F*>(p);
}
#define XGM(name) symbol<decltype(name)>(#name)
int failures = 0;
void check(bool ok, const std::string& what) {
  if (ok) return;
  ++failures;
  std::printf("FAILED: %s\n", what.c_str());
}

// A copy or fill of a build that cannot be launched ends the build there: nothing that needs it is launched.
void moves_that_fail() {
  const std::string text = "root ::= \"a\" [0-9]* list?\nlist ::= \"[\" root (\",\" root)* \"]\"\n";
  xgm_grammar* g = nullptr;
  check(XGM(xgm_grammar_compile)(text.data(), text.size(), "root", &g) == XGM_OK, "compile");
  const uint8_t bytes[] = "a1[],";
  const int64_t offsets[] = {0, 1, 2, 3, 4, 5, 5};
  const int32_t stop = 5;
  xgm_vocab* v = nullptr;
  check(XGM(xgm_vocab_create)(bytes, offsets, 6, &stop, 1, &v) == XGM_OK, "vocabulary");
  auto build = [&](int fail) {
    xgm_cache* c = nullptr;
    n_launches = n_moves = 0;
    fail_at = fail;
    launches_when_it_failed = -1;
    last_error = hipSuccess;
    const int status = XGM(xgm_cache_build)(g, v, nullptr, &c);
    check((status == XGM_OK) == (c != nullptr), "a cache if and only if there is no error");
    if (c) XGM(xgm_cache_destroy)(c);
    return status;
  };
  const int status = build(-1);
  check(status == XGM_OK, std::string("a build without failures: ") + XGM(xgm_last_error)());
  const int of_a_build = n_moves;
  check(of_a_build >= 3, "copies and fills of a build");
  for (int k = 0; k < of_a_build; ++k) {
    const int failed = build(k);
    check(failed == XGM_ERR_HIP, "launch " + std::to_string(k) + " of moves_kernel failed, status " + std::to_string(failed));
    check(n_launches == launches_when_it_failed, "launch " + std::to_string(k) + " of moves_kernel failed, launches after it: " + std::to_string(n_launches - launches_when_it_failed));
  }
  check(build(-1) == XGM_OK, "a build after those that failed");
}
// There is room for kMost of them, and one too many is an error, not a write beyond the room.
void moves_that_are_too_many() {
  struct { xgm::Moves moves; unsigned char behind[64]; } m;
  std::memset(m.behind, 0xAB, sizeof(m.behind));
  alignas(16) static char memory[64];
  for (int k = 0; k < xgm::Moves::kMost; ++k) m.moves.add(memory, memory + 16 * k, 16);
  m.moves.add(memory, nullptr, 0);  // (nothing to do)
  check(m.moves.count == xgm::Moves::kMost, "as many as there is room for");
  for (int k = 0; k < xgm::Moves::kMost; ++k) check((char*)m.moves.move[k].src == memory + 16 * k && m.moves.move[k].n == 1, "a move as it was given");
  bool refused = false;
  try {
    m.moves.add(memory, memory + 48, 16);
  } catch (const std::length_error&) {
    refused = true;
  }
  check(refused && m.moves.count == xgm::Moves::kMost, "one too many is refused");
  bool untouched = true;
  for (unsigned char c : m.behind) untouched = untouched && c == 0xAB;
  check(untouched, "nothing is written beyond the room");
}
// Where the sections in front of the headers count as staged, a header is staged too: walk_wave reads the first of them
// whether a lane needs one or not.
void staging_of_tables() {
  for (int32_t budget : {xgm::kFillLdsBudget, xgm::kAcceptLdsBudget, xgm::kContextLdsBudget, xgm::kClassifyLdsBudget})
    for (int32_t off_hdr = budget - 64; off_hdr <= budget + 64; off_hdr += 16)
      for (int32_t n_nodes : {1, 2, 3, 5, 9, 1000}) {
        xgm::DevTables t{};
        t.off_shapes = 256; t.off_targets = 1024; t.off_follow = 2048; t.off_alts = 4096;
        t.off_hdr = (uint32_t)off_hdr;
        t.n_nodes = n_nodes;
        const xgm::DevTables s = xgm::staged_for(t, budget);
        const std::string what = "tables of " + std::to_string(off_hdr) + " bytes and " + std::to_string(n_nodes) + " headers in " + std::to_string(budget);
        check(s.stage_bytes <= (uint32_t)budget && s.stage_bytes >= s.lds_end && s.stage_bytes - s.lds_end < 16, what + ": bytes");
        check(s.n_near <= (uint32_t)n_nodes, what + ": headers");
        if (s.lds_end >= t.off_hdr) check(s.n_near >= 1 && s.lds_end == t.off_hdr + s.n_near * 8, what + ": sections without a header");
        else check(off_hdr + 8 > budget && s.lds_end == t.off_alts && s.n_near == 0, what + ": a section less than there is room for");
      }
}
std::string input() {
  std::string text;
  for (int c; (c = std::getchar()) != EOF;) text += (char)c;
  return text;
}
// Where the headers of a grammar's tables begin (the grammar's text from stdin, its root rule "root").
void headers_begin() {
  const std::string text = input();
  xgm_grammar* g = nullptr;
  xgm_vocab* v = nullptr;
  xgm_cache* cache = nullptr;
  const uint8_t bytes[] = "a";
  const int64_t offsets[] = {0, 1, 1};
  const int32_t stop = 1;
  check(XGM(xgm_grammar_compile)(text.data(), text.size(), "root", &g) == XGM_OK && XGM(xgm_vocab_create)(bytes, offsets, 2, &stop, 1, &v) == XGM_OK &&
        XGM(xgm_cache_build)(g, v, nullptr, &cache) == XGM_OK, XGM(xgm_last_error)());
  std::printf("%u\n", tables.off_hdr);
}
// Compiles of a grammar in `callers` threads, confined to `cpus` CPUs: how many threads the compiles started, and how many
// there were at the same time.
void compile_threads(int cpus, int callers) {
  const std::string text = input();
  cpu_set_t all, some;
  CPU_ZERO(&some);
  check(sched_getaffinity(0, sizeof(all), &all) == 0, "sched_getaffinity");
  for (int k = 0, n = 0; k < CPU_SETSIZE && n < cpus; ++k)
    if (CPU_ISSET(k, &all)) { CPU_SET(k, &some); ++n; }
  if (CPU_COUNT(&some) < cpus) { std::printf("-1 -1\n"); return; }
  check(sched_setaffinity(0, sizeof(some), &some) == 0, "sched_setaffinity");
  auto work = [&] {
    own = false;
    for (int k = 0; k < 20; ++k) {
      xgm_grammar* g = nullptr;
      if (XGM(xgm_grammar_compile)(text.data(), text.size(), "root", &g) != XGM_OK) std::exit(3);
      XGM(xgm_grammar_destroy)(g);
    }
  };
  std::vector<std::thread> threads;
  own = true;
  for (int k = 1; k < callers; ++k) threads.emplace_back(work);
  work();
  for (std::thread& t : threads) t.join();
  std::printf("%d %d\n", started.load(), most.load());
}
}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 2 ? argv[2] : "";
  library = argc > 2 ? dlopen(argv[1], RTLD_NOW | RTLD_GLOBAL) : nullptr;
  if (!library) { std::fprintf(stderr, "%s\n", dlerror()); return 2; }
  if (what == "moves") moves_that_fail();
  else if (what == "staging") staging_of_tables();
  else if (what == "headers") headers_begin();
  else if (what == "threads" && argc == 5) compile_threads(std::atoi(argv[3]), std::atoi(argv[4]));
  else if (what == "too_many_moves") moves_that_are_too_many();
  else { std::fprintf(stderr, "no check of this name: %s\n", what.c_str()); return 2; }
  std::printf("%s: %d failures\n", what.c_str(), failures);
  return failures ? 1 : 0;
}
