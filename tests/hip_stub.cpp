// A HIP runtime without a device, for CPU tests of the library's launch
// sequences: preloaded over the real one, it keeps "device" memory in host
// memory, writes down the name of every kernel launched (none of them runs) and
// of every replayed graph, and can let a launch fail.
#include <cxxabi.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { unsigned x, y, z; };
struct Capture { std::vector<std::string> log; };
std::map<const void*, std::string> names;
std::vector<std::string> log_;
std::vector<Capture*> capturing;   // of the library's own captures: at most one
bool caller_captures = false;
int fail_in = -1;                  // launches until the one that fails, < 0: none does
int last_error = 0;
Dim3 grid, block;
size_t shared;
void* stream_;
std::string joined;

void write(const std::string& line) {
  (capturing.empty() ? log_ : capturing.back()->log).push_back(line);
}
}  // namespace

extern "C" {
// what the tests call
void stub_reset() { log_.clear(); }
void stub_fail_launch(int n) { fail_in = n; }
void stub_caller_captures(int on) { caller_captures = on != 0; }
const char* stub_log() {
  joined.clear();
  for (const auto& l : log_) joined += l + "\n";
  return joined.c_str();
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void*, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void*, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
  std::string s = st == 0 && d ? d : device;
  free(d);
  const size_t args = s.find("(mf::");
  if (args != std::string::npos) s.resize(args);
  const size_t ns = s.find("mf::");
  names[host] = ns == std::string::npos ? s : s.substr(ns + 4);
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void* st) {
  grid = g, block = b, shared = s, stream_ = st;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
  *g = grid, *b = block, *s = shared, *st = stream_;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3, void**, size_t, void*) {
  if (fail_in >= 0 && fail_in-- == 0) return last_error = 719;
  write(names[f] + " grid " + std::to_string(g.x) + " " + std::to_string(g.y) + " " + std::to_string(g.z));
  return 0;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "stub error"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) { memmove(dst, src, n); return 0; }
int hipMemsetAsync(void* dst, int v, size_t n, void*) { memset(dst, v, n); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamIsCapturing(void*, int* st) { *st = caller_captures ? 1 : 0; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { capturing.push_back(new Capture); return 0; }
int hipStreamEndCapture(void*, void** g) { *g = capturing.back(); capturing.pop_back(); return 0; }
int hipGraphInstantiate(void** e, void* g, void*, char*, size_t) { *e = new Capture(*static_cast<Capture*>(g)); return 0; }
int hipGraphLaunch(void* e, void*) {
  if (fail_in >= 0 && fail_in-- == 0) return 719;
  log_.push_back("graph");
  for (const auto& l : static_cast<Capture*>(e)->log) log_.push_back("  " + l);
  return 0;
}
int hipGraphDestroy(void* g) { delete static_cast<Capture*>(g); return 0; }
int hipGraphExecDestroy(void* e) { delete static_cast<Capture*>(e); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipGetSymbolAddress(void**, const void*) { return 719; }
}
