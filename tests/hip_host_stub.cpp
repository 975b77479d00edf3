// A HIP runtime without a GPU, for host-side tests of liblpic.so: device memory is host memory
// from a budget, kernels do nothing (but for the one that fills with zeros), and what a stream
// would be given is written to a log (launches inside a captured graph when the graph is
// launched).  Loaded before the library under the HIP runtime's soname, it stands in for it.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Graph { std::vector<std::string> log; };

size_t budget = SIZE_MAX, used = 0;
int last_error = 0, fail_instantiate = -1, fail_launch = -1, fail_copy = -1;
bool capturing = false;
std::map<void*, size_t> sizes;
std::vector<void*> order;                 // allocations, oldest first
std::map<const void*, std::string> names;
std::vector<std::string> events, captured;
struct { Dim3 grid, block; size_t shared; void* stream; } config;
std::string text;

void log(const std::string& s) { (capturing ? captured : events).push_back(s); }
int fail(int e) { return last_error = e; }
bool due(int& n) { return n >= 0 && n-- == 0; }
}  // namespace

extern "C" {
// ---- controls ----
void stub_budget(size_t n) { budget = n; }
size_t stub_used() { return used; }
void stub_fail_instantiate(int n) { fail_instantiate = n; }   // the n-th from now (0: the next)
void stub_fail_launch(int n) { fail_launch = n; }
void stub_fail_copy(int n) { fail_copy = n; }
void* stub_newest(size_t size) {          // the newest live allocation of that size
  for (size_t i = order.size(); i-- > 0;)
    if (sizes.count(order[i]) && sizes[order[i]] == size) return order[i];
  return nullptr;
}
const char* stub_events() {
  text.clear();
  for (const auto& e : events) text += e + "\n";
  events.clear();
  return text.c_str();
}

// ---- the runtime ----
int hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (n > budget - used) return fail(2);
  *p = malloc(n);
  sizes[*p] = n;
  order.push_back(*p);
  used += n;
  return 0;
}
int hipFree(void* p) {
  used -= sizes[p];
  sizes.erase(p);
  free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  memcpy(d, s, n);
  log("wait copy");
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  if (due(fail_copy)) return fail(1);
  memcpy(d, s, n);
  log("copy");
  return 0;
}
int hipMemset(void* p, int v, size_t n) {
  memset(p, v, n);
  log("memset");
  return 0;
}
int hipStreamSynchronize(void* st) {
  log(st ? "sync" : "wait null stream");
  return 0;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "stub error"; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = malloc(64); return 0; }

int hipStreamBeginCapture(void*, int) {
  capturing = true;
  captured.clear();
  return 0;
}
int hipStreamEndCapture(void*, void** g) {
  capturing = false;
  *g = new Graph{captured};
  return 0;
}
int hipGraphInstantiate(void** exec, void* g, void*, void*, size_t) {
  if (due(fail_instantiate)) return fail(2);
  *exec = new Graph(*(Graph*)g);
  return 0;
}
int hipGraphLaunch(void* exec, void*) {
  for (const auto& e : ((Graph*)exec)->log) events.push_back(e);
  return 0;
}
int hipGraphDestroy(void* g) { delete (Graph*)g; return 0; }
int hipGraphExecDestroy(void* g) { delete (Graph*)g; return 0; }

void** __hipRegisterFatBinary(const void*) { return (void**)malloc(8); }
void __hipUnregisterFatBinary(void** p) { free(p); }
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void* stream) {
  config = {grid, block, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void** args, size_t shared, void*) {
  if (due(fail_launch)) return fail(1);
  if (!capturing && names[f].find("k_fill_zero_u32") != std::string::npos)
    memset(*(void**)args[0], 0, 4 * *(int64_t*)args[1]);
  log("launch " + names[f] + " " + std::to_string(grid.x) + " " + std::to_string(shared));
  return 0;
}
}
