// Stands in for the HIP runtime under the host side of libmadakv.so, so that what a call allocates, clears, launches and
// waits for can be looked at without a GPU: every function the library imports, none of which does anything but leave a line
// in a log.  Device memory is host memory that nobody touches.  Loaded before the library with its symbols global.
#include <algorithm>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 { unsigned x, y, z; };
struct Launch { Dim3 grid, block; size_t lds; void* stream; };
std::string text;                    // the log
std::map<const void*, std::string> names;
Launch pushed;
std::string failing;                 // launches of kernels whose name contains one of these parts, separated by |, fail
void* capturing = nullptr;           // the stream under capture
int last_error = 0;
long made = 0;                       // streams and events

template <typename... A> void note(const char* f, A... a) {
  char line[256];
  snprintf(line, sizeof line, f, a...);
  text += line;
  text += '\n';
}
bool fails(const std::string& name) {
  for (size_t i = 0; i < failing.size();) {
    const size_t j = std::min(failing.find('|', i), failing.size());
    if (name.find(failing.substr(i, j - i)) != std::string::npos) return true;
    i = j + 1;
  }
  return false;
}
void* next_object() { return reinterpret_cast<void*>(0x1000 + 16 * ++made); }
}  // namespace

extern "C" {
// ---- for the test
const char* fake_log() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_fail(const char* part) { failing = part; }
void fake_capture(void* stream) { capturing = stream; }

// ---- the runtime
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
int hipMalloc(void** p, size_t n) { *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096); note("malloc %p %zu", *p, n); return *p ? 0 : 2; }
int hipFree(void* p) { note("free %p", p); free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* p, unsigned) { *d = p; return 0; }
int hipMemset(void* p, int v, size_t n) { note("memset %p %d %zu (nil)", p, v, n); note("stream_wait %s", "(nil)"); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* st) { note("memset %p %d %zu %p", p, v, n, st); return 0; }
int hipStreamCreateWithFlags(void** st, unsigned flags) { *st = next_object(); note("stream %p %u", *st, flags); return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void* st) { note("stream_wait %p", st); return 0; }
int hipStreamWaitEvent(void* st, void* ev, unsigned) { note("wait %p %p", st, ev); return 0; }
int hipStreamIsCapturing(void* st, int* status) { *status = st && st == capturing ? 1 : 0; return 0; }
int hipEventCreateWithFlags(void** ev, unsigned) { *ev = next_object(); return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* ev, void* st) { note("record %p %p", ev, st); return 0; }
int hipEventQuery(void* ev) { note("query %p", ev); return 600; }             // not ready
int hipEventSynchronize(void*) { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t lds, void* st) {
  const std::string& name = names[f];
  if (fails(name)) { last_error = 1; note("failed %s", name.c_str()); return 1; }
  // the first argument's leading 256 bytes: the kernels take one struct, which starts with its pointers
  std::string words;
  for (int i = 0; args && i < 32; ++i) {
    unsigned long long w;
    memcpy(&w, static_cast<const char*>(args[0]) + 8 * i, 8);
    char one[20];
    snprintf(one, sizeof one, " %llx", w);
    words += one;
  }
  char head[128];
  snprintf(head, sizeof head, "launch %p %u,%u,%u %zu ", st, grid.x, grid.y, grid.z, lds);
  text += head + name + words + "\n";
  return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* st) { pushed = {grid, block, lds, st}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** st) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *st = pushed.stream;
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* one; return &one; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return 0; }
}
