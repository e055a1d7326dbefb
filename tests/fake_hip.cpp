// A HIP runtime without a GPU (test infrastructure): the calls that the
// library's host code makes, kernels left out.  Device memory is host memory.
// It keeps count of what each stream has been given and of what each stream
// and the host have waited for, so that a test can ask whether work was given
// to a stream that does not wait for another stream's.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "fake_hip.h"

namespace {
using Seen = std::map<void*, uint64_t>;   // stream -> its operations waited for
Seen given, host;
std::map<void*, Seen> waits;              // per stream
std::map<void*, Seen> events;
long loose = 0;
struct Dim { uint32_t x, y, z; };
struct Config { Dim grid, block; size_t shmem; void* stream; };
std::vector<Config> configs;

void join(Seen& a, const Seen& b) {
  for (const auto& s : b)
    if (a[s.first] < s.second) a[s.first] = s.second;
}
// One operation given to a stream; `loose` counts those that some other
// stream's earlier operation may still run beside.
void give(void* st) {
  Seen known = waits[st];
  join(known, host);
  for (const auto& s : given)
    if (s.first != st && known[s.first] < s.second) {
      ++loose;
      break;
    }
  ++given[st];
}
void host_waits(void* st) {
  Seen s = waits[st];
  s[st] = given[st];
  join(host, s);
}
}  // namespace

namespace fake {
std::function<void(void*, const void*, size_t)> on_readback;
void reset() {
  given.clear();
  host.clear();
  waits.clear();
  events.clear();
  loose = 0;
}
long loose_operations() { return loose; }
bool host_waited_for(void* st) { return host[st] == given[st]; }
}  // namespace fake

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle[4];
  return handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t shmem, void* st) {
  configs.push_back(Config{grid, block, shmem, st});
  return 0;
}
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* shmem, void** st) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid;
  *block = c.block;
  *shmem = c.shmem;
  *st = c.stream;
  return 0;
}
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void* st) {
  give(st);
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, void* st) {
  give(st);
  std::memmove(dst, src, bytes);
  if (kind == 2 && fake::on_readback) fake::on_readback(dst, src, bytes);
  return 0;
}
int hipMemcpy(void* dst, const void* src, size_t bytes, int) {
  std::memmove(dst, src, bytes);
  return 0;
}
int hipMemsetAsync(void* dst, int v, size_t bytes, void* st) {
  give(st);
  std::memset(dst, v, bytes);
  return 0;
}
int hipStreamSynchronize(void* st) {
  host_waits(st);
  return 0;
}
int hipDeviceSynchronize() {
  join(host, given);
  return 0;
}
int hipStreamWaitEvent(void* st, void* e, unsigned) {
  join(waits[st], events[e]);
  return 0;
}
int hipEventCreate(void** e) {
  *e = std::malloc(1);
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) {
  events.erase(e);
  std::free(e);
  return 0;
}
int hipEventRecord(void* e, void* st) {
  events[e] = waits[st];
  events[e][st] = given[st];
  return 0;
}
int hipEventSynchronize(void* e) {
  join(host, events[e]);
  return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 0.0f;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* b, const void*, int, size_t) {
  *b = 4;
  return 0;
}
const char* hipGetErrorString(int) { return "fake"; }
int hipGetLastError() { return 0; }
int hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = std::malloc(bytes);
  return *p ? 0 : 2;
}
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static char* array = (char*)std::calloc(1, (size_t)80 << 20);
  *p = array;
  return 0;
}
}  // extern "C"
