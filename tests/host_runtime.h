// A stand-in for the HIP runtime, for checks of the library's host code on a
// machine without a GPU.  A program that defines these functions and links
// liblbm.so has the library call them instead of the runtime's.  Device
// memory is host memory, copies are done at once, kernels are only written
// down.  There are two devices; as in the runtime, an event can be recorded
// only on a stream of the device it was made on.  Include in one file.
#ifndef LBM_TEST_HOST_RUNTIME_H
#define LBM_TEST_HOST_RUNTIME_H

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace fake {
enum { kOk = 0, kInvalid = 1, kNoMemory = 2, kInvalidHandle = 400, kUnknown = 999 };

struct Stream {
  int device;
  bool capturing = false;
};
struct Event {
  int device;
};
struct Dim3 {
  uint32_t x, y, z;
};

inline std::recursive_mutex mu;
inline thread_local int device = 0;
inline std::vector<std::string> launched;            // kernels, in order
inline std::map<char *, size_t> pinned;              // live pinned memory
inline size_t pinned_made = 0;                       // bytes ever allocated
inline int streams = 0, events = 0, graphs = 0;      // live objects
inline int graph_launches = 0;
inline int fail_graph_launch = -1;  // that launch of a graph fails (counted down)
inline int fail_stream_create = 0;  // so many creations fail
struct Copy {
  const char *dst, *src;
  size_t n;
};
inline std::vector<Copy> copied;  // hipMemcpyAsync, in order
inline Dim3 cfg_grid, cfg_block;
inline size_t cfg_shared;
inline void *cfg_stream;

// Host function -> name.  The library registers its kernels before this
// program's own objects are made.
inline std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> names;
  return names;
}
inline int device_of(const void *s) { return s ? static_cast<const Stream *>(s)->device : device; }
inline int launches(const char *part) {
  int n = 0;
  for (const auto &k : launched) n += k.find(part) != std::string::npos;
  return n;
}
}  // namespace fake

extern "C" {
using namespace fake;
using Lock = std::lock_guard<std::recursive_mutex>;

void **__hipRegisterFatBinary(const void *) {
  static void *module;
  return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) {
  cfg_grid = grid, cfg_block = block, cfg_shared = shared, cfg_stream = stream;
  return kOk;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
  *grid = cfg_grid, *block = cfg_block, *shared = cfg_shared, *stream = cfg_stream;
  return kOk;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **, size_t, void *) {
  Lock lock(mu);
  launched.push_back(kernels()[f]);
  return kOk;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int, size_t) {
  const std::string &k = kernels()[f];
  *n = k.find("pair_kernel") == std::string::npos ? 2 : k.find("F64") != std::string::npos ? 4 : 8;
  return kOk;
}
int hipGetDevice(int *d) { return *d = device, kOk; }
int hipSetDevice(int d) { return d == 0 || d == 1 ? (device = d, kOk) : kInvalid; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, kOk; }
const char *hipGetErrorString(int) { return "an error of the stand-in runtime"; }
int hipGetLastError() { return kOk; }
int hipGetSymbolAddress(void **p, const void *) {
  static std::vector<char> symbol(size_t(40) << 20);
  return *p = symbol.data(), kOk;
}
int hipHostMalloc(void **p, size_t n, unsigned) {
  Lock lock(mu);
  char *m = static_cast<char *>(std::malloc(n));
  if (!m) return kNoMemory;
  pinned[m] = n;
  pinned_made += n;
  return *p = m, kOk;
}
int hipHostFree(void *p) {
  Lock lock(mu);
  if (!pinned.erase(static_cast<char *>(p))) return kInvalid;
  std::free(p);
  return kOk;
}
int hipMemcpyAsync(void *dst, const void *src, size_t n, int, void *) {
  Lock lock(mu);
  copied.push_back({static_cast<const char *>(dst), static_cast<const char *>(src), n});
  std::memcpy(dst, src, n);
  return kOk;
}
struct Attributes {
  int type, device;
  void *device_pointer, *host_pointer;
  int managed;
  unsigned flags;
};
int hipPointerGetAttributes(Attributes *a, const void *p) {
  Lock lock(mu);
  std::memset(a, 0, sizeof *a);  // type 0: memory that the runtime does not know
  for (const auto &m : pinned)
    if (p >= m.first && p < m.first + m.second) a->type = 1;
  return kOk;
}
int hipMemsetAsync(void *dst, int v, size_t n, void *) {
  std::memset(dst, v, n);
  return kOk;
}
int hipStreamCreateWithFlags(void **s, unsigned) {
  Lock lock(mu);
  if (fail_stream_create > 0) return --fail_stream_create, kNoMemory;
  ++streams;
  return *s = new Stream{device}, kOk;
}
int hipStreamDestroy(void *s) {
  Lock lock(mu);
  --streams;
  delete static_cast<Stream *>(s);
  return kOk;
}
int hipStreamGetDevice(void *s, int *d) { return *d = device_of(s), kOk; }
int hipStreamIsCapturing(void *s, int *status) {
  return *status = s && static_cast<Stream *>(s)->capturing, kOk;
}
int hipStreamSynchronize(void *) { return kOk; }
int hipEventCreateWithFlags(void **e, unsigned) {
  Lock lock(mu);
  ++events;
  return *e = new Event{device}, kOk;
}
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *e) {
  Lock lock(mu);
  --events;
  delete static_cast<Event *>(e);
  return kOk;
}
int hipEventRecord(void *e, void *s) {
  return static_cast<Event *>(e)->device == device_of(s) ? kOk : kInvalidHandle;
}
int hipEventSynchronize(void *) { return kOk; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 1.0f, kOk; }
int hipStreamWaitEvent(void *, void *, unsigned) { return kOk; }
int hipStreamBeginCapture(void *, int) { return kOk; }
int hipStreamEndCapture(void *, void **g) { return *g = new int(0), kOk; }
int hipGraphInstantiate(void **x, void *, void **, char *, size_t) {
  Lock lock(mu);
  ++graphs;
  return *x = new int(0), kOk;
}
int hipGraphDestroy(void *g) {
  delete static_cast<int *>(g);
  return kOk;
}
int hipGraphExecDestroy(void *x) {
  Lock lock(mu);
  --graphs;
  delete static_cast<int *>(x);
  return kOk;
}
int hipGraphLaunch(void *, void *) {
  Lock lock(mu);
  ++graph_launches;
  return fail_graph_launch >= 0 && fail_graph_launch-- == 0 ? kUnknown : kOk;
}
}  // extern "C"

#endif  // LBM_TEST_HOST_RUNTIME_H
