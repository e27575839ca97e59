// Stand-in for the HIP runtime, for tests of the host driver without a GPU:
// device memory is host memory, work is queued per process and runs when the
// host waits or asks, and a kernel is whatever the test says it does.
#pragma once
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <memory>
#include <map>
#include <string>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
#define __align__(n) alignas(n)

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorNotReady = 600, hipErrorUnknown = 999 };
typedef struct FakeStream* hipStream_t;
typedef struct FakeEvent* hipEvent_t;
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2, hipDeviceAttributeMultiprocessorCount = 0 };
enum hipMemoryType { hipMemoryTypeUnregistered, hipMemoryTypeHost, hipMemoryTypeDevice, hipMemoryTypeManaged };
struct hipPointerAttribute_t {
  hipMemoryType type;
  int device;
};
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct uint4 {
  uint32_t x, y, z, w;
};
struct int4 {
  int32_t x, y, z, w;
};

namespace fake {
// What a kernel does, given its arguments; it copies what it needs of them and
// returns the work to queue.
using Kernel = std::function<std::function<void()>(void**)>;
struct Runtime {
  std::map<const void*, std::string> names;
  std::map<std::string, Kernel> kernels;
  std::map<std::string, int> launched;             // by kernel, graph nodes included
  std::map<std::string, int> copies;               // by kind
  std::deque<std::function<void()>> queue;
  std::string fail_launch;                         // this kernel's launch fails
  std::map<const void*, hipPointerAttribute_t> attributes;  // others: this device's memory
};
inline Runtime& rt() {
  static Runtime r;
  return r;
}
inline const void* kernel(const char* name) {
  static std::map<std::string, char> at;
  char* p = &at[name];
  rt().names[p] = name;
  return p;
}
inline void drain() {
  while (!rt().queue.empty()) {
    auto f = rt().queue.front();
    rt().queue.pop_front();
    if (f) f();
  }
}
inline hipError_t launch(const void* fn, void** params) {
  const std::string& n = rt().names[fn];
  if (n == rt().fail_launch) return hipErrorUnknown;
  ++rt().launched[n];
  auto k = rt().kernels.find(n);
  if (k != rt().kernels.end()) rt().queue.push_back(k->second(params));
  return hipSuccess;
}
}  // namespace fake

// A captured graph keeps its nodes' work as made from their arguments.
struct FakeGraph {
  std::vector<std::pair<std::string, std::function<void()>>> nodes;
};
typedef FakeGraph* hipGraph_t;
typedef FakeGraph* hipGraphExec_t;
typedef void* hipGraphNode_t;
struct hipKernelNodeParams {
  void* func;
  dim3 gridDim, blockDim;
  unsigned sharedMemBytes;
  void** kernelParams;
  void** extra;
};

inline hipError_t hipGraphCreate(hipGraph_t* g, unsigned) { *g = new FakeGraph; return hipSuccess; }
inline hipError_t hipGraphDestroy(hipGraph_t g) { delete g; return hipSuccess; }
inline hipError_t hipGraphAddKernelNode(hipGraphNode_t* node, hipGraph_t g, const hipGraphNode_t*, size_t,
                                        const hipKernelNodeParams* p) {
  const std::string& n = fake::rt().names[p->func];
  auto k = fake::rt().kernels.find(n);
  g->nodes.push_back({n, k != fake::rt().kernels.end() ? k->second(p->kernelParams) : nullptr});
  *node = g;
  return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, void*, void*, size_t) {
  *e = new FakeGraph(*g);
  return hipSuccess;
}
inline hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete e; return hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (auto& n : e->nodes) {
    ++fake::rt().launched[n.first];
    fake::rt().queue.push_back(n.second);
  }
  return hipSuccess;
}
inline hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void** params, size_t, hipStream_t) {
  return fake::launch(fn, params);
}
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return hipSuccess; }
inline hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 4;
  return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
inline hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  ++fake::rt().copies[k == hipMemcpyHostToDevice ? "up" : k == hipMemcpyDeviceToHost ? "down" : "device"];
  if (k == hipMemcpyHostToDevice) {  // the source may be gone by then
    std::string bytes((const char*)s, n);
    fake::rt().queue.push_back([=] { memcpy(d, bytes.data(), n); });
  } else {
    fake::rt().queue.push_back([=] { memcpy(d, s, n); });
  }
  return hipSuccess;
}
inline hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
  fake::rt().queue.push_back([=] { memset(p, v, n); });
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { fake::drain(); return hipSuccess; }
inline hipError_t hipStreamQuery(hipStream_t) { fake::drain(); return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { fake::drain(); return hipSuccess; }
inline hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  auto it = fake::rt().attributes.find(p);
  *a = it == fake::rt().attributes.end() ? hipPointerAttribute_t{hipMemoryTypeDevice, 0} : it->second;
  return hipSuccess;
}
#define HIP_SYMBOL(x) ((const void*)(x))
