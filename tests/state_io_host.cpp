// State arrays in and out on a machine of two devices, without one: this
// program stands in for the HIP runtime (its definitions come before the
// library's, which is loaded afterwards), records every launch and copy with
// the device that is current, and runs nothing.  One line per call:
//   name | status | current device afterwards | launches "kernel@device" | 2D copies
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

#include "../include/fdcgks.h"

namespace {
struct Block {
  size_t size;
  int device;
  hipMemoryType type;
};
std::map<char*, Block> g_mem;
std::map<const void*, std::string> g_kernels;
int g_dev = 0, g_copies2d = 0;
std::string g_launches;
dim3 g_grid, g_block;
size_t g_shm;
hipStream_t g_stream;

hipError_t allocate(void** p, size_t n, hipMemoryType type) {
  *p = std::calloc(n ? n : 1, 1);
  if (!*p) return hipErrorOutOfMemory;
  g_mem[static_cast<char*>(*p)] = {n, g_dev, type};
  return hipSuccess;
}
const std::pair<char* const, Block>* find(const void* p) {
  auto it = g_mem.upper_bound(static_cast<char*>(const_cast<void*>(p)));
  if (it == g_mem.begin()) return nullptr;
  --it;
  return static_cast<const char*>(p) < it->first + it->second.size ? &*it : nullptr;
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return allocate(p, n, hipMemoryTypeDevice); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return allocate(p, n, hipMemoryTypeHost); }
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostFree(void*) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = g_dev, hipSuccess; }
hipError_t hipSetDevice(int d) { return g_dev = d, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* v, const void*, int, size_t) { return *v = 1, hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy2DAsync(void*, size_t dpitch, const void*, size_t spitch, size_t width, size_t, hipMemcpyKind,
                            hipStream_t) {
  if (dpitch < width || spitch < width) return hipErrorInvalidValue;
  ++g_copies2d;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void* p) {
  const auto* b = find(p);
  *at = hipPointerAttribute_t{};
  if (!b) return hipErrorInvalidValue;
  at->type = b->second.type;
  at->device = b->second.device;
  at->devicePointer = const_cast<void*>(p);
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* lo, size_t* n, hipDeviceptr_t p) {
  const auto* b = find(p);
  if (!b) return hipErrorInvalidValue;
  *lo = b->first;
  *n = b->second.size;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  g_launches += " " + g_kernels[f] + "@" + std::to_string(g_dev);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t q) {
  g_grid = g, g_block = b, g_shm = s, g_stream = q;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* q) {
  *g = g_grid, *b = g_block, *s = g_shm, *q = g_stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}

int main(int, char** argv) {
  void* lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) return std::fprintf(stderr, "%s\n", dlerror()), 1;
#define F(name) auto name = reinterpret_cast<decltype(&::name)>(dlsym(lib, #name))
  F(fdcgks_default_params);
  F(fdcgks_create);
  F(fdcgks_set_state);
  F(fdcgks_get_state);
  F(fdcgks_batch_create);
  F(fdcgks_batch_set_state);
  F(fdcgks_batch_get_state);
  fdcgks_params p;
  fdcgks_default_params(&p);
  p.nx = 8;
  p.ny = 6;
  p.ly = 0.75;
  fdcgks_problem* pb = nullptr;
  fdcgks_batch* b = nullptr;
  if (fdcgks_create(&p, nullptr, &pb) || fdcgks_batch_create(1, &p, nullptr, &b)) return 2;
  const size_t field = 4 * 48;
  static double host[3 * field];
  void *mine, *peer, *pinned;
  hipMalloc(&mine, sizeof host);
  hipHostMalloc(&pinned, sizeof host, 0);
  hipSetDevice(1);
  hipMalloc(&peer, sizeof host);
  auto call = [&](const std::string& name, int dev, auto&& fn) {
    g_dev = dev;
    g_launches.clear();
    g_copies2d = 0;
    const int st = fn();
    std::printf("%s|%d|%d|%s|%d\n", name.c_str(), st, g_dev, g_launches.c_str(), g_copies2d);
  };
  for (int dev = 0; dev < 2; ++dev)
    for (const auto& [where, q, on] : {std::tuple<const char*, double*, int>{"host", host, 0},
                                       {"mine", static_cast<double*>(mine), 1},
                                       {"peer", static_cast<double*>(peer), 1},
                                       {"pinned", static_cast<double*>(pinned), 1}}) {
      double* const a[3] = {q, q + field, q + 2 * field};
      const std::string t = std::string(where) + (dev ? "_other" : "");
      call("set_" + t, dev, [&] { return fdcgks_set_state(pb, 0, a[0], a[1], a[2], 0, on); });
      call("get_" + t, dev, [&] { return fdcgks_get_state(pb, 1, a[0], a[1], a[2], 0, on); });
      call("batch_set_" + t, dev, [&] { return fdcgks_batch_set_state(b, 0, 0, a[0], a[1], a[2], on); });
      call("batch_get_" + t, dev, [&] { return fdcgks_batch_get_state(b, 0, 1, a[0], a[1], a[2], on); });
    }
  double* m = static_cast<double*>(mine);
  for (int e : {59, 60, 61, 62})
    call("get_stride" + std::to_string(e), 0,
         [&] { return fdcgks_get_state(pb, 0, m, m + field, m + 2 * field, (int64_t)1 << e, 1); });
  return 0;
}
