// Plans on a device with a set amount of memory, without a device: plan.cpp and capi.cpp of the
// library on stand-ins for the HIP calls they make.  hipMalloc hands out host addresses and counts the
// bytes; kernels are not run.  Built by the CPU tests with g++; never part of libpin.so.
#include <cstdlib>
#include <map>

#include "launch.hpp"
#include "plan.hpp"

namespace {

size_t g_total = 0, g_used = 0;
std::map<char*, size_t> g_blocks;
int g_bad = 0;   // frees of something else than a block

}  // namespace

extern "C" {

void fake_memory(size_t bytes) { g_total = bytes; }
size_t fake_used() { return g_used; }
int fake_bad() { return g_bad; }
int fake_batch(pin_plan p) { return p->batch; }
int fake_batch_v(pin_plan p) { return p->batch_v; }
// a caller's own buffer
void* fake_buffer(size_t bytes) {
  void* p = nullptr;
  return hipMalloc(&p, bytes) == hipSuccess ? p : nullptr;
}

hipError_t hipMalloc(void** p, size_t bytes) {
  // address space only: nothing is touched
  if (bytes > g_total - g_used) return hipErrorOutOfMemory;
  static size_t at = size_t(1) << 44;
  *p = reinterpret_cast<void*>(at);
  at += (bytes + 4095) / 4096 * 4096;
  g_blocks[static_cast<char*>(*p)] = bytes;
  g_used += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_blocks.find(static_cast<char*>(p));
  if (it == g_blocks.end()) {
    ++g_bad;
    return hipErrorInvalidValue;
  }
  g_used -= it->second;
  g_blocks.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_bytes, size_t* total) {
  *free_bytes = g_total - g_used;
  *total = g_total;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  auto it = g_blocks.upper_bound(static_cast<char*>(p));
  if (it == g_blocks.begin()) return hipErrorInvalidValue;
  --it;
  *base = it->first;
  *size = it->second;
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t*, unsigned) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t*, hipGraph_t, const hipGraphNode_t*, size_t, const hipKernelNodeParams*) {
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipSuccess; }
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }

}  // extern "C"

namespace pin {

// the launchers of a size: what the kernels would be given has to lie in a block
namespace {

bool inside(const void* p, size_t bytes) {
  hipDeviceptr_t base;
  size_t size;
  return hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) == hipSuccess &&
         static_cast<const char*>(p) + bytes <= static_cast<char*>(base) + size;
}
int g_n = 0;
size_t g_rb = 4;
size_t half() { return (size_t)g_n * g_n * g_n * g_rb; }
void need(const void* p, size_t bytes) {
  if (!inside(p, bytes)) ++g_bad;
}

void prep(const void*, void* g0, double, hipStream_t) { need(g0, half()); }
void xpass(int mode, const void* in, void* out, const void*, const void*, double, int nb, hipStream_t) {
  need(in, half());
  need(out, (mode == 0 ? 3 : 2) * nb * half());
}
void xpass_fwdinv(bool, const void*, void*, const void*, double, hipStream_t) {}
void xpass_lpt3(const void*, void* out, const void*, double, hipStream_t) { need(out, 3 * half()); }
void ypass(int, const void* in, void* out, const void*, int nb, hipStream_t) {
  need(in, nb * half());
  need(out, nb * half());
}
void ypass_hess_grad(const void* in, void* out, void* gout, const void*, int nb, hipStream_t) {
  need(in, 3 * nb * half());
  need(out, 6 * nb * half());
  need(gout, 4 * nb * half());
}
void zcollapse(const CollapseStep& c, hipStream_t) {
  need(c.in, 6 * c.nb * half());
  if (c.gin) need(c.gin, 4 * c.nb * half());
  if (c.groups > 1) need(c.part, (size_t)c.groups * g_n * g_n * g_n * (g_rb + 1));
}
void zpass_store(int, const void*, const void*, void*, hipStream_t) {}
void zpass_mu2(const void*, const void*, void* out, void*, hipStream_t) { need(out, half()); }
void zpass_lpt3(const void*, const void*, const void*, void* out, hipStream_t) { need(out, 4 * half()); }
void grf(void*, uint64_t, const double*, hipStream_t) {}
void reset(void*, uint8_t*, hipStream_t) {}
void redshift(const void*, size_t, const GrowthTables*, void*, hipStream_t) {}
void zero(void*, size_t, hipStream_t) {}
void collapse_points(const void*, size_t, void*, double, hipStream_t) {}

}  // namespace

const SizeOps* find_ops(int n, bool fp64) {
  if (n != 32 && n != 64 && n != 96 && n != 128 && n != 256) return nullptr;
  g_n = n;
  g_rb = fp64 ? 8 : 4;
  static SizeOps ops;
  const auto most = [&](int slots) {
    const size_t fit = ((size_t)256 << 20) / (slots * half());
    return (int)(fit < 1 ? 1 : fit < 16 ? fit : 16);
  };
  ops = SizeOps{n, fp64, prep, xpass, xpass_fwdinv, xpass_lpt3, ypass, ypass_hess_grad, zcollapse, 64, most(9), most(13),
                zpass_store, zpass_mu2, zpass_lpt3, grf, reset, redshift, zero, collapse_points, {}, {}, {}};
  return &ops;
}

void fragment_free(FragWorkspace&) {}
size_t fragment_workspace_bytes(int) { return 0; }
void fragment_prepare(FragWorkspace&, int, double, double, double, double, hipStream_t) {}
int fragment_run(FragWorkspace&, bool, int, const void*, const void*, double, double, const FragParams&, int32_t*, int32_t*,
                 hipStream_t) {
  return 0;
}
int fragment_catalog(FragWorkspace&, double, int32_t*, int32_t*, double*, double*, int, hipStream_t) { return 0; }
int fragment_mergers(FragWorkspace&, double*, int32_t*, int32_t*, int32_t*, int32_t*, int, hipStream_t) { return 0; }

}  // namespace pin
