// The few HIP runtime functions that the host code of the library calls, as recorders: linked with the host halves of the
// sources alone they make a library whose entry points run on any machine and launch nothing. What they would have launched
// (kernel, grid, workgroup, dynamic LDS and the kernel's LDS limit at that moment) is read through launch_record(). Built by
// paper_2602_11562_amd.build.build_launch_recorder(), used by tests/test_launches_cpu.py.
#ifndef _GNU_SOURCE
#define _GNU_SOURCE
#endif
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <map>
#include <vector>

struct LaunchRecord {
  const char* kernel;
  unsigned grid, block;
  unsigned long long lds;
  int limit;   // what hipFuncSetAttribute last set for the kernel, -1: never called
};

static std::vector<LaunchRecord> records;
static std::map<const void*, int> limits;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } pending;

extern "C" {

// (no device code is there to register)
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}

int launch_count() { return (int)records.size(); }
void launch_clear() { records.clear(); }
const LaunchRecord* launch_record(int i) { return &records[i]; }

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  pending = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = pending.grid;
  *block = pending.block;
  *lds = pending.lds;
  *stream = pending.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  Dl_info info;
  const auto at = limits.find(f);
  records.push_back({dladdr(f, &info) && info.dli_sname ? info.dli_sname : "", grid.x, block.x, lds,
                     at == limits.end() ? -1 : at->second});
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value) {
  limits[f] = value;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* device) {
  *device = 0;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  *p = const_cast<void*>(symbol);
  return hipSuccess;
}

}  // extern "C"
