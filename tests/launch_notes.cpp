// The host side of libfp8lm with a HIP runtime that launches nothing and takes notes instead: device memory is host memory, a
// launch is its kernel's name, its grid and, for a kernel that walks the tensors, the tables it was given.  For tests of what
// is launched, on machines without a GPU.  Compiled for the host only (launch_notes_build.py).
#include "fp8lm.hip"

#include <cstdlib>
#include <map>

namespace {
struct Note {
  std::string kernel;
  unsigned grid;
  bool walks;
  Tables tables;
};
std::vector<Note> notes;
std::map<const void*, std::string> kernels;
struct Launch { dim3 grid, block; size_t shared; hipStream_t stream; } pending;
int compute_units = 256;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* one; return &one; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  pending = {grid, block, shared, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = pending.grid; *block = pending.block; *shared = pending.shared; *stream = pending.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  Note n{kernels[f], grid.x, false, Tables{}};
  n.walks = n.kernel.find("vNS_6TablesE") != std::string::npos;
  if (n.walks) std::memcpy(&n.tables, args[0], sizeof(Tables));
  notes.push_back(n);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) { return (*p = std::malloc(bytes)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t bytes, hipMemcpyKind) { std::memcpy(to, from, bytes); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t bytes) { std::memset(p, v, bytes); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  *p = hipDeviceProp_t{};
  p->multiProcessorCount = compute_units;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = compute_units; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static std::vector<unsigned char> arena(sizeof(StaticArena) + 256);
  *p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(arena.data()) + 255) & ~(uintptr_t)255);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "noted"; }
// nothing here is called by a launch
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipMemAddressReserve(void**, size_t, size_t, void*, unsigned long long) { return hipErrorNotSupported; }
hipError_t hipMemAddressFree(void*, size_t) { return hipErrorNotSupported; }
hipError_t hipMemCreate(hipMemGenericAllocationHandle_t*, size_t, const hipMemAllocationProp*, unsigned long long) { return hipErrorNotSupported; }
hipError_t hipMemRelease(hipMemGenericAllocationHandle_t) { return hipErrorNotSupported; }
hipError_t hipMemGetAllocationGranularity(size_t*, const hipMemAllocationProp*, hipMemAllocationGranularity_flags) { return hipErrorNotSupported; }
hipError_t hipMemMap(void*, size_t, size_t, hipMemGenericAllocationHandle_t, unsigned long long) { return hipErrorNotSupported; }
hipError_t hipMemUnmap(void*, size_t) { return hipErrorNotSupported; }
hipError_t hipMemSetAccess(void*, size_t, const hipMemAccessDesc*, size_t) { return hipErrorNotSupported; }

// ---- reading the notes --------------------------------------------------------------------------
int notes_count() { return (int)notes.size(); }
void notes_clear() { notes.clear(); }
const char* notes_kernel(int i) { return notes[i].kernel.c_str(); }
// grid; then, for a kernel that walks: 1, unit_elems, unit_shift, one_unit, deferred, n_chunks
void notes_launch(int i, int64_t* out) {
  const Note& n = notes[i];
  const int64_t v[7] = {n.grid, n.walks, n.tables.unit_elems, n.tables.unit_shift, n.tables.one_unit, n.tables.deferred, n.tables.n_chunks};
  std::memcpy(out, v, sizeof(v));
}
}  // extern "C"
