#include "host_hip.h"

#include <stdlib.h>
#include <string.h>

#include <algorithm>

FakeHip fake;

namespace {
struct Block {
  size_t bytes, cleared;  // cleared: from its start on
};
std::map<uintptr_t, Block> blocks;
uintptr_t next_address = (uintptr_t)1 << 40;
hipError_t last = hipSuccess;
bool capturing = false;
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
hipError_t done(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
std::map<uintptr_t, Block>::iterator find(const void* p) {
  auto it = blocks.upper_bound((uintptr_t)p);
  if (it == blocks.begin()) return blocks.end();
  --it;
  return (uintptr_t)p < it->first + it->second.bytes ? it : blocks.end();
}
hipError_t clear(void* p, int v, size_t n) {
  auto it = find(p);
  if (it == blocks.end() || v != 0) return hipSuccess;
  const size_t at = (uintptr_t)p - it->first;
  if (at + n > it->second.bytes) return done(hipErrorInvalidValue);
  if (at <= it->second.cleared) it->second.cleared = std::max(it->second.cleared, at + n);
  return hipSuccess;
}
struct Call {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} pushed;
}  // namespace

bool FakeHip::cleared(const void* p, size_t bytes) const {
  auto it = find(p);
  return it != blocks.end() && (uintptr_t)p - it->first + bytes <= it->second.cleared;
}
size_t FakeHip::live() const { return blocks.size(); }

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* m = nullptr;
  return &m;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  pushed = Call{grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = pushed.grid;
  *block = pushed.block;
  *shared = pushed.shared;
  *s = pushed.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  const Launch l{names()[f], grid.x, block.x, args};
  fake.launches[l.kernel] += 1;
  if (grid.x == 0 || (uint64_t)grid.x * block.x >= (uint64_t)1 << 32) {
    fake.too_large.push_back(l.kernel);
    return done(hipErrorInvalidConfiguration);
  }
  if (fake.on_launch) fake.on_launch(l);
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  const long k = fake.allocations++;
  if (k == fake.fail_at || n > fake.most) {
    fake.refused += 1;
    *p = nullptr;
    return done(hipErrorOutOfMemory);
  }
  blocks[next_address] = Block{n, 0};
  *p = (void*)next_address;
  next_address += (n + 4095) / 4096 * 4096 + 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (p && !blocks.erase((uintptr_t)p)) return done(hipErrorInvalidValue);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = nullptr;
  if (!scratch) {
    blocks[next_address] = Block{(size_t)1 << 30, 0};
    scratch = (void*)next_address;
    next_address += (size_t)1 << 31;
  }
  *p = scratch;
  return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) { return clear(p, v, n); }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return clear(p, v, n); }
hipError_t hipMemcpy(void* d, const void*, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) memset(d, 0, n);
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "an error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;  // compute units
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 8;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  fake.waits += 1;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  if (capturing) return done(hipErrorIllegalState);
  capturing = true;
  fake.captures += 1;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  capturing = false;
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  fake.replays += 1;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)1;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
}
