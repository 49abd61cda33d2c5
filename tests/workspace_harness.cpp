// A recording stand-in for the HIP calls of csrc/workspace.cpp, so that the
// rules of the kept workspaces run without a GPU.  Memory is numbered, never
// touched; streams are any non-null values.
#include <hip/hip_runtime_api.h>

#include <map>

#include "conv_internal.h"

namespace {
std::map<void*, size_t> live;  // allocations not freed
size_t room = ~size_t(0);      // bytes that all live allocations may take
bool capturing = false;
int last_error = 0, graph_allocs = 0, graph_frees = 0, bad_frees = 0;
uintptr_t next_ptr = 0x100000;
size_t used() {
  size_t s = 0;
  for (const auto& a : live) s += a.second;
  return s;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) {
  return *p = reinterpret_cast<hipMemPool_t>(1), hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** out, size_t bytes, hipMemPool_t, hipStream_t) {
  if (bytes > room || used() > room - bytes) {
    last_error = hipErrorOutOfMemory;
    return hipErrorOutOfMemory;
  }
  *out = reinterpret_cast<void*>(next_ptr);
  next_ptr += 0x1000;
  live[*out] = bytes;
  graph_allocs += capturing;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
  bad_frees += live.erase(p) == 0;
  graph_frees += capturing;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return static_cast<hipError_t>(e);
}

// One call's use of a workspace: its address, or 0 if it could not be had.
uint64_t t_call(int level, uint64_t bytes, uint64_t stream) {
  convfwd::Workspace w;
  void* st = reinterpret_cast<void*>(stream);
  if (convfwd::workspace_acquire(level, bytes, st, &w) != CONV_OK) return 0;
  const uint64_t p = reinterpret_cast<uint64_t>(w.ptr);
  return convfwd::workspace_release(w, st) == CONV_OK ? p : 0;
}
void t_reserve(int level, uint64_t bytes, uint64_t stream) {
  convfwd::workspace_reserve(level, bytes, reinterpret_cast<void*>(stream));
}
int t_release(uint64_t stream) { return convfwd::workspace_release_stream(reinterpret_cast<void*>(stream)); }
void t_capturing(int on) { capturing = on != 0; }
void t_room(uint64_t bytes) { room = bytes; }
int t_live(uint64_t p) { return live.count(reinterpret_cast<void*>(p)) != 0; }
uint64_t t_used() { return used(); }
int t_last_error() { return last_error; }
int t_graph_allocs() { return graph_allocs; }
int t_graph_frees() { return graph_frees; }
int t_bad_frees() { return bad_frees; }
}
