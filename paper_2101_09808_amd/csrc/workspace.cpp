// Device memory of the compute calls (host code): the stream-ordered pool and
// the workspaces kept per stream.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "conv_internal.h"

namespace convfwd {

// Workspaces come from a memory pool the library owns, one per device,
// which keeps up to 1 GB of freed blocks for reuse (the default pool hands
// freed memory back at each synchronisation, so every call would map fresh
// pages).  The calling thread's current device must own the stream.
int stream_alloc(size_t bytes, void* stream, void** out) {
  static std::mutex mu;
  static hipMemPool_t pools[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CONV_EHIP;
  hipMemPool_t pool = nullptr;
  {
    std::lock_guard<std::mutex> lk(mu);
    if (!pools[dev]) {
      hipMemPoolProps props = {};
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      hipMemPool_t p = nullptr;
      if (hipMemPoolCreate(&p, &props) != hipSuccess) return CONV_EHIP;
      uint64_t keep = uint64_t(1) << 30;
      if (hipMemPoolSetAttribute(p, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) return CONV_EHIP;
      pools[dev] = p;
    }
    pool = pools[dev];
  }
  return hipMallocFromPoolAsync(out, bytes, pool, reinterpret_cast<hipStream_t>(stream)) == hipSuccess ? CONV_OK
                                                                                                      : CONV_EHIP;
}

int stream_free(void* p, void* stream) {
  return hipFreeAsync(p, reinterpret_cast<hipStream_t>(stream)) == hipSuccess ? CONV_OK : CONV_EHIP;
}

bool stream_capturing(void* stream) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(reinterpret_cast<hipStream_t>(stream), &cs) != hipSuccess) {
    (void)hipGetLastError();  // (not this call's error to report)
    return true;
  }
  return cs != hipStreamCaptureStatusNone;
}

namespace {
// Workspaces kept per (device, stream, nesting level): the kernels of the
// calls on one stream run in stream order, so a call can reuse the buffer
// the previous call on that stream used.  A buffer grows by a new allocation
// and a stream-ordered free; while another host thread holds it, a call takes
// a fresh stream-ordered allocation instead.
//
// A call that is captured hands the kept buffer's address to the graph, so
// that buffer is not freed when a later, larger call needs more: it is
// retained, and the new one is at least twice its size, which bounds the
// retained ones by the kept one.  A captured call that needs more than is
// kept allocates and frees within the graph, and keeps nothing.
struct CachedWorkspace {
  void* ptr = nullptr;
  size_t size = 0;
  bool busy = false;
  bool captured = false;        // a graph holds its address
  std::vector<void*> retained;  // earlier buffers that graphs hold
};
std::mutex g_ws_mu;
std::map<std::tuple<int, void*, int>, CachedWorkspace> g_ws;

// The arena of the calling thread's allocation-free call, if one is running.
thread_local ScratchArena* t_arena = nullptr;

// Grows the kept buffer.  If both buffers do not fit at once, a call that
// needs the larger one (`must`) gives the smaller back first; otherwise the
// smaller one stays.  No error of an attempt is left for the runtime to report.
int grow_kept(CachedWorkspace& c, size_t bytes, bool must, void* stream) {
  if (c.size >= bytes) return CONV_OK;
  const size_t want = c.captured ? std::max(bytes, 2 * c.size) : bytes;
  const size_t sz = (want + (size_t(1) << 20) - 1) >> 20 << 20;  // whole MiB
  void* p = nullptr;
  if (stream_alloc(sz, stream, &p) != CONV_OK) {
    (void)hipGetLastError();
    if (!must || !c.ptr || c.captured) return CONV_EHIP;
    if (stream_free(c.ptr, stream) != CONV_OK) return CONV_EHIP;
    c.ptr = nullptr;
    c.size = 0;
    if (stream_alloc(sz, stream, &p) != CONV_OK) {
      (void)hipGetLastError();
      return CONV_EHIP;
    }
  }
  void* const old = c.ptr;
  const bool held = c.captured;
  c.ptr = p;
  c.size = sz;
  c.captured = false;
  if (held) c.retained.push_back(old);
  else if (old) return stream_free(old, stream);
  return CONV_OK;
}
}  // namespace

void set_thread_arena(ScratchArena* a) { t_arena = a; }

void workspace_reserve(int level, size_t bytes, void* stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return;
  std::lock_guard<std::mutex> lk(g_ws_mu);
  CachedWorkspace& c = g_ws[std::make_tuple(dev, stream, level)];
  if (!c.busy) (void)grow_kept(c, bytes, false, stream);
}

int workspace_acquire(int level, size_t bytes, void* stream, Workspace* w) {
  w->cached = false;
  w->arena = false;
  w->level = level;
  if (t_arena) {
    // bump allocation from the caller's scratch, 256-byte aligned
    const size_t off = (t_arena->used + 255) / 256 * 256;
    if (off > t_arena->cap || bytes > t_arena->cap - off) return CONV_ESCRATCH;
    w->ptr = t_arena->base + off;
    w->arena = true;
    t_arena->used = off + bytes;
    return CONV_OK;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CONV_EHIP;
  const bool capturing = stream_capturing(stream);
  {
    std::lock_guard<std::mutex> lk(g_ws_mu);
    CachedWorkspace& c = g_ws[std::make_tuple(dev, stream, level)];
    if (!c.busy && (!capturing || c.size >= bytes)) {
      if (grow_kept(c, bytes, true, stream) != CONV_OK) return CONV_EHIP;
      c.busy = true;
      if (capturing) c.captured = true;
      w->ptr = c.ptr;
      w->cached = true;
      return CONV_OK;
    }
  }
  return stream_alloc(bytes, stream, &w->ptr);
}

int workspace_release(const Workspace& w, void* stream) {
  if (w.arena) return CONV_OK;
  if (!w.cached) return stream_free(w.ptr, stream);
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CONV_EHIP;
  std::lock_guard<std::mutex> lk(g_ws_mu);
  g_ws[std::make_tuple(dev, stream, w.level)].busy = false;
  return CONV_OK;
}

int workspace_release_stream(void* stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CONV_EHIP;
  std::lock_guard<std::mutex> lk(g_ws_mu);
  int rc = CONV_OK;
  for (auto it = g_ws.begin(); it != g_ws.end();) {
    CachedWorkspace& c = it->second;
    if (std::get<0>(it->first) == dev && std::get<1>(it->first) == stream && !c.busy) {
      if (c.ptr) c.retained.push_back(c.ptr);
      for (void* p : c.retained)
        if (stream_free(p, stream) != CONV_OK) rc = CONV_EHIP;
      it = g_ws.erase(it);
    } else {
      ++it;
    }
  }
  return rc;
}

}  // namespace convfwd
