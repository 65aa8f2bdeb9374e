// A small host model of the HIP runtime calls the library makes: streams and
// events are heap objects (a use after destroy is a heap-use-after-free for
// AddressSanitizer), stream capture follows the fork/join rules of the real
// runtime (a stream joins a capture by waiting on an event recorded in it; all
// forked work must be joined back before the capture ends; synchronising or
// destroying a capturing stream is an error), and device memory is host memory
// of the exact size asked for.
#include "hip_stub.h"

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <unordered_set>
#include <vector>

struct ihipStream_t {
  unsigned magic = 0x57AEA3u;
  ihipStream_t* origin = nullptr;         // capture this stream belongs to (itself for the origin)
  std::set<ihipStream_t*> forked;         // origin only: streams that joined its capture
  std::set<ihipStream_t*> unjoined;       // origin only: forked streams with work not yet joined back
  long last_work = 0;                     // sequence number of the last work enqueued
  long finished = 0;                      // and of the last that the host has waited for
};
struct ihipEvent_t {
  unsigned magic = 0xE7E27u;
  ihipStream_t* origin = nullptr;         // capture the last record belongs to
  ihipStream_t* from = nullptr;           // stream of the last record
  long seq = 0;
  bool recorded = false;
  bool reached = false;                   // the last record is known to have been reached
};

namespace {
int g_cu = 256;
bool g_tensor_checks = true;
bool g_strict_destroy = false;
int g_violations = 0;
long g_launches = 0, g_nodes = 0, g_seq = 0;
std::map<std::string, long> g_launches_of;
long g_streams = 0;                        // created by the library
int g_captures = 0;                        // captures in progress
std::map<const char*, size_t> g_allocs;
// Copies out of page-locked memory (or kernels that read it): the model makes them at once, the device at any time until an event
// behind them is known to have been reached, so their source must not change before that.
struct PendingCopy {
  const char* src;
  std::vector<char> bytes;
  ihipStream_t* stream;
  long seq;
};
std::vector<PendingCopy> g_pending;
struct Wait { long at; ihipStream_t* from; long seq; };   // work enqueued after `at` runs behind what `from` had been given by `seq`
std::map<ihipStream_t*, std::vector<Wait>> g_waits;
std::map<const char*, size_t> g_pinned;
ihipStream_t g_null_stream;               // the default stream

ihipStream_t* resolve(hipStream_t s) { return s ? s : &g_null_stream; }
bool alive(ihipStream_t* s) { return s->magic == 0x57AEA3u; }   // reads the object: ASan reports a freed one
bool alive(ihipEvent_t* e) { return e->magic == 0xE7E27u; }

bool pinned(const char* p) {
  auto it = g_pinned.upper_bound(p);
  if (it == g_pinned.begin()) return false;
  --it;
  return p < it->first + it->second;
}
// The copies of `stream` (nullptr: of every stream) up to `seq` are over, and with them those that `stream` has waited for.
void copies_made(ihipStream_t* stream, long seq) {
  for (size_t i = 0; i < g_pending.size();) {
    const PendingCopy& c = g_pending[i];
    if ((stream && c.stream != stream) || c.seq > seq) {
      ++i;
      continue;
    }
    if (std::memcmp(c.src, c.bytes.data(), c.bytes.size()) != 0) stub::violation("the source of a copy changed before the copy was made");
    g_pending.erase(g_pending.begin() + i);
  }
  const auto it = g_waits.find(stream);
  if (it != g_waits.end())
    for (const Wait& w : it->second)   // (their sequence numbers descend: this ends)
      if (w.at <= seq) copies_made(w.from, w.seq);
}

void work_on(ihipStream_t* s) {
  s->last_work = ++g_seq;
  if (s->origin && s->origin != s) s->origin->unjoined.insert(s);
}
}  // namespace

namespace stub {

void violation(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::fprintf(stderr, "hip model violation: ");
  std::vfprintf(stderr, fmt, ap);
  std::fprintf(stderr, "\n");
  va_end(ap);
  ++g_violations;
}
int violations() { return g_violations; }
long launches() { return g_launches; }
long captured_nodes() { return g_nodes; }
long streams_created() { return g_streams; }
long launches_of(const char* what) { return g_launches_of[what]; }
void set_compute_units(int n) { g_cu = n; }

namespace {
std::unordered_set<const void*> g_out_rows;
long g_tiles = 0;
}
void new_forward() {
  g_out_rows.clear();
  g_tiles = 0;
}
void note_tiles(long n) { g_tiles += n; }
long tiles_walked() { return g_tiles; }
void note_out_row(const void* row) {
  if (!g_out_rows.insert(row).second) violation("an output row is stored twice in one forward pass (launch %ld)", launches());
}
size_t out_rows_written() { return g_out_rows.size(); }
void set_tensor_checks(bool on) { g_tensor_checks = on; }
void set_strict_destroy(bool on) { g_strict_destroy = on; }
bool tensor_checks() { return g_tensor_checks; }

void* device_alloc(size_t bytes) {
  char* p = static_cast<char*>(std::malloc(bytes ? bytes : 1));
  std::memset(p, 0xCD, bytes);
  g_allocs[p] = bytes;
  return p;
}
void device_free(void* p) {
  g_allocs.erase(static_cast<const char*>(p));
  std::free(p);
}
bool in_device(const void* p, size_t bytes) {
  const char* c = static_cast<const char*>(p);
  auto it = g_allocs.upper_bound(c);
  if (it == g_allocs.begin()) return false;
  --it;
  return c >= it->first && c + bytes <= it->first + it->second;
}

hipStream_t create_stream() { return new ihipStream_t(); }
void destroy_stream(hipStream_t s) { (void)hipStreamDestroy(s); }

void begin_capture(hipStream_t s) {
  ihipStream_t* st = resolve(s);
  if (st->origin) violation("begin_capture on a stream that is already capturing");
  st->origin = st;
  st->forked.clear();
  st->unjoined.clear();
  ++g_captures;
}

hipError_t end_capture(hipStream_t s) {
  ihipStream_t* st = resolve(s);
  if (st->origin != st) {
    violation("end_capture on a stream that is not the origin of a capture");
    return hipErrorInvalidValue;
  }
  const bool unjoined = !st->unjoined.empty();
  for (ihipStream_t* f : st->forked)
    if (alive(f)) f->origin = nullptr;
  st->forked.clear();
  st->unjoined.clear();
  st->origin = nullptr;
  --g_captures;
  if (unjoined) violation("capture ended with forked work that was not joined back");
  return unjoined ? hipErrorStreamCaptureUnjoined : hipSuccess;
}

void note_launch(hipStream_t s, const char* what) {
  ihipStream_t* st = resolve(s);
  if (!alive(st)) violation("launch of %s on a dead stream", what);
  ++g_launches;
  ++g_launches_of[what];
  if (st->origin) ++g_nodes;
  work_on(st);
}

void note_pinned_read(hipStream_t s, const void* src, size_t bytes) {
  const char* c = static_cast<const char*>(src);
  if (!pinned(c) || !pinned(c + bytes - 1)) violation("a copy reads %zu bytes that are not all page-locked", bytes);
  g_pending.push_back({c, std::vector<char>(c, c + bytes), resolve(s), ++g_seq});
}

}  // namespace stub

hipError_t hipGetDevice(int* device) {
  if (g_cu <= 0) return hipErrorUnknown;   // a box without a GPU
  *device = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t attr, int) {
  if (attr != hipDeviceAttributeMultiprocessorCount) return hipErrorInvalidValue;
  *value = g_cu;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }

hipError_t hipStreamCreateWithFlags(hipStream_t* stream, unsigned) {
  ++g_streams;
  *stream = new ihipStream_t();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t stream) {
  if (!stream) return hipErrorInvalidResourceHandle;
  if (!alive(stream)) stub::violation("hipStreamDestroy of a dead stream");
  if (stream->origin) stub::violation("hipStreamDestroy of a stream that is capturing");
  if (g_strict_destroy && stream->last_work > stream->finished) stub::violation("hipStreamDestroy of a stream whose work may be under way");
  copies_made(stream, g_seq);   // what it holds is finished first
  g_waits.erase(stream);
  stream->magic = 0;
  delete stream;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t stream) {
  ihipStream_t* st = resolve(stream);
  if (!alive(st)) stub::violation("hipStreamSynchronize on a dead stream");
  if (st->origin) {
    stub::violation("hipStreamSynchronize on a capturing stream");
    return hipErrorStreamCaptureUnsupported;
  }
  copies_made(st, g_seq);
  st->finished = g_seq;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  if (g_captures > 0) {
    stub::violation("hipDeviceSynchronize while a capture is active");
    return hipErrorStreamCaptureUnsupported;
  }
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus* status) {
  ihipStream_t* st = resolve(stream);
  if (!alive(st)) stub::violation("hipStreamIsCapturing on a dead stream");
  *status = st->origin ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* event, unsigned) {
  *event = new ihipEvent_t();
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t event) {
  if (!event) return hipErrorInvalidResourceHandle;
  if (!alive(event)) stub::violation("hipEventDestroy of a dead event");
  event->magic = 0;
  delete event;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t event, hipStream_t stream) {
  ihipStream_t* st = resolve(stream);
  if (!event || !alive(event) || !alive(st)) {
    stub::violation("hipEventRecord with a dead handle");
    return hipErrorInvalidResourceHandle;
  }
  event->origin = st->origin;
  event->from = st;
  event->seq = ++g_seq;
  event->recorded = true;
  event->reached = false;
  return hipSuccess;
}
// Never ready by itself: what the host may do early it must be able to do late.
hipError_t hipEventQuery(hipEvent_t event) {
  if (!event || !alive(event)) stub::violation("hipEventQuery with a dead handle");
  return !event->recorded || event->reached ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t event) {
  if (!event || !alive(event)) stub::violation("hipEventSynchronize with a dead handle");
  if (event->recorded && event->origin) stub::violation("hipEventSynchronize on an event of a capture");
  if (event->recorded) copies_made(event->from, event->seq);
  event->reached = true;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** ptr, size_t bytes, unsigned) {
  if (g_captures > 0) stub::violation("hipHostMalloc while a capture is active");
  *ptr = std::malloc(bytes);
  g_pinned[static_cast<const char*>(*ptr)] = bytes;
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** device_ptr, void* host_ptr, unsigned) {
  *device_ptr = host_ptr;
  return pinned(static_cast<const char*>(host_ptr)) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipHostFree(void* ptr) {
  copies_made(nullptr, g_seq);   // the real call waits for the device
  g_pinned.erase(static_cast<const char*>(ptr));
  std::free(ptr);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t event, unsigned) {
  ihipStream_t* st = resolve(stream);
  if (!event || !alive(event) || !alive(st)) {
    stub::violation("hipStreamWaitEvent with a dead handle");
    return hipErrorInvalidResourceHandle;
  }
  if (!event->recorded) return hipSuccess;
  if (!event->origin && !g_pending.empty()) g_waits[st].push_back({++g_seq, event->from, event->seq});
  if (event->origin) {
    ihipStream_t* o = event->origin;
    if (!alive(o) || o->origin != o) {
      stub::violation("wait on an event recorded in a capture that has ended");
      return hipErrorStreamCaptureIsolation;
    }
    if (st->origin && st->origin != o) {
      stub::violation("a stream of one capture waits on an event of another");
      return hipErrorStreamCaptureIsolation;
    }
    if (!st->origin) {   // joins the capture
      st->origin = o;
      o->forked.insert(st);
    }
    // the origin (or any stream of the capture) waiting on a forked stream's event joins that
    // stream's work up to the record
    ihipStream_t* f = event->from;
    if (f != o && f != st && alive(f) && f->last_work <= event->seq) o->unjoined.erase(f);
  } else if (st->origin) {
    stub::violation("a capturing stream waits on an event recorded outside the capture");
    return hipErrorStreamCaptureIsolation;
  }
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t stream) {
  ihipStream_t* st = resolve(stream);
  if (!alive(st)) stub::violation("hipMemcpyAsync on a dead stream");
  if (st->origin) stub::violation("hipMemcpyAsync recorded into a capture (the forward pass promises launches only)");
  if (kind == hipMemcpyHostToDevice && !stub::in_device(dst, bytes)) stub::violation("H2D copy outside a device allocation");
  if (kind == hipMemcpyDeviceToHost && !stub::in_device(src, bytes)) stub::violation("D2H copy outside a device allocation");
  std::memcpy(dst, src, bytes);
  if (kind == hipMemcpyHostToDevice && pinned(static_cast<const char*>(src))) stub::note_pinned_read(stream, src, bytes);
  return hipSuccess;
}
