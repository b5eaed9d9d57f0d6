// The kept device blocks on a host model of streams: csrc/devmem.hip compiled with a
// runtime that runs nothing and only tracks order. Every use of a buffer on a stream
// is a numbered item of that stream; a stream "knows" the items of the others that are
// ordered ahead of what it queues next (by events and by waits of the host). A block
// handed out while an item that uses it is not known to the new stream is a race.
//
// usage: devmem_host SCENARIO; prints "ok" or the faults found.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <unistd.h>

#include <chrono>
#include <functional>
#include <future>
#include <map>
#include <memory>
#include <thread>

#include "../paper_2505_08174_amd/csrc/devmem.hip"

namespace model {
using Clock = std::map<hipStream_t, int>;   // items of each stream that are known
struct Stream {
  int device = 0, items = 0;
  bool capturing = false;
  Clock knows;
};
struct Mem {
  size_t bytes;
  int device;
  bool freed = false, graph = false;   // graph: allocated in a capture
  Clock uses;   // last item of each stream that uses it
};
std::map<hipStream_t, Stream> streams = {{nullptr, Stream{}}};   // and the null stream
std::map<void*, Mem> mem;
std::map<hipEvent_t, Clock> events;
int current = 0, bad = 0, mallocs = 0;
bool no_host_memory = false;
size_t live[2] = {0, 0}, total = (size_t)64 << 20;
std::function<void()> after_wait;   // another thread, between a wait of this one and what follows

std::function<void()> other;   // what another thread does while the runtime is busy
void fault(const char* what);
void meanwhile() {
  if (!other) return;
  auto f = other;
  other = nullptr;
  auto done = std::make_shared<std::promise<void>>();
  std::thread([f, done] {
    f();
    done->set_value();
  }).detach();
  if (done->get_future().wait_for(std::chrono::seconds(10)) != std::future_status::ready) {
    fault("another device's thread has to wait");
    printf("\n");
    fflush(stdout);
    _exit(1);
  }
}

void fault(const char* what) {
  printf("%s\n", what);
  ++bad;
}
hipStream_t stream(long id, int device = 0) {
  hipStream_t s = (hipStream_t)id;
  streams[s].device = device;
  return s;
}
void merge(Clock& to, const Clock& from) {
  for (auto& k : from) to[k.first] = std::max(to[k.first], k.second);
}
Clock tail(hipStream_t s) {
  Clock c = streams[s].knows;
  c[s] = streams[s].items;
  return c;
}
void host_knows(const Clock& c) {
  for (auto& s : streams) merge(s.second.knows, c);
}
// the work of this buffer that is not ahead of what stream s queues next
bool pending(const Mem& m, hipStream_t s) {
  for (auto& u : m.uses)
    if (u.first != s && u.second > streams[s].knows[u.first]) return true;
  return false;
}
void use(const DevBuf& b, hipStream_t s) {
  Mem& m = mem[b.p];
  if (m.freed) fault("use of freed memory");
  if (m.graph && !streams[s].capturing) fault("a graph's memory is used outside it");
  if (pending(m, s)) fault("a block is used on a stream that its earlier work is not ahead of");
  m.uses[s] = ++streams[s].items;
}
void drop(void* p, hipStream_t s, bool wait) {
  Mem& m = mem[p];
  if (m.freed) fault("memory freed twice");
  if (!wait && pending(m, s)) fault("memory returned while its work may be running");
  m.freed = true;
  live[m.device] -= m.bytes;
}
}  // namespace model

void* operator new(size_t n) {
  void* p = model::no_host_memory ? nullptr : malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

// ------------------------------------------------------------ the runtime calls
extern "C" {
hipError_t hipGetDevice(int* d) {
  *d = model::current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  model::current = d;
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* fr, size_t* tot) {
  *tot = model::total;
  *fr = model::total - model::live[model::current];
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) {
  model::meanwhile();
  const int dev = s ? model::streams[s].device : model::current;
  const bool graph = model::streams[s].capturing;
  if (model::live[dev] + n > model::total) return hipErrorOutOfMemory;
  static uintptr_t next = 1 << 20;
  *p = (void*)(next += 256);
  model::mem[*p] = model::Mem{n, dev, false, graph, {}};
  model::live[dev] += n;
  ++model::mallocs;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t s) {
  // the null stream of the current device, not of the memory's
  if (!s && model::mem[p].device != model::current) model::fault("memory freed on another device");
  model::drop(p, s, false);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  model::meanwhile();
  model::host_knows(model::tail(s));
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* cs) {
  *cs = model::streams[s].capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (model::streams[s].capturing) model::fault("an event outside the graph in a capture");
  model::events[e] = model::tail(s);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (model::streams[s].capturing) model::fault("a wait for work outside the graph in a capture");
  model::merge(model::streams[s].knows, model::events[e]);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
  model::meanwhile();
  model::Clock c;
  for (auto& s : model::streams)
    if (s.second.device == model::current) model::merge(c, model::tail(s.first));
  model::host_knows(c);
  return hipSuccess;
}
}

// ------------------------------------------------------------------ scenarios
using model::stream;
using model::use;

static hh_ctx_s* context(hipStream_t s, int device = 0) {
  hh_ctx_s* c = new hh_ctx_s();
  c->device = device;
  c->stream = s;
  model::current = device;
  devmem_attach(c);
  return c;
}
static void destroy(hh_ctx_s* c) {
  model::current = c->device;
  const bool waited = devmem_wait(c);
  if (model::after_wait) model::after_wait();
  model::after_wait = nullptr;
  devmem_detach(c, waited);
  delete c;
}
static void set_stream(hh_ctx_s* c, hipStream_t s) { devmem_restream(c, s); }

// No host memory for the lists while a buffer is freed (handles are freed by calls that
// cannot report an error): nothing is thrown, and the memory goes back.
static void no_host_memory() {
  hipStream_t S = stream(1);
  hh_ctx_s* x = context(S);
  DevBuf a;
  a.alloc(x, 4096);
  use(a, S);
  model::no_host_memory = true;
  a.release();
  model::no_host_memory = false;
  if (model::live[0] != 0) model::fault("the buffer's memory is lost");
  destroy(x);
}

// Another thread frees a buffer with work queued while a context is destroyed, between
// that context's wait and the return of its blocks; a third stream allocates. With two
// contexts on one stream, and with streams of their own where the destroyed context
// has changed its stream.
static void destroy_race(bool same_stream) {
  hipStream_t S = stream(1), T = stream(2), V = stream(3);
  hh_ctx_s *x = context(S), *y = context(same_stream ? S : V), *z = context(T);
  if (!same_stream) set_stream(x, stream(4));
  DevBuf a, b;
  a.alloc(y, 4096);
  model::after_wait = [&] {
    use(a, y->stream);
    a.release();
  };
  destroy(x);
  b.alloc(z, 4096);
  use(b, T);
  b.release();
  destroy(y);
  destroy(z);
}

// A buffer made on one stream, used on another after the context went there, and freed:
// neither a second context on the first stream nor the same one back there may be
// ahead of that use.
static void restream() {
  hipStream_t A = stream(1), B = stream(2);
  hh_ctx_s *x = context(A), *y = context(A);
  DevBuf a, b, c;
  a.alloc(x, 4096);
  use(a, A);
  set_stream(x, B);
  use(a, B);
  a.release();
  b.alloc(y, 4096);
  use(b, A);
  b.release();
  set_stream(x, A);
  c.alloc(x, 4096);
  use(c, A);
  c.release();
  destroy(x);
  destroy(y);
}

// The same through a stream in capture: nothing is ordered in it, and the stream after
// it comes behind the one before it.
static void restream_capture() {
  hipStream_t A = stream(1), S = stream(2), B = stream(3);
  hh_ctx_s *x = context(A), *y = context(B);
  DevBuf a, b, c;
  a.alloc(x, 4096);
  use(a, A);
  model::streams[S].capturing = true;
  set_stream(x, S);
  a.release();
  b.alloc(y, 4096);
  use(b, B);
  b.release();
  model::streams[S].capturing = false;
  set_stream(x, B);
  c.alloc(y, 4096);
  use(c, B);
  b.alloc(x, 4096);
  use(b, B);
  b.release();
  c.release();
  set_stream(x, S);
  destroy(x);
  destroy(y);
}

// Above the limit the largest blocks go back to the runtime, with kernels that use them
// still queued and another device current; those of a context elsewhere stay.
static void trim_other_device() {
  hipStream_t S = stream(1), T = stream(2), V = stream(3, 1);
  hh_ctx_s *x = context(S), *y = context(T), *z = context(V, 1);
  const size_t big = (size_t)14 << 20;   // the limit is 25.6 MiB
  DevBuf a, b, c;
  a.alloc(y, big);
  use(a, T);
  b.alloc(x, big);
  use(b, S);
  c.alloc(x, 4096);
  use(c, S);
  model::current = 1;
  a.release();
  b.release();
  c.release();
  if (model::live[0] > model::total * 4 / 10) model::fault("more is kept than the limit");
  destroy(x);
  destroy(y);
  destroy(z);
  if (model::live[0] + model::live[1] != 0) model::fault("memory is left after the last context");
}

// While one device's thread allocates, and while it returns its kept blocks after a
// failed allocation, which waits for their work, another device's thread allocates and
// frees; and the failed allocation succeeds then.
static void other_device_goes_on() {
  hipStream_t S = stream(1), T = stream(2), V = stream(3, 1);
  hh_ctx_s *x = context(S), *y = context(T), *z = context(V, 1);
  DevBuf a, b, c, d;
  a.alloc(z, 4096);
  const auto step = [&] {
    d.alloc(z, 4096);
    d.release();
  };
  a.release();
  model::current = 0;
  model::other = step;
  b.alloc(x, (size_t)20 << 20);
  use(b, S);
  b.release();
  b.alloc(y, (size_t)20 << 20);
  use(b, T);
  model::other = nullptr;
  model::mallocs = 0;
  hipMallocAsync(&a.p, 20 << 20, S);   // the caller's own memory
  model::other = step;
  c.alloc(y, (size_t)24 << 20);
  use(c, T);
  if (model::other) model::fault("no allocation failed");
  hipFreeAsync(a.p, S);
  a.p = nullptr;
  for (DevBuf* f : {&b, &c}) f->release();
  destroy(x);
  destroy(y);
  destroy(z);
  if (model::live[0] + model::live[1] != 0) model::fault("memory is left after the last context");
}

// A buffer allocated in a capture (the first product of a handle, recorded) is not
// handed out after it.
static void graph_memory() {
  hipStream_t S = stream(1), G = stream(2);
  hh_ctx_s* x = context(S);
  DevBuf a, b;
  model::streams[G].capturing = true;
  set_stream(x, G);
  a.alloc(x, 4096);
  use(a, G);
  model::streams[G].capturing = false;
  set_stream(x, S);
  a.release();
  b.alloc(x, 4096);
  use(b, S);
  b.release();
  destroy(x);
}

// A context that stays on the stream after its capture: what it allocates there then
// comes behind its work on the stream before.
static void stay_after_capture() {
  hipStream_t A = stream(1), S = stream(2);
  hh_ctx_s* x = context(A);
  DevBuf a, b;
  a.alloc(x, 4096);
  use(a, A);
  model::streams[S].capturing = true;
  set_stream(x, S);
  a.release();
  model::streams[S].capturing = false;
  b.alloc(x, 4096);
  use(b, S);
  b.release();
  destroy(x);
}

// A context's own blocks come back to it at once, to another context on its stream,
// and to any once it was destroyed: no allocation after the first.
static void reuse() {
  hipStream_t S = stream(1), T = stream(2);
  hh_ctx_s *x = context(S), *y = context(S), *z = context(T);
  DevBuf a;
  for (hh_ctx_s* c : {x, x, y, y}) {
    a.alloc(c, 4096);
    use(a, S);
    a.release();
  }
  if (model::mallocs != 1) model::fault("a kept block was not reused on its stream");
  a.alloc(z, 4096);
  if (model::mallocs != 2) model::fault("a block in use elsewhere was handed out");
  use(a, T);
  a.release();
  destroy(x);
  destroy(y);
  DevBuf b, c;
  b.alloc(z, 4096);
  use(b, T);
  c.alloc(z, 4096);
  use(c, T);
  if (model::mallocs != 2) model::fault("a destroyed context's block was not reused");
  b.release();
  c.release();
  destroy(z);
  if (model::live[0] != 0) model::fault("memory is left after the last context");
}

int main(int argc, char** argv) {
  const std::string s = argc > 1 ? argv[1] : "";
  if (s == "destroy_same_stream") destroy_race(true);
  else if (s == "destroy_restreamed") destroy_race(false);
  else if (s == "restream") restream();
  else if (s == "restream_capture") restream_capture();
  else if (s == "trim_other_device") trim_other_device();
  else if (s == "other_device_goes_on") other_device_goes_on();
  else if (s == "graph_memory") graph_memory();
  else if (s == "stay_after_capture") stay_after_capture();
  else if (s == "no_host_memory") no_host_memory();
  else if (s == "reuse") reuse();
  else return 2;
  if (model::bad == 0) printf("ok\n");
  return model::bad != 0;
}
