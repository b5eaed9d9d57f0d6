// Device memory of the library: blocks of size classes, kept when freed.
//
// Every call builds and drops some hundreds of buffers (190 allocations and
// frees per time step), and the sizes of the large ones (the ACA's factor pool,
// tens of GiB, its arenas, the block lists) change a little from step to step
// as the particles move. From hipMallocAsync each of them costs 5 + 14 us of
// host time, and a pool that is a little larger than the freed one is mapped
// anew: steps of 90 ms of kernels took 0.8 s, and of 0.4 s took 1.7 s. Freed
// blocks therefore stay here, one list per size class: eight classes per power of
// two, so a class is at most an eighth larger than what is asked for, and a kept block
// may be a quarter larger than the class (1.41 times the request in all: a pool that
// shrinks a little from step to step keeps its block).
//
// A kept block belongs to the context whose buffer it was, and a later buffer takes
// it if the order of streams puts the block's earlier work ahead: the same context's
// buffers (a context that changes its stream orders the new one after the old one),
// those of another context on the same stream, and, once the context has been waited
// for and destroyed, any. That wait says nothing about another context's blocks: their
// work may have been queued after it, by another thread. The lists of a device hold at most
// KEEP_SHARE of its memory, or the largest budget a caller granted a context up to
// KEEP_MOST of it (the largest blocks go first: with KEEP_SHARE alone, a budget of
// 280 GB and a factor pool above 115 GB, the pool was mapped anew in every other
// step, 3.9 s of a 4.2 s training step at 200,000 particles), and everything is
// returned when the last context on the device is destroyed or when an
// allocation fails. Contexts may live in any thread: one lock per device, not held
// while the runtime allocates.
#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <vector>

#include "internal.h"

namespace {

constexpr int MAX_DEVICES = 64;
constexpr double KEEP_SHARE = 0.4, KEEP_MOST = 0.75;

// Owners of kept blocks besides the contexts' numbers.
constexpr uint64_t IDLE = 0;               // nothing queued uses it any more
constexpr uint64_t LOST = ~(uint64_t)0;    // of a context that could not be waited for
// Of a buffer that was allocated while its stream was captured: the memory belongs to
// the graph, is there during its replays only, and is not kept.
constexpr uint64_t GRAPH = LOST - 1;

struct Block {
  void* p;
  uint64_t owner;
};

struct Owner {
  hipStream_t stream;
  bool behind;   // it queued work elsewhere that this stream is not ordered after
};

struct DeviceBlocks {
  std::mutex mu;
  std::map<size_t, std::vector<Block>> free;
  std::map<uint64_t, Owner> contexts;   // the living ones by number
  size_t kept = 0, limit = 0, most = 0;
};
std::atomic<uint64_t> g_contexts{0};   // contexts so far

// Whether the work of context `owner`'s blocks is ahead of what context `next` queues.
bool ordered(const DeviceBlocks* d, uint64_t owner, uint64_t next) {
  if (owner == IDLE || owner == next) return true;
  const auto a = d->contexts.find(owner), b = d->contexts.find(next);
  return a != d->contexts.end() && b != d->contexts.end() && !a->second.behind &&
         a->second.stream == b->second.stream;
}

// Also where the runtime cannot say (the null stream while another one is captured).
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) == hipSuccess) return cs != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// never destroyed: handles may be freed while the process ends
DeviceBlocks* device_blocks(int dev) {
  static DeviceBlocks* all = new DeviceBlocks[MAX_DEVICES];
  return dev >= 0 && dev < MAX_DEVICES ? all + dev : nullptr;
}

size_t size_class(size_t n) {
  if (n <= 512) return 512;
  const size_t step = (size_t)1 << (60 - __builtin_clzll(n - 1));   // an eighth of the power of two below
  return (n + step - 1) / step * step;
}

// Returns kept blocks above the limit, the largest first, in the stream order of the
// context that released the last one: its own and those ordered ahead of it. That
// order holds whichever device is current (handles are freed from any thread, also by
// a garbage collector), and nothing waits.
void trim(DeviceBlocks* d, uint64_t owner) {
  const auto c = d->contexts.find(owner);
  if (c == d->contexts.end() || c->second.behind || capturing(c->second.stream)) return;
  for (auto it = d->free.end(); d->kept > d->limit && it != d->free.begin();) {
    std::vector<Block>& v = (--it)->second;
    for (size_t i = v.size(); i-- > 0 && d->kept > d->limit;) {
      if (!ordered(d, v[i].owner, owner)) continue;
      (void)hipFreeAsync(v[i].p, c->second.stream);
      d->kept -= it->first;
      v.erase(v.begin() + i);
    }
    if (v.empty()) it = d->free.erase(it);
  }
}

// Returns kept blocks to the runtime through stream s, which is waited for: those of
// no living context, and those of the contexts whose stream can be waited for.
void give_back(DeviceBlocks* d, hipStream_t s) {
  if (capturing(s)) return;   // a graph would record the frees
  std::map<uint64_t, bool> done;
  for (auto& c : d->contexts)
    done[c.first] = !c.second.behind && !capturing(c.second.stream) &&
                    hipStreamSynchronize(c.second.stream) == hipSuccess;
  for (auto it = d->free.begin(); it != d->free.end();) {
    std::vector<Block>& v = it->second;
    for (size_t i = v.size(); i-- > 0;) {
      if (v[i].owner == LOST || (v[i].owner != IDLE && !done[v[i].owner])) continue;
      (void)hipFreeAsync(v[i].p, s);
      d->kept -= it->first;
      v.erase(v.begin() + i);
    }
    it = v.empty() ? d->free.erase(it) : std::next(it);
  }
  (void)hipStreamSynchronize(s);
  (void)hipGetLastError();
}

bool keep(DeviceBlocks* d, void* p, size_t bytes, uint64_t owner) {
  if (!d || owner == GRAPH) return false;
  std::lock_guard<std::mutex> lock(d->mu);
  if (d->contexts.empty()) return false;
  try {
    // (a context that is gone was waited for)
    d->free[bytes].push_back(Block{p, d->contexts.count(owner) ? owner : IDLE});
  } catch (const std::bad_alloc&) {   // no host memory for the list
    return false;
  }
  d->kept += bytes;
  if (d->kept > d->limit) trim(d, owner);
  return true;
}

// A kept block of class c, or of the next ones up to a quarter more memory, for a
// buffer of context `owner`: its size, 0 without one.
size_t take_kept(DeviceBlocks* d, size_t c, uint64_t owner, void** p) {
  if (!d) return 0;
  std::lock_guard<std::mutex> lock(d->mu);
  for (auto it = d->free.lower_bound(c); it != d->free.end() && it->first <= c + c / 4; ++it) {
    std::vector<Block>& v = it->second;
    for (size_t i = v.size(); i-- > 0;) {
      if (!ordered(d, v[i].owner, owner)) continue;
      const size_t bytes = it->first;
      *p = v[i].p;
      v.erase(v.begin() + i);
      d->kept -= bytes;
      if (v.empty()) d->free.erase(it);
      return bytes;
    }
  }
  return 0;
}

}  // namespace

void DevBuf::release() {
  if (!p) return;
  if (!keep(device_blocks(dev), p, bytes, owner)) (void)hipFreeAsync(p, s);
  p = nullptr;
  bytes = 0;
}

void DevBuf::take(DevBuf& src) {
  release();
  p = src.p;
  bytes = src.bytes;
  owner = src.owner;
  s = src.s;
  dev = src.dev;
  src.p = nullptr;
  src.bytes = 0;
}

static void follow(hh_ctx ctx, hipStream_t stream);

void DevBuf::alloc(hh_ctx ctx, size_t nbytes) {
  release();
  if (!ctx->behind.empty()) follow(ctx, ctx->stream);
  owner = ctx->mem;
  s = ctx->stream;
  dev = ctx->device;
  const size_t c = size_class(nbytes);
  DeviceBlocks* d = device_blocks(dev);
  bytes = take_kept(d, c, owner, &p);
  if (bytes > 0) return;
  if (capturing(s)) owner = GRAPH;
  hipError_t e = hipMallocAsync(&p, c, s);
  if (e != hipSuccess && d) {
    (void)hipGetLastError();
    {
      std::lock_guard<std::mutex> lock(d->mu);
      give_back(d, s);
    }
    e = hipMallocAsync(&p, c, s);
  }
  if (e != hipSuccess) {
    p = nullptr;
    (void)hipGetLastError();
    throw hh_error{HH_ERR_OUT_OF_MEMORY,
                   "device allocation of " + std::to_string(nbytes) + " bytes failed"};
  }
  bytes = c;
}

size_t devmem_attach(hh_ctx ctx) {
  DeviceBlocks* d = device_blocks(ctx->device);
  size_t fr = 0, tot = 0;
  HIP_OK(hipMemGetInfo(&fr, &tot));
  if (!d) return fr;
  std::lock_guard<std::mutex> lock(d->mu);
  if (d->contexts.empty()) d->limit = (size_t)(KEEP_SHARE * (double)tot);
  d->most = (size_t)(KEEP_MOST * (double)tot);
  const uint64_t number = ++g_contexts;
  d->contexts[number] = Owner{ctx->stream, false};
  ctx->mem = number;
  return fr + d->kept;
}

void devmem_grant(int dev, size_t bytes) {
  DeviceBlocks* d = device_blocks(dev);
  if (!d) return;
  std::lock_guard<std::mutex> lock(d->mu);
  d->limit = std::max(d->limit, std::min(bytes, d->most));
}

// A stream in capture runs nothing and cannot wait for work outside: it is ordered
// after nothing, its replays by whoever launches them. The streams left out then, and
// one that is captured itself now, are waited for by a later stream, or by the same one
// when it allocates after the capture.
void devmem_restream(hh_ctx ctx, hipStream_t stream) {
  if (stream == ctx->stream) return;
  ctx->behind.push_back(ctx->stream);
  follow(ctx, stream);
}
static void follow(hh_ctx ctx, hipStream_t stream) {
  std::vector<hipStream_t> left;
  if (capturing(stream)) {
    left = ctx->behind;
  } else {
    for (hipStream_t s : ctx->behind) {
      if (s == stream) continue;
      if (capturing(s)) {
        left.push_back(s);
      } else if (hipEventRecord(ctx->fork, s) != hipSuccess ||
                 hipStreamWaitEvent(stream, ctx->fork, 0) != hipSuccess) {
        (void)hipGetLastError();   // a stream that is gone: its work was the device's
        HIP_OK(hipDeviceSynchronize());
      }
    }
  }
  ctx->behind = left;
  ctx->stream = stream;
  DeviceBlocks* d = device_blocks(ctx->device);
  if (!d) return;
  std::lock_guard<std::mutex> lock(d->mu);
  const auto c = d->contexts.find(ctx->mem);
  if (c != d->contexts.end()) c->second = Owner{stream, !left.empty()};
}

bool devmem_wait(hh_ctx ctx) {
  bool ok = hipStreamSynchronize(ctx->stream) == hipSuccess;
  for (hipStream_t s : ctx->behind) ok &= hipStreamSynchronize(s) == hipSuccess;
  if (!ok && !capturing(ctx->stream)) ok = hipDeviceSynchronize() == hipSuccess;
  (void)hipGetLastError();
  return ok;
}

void devmem_detach(hh_ctx ctx, bool waited) {
  DeviceBlocks* d = device_blocks(ctx->device);
  if (!d) return;
  std::lock_guard<std::mutex> lock(d->mu);
  if (!d->contexts.erase(ctx->mem)) return;
  for (auto& c : d->free)
    for (Block& b : c.second)
      if (b.owner == ctx->mem) b.owner = waited ? IDLE : LOST;
  if (d->contexts.empty()) give_back(d, ctx->stream);
}
