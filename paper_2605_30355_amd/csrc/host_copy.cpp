// host_copy.cpp -- results from device memory to the caller's arrays.
//
// A copy to pageable memory goes through the runtime's staging in one thread, with a
// wait per call: some 10 us for the smallest, and 10 GB/s for the largest, where the
// link gives five times that and most of the time goes to the first touch of a fresh
// array's pages.  Here the small pieces of a call go to pinned memory, neighbours in
// one copy, and from there to the caller; the large ones in chunks through pinned
// memory, the device filling one while several threads empty those before it.
#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "internal.hpp"

namespace cosm {

namespace {

// Pieces up to kShort share a copy, pieces of kLong and more go in chunks; between
// them the runtime's own staging is as fast or faster.  Spins of a 10000-spin graph,
// us over a call without them, runtime's | here, into pages used before and into
// fresh ones: 0.16 MB 78 | 14 and 82 | 17; 2 MB 127 | 219 and 438 | 379; 4 MB 280 | 345
// and 897 | 626; 16 MB 1165 | 929 and 1703 | 717; 64 MB 6148 | 2531 and 6287 | 2283.
constexpr size_t kShort = (size_t)192 << 10;
constexpr size_t kLong = (size_t)5 << 19;
constexpr size_t kGap = 4096;                 // pieces this near each other are neighbours
constexpr size_t kShorts = kHostPieces * (kShort + kGap);
constexpr size_t kChunkMax = (size_t)2 << 20;
constexpr int kChunks = 4;
constexpr size_t kBlock = kChunkMax * kChunks + kShorts;  // the chunks, then the short pieces
constexpr int kPoolMax = 4;  // pinned blocks kept for the next state
constexpr int kThreadsMax = 8;

// A pinned block with the events of its chunks.
struct Block {
  char *mem = nullptr;
  hipEvent_t ev[kChunks] = {};
  int device = 0;
};

void free_block(Block *b) {
  for (hipEvent_t e : b->ev)
    if (e) (void)hipEventDestroy(e);
  if (b->mem) (void)hipHostFree(b->mem);
  delete b;
}

std::mutex g_mu;
Block *g_pool[kPoolMax];
int g_count = 0;

// A block of the current device, or null: out of memory, or the stream is another
// device's (whose events would have to be made with that device current).
Block *take_block(hipStream_t stream) {
  int dev = 0;
  hipDevice_t own = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  if (stream != nullptr) {
    if (hipStreamGetDevice(stream, &own) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    if (own != dev) return nullptr;
  }
  {
    std::lock_guard<std::mutex> lk(g_mu);
    for (int i = 0; i < g_count; i++)
      if (g_pool[i]->device == dev) {
        Block *b = g_pool[i];
        g_pool[i] = g_pool[--g_count];
        return b;
      }
  }
  Block *b = new (std::nothrow) Block();
  if (b == nullptr) return nullptr;
  b->device = dev;
  bool ok = hipHostMalloc((void **)&b->mem, kBlock, hipHostMallocDefault) == hipSuccess;
  for (hipEvent_t &e : b->ev)
    ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    free_block(b);
    return nullptr;
  }
  return b;
}

void give_block(Block *b) {
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_count < kPoolMax) {
      g_pool[g_count++] = b;
      return;
    }
  }
  free_block(b);
}

// One long piece in chunks through the block, emptied by a thread per two megabytes
// (two at least).  idle: nothing else was in the stream.
int copy_long(hipStream_t stream, Block *b, char *dst, const char *src, size_t bytes, bool idle) {
  const size_t kChunk = bytes < ((size_t)8 << 20) ? kChunkMax / 4 : kChunkMax;
  const int threads = (int)std::min<size_t>(
      {(size_t)kThreadsMax, std::max<size_t>(2, bytes >> 21), (size_t)std::thread::hardware_concurrency() / 2});
  const size_t n = (bytes + kChunk - 1) / kChunk;
  auto len = [&](size_t c) { return std::min(kChunk, bytes - c * kChunk); };
  std::atomic<size_t> ready{0};                 // chunks that have arrived
  std::atomic<bool> stop{false};
  // threads done with a chunk
  const std::unique_ptr<std::atomic<int>[]> emptied(new (std::nothrow) std::atomic<int>[n]);
  if (!emptied) return set_error(COSM_ENOMEM, "out of host memory");
  for (size_t c = 0; c < n; c++) emptied[c].store(0, std::memory_order_relaxed);
  auto part = [&](size_t c, int k, int of) {
    // (the share rounded up twice: to whole bytes, then to pages)
    const size_t l = len(c), p = ((l + (size_t)of - 1) / (size_t)of + 4095) / 4096 * 4096;
    const size_t at = p * (size_t)k;
    if (at < l)
      std::memcpy(dst + c * kChunk + at, b->mem + (c % kChunks) * kChunk + at, std::min(p, l - at));
  };
  // While the device has work left (sweeps may take seconds) the threads sleep; they wake
  // while the first chunk is on its way and follow the chunks, some tens of us apart.
  std::mutex mu;
  std::condition_variable first;
  bool go = idle;
  auto start = [&] {
    if (idle) return;
    {
      std::lock_guard<std::mutex> lk(mu);
      go = true;
    }
    first.notify_all();
  };
  std::vector<std::thread> workers;
  int of = 1;
  auto work = [&](int k, int of) {
    if (!idle) {
      std::unique_lock<std::mutex> lk(mu);
      first.wait(lk, [&] { return go; });
    }
    for (size_t c = 0; c < n; c++) {
      while (ready.load(std::memory_order_acquire) <= c) {
        if (stop.load(std::memory_order_relaxed)) return;
        std::this_thread::yield();
      }
      part(c, k, of);
      emptied[c].fetch_add(1, std::memory_order_release);
    }
  };
  if (threads > 1) try {
    workers.reserve((size_t)threads);
    for (int k = 0; k < threads; k++) workers.emplace_back(work, k, threads);
    of = threads;
  } catch (...) {  // fewer threads than parts: none, and this one copies
    stop.store(true);
    start();
    for (std::thread &w : workers) w.join();
    workers.clear();
    of = 1;
  }
  hipError_t err = hipSuccess;
  // (the last event is not a chunk's before the first has arrived)
  const hipEvent_t before = b->ev[kChunks - 1];
  if (!idle) err = hipEventRecord(before, stream);
  size_t issued = 0, arrived = 0;
  while (arrived < n && err == hipSuccess) {
    // a chunk's place is free once every thread has emptied the one before it
    while (issued < n && issued < arrived + kChunks - 1 && err == hipSuccess) {
      if (issued >= (size_t)kChunks && !workers.empty())
        while (emptied[issued - kChunks].load(std::memory_order_acquire) < of)
          std::this_thread::yield();
      err = hipMemcpyAsync(b->mem + (issued % kChunks) * kChunk, src + issued * kChunk, len(issued),
                           hipMemcpyDeviceToHost, stream);
      if (err == hipSuccess) err = hipEventRecord(b->ev[issued % kChunks], stream);
      issued++;
    }
    if (err == hipSuccess && arrived == 0 && !idle) {
      err = hipEventSynchronize(before);
      start();
    }
    if (err == hipSuccess) err = hipEventSynchronize(b->ev[arrived % kChunks]);
    if (err != hipSuccess) break;
    if (workers.empty()) part(arrived, 0, 1);
    arrived++;
    ready.store(arrived, std::memory_order_release);
  }
  if (err != hipSuccess) {
    stop.store(true);
    start();
  }
  for (std::thread &w : workers) w.join();
  if (err != hipSuccess) {
    (void)hipStreamSynchronize(stream);  // no copy into the block is left
    return set_error(COSM_EDEVICE, std::string("copying results: ") + hipGetErrorString(err));
  }
  return COSM_OK;
}

int plain(hipStream_t stream, const HostPiece *p, int count) {
  for (int i = 0; i < count; i++)
    if (p[i].bytes > 0)
      COSM_HIP_CHECK(hipMemcpyAsync(p[i].dst, p[i].src, p[i].bytes, hipMemcpyDeviceToHost, stream));
  COSM_HIP_CHECK(hipStreamSynchronize(stream));
  return COSM_OK;
}

}  // namespace

int copy_to_host(hipStream_t stream, HostPiece *p, int count, bool may_allocate) {
  Block *b = may_allocate ? take_block(stream) : nullptr;
  if (b == nullptr) return plain(stream, p, count);
  bool idle = true;  // (asked only where it matters: the question takes some 8 us)
  if (std::any_of(p, p + count, [](const HostPiece &x) { return x.bytes >= kLong; })) {
    idle = hipStreamQuery(stream) == hipSuccess;
    if (!idle) (void)hipGetLastError();  // (not ready is no error)
  }
  std::sort(p, p + count, [](const HostPiece &x, const HostPiece &y) { return x.src < y.src; });
  // the short pieces: neighbours in one copy, waited for with the long ones' or last
  char *const shorts = b->mem + kChunkMax * kChunks;
  size_t used = 0, at[kHostPieces] = {};
  int rc = COSM_OK;
  for (int i = 0; i < count && rc == COSM_OK;) {
    if (p[i].bytes > kShort) {
      i++;
      continue;
    }
    const char *lo = (const char *)p[i].src;
    const char *hi = lo + p[i].bytes;
    int j = i + 1;
    while (j < count && p[j].bytes <= kShort && (const char *)p[j].src >= hi &&
           (const char *)p[j].src < hi + kGap) {
      hi = (const char *)p[j].src + p[j].bytes;
      j++;
    }
    for (int k = i; k < j; k++) at[k] = used + (size_t)((const char *)p[k].src - lo);
    if (hi > lo && hipMemcpyAsync(shorts + used, lo, (size_t)(hi - lo), hipMemcpyDeviceToHost,
                                  stream) != hipSuccess)
      rc = set_error(COSM_EDEVICE, "copying results failed");
    used += (size_t)(hi - lo);
    i = j;
  }
  for (int i = 0; i < count && rc == COSM_OK; i++)
    if (p[i].bytes >= kLong)
      rc = copy_long(stream, b, (char *)p[i].dst, (const char *)p[i].src, p[i].bytes, idle);
    else if (p[i].bytes > kShort &&
             hipMemcpyAsync(p[i].dst, p[i].src, p[i].bytes, hipMemcpyDeviceToHost, stream) !=
                 hipSuccess)
      rc = set_error(COSM_EDEVICE, "copying results failed");
  if (hipStreamSynchronize(stream) != hipSuccess && rc == COSM_OK)
    rc = set_error(COSM_EDEVICE, "hipStreamSynchronize");
  for (int i = 0; i < count && rc == COSM_OK; i++)
    if (p[i].bytes <= kShort) std::memcpy(p[i].dst, shorts + at[i], p[i].bytes);
  give_block(b);
  return rc;
}

}  // namespace cosm
