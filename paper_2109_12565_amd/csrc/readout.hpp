// Copies of device results into the caller's ordinary memory, through
// page-locked memory of the handle.
//
// A copy to ordinary memory is staged by the runtime, one thread filling the
// destination, whose fresh pages are mapped and cleared on the way: 4096 x 2048
// fields (336 MB) take 34 ms of it, where the link needs 6. From 48 MiB in all,
// or 32 MiB a block (which an allocator maps afresh each time), the copy
// engine fills a ring of page-locked chunks and several threads empty it: 9 to
// 12 ms; 32 MiB of droplet labels 1 ms (2). Up to 2 MiB all blocks come in one
// copy: 128 x 64 fields, with the fields pass, 50 us (210 in five). Between
// the two, where blocks are often recycled pages, the threads only compete
// with the program's own: a run with its snapshot, ring / runtime, 17 MiB 2.7 /
// 1.9 ms, 33 MiB 4.0 / 3.4, 49 MiB 4.0 / 4.7; without threads 2 to 4% slower.
// Where there is no page-locked memory (or no host memory for the lists), the
// runtime copies block by block, whatever the size.
#pragma once

#include <hip/hip_runtime.h>
#include <sched.h>
#include <stdint.h>
#include <sys/mman.h>

#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace tlbh {

class Readout {
 public:
  ~Readout() {
    for (hipEvent_t e : landed_)
      if (e) (void)hipEventDestroy(e);
    if (page_) (void)hipHostFree(page_);
    if (ring_) (void)hipHostFree(ring_);
  }

  // 64 KiB of page-locked memory that a kernel may write, for results read
  // after the stream is waited for and before the next use of this object; null
  // when there is none. Allocated at the first call (10 us or more: tlb_init
  // makes it).
  void* page() {
    if (!page_ && hipHostMalloc(&page_, kPage, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      page_ = nullptr;
    }
    return page_;
  }

  // `parts` blocks of `bytes` bytes, one after the other in device memory, to
  // dst[0 .. parts - 1] (those that are not null), after the work on `stream`;
  // returns when they are there.
  hipError_t fetch(const void* src, size_t bytes, int parts, void* const* dst, hipStream_t stream) {
    for (int k = 0; k < parts;) {
      int e = k;
      while (e < parts && dst[e]) ++e;
      if (e > k) {
        const char* from = static_cast<const char*>(src) + k * bytes;
        hipError_t err;
        try {
          err = run(from, bytes, e - k, dst + k, stream);
        } catch (const std::exception&) {  // no host memory for the lists; nothing was begun
          err = each(from, bytes, e - k, dst + k, stream);
        }
        if (err != hipSuccess) return err;
      }
      k = e + 1;
    }
    return hipStreamSynchronize(stream);
  }

 private:
  // A copy costs the issuing thread about 35 us whatever its size, 4 MiB take
  // the link 73 us. Threads that fault in one huge page of a destination each
  // clear it, so a piece is what lies in one 2 MiB window of it.
  static constexpr size_t kChunk = (size_t)4 << 20, kWindow = (size_t)2 << 20;
  static constexpr size_t kPage = (size_t)64 << 10;
  static constexpr size_t kOneCopy = (size_t)2 << 20, kThreaded = (size_t)48 << 20, kFresh = (size_t)32 << 20;
  static constexpr int kSlots = 4;
  static constexpr size_t kPerThread = (size_t)8 << 20;
  static constexpr int kMaxThreads = 8;

  struct Piece {
    char* dst;
    size_t off, len;  // of the blocks' bytes
  };

  // A piece into place. Pages that are not there yet are mapped in one call,
  // at half the cost of a fault each (where the kernel cannot, by faults).
  static void place(const Piece& p, const char* ring) {
#ifdef MADV_POPULATE_WRITE
    constexpr uintptr_t kUnit = 4096;
    const uintptr_t a = (reinterpret_cast<uintptr_t>(p.dst) + kUnit - 1) & ~(kUnit - 1);
    const uintptr_t b = (reinterpret_cast<uintptr_t>(p.dst) + p.len) & ~(kUnit - 1);
    if (b > a + 16 * kUnit) (void)madvise(reinterpret_cast<void*>(a), b - a, MADV_POPULATE_WRITE);
#endif
    const size_t at = p.off % (kSlots * kChunk), m1 = std::min(p.len, kSlots * kChunk - at);
    std::memcpy(p.dst, ring + at, m1);
    std::memcpy(p.dst + m1, ring, p.len - m1);
  }

  // The ring of at least `need` bytes, or null: kOneCopy at first, so that it
  // grows once at most.
  char* reserve(size_t need) {
    need = std::max(need, kOneCopy);
    if (need > size_) {
      if (ring_) (void)hipHostFree(ring_);
      ring_ = nullptr;
      size_ = 0;
      if (hipHostMalloc(&ring_, need, hipHostMallocDefault) == hipSuccess) {
        size_ = need;
      } else {
        (void)hipGetLastError();
        ring_ = nullptr;
      }
    }
    return static_cast<char*>(ring_);
  }

  // By the runtime's own copy.
  static hipError_t each(const char* src, size_t bytes, int parts, void* const* dst, hipStream_t stream) {
    hipError_t e = hipSuccess;
    for (int k = 0; k < parts && e == hipSuccess; ++k)
      e = hipMemcpyAsync(dst[k], src + k * bytes, bytes, hipMemcpyDeviceToHost, stream);
    return e;
  }

  hipError_t run(const char* src, size_t bytes, int parts, void* const* dst, hipStream_t stream) {
    const size_t total = bytes * parts;
    if (total == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    // (one block gains nothing that would pay for page-locked memory)
    if (total <= kOneCopy ? total > kPage && total > size_ && parts == 1
                          : total < kThreaded && bytes < kFresh)
      return each(src, bytes, parts, dst, stream);
    const size_t n = (total + kChunk - 1) / kChunk;
    char* ring = total <= kPage      ? static_cast<char*>(page())
                 : total <= kOneCopy ? reserve(total)
                                     : reserve(kSlots * kChunk);
    if (!ring) return each(src, bytes, parts, dst, stream);
    if (total <= kOneCopy) {
      e = hipMemcpyAsync(ring, src, total, hipMemcpyDeviceToHost, stream);
      if (e == hipSuccess) e = hipStreamSynchronize(stream);
      if (e == hipSuccess)
        for (int k = 0; k < parts; ++k) std::memcpy(dst[k], ring + k * bytes, bytes);
      return e;
    }
    std::vector<Piece> pieces;
    for (int k = 0; k < parts; ++k)
      for (size_t at = 0, len; at < bytes; at += len) {
        char* to = static_cast<char*>(dst[k]) + at;
        len = std::min(bytes - at, kWindow - reinterpret_cast<uintptr_t>(to) % kWindow);
        pieces.push_back({to, k * bytes + at, len});
      }
    std::vector<size_t> left(n, 0);  // pieces of a chunk not yet in place
    for (const Piece& p : pieces)
      for (size_t c = p.off / kChunk; c <= (p.off + p.len - 1) / kChunk; ++c) ++left[c];
    for (hipEvent_t& ev : landed_)
      if (!ev && (e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return e;

    // This thread issues the copies and reports the chunks that have landed;
    // the threads (and this one at the end) take their pieces in order.
    std::mutex m;
    std::condition_variable work, freed;
    size_t landed = 0, taken = 0;  // chunks, pieces
    bool stop = false;
    auto ready = [&]() {
      return taken < pieces.size() && pieces[taken].off + pieces[taken].len <= std::min(landed * kChunk, total);
    };
    auto place_one = [&](std::unique_lock<std::mutex>& lock) {
      const Piece p = pieces[taken++];
      lock.unlock();
      place(p, ring);
      lock.lock();
      for (size_t c = p.off / kChunk; c <= (p.off + p.len - 1) / kChunk; ++c)
        if (--left[c] == 0) freed.notify_one();
    };
    // (the slot of chunk c is free when chunk c - kSlots is in place)
    auto slot_free = [&](size_t c) { return c < (size_t)kSlots || left[c - kSlots] == 0; };
    std::vector<std::thread> threads;
    try {
      const int want = (int)std::min<size_t>(std::min(kMaxThreads, cpus()), total / kPerThread);
      threads.reserve(want);
      for (int k = 0; k < want; ++k)
        threads.emplace_back([&]() {
          std::unique_lock<std::mutex> lock(m);
          for (;;) {
            work.wait(lock, [&]() { return ready() || stop; });
            if (!ready()) return;
            place_one(lock);
          }
        });
    } catch (const std::exception&) {  // as many threads as there could be
    }
    for (size_t issued = 0; landed < n && e == hipSuccess;) {
      std::unique_lock<std::mutex> lock(m);
      if (issued < n && slot_free(issued)) {
        const size_t slot = issued % kSlots, off = issued * kChunk;
        ++issued;
        lock.unlock();
        e = hipMemcpyAsync(ring + slot * kChunk, src + off, std::min(kChunk, total - off),
                           hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipEventRecord(landed_[slot], stream);
      } else if (landed < issued) {
        lock.unlock();
        e = hipEventSynchronize(landed_[landed % kSlots]);
        if (e == hipSuccess) {
          lock.lock();
          ++landed;
          work.notify_all();
        }
      } else if (ready()) {
        place_one(lock);
      } else {
        freed.wait(lock, [&]() { return slot_free(issued); });
      }
    }
    {
      std::unique_lock<std::mutex> lock(m);
      stop = true;
      work.notify_all();
      while (e == hipSuccess && ready()) place_one(lock);
    }
    for (std::thread& t : threads) t.join();
    if (e != hipSuccess) (void)hipStreamSynchronize(stream);  // no copy is left under way
    return e;
  }

  static int cpus() {
    cpu_set_t set;
    return sched_getaffinity(0, sizeof set, &set) == 0 ? std::max(1, CPU_COUNT(&set)) : 1;
  }

  void* page_ = nullptr;
  void* ring_ = nullptr;
  size_t size_ = 0;  // of the ring
  hipEvent_t landed_[kSlots] = {};
};

}  // namespace tlbh
