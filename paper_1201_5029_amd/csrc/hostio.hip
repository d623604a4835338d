// Pinned read-backs and staged host copies (see hostio.h).

#include "hostio.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <new>
#include <thread>

namespace symlat {

ReadBack::~ReadBack() {
  if (pin_) (void)hipHostFree(pin_);
}

void ReadBack::reserve(size_t bytes) {
  void* p = nullptr;
  if (hipHostMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  pin_ = static_cast<unsigned char*>(p);
  cap_ = bytes;
}

unsigned char* ReadBack::room(size_t bytes) {
  if (bytes <= cap_) return pin_;
  if (plain_cap_ < bytes) {
    plain_.reset(new (std::nothrow) unsigned char[bytes]);
    plain_cap_ = plain_ ? bytes : 0;
  }
  return plain_.get();
}

hipError_t ReadBack::one(const void* src, size_t bytes, hipStream_t s, const unsigned char** out) {
  unsigned char* dst = room(bytes);
  *out = dst;
  if (!dst) return hipErrorOutOfMemory;
  const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
  return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

HostRing::~HostRing() {
  for (hipEvent_t e : ev_)
    if (e) (void)hipEventDestroy(e);
  if (pin_) (void)hipHostFree(pin_);
}

bool HostRing::ready() {
  if (pin_) return true;
  for (hipEvent_t& e : ev_)
    if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      e = nullptr;
      (void)hipGetLastError();
      return false;
    }
  void* p = nullptr;
  if (hipHostMalloc(&p, kThreads * kSlots * kChunk) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  pin_ = static_cast<unsigned char*>(p);
  return true;
}

hipError_t HostRing::run(const HostRange* r, int nr, hipStream_t s, bool in) {
  size_t total = 0;
  for (int i = 0; i < nr; ++i) total += r[i].bytes;
  if (total < kLeast || !ready()) {
    for (int i = 0; i < nr; ++i) {
      const HostRange& q = r[i];
      const hipError_t e = in ? hipMemcpyAsync(q.dev, q.host, q.bytes, hipMemcpyHostToDevice, s)
                              : hipMemcpyAsync(q.host, q.dev, q.bytes, hipMemcpyDeviceToHost, s);
      if (e != hipSuccess) return e;
    }
    return hipStreamSynchronize(s);
  }
  // chunk c of the ranges; no bytes past the last
  auto chunk = [&](size_t c) {
    for (int i = 0; i < nr; ++i) {
      const size_t m = (r[i].bytes + kChunk - 1) / kChunk;
      if (c < m) {
        const size_t o = c * kChunk;
        return HostRange{static_cast<unsigned char*>(r[i].dev) + o, static_cast<unsigned char*>(r[i].host) + o,
                         std::min(kChunk, r[i].bytes - o)};
      }
      c -= m;
    }
    return HostRange{};
  };
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  std::atomic<int> err{int(hipSuccess)};
  std::atomic<size_t> next{0};
  // Each worker takes chunks in turn and has kSlots of them under way.
  auto work = [&](int t) {
    HostRange held[kSlots] = {};
    auto check = [&](hipError_t x) {
      if (x != hipSuccess) err.store(int(x));
      return x == hipSuccess;
    };
    if (t > 0 && !check(hipSetDevice(device))) return;
    // a slot's earlier copy is done; what it read goes to the caller
    auto settle = [&](int k) {
      if (!held[k].bytes) return true;
      if (!check(hipEventSynchronize(ev_[t * kSlots + k]))) return false;
      if (!in) std::memcpy(held[k].host, pin_ + (t * kSlots + k) * kChunk, held[k].bytes);
      held[k].bytes = 0;
      return true;
    };
    for (int k = 0; err.load() == int(hipSuccess); k = (k + 1) % kSlots) {
      if (!settle(k)) return;
      const HostRange q = chunk(next.fetch_add(1));
      if (!q.bytes) break;
      unsigned char* slot = pin_ + (t * kSlots + k) * kChunk;
      if (in) std::memcpy(slot, q.host, q.bytes);
      if (!check(in ? hipMemcpyAsync(q.dev, slot, q.bytes, hipMemcpyHostToDevice, s)
                    : hipMemcpyAsync(slot, q.dev, q.bytes, hipMemcpyDeviceToHost, s)) ||
          !check(hipEventRecord(ev_[t * kSlots + k], s)))
        return;
      held[k] = q;
    }
    for (int k = 0; k < kSlots; ++k)
      if (!settle(k)) return;
  };
  std::thread team[kThreads - 1];
  for (int t = 1; t < kThreads; ++t) {
    try {
      team[t - 1] = std::thread(work, t);
    } catch (...) {
      break;  // the workers there are take every chunk
    }
  }
  work(0);
  for (std::thread& t : team)
    if (t.joinable()) t.join();
  // after an error copies may still be under way in the slots
  e = hipStreamSynchronize(s);
  return err.load() != int(hipSuccess) ? hipError_t(err.load()) : e;
}

}  // namespace symlat
