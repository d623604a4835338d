// Copies between the device and the caller's memory through pinned memory
// that a handle owns.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <memory>

namespace symlat {

// Where a handle's small results land.  A copy into the caller's pageable
// memory took 11.4 us more than the kernel before it and the wait, one into
// pinned memory 3 us: one step of a 32^3 lattice and a look at its background
// 43.4 -> 35.7 us.  A kernel that ends a call's work stores its results there
// itself: a read-out of the energies, with two copies 46.8 us, with one kernel
// that gathered them 28.1, now takes 26.3.  Where no pinned memory is to
// be had, ordinary memory.
class ReadBack {
 public:
  ~ReadBack();
  void reserve(size_t bytes);
  // One copy, then a wait for the stream; the result stays until the next.
  hipError_t one(const void* src, size_t bytes, hipStream_t s, const unsigned char** out);
  // Where a kernel may store `bytes` for the host; NULL without pinned memory.
  unsigned char* direct(size_t bytes) { return bytes <= cap_ ? pin_ : nullptr; }

 private:
  unsigned char* room(size_t bytes);
  unsigned char* pin_ = nullptr;
  size_t cap_ = 0, plain_cap_ = 0;
  std::unique_ptr<unsigned char[]> plain_;
};

// Large arrays in and out: chunks through a ring of pinned slots, copied to
// and from the caller's memory by a few threads while the DMA runs.  What it
// saves is mostly the caller's page faults, which one thread takes one after
// another: 14 MB out of the device into memory not touched before took 1490 us
// by a pageable copy and 650 so (into touched memory 870 and 510; in 530 and
// 510), a linearized handle's fields at 96^3 1900-3700 and 1240-1430.
// The slots (8 MiB) are taken at the first use and kept.
struct HostRange {
  void* dev;
  void* host;
  size_t bytes;
};
class HostRing {
 public:
  ~HostRing();
  // Both return when the copies are done; the stream's earlier work is
  // waited for with them.
  hipError_t read(const HostRange* r, int nr, hipStream_t s) { return run(r, nr, s, false); }
  hipError_t write(const HostRange* r, int nr, hipStream_t s) { return run(r, nr, s, true); }

 private:
  static constexpr int kThreads = 4, kSlots = 2;
  static constexpr size_t kChunk = size_t(1) << 20;
  // below this a pageable copy: too few chunks to fill the ring
  static constexpr size_t kLeast = 8 * kChunk;
  bool ready();
  hipError_t run(const HostRange* r, int nr, hipStream_t s, bool in);
  unsigned char* pin_ = nullptr;
  hipEvent_t ev_[kThreads * kSlots] = {};
};

}  // namespace symlat
