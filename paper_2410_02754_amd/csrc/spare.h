// Device memory that a call can do without: with it a faster route runs, without it
// another one with the same results.  So it is never taken where it could be missed:
// all such buffers of a device hold at most kSpareMax together, one above kSpareSmall is
// only taken where a sixteenth of the device's memory stays free beside it (asking cost
// a context's first pass 9 to 10 us of 218 and 289), and an allocation that fails takes
// its context's back (DevBuf::spare).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace chfsi {

constexpr size_t kSpareMax = (size_t)8 << 30, kSpareSmall = (size_t)32 << 20;

class SpareBuf {
 public:
  SpareBuf() = default;
  SpareBuf(const SpareBuf&) = delete;
  SpareBuf& operator=(const SpareBuf&) = delete;
  ~SpareBuf() { release(); }
  // At least `bytes`, or null.  A growing buffer takes its new memory beside the old and
  // keeps the old where that fails (its address stays good); a size that failed is not
  // asked for again, nor any larger one, until retry().
  void* get(size_t bytes);
  void retry() { refused_ = SIZE_MAX; }
  void release();
  size_t bytes() const { return bytes_; }

 private:
  void* ptr_ = nullptr;
  size_t bytes_ = 0, refused_ = SIZE_MAX;
  int device_ = -1;
};

}  // namespace chfsi
