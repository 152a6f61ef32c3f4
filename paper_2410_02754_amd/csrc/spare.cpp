#include "spare.h"

#include <map>
#include <mutex>

namespace chfsi {

// bytes held per device by the buffers of all contexts and batches (never destroyed: a
// context may outlive the static objects)
static std::mutex& g_mu = *new std::mutex;
static std::map<int, size_t>& g_held = *new std::map<int, size_t>;

void* SpareBuf::get(size_t bytes) {
  if (bytes <= bytes_ && ptr_) return ptr_;
  if (bytes >= refused_ || bytes == 0) return nullptr;
  int dev = 0;
  void* p = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    size_t avail = 0, total = 0;
    const bool known = hipGetDevice(&dev) == hipSuccess;
    const size_t mine = dev == device_ ? bytes_ : 0;      // given back once p is there
    const auto room = [&]() {
      return bytes <= kSpareSmall ||
             (hipMemGetInfo(&avail, &total) == hipSuccess && avail >= bytes + total / 16);
    };
    if (known && g_held[dev] - mine + bytes <= kSpareMax && room() && hipMalloc(&p, bytes) == hipSuccess)
      g_held[dev] += bytes;
    else
      p = nullptr;
  }
  if (!p) {
    (void)hipGetLastError();
    refused_ = bytes;
    return nullptr;
  }
  release();
  ptr_ = p;
  bytes_ = bytes;
  device_ = dev;
  return p;
}

void SpareBuf::release() {
  if (!ptr_) return;
  (void)hipFree(ptr_);
  {
    std::lock_guard<std::mutex> lk(g_mu);
    g_held[device_] -= bytes_;
  }
  ptr_ = nullptr;
  bytes_ = 0;
}

}  // namespace chfsi
