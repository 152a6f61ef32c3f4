#include "spare.h"

namespace chfsi {

void* SpareBuf::get(size_t bytes) {
  if (bytes <= bytes_ && ptr_) return ptr_;
  if (bytes >= refused_ || bytes == 0) return nullptr;
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    refused_ = bytes;
    return nullptr;
  }
  release();
  ptr_ = p;
  bytes_ = bytes;
  return p;
}

void SpareBuf::release() {
  if (ptr_) (void)hipFree(ptr_);
  ptr_ = nullptr;
  bytes_ = 0;
}

}  // namespace chfsi
