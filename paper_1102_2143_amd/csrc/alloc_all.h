// Sets of device buffers that are used together.
#pragma once

#include <cstddef>
#include <initializer_list>

namespace msc {

struct BufferSpec {
  void** ptr;
  size_t bytes;
};

// Allocates every buffer of the list, or none: when one fails, those before it are freed and
// all the pointers are null, so a set whose first pointer is set is whole.  alloc(void**,
// size_t) returns a status that is 0 on success, the value returned; release(void*).
template <class Alloc, class Release>
auto alloc_all(std::initializer_list<BufferSpec> list, Alloc alloc, Release release)
    -> decltype(alloc(static_cast<void**>(nullptr), size_t(0))) {
  for (const BufferSpec& b : list) *b.ptr = nullptr;
  for (const BufferSpec& b : list) {
    const auto e = alloc(b.ptr, b.bytes);
    if (int(e) != 0) {
      *b.ptr = nullptr;
      for (const BufferSpec& c : list) {
        if (*c.ptr) release(*c.ptr);
        *c.ptr = nullptr;
      }
      return e;
    }
  }
  return decltype(alloc(static_cast<void**>(nullptr), size_t(0)))(0);
}

}  // namespace msc
