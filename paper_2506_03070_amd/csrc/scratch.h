// Scratch that an operation can run faster with and does without where it
// cannot be had.  Host code only; Mem allocates (HIP in api.hip, a model of a
// device in the CPU tests).
#pragma once

#include <cstddef>

namespace sap {

// One buffer per context, beside its workspace: what a call needs never waits
// for, and is never given up for, what it would like to have.  A size that the
// device had no room for is not asked for again until it reports that much free,
// so that a full device costs a call one query and no allocation, free or wait.
//
// Mem: bool alloc(void **, size_t); void free(void *) (waits for the buffer's
// last use); size_t available().
template <typename Mem>
struct OptionalScratch {
  void *base = nullptr;
  size_t size = 0;
  size_t refused = 0;  // the smallest size the device had no room for

  // Whether the buffer holds `bytes` now; room: what the budget leaves for it.
  bool reserve(Mem &mem, size_t bytes, size_t room) {
    if (bytes <= size) return true;
    bytes = (bytes + 4095) & ~size_t(4095);
    if (bytes > room) return false;
    if (refused != 0 && bytes >= refused && mem.available() + size < bytes) return false;
    release(mem);
    void *p = nullptr;
    if (!mem.alloc(&p, bytes)) {
      refused = bytes;
      return false;
    }
    base = p;
    size = bytes;
    if (bytes >= refused) refused = 0;
    return true;
  }
  void release(Mem &mem) {
    if (base) mem.free(base);
    base = nullptr;
    size = 0;
  }
};

}  // namespace sap
