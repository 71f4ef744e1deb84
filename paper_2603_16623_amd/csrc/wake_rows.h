// Which device destinations the read-out kernels may write (no HIP types: the
// rule is host arithmetic on pointers and what the runtime says of them).
#pragma once
#include <cstddef>
#include <cstdint>

// What the runtime knows of an output pointer: the allocation it lies in and
// the device that holds it (device < 0: not device memory, or not known).
struct OutMem {
  uintptr_t base;
  size_t size;
  int device;
};

// Whether one kernel on `device` may write n doubles to each of outs (null
// ones skipped): every output aligned and whole inside an allocation of that
// device, and no two of them sharing memory.  Anything else (another GPU's
// memory, host memory, a range past its allocation, outputs that overlap) goes
// through copies on the stream, row by row in order, which reach other devices
// and answer a bad pointer with an error where a kernel's stores would fault.
inline bool rows_by_kernel(double* const* outs, const OutMem* mem, int rows, size_t n, int device) {
  const size_t bytes = n * sizeof(double);
  for (int q = 0; q < rows; ++q) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(outs[q]);
    if (!p) continue;
    if (mem[q].device != device || p % alignof(double) != 0) return false;
    if (p < mem[q].base || p - mem[q].base > mem[q].size || bytes > mem[q].size - (p - mem[q].base)) return false;
    for (int o = 0; o < q; ++o) {
      const uintptr_t x = reinterpret_cast<uintptr_t>(outs[o]);
      if (x && p < x + bytes && x < p + bytes) return false;
    }
  }
  return true;
}
