// Host side of the stage report of Algorithm 1: the wait for a word that the device writes to pinned host memory.
#pragma once
#include <cstdint>

namespace adac {

// Waits until *word is `value`.  A stream that has run dry (or failed) without it ends the wait with false.
inline bool report_landed(const int32_t* word, int32_t value, hipStream_t st) {
  for (unsigned spin = 1;; ++spin) {
    if (__atomic_load_n(word, __ATOMIC_ACQUIRE) == value) return true;
    if ((spin & 0xFFF) == 0) {
      if (hipStreamQuery(st) != hipErrorNotReady) return __atomic_load_n(word, __ATOMIC_ACQUIRE) == value;
      (void)hipGetLastError();       // "not ready" is an answer: it must not be taken for the error of a later launch
    }
    __builtin_ia32_pause();
  }
}

}  // namespace adac
