// How a call of the short conv is cut into runs, and where its end state goes (host code, no HIP).  Kernel: rom_seq.hip.
#pragma once

#include <cstdint>

namespace rom {

// a sequence of at most this many steps is one run of one conv thread: its state may be updated in place
constexpr int kConvInPlaceMaxLen = 32;

// Whether the end state of n floats goes beside its place and is copied over, float by float.  It may be the incoming one
// (rom_step): a sequence of up to kConvInPlaceMaxLen steps is one run of one thread, which reads the old state before it writes
// the new one; longer ones are cut into runs for different threads, so a new state that shares memory with the old one is not
// written directly, nor one that does not take the kernel's 16-byte stores.
inline bool conv_state_beside(const float *in, const float *out, int64_t L, int64_t n) {
  if (!out || L <= kConvInPlaceMaxLen) return false;
  return reinterpret_cast<uintptr_t>(out) % 16 != 0 || (in && in < out + n && out < in + n);
}

}  // namespace rom
