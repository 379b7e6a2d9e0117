// How the adjoint scan cuts a call into chunks (host code, no HIP).
#pragma once

#include <cstdint>

namespace rom {

// Steps per chunk of the adjoint scan (kernels in rom_bwd.hip), a multiple of 16.  A unit is one chunk of 64 channels, a
// workgroup of its own; its kernels walk their chunk step by step, some 0.3 us each.
//   * two units per CU and more: 128 steps.  2048 steps x 2048 channels (512 units) 126 us, in 32-step chunks 106, but
//     16384 x 1024 (2048 units) 355 / 438: the carries are half of the work then.
//   * fewer: what counts is the walk.  1024 x 2048 (256 units) 102 us, in 32 steps 65; 300 x 1536, four sequences, 123 / 65;
//     with next to none also the fold over the chunks is short: 200 x 512, two sequences, 101 us, 38 in 32 and 28 in 16 steps,
//     but 4000 x 128 105, 64 and 83.
//   * one chunk needs no carries, which weighs more than its length unless the chip is all but idle: 128 x 2048, eight
//     sequences, 52 us, 64 cut; 128 x 512 49 us, 23 in 16-step chunks; 33 x 128 21.7 / 22.6.
inline int scan_bwd_chunk(int64_t B, int64_t L, int d_inner) {
  const int64_t units = B * ((L + 127) / 128) * ((d_inner + 63) / 64);
  if (units >= 512) return 128;
  if (L <= 128) return L <= 32 || units >= 128 ? 128 : 16;
  return units <= 32 ? 16 : 32;
}

}  // namespace rom
