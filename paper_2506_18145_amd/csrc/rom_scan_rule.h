// Which selective scan takes a call, and how its adjoint cuts a call into chunks (host code, no HIP).
#pragma once

#include <cstdint>

namespace rom {

// Whether the lane = channel scan takes a call (kernels in rom_seq.hip; us, lane = (channel, state) first):
//   * with 2048 wavefronts' worth of channels it needs no time chunks: 64 sequences x 256 steps x 4096 channels 300 / 203,
//     128 x 2 x 2048 74 / 12, 512 x 64 x 3072 471 / 347 in bf16, 514 / 400 in fp32; at one 64-step tile and just 2048
//     wavefronts the two are about even (64 x 64 x 2048 39 / 35, in fp32 41 / 45).  Channels count, not wavefronts: with
//     16 channels a sequence three lanes in four idle (4096 x 40 x 16 22 / 49);
//   * few (sequence, 16 channel) blocks, at most three per CU, leave the lane = (channel, state) kernels at one or two
//     wavefronts per SIMD: with enough steps to cut, lane = channel wins in spite of its second pass
//     (1 x 16384 x 4096: 385 / 351, 1 x 16384 x 3072 521 / 282, 2 x 4096 x 3072 192 / 149, 4 x 4096 x 2048 194 / 183, in
//     fp32 449 / 410, 620 / 309, 200 / 157, 220 / 215; below about 24 M (step, channel) pairs its three launches and
//     short chunks cost the gain: 4 x 2048 x 2048 105 / 108);
//   * in between (8 x 2048 x 4096: 312 / 338) and for short calls the lane = (channel, state) kernels stay.
inline bool scan_by_lane(int64_t B, int64_t L, int d_inner) {
  if (B * d_inner >= 2048 * 64) return true;
  return B * (d_inner / 16) <= 768 && B * L * d_inner >= (int64_t{24} << 20);
}

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
