// Which selective scan takes a call, and how its adjoint cuts a call into chunks (host code, no HIP).
#pragma once

#include <cstdint>

namespace rom {

// Time chunks of the lane = (channel, state) scan: only when there are fewer workgroups than CUs (the state-only pass costs about as much
// as the better occupancy of the full pass gains once every SIMD has a wavefront), whole tiles and at least 256 steps long
constexpr int kScanCh = 16;              // channels per workgroup
inline int scan_chunks(int64_t B, int64_t L, int d_inner) {
  const int64_t blocks = B * (d_inner / kScanCh) > 0 ? B * (d_inner / kScanCh) : 1, by_len = L / 256;
  int64_t nc = (256 + blocks - 1) / blocks;
  if (nc > by_len) nc = by_len;
  if (nc > 8) nc = 8;
  return nc < 1 ? 1 : static_cast<int>(nc);
}

// Time chunks of the lane = channel scan: enough for kLaneWaves wavefronts, of at least 64 steps; small calls, which have too few of those,
// of 32 (us, 32 / 64 steps: 1 x 2048 x 1536 45 / 55, 2 x 2048 x 1280 56 / 63, 1 x 4096 x 2048 74 / 69, 1 x 8192 x 1536 106 / 98).
constexpr int kLaneWaves = 4096;
inline int scan_lane_chunks(int64_t B, int64_t L, int d_inner) {
  const int64_t waves = B * ((d_inner + 63) / 64);
  if (waves >= 2048) return 1;
  const int64_t min_len = B * L * d_inner < (int64_t{7} << 20) ? 32 : 64;
  int64_t nc = kLaneWaves / (waves > 0 ? waves : 1);
  if (nc > L / min_len) nc = L / min_len;
  return nc < 1 ? 1 : static_cast<int>(nc);
}

// Whether the lane = channel scan takes a call (kernels in rom_seq.hip; us, lane = (channel, state) first):
//   * with 2048 wavefronts' worth of channels it needs no time chunks: 64 sequences x 256 steps x 4096 channels 300 / 203,
//     128 x 2 x 2048 74 / 12, 512 x 64 x 3072 471 / 347 in bf16, 514 / 400 in fp32; at one 64-step tile and just 2048
//     wavefronts the two are about even (64 x 64 x 2048 39 / 35, in fp32 41 / 45).  Channels count, not wavefronts: with
//     16 channels a sequence three lanes in four idle (4096 x 40 x 16 22 / 49);
//   * few (sequence, 16 channel) blocks, at most three per CU: lane = (channel, state) takes its time per step, whatever the width: 25.7 ns
//     up to one workgroup per CU, 51 up to two, 70 beyond, 17 more for the state-only pass where it cuts the sequences, too.  Lane = channel
//     takes 24 us for its three launches, 0.08 per chunk in the fold, and 5.4 per Mi (step, channel) pairs.  That line against what was
//     measured (115 shapes): 1 x 8192 x 768 91 / 77, 4096 49 / 54; 1 x 2048 x 1536 50 / 45, 1536 40 / 42; 1 x 3072 x 2048 69 / 59;
//     2 x 1536 x 1280 56 / 45, 2 x 1024 x 1536 39 / 41; 1 x 16384 x 4096 385 / 351, 2 x 3072 x 2048 77 / 86; 4 x 1536 x 1280 77 / 66, 4 x 1024
//     x 1536 53 / 54, 4 x 3072 x 1792 160 / 146, 4 x 2048 x 2048 106 / 108, 4 x 3072 x 2048 164 / 159; 4 x 1536 x 2304 107 / 99, 1024 72 / 75;
//     8 x 2048 x 1536 152 / 163;
//   * in between (8 x 2048 x 4096: 312 / 338) and for short calls the lane = (channel, state) kernels stay.
//   * fp32 calls go over from 24 Mi pairs on only: what lane = channel gains there is small (2 x 3000 x 1280 847 / 816 us a call, 4 x 1500 x 1536
//     1070 / 1075), and its sums over the states in two chains have an error of 9.8e-8 against the butterfly's 6.4e-8.  (In bf16 the rounding
//     of the outputs hides either, 1.657e-3; the states' is smaller, 4e-7 ... 9e-7 against 1e-6 ... 4e-6.)
inline bool scan_by_lane(int64_t B, int64_t L, int d_inner, bool f32 = false) {
  if (B * d_inner >= 2048 * 64) return true;
  const int64_t blocks = B * (d_inner / kScanCh), chunks = scan_chunks(B, L, d_inner), wgs = blocks * chunks;
  if (blocks > 768) return false;
  if (f32) return B * L * d_inner >= (int64_t{24} << 20);
  const double step = (wgs <= 256 ? 25.7 : wgs <= 512 ? 51.0 : 70.0) + (chunks > 1 ? 17.0 : 0.0);
  const double pair = 5.4e3 / (1 << 20);                           // ns
  return static_cast<double>(L) * (step / static_cast<double>(chunks) - pair * kScanCh * static_cast<double>(blocks)) >
         24e3 + 80.0 * scan_lane_chunks(B, L, d_inner);
}

// Chunks over all sequences whose states a call keeps, or any of fewer or shorter sequences would: one workspace serves them all.  (The
// other scan's are fewer: at most 8 a sequence, of 256 steps, and two per CU.)
inline int64_t scan_most_chunks(int64_t B, int64_t L, int d_inner) {
  const int64_t waves = (d_inner + 63) / 64, by_waves = (kLaneWaves + waves - 1) / waves, by_len = B * (L / 32);
  return L < 64 ? 0 : by_len < by_waves ? by_len : by_waves;
}

// The same where a call or one of fewer or shorter sequences is cut, else none: 64 sequences of 64 steps keep no states.  (No call of fewer
// than 512 steps is cut, and one that a shorter one of as many sequences is cut like is cut itself.)
inline int64_t scan_room_chunks(int64_t B, int64_t L, int d_inner, bool f32) {
  if (L < 512 || d_inner < kScanCh) return 0;
  int64_t most = 0, by_lane = 0;
  for (int64_t b = 1; b <= B && b * (d_inner / kScanCh) <= 768; ++b) {         // beyond that only calls without chunks
    const int64_t n = scan_chunks(b, L, d_inner) > 1 ? b * scan_chunks(b, L, d_inner) : 0;
    if (n > most) most = n;
    if (scan_by_lane(b, L, d_inner, f32)) by_lane = b;
  }
  const int64_t lane = by_lane > 0 ? scan_most_chunks(by_lane, L, d_inner) : 0;
  return lane > most ? lane : most;
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
