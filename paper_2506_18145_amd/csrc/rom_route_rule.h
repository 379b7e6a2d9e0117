// Which kernels route a call's tokens and group its slots by expert (host code, no HIP).  Kernels: rom_route.hip.
#pragma once

#include <cstdint>

namespace rom {

// Four wavefronts for a token, a quarter of d_model each, so that the launch spreads over the chip and no wavefront walks all of d_model
// for all experts alone; from a line that lies the higher the more a token has to multiply, one wavefront a token.  Layer calls in us, one /
// four: 8 experts, 1200 tokens x 576 92.0 / 90.1, 3072 x 768 154.7 / 153.6, 4096 x 1024 204.8 / 204.5, 4096 x 2048 420 / 414;
// 16 experts, 2000 x 1536 282 / 271; 6 experts, 3000 x 768 153.7 / 153.9, x 1024 149.1 / 149.8, x 2048 335 / 331; 2 experts,
// 2000 x 768 105.9 / 105.4, 3000 x 768 133.3 / 134.1; one expert, 2000 x 1024 102.8 / 103.7, 3000 x 768 131.2 / 132.2.  fp32
// likewise: 16 experts, 2000 x 1536 1974 / 1967, one, 3000 x 1024 814 / 816.
// (The router alone: 16 experts, 4096 x 768 18.4 / 19.5, 6000 x 1536 29.2 / 28.7.)
inline int64_t route_four_most(int d_model, int n_experts) {
  if (d_model <= 512) return 1024;
  const int64_t least = n_experts == 1 ? 1024 : 2048, most = n_experts <= 8 ? 4096 : 3072, line = static_cast<int64_t>(d_model) * n_experts / 2;
  return line < least ? least : line < most ? line : most;
}

// More tokens than this take the kernels with 64 and more tokens a workgroup: the matrix pipe (bf16, up to 16 experts) or router weights in
// LDS.  The matrix pipe's fp32 sums are chains of d_model / 32 terms: its logits are 1.8e-7 of their size off the 64-bit ones at
// d_model 1024 and 2.7e-7 at 2048 where the other kernels' are 0.7e-7, those of a block, whose scale is folded into the
// weights, 3.7e-7 and 7.0e-7 (1.1e-7 and 1.4e-7).  It would be faster from 4096 tokens of 8 experts and 3072 of 16 on (the router of 6000 x 2048
// 21.5 / 19.0 us, 16 experts, 6000 x 1536 29.2 / 21.3), and is not taken there.
constexpr int64_t kRouteFewMost = 8192;

// Whether one workgroup groups a call's slots, else three launches.  One workgroup is bound by its scattered stores, about an address a
// clock.  Layer calls in us, three launches / one: 8 experts, 1024 slots 67.7 / 64.8, 2048 75.6 / 73.6, 4096 93.7 / 93.2, 5000 95.0 / 97.1,
// 8192 129.9 / 133.7; 4 experts, 4096 90.5 / 89.3, 8192 125.7 / 127.3; 16 experts, 2048 82.4 / 80.1, 3000 93.9 / 93.8, 4096 98.4 / 99.1;
// 64 experts, 2048 129.5 / 125.9.
inline bool grouping_in_one(int64_t n_slots, int n_experts) { return n_slots <= (n_experts <= 8 ? 4096 : 2048); }

}  // namespace rom
