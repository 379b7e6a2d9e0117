// Which kernel routes a call's tokens (host code, no HIP).  Kernels: rom_route.hip.
#pragma once

#include <cstdint>

namespace rom {

// Four wavefronts for a token, a quarter of d_model each, so that the launch spreads over the chip and no wavefront walks all of d_model
// for all experts alone; from some thousand tokens on one wavefront a token (us, four / one: 8 experts, 3063 tokens x 1536 10.8 / 14.5,
// 4096 x 2048 13.7 / 19.7, 4096 x 768 9.6 / 8.7; 16 experts, 3063 x 2048 18.8 / 33.8, 4096 x 768 19.5 / 18.4, 6000 x 1536 28.7 / 29.2).
inline int64_t route_four_most(int d_model, int n_experts) {
  return d_model <= 512 ? 1024 : n_experts <= 8 && d_model >= 1024 ? 4096 : 3072;
}

// More tokens than this take the kernels with 64 and more tokens a workgroup: the matrix pipe (bf16, up to 16 experts) or router weights in
// LDS.  The matrix pipe's fp32 sums are chains of d_model / 32 terms: its logits are 1.8e-7 of their size off the 64-bit ones at
// d_model 1024 and 2.7e-7 at 2048 where the other kernels' are 0.7e-7, those of a block, whose scale is folded into the
// weights, 3.7e-7 and 7.0e-7 (1.1e-7 and 1.4e-7).  It would be faster from 4096 tokens of 8 experts and 3072 of 16 on (the router of 6000 x 2048
// 21.5 / 19.0 us, 16 experts, 6000 x 1536 29.2 / 21.3), and is not taken there.
constexpr int64_t kRouteFewMost = 8192;

}  // namespace rom
