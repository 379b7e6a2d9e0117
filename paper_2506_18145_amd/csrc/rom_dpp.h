// Sums over the 16 lanes of a row by data-parallel primitives, shared by the scan (rom_seq.hip) and its adjoint (rom_bwd.hip).
// gfx950 only.
#pragma once

#include <hip/hip_runtime.h>

namespace rom {
namespace {

template <int CTRL> __device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sixteen values per lane, each to be summed over the 16 lanes of a row: a butterfly that halves
// the number of live values at every stage (the lanes with bit 3 / 2 / 1 / 0 of n set keep the upper
// half) leaves the row total of p[n] in lane n - 30 DPP adds and 3 selects instead of 64 adds.  In the first two stages
// the upper half's adds are written by their lanes' banks alone; with selects, 12 more instructions, the adjoint scan's main kernel took 1064 us on
// 16384 x 4096 (now 1016), the scan of 3 x 1021 x 3072 73.5 (70.7).  The compiler has no form for an add whose other lanes keep their
// value, hence the asm.  A DPP read wants two instructions between it and the write of its source: the block starts with a wait
// for what its caller wrote, and within it a source is five and more instructions old.
__device__ __forceinline__ float transpose_sum16(const float *p, int n) {
#pragma clang fp contract(off)
  float a[8], c[2];
  const bool hi2 = (n & 2) != 0, hi1 = (n & 1) != 0;
#define ROM_MIRROR(d, lo, hi)                                                      \
  "v_add_f32_dpp " d ", " lo ", " lo " row_mirror row_mask:0xf bank_mask:0xf\n\t" \
  "v_add_f32_dpp " d ", " hi ", " hi " row_mirror row_mask:0xf bank_mask:0xc\n\t"
#define ROM_HALF_MIRROR(lo, hi)                                                           \
  "v_add_f32_dpp " lo ", " lo ", " lo " row_half_mirror row_mask:0xf bank_mask:0xf\n\t"  \
  "v_add_f32_dpp " lo ", " hi ", " hi " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
  asm("s_nop 1\n\t"
      ROM_MIRROR("%0", "%8", "%16") ROM_MIRROR("%4", "%12", "%20") ROM_MIRROR("%1", "%9", "%17") ROM_MIRROR("%5", "%13", "%21")
      ROM_MIRROR("%2", "%10", "%18") ROM_MIRROR("%6", "%14", "%22") ROM_MIRROR("%3", "%11", "%19") ROM_MIRROR("%7", "%15", "%23")
      ROM_HALF_MIRROR("%0", "%4") ROM_HALF_MIRROR("%1", "%5") ROM_HALF_MIRROR("%2", "%6") ROM_HALF_MIRROR("%3", "%7")
      "s_nop 1"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]), "=&v"(a[6]), "=&v"(a[7])
      : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7]), "v"(p[8]), "v"(p[9]), "v"(p[10]),
        "v"(p[11]), "v"(p[12]), "v"(p[13]), "v"(p[14]), "v"(p[15]));
#undef ROM_HALF_MIRROR
#undef ROM_MIRROR
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float lo = dpp<0x1B>(a[j]) + a[j];
    const float hi = dpp<0x1B>(a[j + 2]) + a[j + 2];
    c[j] = hi2 ? hi : lo;
  }
  const float lo = dpp<0xB1>(c[0]) + c[0];
  const float hi = dpp<0xB1>(c[1]) + c[1];
  return hi1 ? hi : lo;
}

}  // namespace
}  // namespace rom
