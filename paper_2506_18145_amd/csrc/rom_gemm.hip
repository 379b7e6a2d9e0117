// Expert-grouped GEMM for the routed projections of the RoM layer (Eq. (10), (11), (13)):
//   C[c_row(p), :] = epilogue( A[a_row(p), :] . W[e(p)]^T )   for every sorted position p,
// where positions are grouped by expert (offsets[]) and both operands are K-contiguous
// (activations [rows, K], weights [expert][N, K]).  Rows are gathered / scattered through
// index maps, so no separate token-permute pass is needed.
//
// bf16 path: v_mfma_f32_32x32x16_bf16, 64-lane wavefronts, a workgroup of WM x WN waves owns a
// BM x BN tile; K is walked in slabs of 64 staged through double-buffered, XOR-swizzled LDS.
// Group sizes live in device memory: every workgroup finds its (expert, row tile) by walking
// the offsets, so skewed loads only change how many tiles an expert contributes.
// Epilogues (compile-time variants): plain store, bias + softplus, per-row scale (gate weight or
// 1 / rms), per-row scale + skip rows added, fp32 partial sums of inner-dimension slices, and
// SiLU(gate) * up over a weight whose rows interleave the two halves of a SwiGLU expert.
// fp32 path (and shapes the bf16 kernels do not take): v_mfma_f32_16x16x4_f32, operands straight from memory.
#include <atomic>
#include <mutex>
#include <type_traits>

#include "rom_gemm_rule.h"
#include "rom_internal.h"

namespace rom {

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

__device__ __forceinline__ float softplus_f32(float v) { return v > 20.0f ? v : log1pf(__expf(v)); }
// branch-free softplus for the bf16 epilogues: max(v, 0) + log(1 + e) with e = exp(-|v|) in (0, 1].
// Where 1 + e would lose e to rounding, log(1 + e) = e - e^2/2 + ... is replaced by e itself; at the
// switch point (e = 2^-12) either form is within 1.3e-4 relative of the true value, an order of
// magnitude below the bf16 rounding of the stored result.  The raw exp2 / log2 instructions are used
// on purpose: their arguments are never denormal here, so the library's range fix-ups are dead weight
// in an epilogue that is bound by ALU issue.
__device__ __forceinline__ float softplus_fast(float v) {
  const float e = __builtin_amdgcn_exp2f(-1.44269504088896341f * fabsf(v));
  const float lg = __builtin_amdgcn_logf(1.0f + e) * 0.693147180559945309f;
  return fmaxf(v, 0.0f) + (e < 2.44140625e-4f ? e : lg);
}

struct TileCoord {
  int group;
  int64_t row0, row_end;   // sorted positions covered by this tile: [row0, row_end)
  int n0;
  bool valid;
};

// logical tile id -> (global row tile, column tile) in patches of 32 tiles, PM x PN with PN = up
// to 8 column tiles (fewer when the output is narrower), so that workgroups that run together
// share activation row tiles and weight column tiles.
constexpr int kPatchTiles = 32, kPatchNMax = 8;
constexpr bool kXcdRemap = true;    // hand each XCD (workgroup id mod 8) a contiguous run of tiles

__host__ __device__ __forceinline__ int patch_n_for(int n_tiles) {
  int pn = 1;
  while (pn < kPatchNMax && pn < n_tiles) pn *= 2;
  return pn;
}

__device__ __forceinline__ TileCoord locate_tile(const GemmArgs &a, int BM, int BN) {
  TileCoord tc;
  tc.valid = false;
  const int n_tiles = (a.N + BN - 1) / BN;
  const int pn = patch_n_for(n_tiles), pm = kPatchTiles / pn;
  const int patches_n = (n_tiles + pn - 1) / pn;
  const int G = gridDim.x;
  const int bid = blockIdx.x;
  int t = bid;
  if (kXcdRemap && !a.no_xcd_remap && G % 8 == 0) t = (bid % 8) * (G / 8) + bid / 8;
  const int patch = t / kPatchTiles, in_patch = t % kPatchTiles;
  const int mt = (patch / patches_n) * pm + in_patch % pm;
  const int nt = (patch % patches_n) * pn + in_patch / pm;
  if (nt >= n_tiles) return tc;
  tc.n0 = nt * BN;
  if (a.offsets == nullptr) {
    tc.group = 0;
    tc.row0 = static_cast<int64_t>(mt) * BM;
    tc.row_end = a.M;
    tc.valid = tc.row0 < a.M;
  } else {
    int rem = mt;
    for (int e = 0; e < a.n_groups; ++e) {
      const int lo = a.offsets[e], hi = a.offsets[e + 1];
      const int tiles = (hi - lo + BM - 1) / BM;
      if (rem < tiles) {
        tc.group = e;
        tc.row0 = lo + static_cast<int64_t>(rem) * BM;
        tc.row_end = hi;
        tc.valid = true;
        break;
      }
      rem -= tiles;
    }
  }
  if (tc.valid && tc.row_end > tc.row0 + BM) tc.row_end = tc.row0 + BM;
  return tc;
}

// epilogue variants of the MFMA kernel (compile-time, so the store loop has no branches)
enum { kEpiPlain = 0, kEpiBiasSoftplus = 1, kEpiRowScale = 2, kEpiPlainF32 = 3, kEpiRowScaleResidual = 4,
       kEpiSwiGLU = 5 };

__device__ __forceinline__ float finish_out(const GemmArgs &a, int64_t crow, int col, float v) {
  if (a.bias) v += a.bias[col];
  if (a.softplus) v = softplus_f32(v);
  if (a.row_scale) v *= a.row_scale[crow];
  if (a.residual)
    v += a.dtype == ROM_DTYPE_F32 ? static_cast<const float *>(a.residual)[crow * a.ldc + col]
                                  : bf16_to_f32(static_cast<const bf16_t *>(a.residual)[crow * a.ldc + col]);
  return v;
}
__device__ __forceinline__ void store_out(const GemmArgs &a, int64_t crow, int col, float v) {
  v = finish_out(a, crow, col, v);
  if (a.c_is_f32 || a.dtype == ROM_DTYPE_F32)
    static_cast<float *>(a.C)[blockIdx.y * a.c_split_stride + crow * a.ldc + col] = v;
  else
    static_cast<bf16_t *>(a.C)[crow * a.ldc + col] = f32_to_bf16(v);
}
// whether C takes stores of four columns, from every fourth one on
__device__ __forceinline__ bool out_in_fours(const GemmArgs &a) {
  const uintptr_t bytes = a.c_is_f32 || a.dtype == ROM_DTYPE_F32 ? 16 : 8;
  return a.N % 4 == 0 && a.ldc % 4 == 0 && a.c_split_stride % 4 == 0 && reinterpret_cast<uintptr_t>(a.C) % bytes == 0;
}
// columns col .. col + 3 of a row, those that exist; whole: out_in_fours
__device__ __forceinline__ void store_out4(const GemmArgs &a, bool whole, int64_t crow, int col, f32x4_t v) {
  if (col >= a.N) return;
  const bool f32 = a.c_is_f32 || a.dtype == ROM_DTYPE_F32;
  const int64_t at = (f32 ? blockIdx.y * a.c_split_stride : 0) + crow * a.ldc + col;
  const int n = a.N - col < 4 ? a.N - col : 4;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (r < n) v[r] = finish_out(a, crow, col + r, v[r]);
  if (whole && f32) {
    *reinterpret_cast<f32x4_t *>(static_cast<float *>(a.C) + at) = v;
  } else if (whole) {
    *reinterpret_cast<u32x2_t *>(static_cast<bf16_t *>(a.C) + at) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r >= n) continue;
      if (f32) static_cast<float *>(a.C)[at + r] = v[r];
      else static_cast<bf16_t *>(a.C)[at + r] = f32_to_bf16(v[r]);
    }
  }
}

// ------------------------------------------------------------------ bf16 MFMA kernel
constexpr int kBK = 64;                 // K slab, 8 chunks of 8 bf16 (16 bytes) per row
constexpr int kRowChunks = kBK / 8;
// LDS swizzle: chunk c of tile row r lives in slot c ^ lds_swizzle(r) of that row.  Two rows span
// the 64 four-byte banks, and a 16-byte-per-lane read is served 16 lanes (rows) at a time, so 16
// consecutive rows reading the same logical chunk must land in 16 different (row parity, slot)
// pairs; (r & 7) ^ ((r >> 3) & 1) does that and stays conflict-free on 8-row groups as well.
__device__ __forceinline__ int lds_swizzle(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Epilogue shared by the MFMA kernels.  The weight fragment is the MFMA's row operand, so a lane
// holds, for ONE output row (tile row lane%32), the output columns 8*q + 4*(lane/32) + r of each
// 32-wide tile in accumulator element 4*q + r: four consecutive columns per q.
template <int EPI, int TM, int TN, int WTM, int WTN>
__device__ __forceinline__ void mfma_epilogue(const GemmArgs &a, const TileCoord &tc, f32x16_t (&acc)[TM][TN],
                                              uint4 *smem, int wave, int wm, int wn, int lane) {
  const int frag_row = lane & 31, frag_half = lane >> 5;
  if constexpr (EPI == kEpiPlainF32) {
    // fp32 output: one 16-byte store per q straight from the accumulators
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t p = tc.row0 + wm * WTM + i * 32 + frag_row;
      const bool row_ok = p < tc.row_end;
      const int64_t crow = row_ok ? (a.c_rows ? a.c_rows[p] : p) : 0;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = tc.n0 + wn * WTN + j * 32 + q * 8 + frag_half * 4;
          if (row_ok && col < a.N)
            *reinterpret_cast<float4 *>(static_cast<float *>(a.C) + blockIdx.y * a.c_split_stride +
                                        crow * a.ldc + col) =
                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        }
      }
    }
  } else if constexpr (EPI == kEpiSwiGLU) {
    // The weight's rows come in blocks of 16: gate features 8b..8b+7, then up features 8b..8b+7.
    // A lane's accumulator elements 8m..8m+3 and 8m+4..8m+7 of a 32-wide tile are then the gate
    // and the up pre-activation of the same four features of the same row, so
    // SiLU(gate) * up is formed in registers and the output tile is half as wide as the product.
    constexpr int kOutW = WTN / 2;
    constexpr int kPitch = kOutW * 2 + 16;
    char *stage = reinterpret_cast<char *>(smem) + wave * (32 * kPitch);
    constexpr int kChunks = kOutW / 8;
    constexpr int kRowsPerPass = 64 / kChunks;
    const int chunk = lane % kChunks, sub = lane / kChunks;
    const int col = (tc.n0 + wn * WTN) / 2 + chunk * 8;
    const int n_out = a.N / 2;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float scale = 1.0f;
      if (a.row_scale) {                   // pre-norm: 1 / rms of the row, before the activation
        const int64_t p = tc.row0 + wm * WTM + i * 32 + frag_row;
        scale = p < tc.row_end ? a.row_scale[a.c_rows ? a.c_rows[p] : p] : 0.0f;
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          float o[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            o[r] = silu_f32(acc[i][j][8 * m + r] * scale) * (acc[i][j][8 * m + 4 + r] * scale);
          uint2 pk;
          pk.x = pack_bf16x2(o[0], o[1]);
          pk.y = pack_bf16x2(o[2], o[3]);
          const int lcol = (j * 2 + m) * 8 + frag_half * 4;
          *reinterpret_cast<uint2 *>(stage + frag_row * kPitch + lcol * 2) = pk;
        }
      }
#pragma unroll 4
      for (int r0 = 0; r0 < 32; r0 += kRowsPerPass) {
        const int row = r0 + sub;
        const int64_t p = tc.row0 + wm * WTM + i * 32 + row;
        if (row < 32 && p < tc.row_end && col < n_out) {
          const int64_t crow = a.c_rows ? a.c_rows[p] : p;
          const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * kPitch + chunk * 16);
          *reinterpret_cast<uint4 *>(static_cast<bf16_t *>(a.C) + crow * a.ldc + col) = v;
        }
      }
    }
  } else {
    // bf16 output: every wave parks 32 rows of its sub-tile at a time (after bias / softplus / row
    // scale) in its own slice of the now idle LDS, then writes them out row by row, 16 bytes per
    // lane, so that each store instruction covers whole 128..256-byte row segments.  No workgroup
    // barrier is needed: after the last slab's barrier nobody reads the operand buffers for real
    // any more, and LDS serves one wave's accesses in program order.
    constexpr int kPitch = WTN * 2 + 16;                 // bytes per parked row (16-byte aligned)
    char *stage = reinterpret_cast<char *>(smem) + wave * (32 * kPitch);
    constexpr int kChunks = WTN / 8;                     // 16-byte chunks per parked row
    constexpr int kRowsPerPass = 64 / kChunks;
    const int chunk = lane % kChunks, sub = lane / kChunks;
    const int col = tc.n0 + wn * WTN + chunk * 8;
    constexpr int kPasses = (32 + kRowsPerPass - 1) / kRowsPerPass;
    // skip connection: the block's input rows, in the output's layout.  All of them are fetched
    // before the first output store: loads and stores retire through one in-order counter, so a
    // load issued behind a store could only be waited for together with that store.
    u32x4_t res[EPI == kEpiRowScaleResidual ? TM : 1][EPI == kEpiRowScaleResidual ? kPasses : 1];
    if constexpr (EPI == kEpiRowScaleResidual) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int ps = 0; ps < kPasses; ++ps) {
          const int row = ps * kRowsPerPass + sub;
          const int64_t p = tc.row0 + wm * WTM + i * 32 + row;
          res[i][ps] = u32x4_t{0u, 0u, 0u, 0u};
          if (row < 32 && p < tc.row_end && col < a.N) {
            const int64_t crow = a.c_rows ? a.c_rows[p] : p;
            res[i][ps] = *reinterpret_cast<const u32x4_t *>(static_cast<const bf16_t *>(a.residual) +
                                                            crow * a.ldc + col);
          }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float scale = 1.0f;
      if (EPI == kEpiRowScale || EPI == kEpiRowScaleResidual) {
        const int64_t p = tc.row0 + wm * WTM + i * 32 + frag_row;
        // (the residual epilogue without a row scale: accumulation into the output, scale 1)
        scale = p < tc.row_end ? (a.row_scale ? a.row_scale[a.c_rows ? a.c_rows[p] : p] : 1.0f) : 0.0f;
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int lcol = j * 32 + q * 8 + frag_half * 4;
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r];
          if (EPI == kEpiBiasSoftplus) {
            const int bcol = tc.n0 + wn * WTN + lcol;
            float4 b4 = make_float4(0.f, 0.f, 0.f, 0.f);
            if (bcol < a.N) b4 = *reinterpret_cast<const float4 *>(a.bias + bcol);
            v[0] = softplus_fast(v[0] + b4.x); v[1] = softplus_fast(v[1] + b4.y);
            v[2] = softplus_fast(v[2] + b4.z); v[3] = softplus_fast(v[3] + b4.w);
          }
          if (EPI == kEpiRowScale || EPI == kEpiRowScaleResidual) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] *= scale;
          }
          uint2 pk;
          pk.x = pack_bf16x2(v[0], v[1]);
          pk.y = pack_bf16x2(v[2], v[3]);
          *reinterpret_cast<uint2 *>(stage + frag_row * kPitch + lcol * 2) = pk;
        }
      }
      if constexpr (EPI == kEpiRowScaleResidual) {
#pragma unroll
        for (int ps = 0; ps < kPasses; ++ps) {
          const int row = ps * kRowsPerPass + sub;
          const int64_t p = tc.row0 + wm * WTM + i * 32 + row;
          if (row < 32 && p < tc.row_end && col < a.N) {
            const int64_t crow = a.c_rows ? a.c_rows[p] : p;
            uint4 v = *reinterpret_cast<const uint4 *>(stage + row * kPitch + chunk * 16);
            // added to the (already rounded) branch output here, where a lane holds 8 consecutive columns
            unsigned int *vw = &v.x;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const float lo = __uint_as_float(vw[w] << 16) + __uint_as_float(res[i][ps][w] << 16);
              const float hi = __uint_as_float(vw[w] & 0xFFFF0000u) + __uint_as_float(res[i][ps][w] & 0xFFFF0000u);
              vw[w] = pack_bf16x2(lo, hi);
            }
            *reinterpret_cast<uint4 *>(static_cast<bf16_t *>(a.C) + crow * a.ldc + col) = v;
          }
        }
      } else {
#pragma unroll 4
        for (int r0 = 0; r0 < 32; r0 += kRowsPerPass) {
          const int row = r0 + sub;
          const int64_t p = tc.row0 + wm * WTM + i * 32 + row;
          if (row < 32 && p < tc.row_end && col < a.N) {
            const int64_t crow = a.c_rows ? a.c_rows[p] : p;
            const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * kPitch + chunk * 16);
            *reinterpret_cast<uint4 *>(static_cast<bf16_t *>(a.C) + crow * a.ldc + col) = v;
          }
        }
      }
    }
  }
}

// Scheduling hints for one 16-wide step: after MFMA number I, one LDS fragment read (while there
// are any) and this MFMA's share of the LDS writes that park the next slab.
template <int MMA, int READS, int PARKS, bool WITH_PARKS, int I> struct InterleaveHints {
  __device__ static __forceinline__ void run() {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // one MFMA
    if constexpr (I < READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one DS read
    if constexpr (WITH_PARKS) {
      constexpr int lo = I * PARKS / MMA, hi = (I + 1) * PARKS / MMA;
      if constexpr (hi > lo) __builtin_amdgcn_sched_group_barrier(0x200, hi - lo, 0);   // DS writes
    }
    InterleaveHints<MMA, READS, PARKS, WITH_PARKS, I + 1>::run();
  }
};
template <int MMA, int READS, int PARKS, bool WITH_PARKS>
struct InterleaveHints<MMA, READS, PARKS, WITH_PARKS, MMA> {
  __device__ static __forceinline__ void run() {}
};

// PA / PB: how many K slabs ahead the global loads of the activation / weight operand run
// (1 or 2; each extra slab costs one more register set for that operand).
// KTAIL: K is not a multiple of the slab, the last slab is zero-filled past K.
template <int BM, int BN, int WM, int WN, int EPI, bool KTAIL, int PA = 2, int PB = 2>
__global__ __launch_bounds__(WM *WN * 64) void gemm_bf16_mfma_kernel(const GemmArgs a) {
  constexpr int NT = WM * WN * 64;
  constexpr int WTM = BM / WM, WTN = BN / WN;       // wave tile
  constexpr int TM = WTM / 32, TN = WTN / 32;       // 32x32 MFMA tiles per wave
  constexpr int A_CH = BM * kRowChunks / NT, B_CH = BN * kRowChunks / NT;
  static_assert(BM * kRowChunks % NT == 0 && BN * kRowChunks % NT == 0, "tile/threads mismatch");
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of 32");

  extern __shared__ __attribute__((aligned(16))) uint4 smem[];
  uint4 *As = smem;                                  // [2][BM * 8] chunks
  uint4 *Bs = smem + 2 * BM * kRowChunks;            // [2][BN * 8] chunks

  const TileCoord tc = locate_tile(a, BM, BN);
  if (!tc.valid) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  const bf16_t *Ap = static_cast<const bf16_t *>(a.A);
  const bf16_t *Wp = static_cast<const bf16_t *>(a.W) + static_cast<int64_t>(tc.group) * a.N * a.K;

  // global source of every 16-byte chunk this thread stages.  Rows past the end of the tile are
  // redirected to its first row (their results are never stored), so the loads need no branch;
  // a K tail is zero-filled by a select.
  // (32-bit element offsets from the operand bases: the launcher checks that both operands span
  // less than 2^32 elements, and registers are scarce here)
  uint32_t a_src[A_CH], b_src[B_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    const int q = tid + i * NT, r = q / kRowChunks;
    int64_t p = tc.row0 + r;
    if (p >= tc.row_end) p = tc.row0;
    a_src[i] = static_cast<uint32_t>((a.a_rows ? a.a_rows[p] : p) * a.lda);
  }
#pragma unroll
  for (int i = 0; i < B_CH; ++i) {
    const int q = tid + i * NT, r = q / kRowChunks;
    const int n = (tc.n0 + r < a.N) ? tc.n0 + r : a.N - 1;
    b_src[i] = static_cast<uint32_t>(n) * static_cast<uint32_t>(a.K);
  }
  // split-K: grid.y slices of k_per_split inner-dimension elements, each with its own fp32 output
  const int k_begin = blockIdx.y * a.k_per_split;
  const int k_len = (a.K - k_begin < a.k_per_split) ? a.K - k_begin : a.k_per_split;
  const int k_chunk = k_begin + (tid % kRowChunks) * 8;
  const int k_last = k_begin + k_len - 8;

  // Register sets for slabs in flight: with depth 2 the global loads of slab kt+2 are issued while
  // slab kt is multiplied, so they have two slab times to land before they are parked in LDS
  // (HBM latency is longer than one slab of MFMA work).
  // (separate arrays with compile-time selection: the compiler keeps them in registers only if
  // every index is a constant and the arrays are never passed around by reference)
  uint4 ra0[A_CH], ra1[A_CH], rb0[B_CH], rb1[B_CH];
  auto load_a = [&](int k0, auto set) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
    const int k = k0 + k_chunk;
    const bool k_ok = !KTAIL || k <= k_last;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (!KTAIL || k0 + kBK <= k_len) v = *reinterpret_cast<const uint4 *>(Ap + a_src[i] + k);
      else if (k_ok) v = *reinterpret_cast<const uint4 *>(Ap + a_src[i] + k);
      if constexpr (S == 0) ra0[i] = v; else ra1[i] = v;
    }
  };
  // 64-row tiles serve launches with a few rows per expert (the recurrent step): every weight is
  // used once or twice, so it is streamed past the caches (non-temporal) and the activations,
  // states and routing arrays keep their place in L2 / the infinity cache (measured: -10 % per step)
  constexpr bool kStreamW = BM == 64;
  auto load_w = [&](const bf16_t *src) __attribute__((always_inline)) {
    if constexpr (kStreamW) {
      const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src));
      return make_uint4(t.x, t.y, t.z, t.w);
    } else {
      return *reinterpret_cast<const uint4 *>(src);
    }
  };
  auto load_b = [&](int k0, auto set) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
    const int k = k0 + k_chunk;
    const bool k_ok = !KTAIL || k <= k_last;
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      uint4 v = make_uint4(0, 0, 0, 0);
      if (!KTAIL || k0 + kBK <= k_len) v = load_w(Wp + b_src[i] + k);
      else if (k_ok) v = load_w(Wp + b_src[i] + k);
      if constexpr (S == 0) rb0[i] = v; else rb1[i] = v;
    }
  };
  auto park_a = [&](int buf, auto set) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int q = tid + i * NT, r = q / kRowChunks, c = q % kRowChunks;
      uint4 v;
      if constexpr (S == 0) v = ra0[i]; else v = ra1[i];
      As[buf * BM * kRowChunks + r * kRowChunks + (c ^ lds_swizzle(r))] = v;
    }
  };
  auto park_b = [&](int buf, auto set) __attribute__((always_inline)) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int q = tid + i * NT, r = q / kRowChunks, c = q % kRowChunks;
      uint4 v;
      if constexpr (S == 0) v = rb0[i]; else v = rb1[i];
      Bs[buf * BN * kRowChunks + r * kRowChunks + (c ^ lds_swizzle(r))] = v;
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  const int KT = (k_len + kBK - 1) / kBK;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  // LDS chunk index of this lane's fragment for 16-wide K step kk: row * 8 + ((2 kk + half) ^ swizzle(row));
  // the wave / tile row offsets are multiples of 32, so the swizzle term depends on the lane only.
  const int a_base = (wm * WTM + frag_row) * kRowChunks, b_base = (wn * WTN + frag_row) * kRowChunks;
  const int swz = lds_swizzle(frag_row);

  bf16x8_t fa[2][TM], fb[2][TN];
  auto load_frags = [&](int buf, int kk, bf16x8_t(&af)[TM], bf16x8_t(&bfr)[TN]) __attribute__((always_inline)) {
    const int c = (kk * 2 + frag_half) ^ swz;
    const uint4 *Ab = As + buf * BM * kRowChunks + a_base + c;
    const uint4 *Bb = Bs + buf * BN * kRowChunks + b_base + c;
    // issue order = order of first use by mma(): A row 0, then every B column, then the other A rows
    {
      const uint4 v = Ab[0];
      af[0] = *reinterpret_cast<const bf16x8_t *>(&v);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint4 v = Bb[j * 32 * kRowChunks];
      bfr[j] = *reinterpret_cast<const bf16x8_t *>(&v);
    }
#pragma unroll
    for (int i = 1; i < TM; ++i) {
      const uint4 v = Ab[i * 32 * kRowChunks];
      af[i] = *reinterpret_cast<const bf16x8_t *>(&v);
    }
  };
  auto mma = [&](const bf16x8_t(&af)[TM], const bf16x8_t(&bfr)[TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
  };
  // ask the scheduler to put the next step's LDS fragment reads (and, in one step per slab, the
  // LDS writes that park the next slab) between the MFMAs of this step, one per MFMA
  auto interleave = [&](auto with_parks) __attribute__((always_inline)) {
    InterleaveHints<TM * TN, TM + TN, A_CH + B_CH, decltype(with_parks)::value, 0>::run();
  };

  load_a(0, Set0{});
  load_b(0, Set0{});
  park_a(0, Set0{});
  park_b(0, Set0{});
  const int k_end = (KT - 1) * kBK;      // loads past the last slab are redirected to it (and never used)
  if (PA == 2) load_a(kBK < k_end ? kBK : k_end, Set1{});
  if (PB == 2) load_b(kBK < k_end ? kBK : k_end, Set1{});
  __syncthreads();
  load_frags(0, 0, fa[0], fb[0]);

  // One K slab, free of conditionals: PAR = kt & 1 selects the LDS buffer being read; slab s of an
  // operand with depth P travels in register set s % P.  The slab after the last one is "loaded"
  // and parked like any other (clamped address, buffer nobody reads again).
  auto slab = [&](int kt, auto par) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par)::value;
    using LoadA = std::integral_constant<int, PA == 2 ? PAR : 0>;
    using LoadB = std::integral_constant<int, PB == 2 ? PAR : 0>;
    using ParkA = std::integral_constant<int, PA == 2 ? (PAR ^ 1) : 0>;
    using ParkB = std::integral_constant<int, PB == 2 ? (PAR ^ 1) : 0>;
    const int ka = (kt + PA) * kBK, kb = (kt + PB) * kBK;
    load_a(ka < k_end ? ka : k_end, LoadA{});
    load_b(kb < k_end ? kb : k_end, LoadB{});
    // The next slab (loaded while the previous one was multiplied) is parked in the middle of
    // this slab, its LDS writes spread between MFMAs, instead of in a burst before the barrier.
    constexpr int kParkAt = 3;       // 0..2: interleaved with that 16-wide step; 3: after the third step.
                                     // Measured: any earlier than 3 stalls on the loads still in flight.
    load_frags(PAR, 1, fa[1], fb[1]);
    if (kParkAt == 0) { park_a(PAR ^ 1, ParkA{}); park_b(PAR ^ 1, ParkB{}); }
    mma(fa[0], fb[0]);
    interleave(std::bool_constant<kParkAt == 0>{});
    load_frags(PAR, 2, fa[0], fb[0]);
    if (kParkAt == 1) { park_a(PAR ^ 1, ParkA{}); park_b(PAR ^ 1, ParkB{}); }
    mma(fa[1], fb[1]);
    interleave(std::bool_constant<kParkAt == 1>{});
    load_frags(PAR, 3, fa[1], fb[1]);
    if (kParkAt == 2) { park_a(PAR ^ 1, ParkA{}); park_b(PAR ^ 1, ParkB{}); }
    mma(fa[0], fb[0]);
    interleave(std::bool_constant<kParkAt == 2>{});
    if (kParkAt == 3) { park_a(PAR ^ 1, ParkA{}); park_b(PAR ^ 1, ParkB{}); }
    // every fragment of this slab is in registers and the next slab is parked: overlap the fetch
    // of its first fragments with the last 16-wide step of this one
    __syncthreads();
    load_frags(PAR ^ 1, 0, fa[0], fb[0]);
    mma(fa[1], fb[1]);
  };
  int kt = 0;
  for (; kt + 1 < KT; kt += 2) {
    slab(kt, Set0{});
    slab(kt + 1, Set1{});
  }
  if (kt < KT) slab(kt, Set0{});

  mfma_epilogue<EPI, TM, TN, WTM, WTN>(a, tc, acc, smem, wave, wm, wn, lane);
}

// ------------------------------------------------------------------ bf16 MFMA kernel, LDS-DMA loads
// The operand slabs travel from global memory straight into LDS (global_load_lds_dwordx4: lane l of
// a wave deposits its 16 bytes at M0 + 16 l), so no registers, no LDS-write instructions and no
// load->store dependency sit in the MFMA loop.
// K is walked in 64-wide slabs so that every row contributes one whole 128-byte cache line per
// slab.  A slab is two "half slabs" of up to 32 KiB (the A rows, then the W rows) and LDS is a
// ring of five such slots: while slab m (two slots) is multiplied, A(m+1), W(m+1) and A(m+2) are in
// flight or landed; the barrier before the last 16-wide step of slab m frees its two slots, which
// then receive W(m+2) and A(m+3).
// The XOR swizzle is applied on the global side: the lane that fills 16-byte position c' of row r
// fetches chunk c' ^ ((r >> 1) & 7), which keeps the 16-lane fragment reads conflict-free for
// 128-byte rows.  The compiler does not see these loads (inline asm), so the waits are explicit:
// every wave issues the same number of loads per half slab, in ring order, and a vmcnt of that number
// therefore means "everything but the newest half slab I asked for has landed".
// dma_tile is one tile of that kind: 256 rows of one narrow column tile (fp32, 161 to 192 columns), a whole 256 x 256 one for the
// epilogues that the stream kernel has not, and the pieces of the stream kernel's last round.
constexpr int kDmaBK = 64, kDmaRC = kDmaBK / 8, kDmaSlots = 5;
constexpr bool kUseDma = true;
constexpr int kSkinnyMinWgs = 100;
constexpr int kSkinnyColsMaxWgs = 600;    // fewer 64 x 128 tiles than this (about two per CU): 64 x 64 tiles instead
constexpr bool kUseSmallK = true;

__device__ __forceinline__ void dma_load_16(unsigned lds_addr, unsigned voff, const void *base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n"
               :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}

// BN < 256 or BM < 256 keep the five 32 KiB ring slots; the half slabs just fill less of theirs.
// grid.y slices the inner dimension (fp32 partial sums, plain epilogue only).
// WT: the weight is stored contraction-major, [group][K][N] (a forward weight used for the input
// gradient without a transposed copy; BN = 128 or 256, N a multiple of 256).  Its half slab is then 64
// contraction rows x BN output columns as they lie in memory, 512 / BN rows per DMA instruction, chunk c
// of row r at position c ^ 4 (r & 3), and the MFMA fragments - eight consecutive contraction indices of
// one output column per lane - come out of it through the transposing LDS read (ds_read_b64_tr_b16:
// the 16 lanes of a group name four rows x 16 columns, lane i receives column i of the four rows).
template <int BN, int WM, int WN, int EPI, bool WT = false, int BM = 256>
__device__ __forceinline__ void dma_tile(const GemmArgs &a, const TileCoord &tc, uint4 *smem) {
  constexpr int NW = WM * WN;
  static_assert(kDmaSlots == 5, "ring of five half-slab slots");
  static_assert((NW == 16 || NW == 8 || NW == 4) && BN <= 256 && BM <= 256 && BN % (32 * WN) == 0, "4, 8 or 16 waves, 32-wide MFMA tiles");
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int kSlotChunks = 256 * kDmaRC;                   // 16-byte chunks per ring slot
  constexpr int kSlotBytes = kSlotChunks * 16;                // 32 KiB
  constexpr int kAInstr = BM / (8 * NW);                      // DMA instructions per wave and half slab: 8 rows each
  constexpr int kWInstr = (BN + 8 * NW - 1) / (8 * NW);       // (rows past BN are clamped re-reads into unused slot space)
  static_assert(!WT || BN == 256 || BN == 128, "contraction-major weights: a row's chunks cover the banks in whole rounds");
  constexpr int kWtChunks = BN / 8;                           // 16-byte chunks per contraction row of a contraction-major W

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  const int k_begin = blockIdx.y * a.k_per_split;
  const int k_len = (a.K - k_begin < a.k_per_split) ? a.K - k_begin : a.k_per_split;
  const bf16_t *Ap = static_cast<const bf16_t *>(a.A) + k_begin;
  const bf16_t *Wp = static_cast<const bf16_t *>(a.W) + static_cast<int64_t>(tc.group) * a.N * a.K +
                     (WT ? static_cast<int64_t>(k_begin) * a.N : k_begin);

  // this lane's share of a half slab: one 16-byte chunk in each of its wave's 8-row groups
  unsigned a_voff[kAInstr], b_voff[kWInstr];
#pragma unroll
  for (int j = 0; j < kAInstr; ++j) {
    const int r = (wave * kAInstr + j) * 8 + (lane >> 3);      // tile row filled by this lane
    const int c = (lane & 7) ^ ((r >> 1) & 7);                 // global chunk that belongs in its position
    int64_t p = tc.row0 + r;
    if (p >= tc.row_end) p = tc.row0;                          // rows past the tile: never stored
    a_voff[j] = static_cast<unsigned>(((a.a_rows ? a.a_rows[p] : p) * a.lda + c * 8) * 2);
  }
#pragma unroll
  for (int j = 0; j < kWInstr; ++j) {
    if constexpr (WT) {
      const int r = (wave * kWInstr + j) * (64 / kWtChunks) + lane / kWtChunks;    // contraction row within the slab
      const int c = (lane % kWtChunks) ^ (4 * (r & 3));
      b_voff[j] = static_cast<unsigned>((static_cast<int64_t>(r) * a.N + tc.n0 + c * 8) * 2);
    } else {
      const int r = (wave * kWInstr + j) * 8 + (lane >> 3);
      const int c = (lane & 7) ^ ((r >> 1) & 7);
      const int n = (tc.n0 + r < a.N) ? tc.n0 + r : a.N - 1;
      b_voff[j] = static_cast<unsigned>((static_cast<int64_t>(n) * a.K + c * 8) * 2);
    }
  }
  const unsigned lds_base =
      static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void *)smem));
  const unsigned lds_wave_a = __builtin_amdgcn_readfirstlane(lds_base + wave * (kAInstr * 1024));
  const unsigned lds_wave_w = __builtin_amdgcn_readfirstlane(lds_base + wave * (kWInstr * 1024));
  const int KT = k_len / kDmaBK;

  // DMA instruction j of half slab h: the A rows (h even) or the W rows (h odd) of slab h / 2, into ring slot h % 5
  auto issue1 = [&](int h, int j) __attribute__((always_inline)) {
    const int m = h >> 1;
    const int sl = m < KT ? m : KT - 1;                        // past the end: harmless reload
    const unsigned slot = static_cast<unsigned>(h % kDmaSlots) * kSlotBytes;
    if (h & 1) dma_load_16(lds_wave_w + slot + j * 1024, b_voff[j], Wp + static_cast<int64_t>(sl) * kDmaBK * (WT ? a.N : 1));
    else dma_load_16(lds_wave_a + slot + j * 1024, a_voff[j], Ap + sl * kDmaBK);
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int a_base = (wm * WTM + frag_row) * kDmaRC, b_base = (wn * WTN + frag_row) * kDmaRC;
  const int swz = (frag_row >> 1) & 7;
  // contraction-major W: byte offset of this lane's 8 bytes in the first of its two 4-row reads
  unsigned wt_off[TN];
  if constexpr (WT) {
    const int i16 = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int chunk = (wn * (WTN / 8) + j * 4 + 2 * (grp & 1) + ((i16 >> 1) & 1)) ^ (4 * (i16 >> 2));
      wt_off[j] = static_cast<unsigned>((8 * (grp >> 1) + (i16 >> 2)) * (2 * BN) + chunk * 16 + (i16 & 1) * 8);
    }
  }
  bf16x8_t fa0[TM], fa1[TM], fb0[TN], fb1[TN];
  auto read_a = [&](int m, int kk, int i) __attribute__((always_inline)) {
    const uint4 v = smem[((2 * m) % kDmaSlots) * kSlotChunks + a_base + i * 32 * kDmaRC + ((kk * 2 + frag_half) ^ swz)];
    return *reinterpret_cast<const bf16x8_t *>(&v);
  };
  auto read_w = [&](int m, int kk, int j) __attribute__((always_inline)) {
    const uint4 *sb = smem + ((2 * m + 1) % kDmaSlots) * kSlotChunks;
    if constexpr (WT) {
      typedef short i16x4_t __attribute__((ext_vector_type(4)));
      typedef short i16x8_t __attribute__((ext_vector_type(8)));
      typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
      const __attribute__((address_space(3))) unsigned char *pb =
          (const __attribute__((address_space(3))) unsigned char *)sb + kk * (16 * 2 * BN) + wt_off[j];
      const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)pb);
      const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(pb + 4 * 2 * BN));
      return __builtin_bit_cast(bf16x8_t, (i16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      const uint4 v = sb[b_base + j * 32 * kDmaRC + ((kk * 2 + frag_half) ^ swz)];
      return *reinterpret_cast<const bf16x8_t *>(&v);
    }
  };
  // One 16-wide step: between its MFMAs, one by one and held there by scheduling fences, the fragment reads of the next
  // step (step kn of slab mn) and DMA instructions j0 .. j1 - 1 of half slab h.  All DMA of a slab issued at once behind
  // its barrier fills the L1's request queue and blocks the wavefronts at issue.
  constexpr int kMma = TM * TN, kReads = TM + TN;
  auto step = [&](const bf16x8_t(&fa)[TM], const bf16x8_t(&fb)[TN], bf16x8_t(&na)[TM], bf16x8_t(&nb)[TN], int mn, int kn, int h,
                  int j0, int j1) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < kMma; ++q) {
      acc[q / TN][q % TN] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[q % TN], fa[q / TN], acc[q / TN][q % TN], 0, 0, 0);
      // in the order of first use: A row 0, the W columns, the other A rows (the last MFMA takes what is left over)
#pragma unroll
      for (int r = q; r < (q == kMma - 1 ? kReads : q + 1) && r < kReads; ++r) {
        if (r == 0) na[0] = read_a(mn, kn, 0);
        else if (r <= TN) nb[r - 1] = read_w(mn, kn, r - 1);
        else na[r - TN] = read_a(mn, kn, r - TN);
      }
#pragma unroll
      for (int j = j0 + (j1 - j0) * q / kMma; j < j0 + (j1 - j0) * (q + 1) / kMma; ++j) issue1(h, j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // A(0), W(0), A(1) and half of W(1): the loop requests the rest
  constexpr int kWh = (kWInstr + 1) / 2, kAh = (kAInstr + 1) / 2;
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int j = 0; j < (h == 3 ? kWh : (h & 1) ? kWInstr : kAInstr); ++j) issue1(h, j);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kAInstr + kWh) : "memory");     // slab 0 is in LDS
  fa0[0] = read_a(0, 0, 0);
#pragma unroll
  for (int j = 0; j < TN; ++j) fb0[j] = read_w(0, 0, j);
#pragma unroll
  for (int i = 1; i < TM; ++i) fa0[i] = read_a(0, 0, i);

  for (int m = 0; m < KT; ++m) {
    step(fa0, fb0, fa1, fb1, m, 1, 2 * m + 3, kWh, kWInstr);      // second half of W(m+1)
    step(fa1, fb1, fa0, fb0, m, 2, 2 * m + 4, 0, kAh);            // A(m+2)
    step(fa0, fb0, fa1, fb1, m, 3, 2 * m + 4, kAh, kAInstr);
    // slab m+1 has landed for everyone (only A(m+2) is outstanding) and nobody reads slab m any more
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kAInstr) : "memory");
    step(fa1, fb1, fa0, fb0, m + 1, 0, 2 * m + 5, 0, kWh);        // first half of W(m+2)
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // LDS is reused by the epilogue
  mfma_epilogue<EPI, TM, TN, WTM, WTN>(a, tc, acc, smem, wave, wm, wn, lane);
}

template <int BN, int WM, int WN, int EPI>
__global__ __launch_bounds__(WM *WN * 64) void gemm_bf16_dma_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint4 smem[];
  const TileCoord tc = locate_tile(a, 256, BN);
  if (!tc.valid) return;
  dma_tile<BN, WM, WN, EPI>(a, tc, smem);
}

// ------------------------------------------------------------------ bf16 MFMA kernel, few rows
// A few sequences' recurrent step (kGemmFewRows positions at most; a row tile holds 16): the call is one pass over the weights of the picked
// experts, bound by how much of it is in flight.  The 64-row tiles of the general kernel park 64 rows for the one or two
// that exist, walk K serially with two slabs in flight and a barrier each.  Here a workgroup of eight wavefronts owns
// 16 CT output columns of one expert's rows (CT = 2 from kFewWideCols columns on); the wavefronts deal the 64-wide units
// of K among themselves, read both operands straight into fragments (no LDS, no barrier; four units of both requested at
// once), and their partial sums are added through LDS in wavefront order.  The weight is the MFMA's row operand: lane
// (c, g) ends with columns 4 g .. 4 g + 3 of position c.  Positions past the group's end repeat its first row and are not
// stored.  One sequence, d_model 2048: with 64 x 64 tiles the in and out projections take 30 us each of a step of 94 us;
// the step took 55 us through twelve layers in turn with this kernel, 47 (91) with one layer whose expert the last step has
// just read; 36 since the launches behind the x projection are one (step_tail_kernel).
constexpr int kFewWideCols = 4096;
constexpr int kFewWaves = 8;
typedef float f32x4_few_t __attribute__((ext_vector_type(4)));

// UNITS: 64-wide units that a wavefront requests together.
template <int CT, int EPI, int UNITS>
__global__ __launch_bounds__(kFewWaves * 64) void gemm_bf16_few_rows_kernel(const GemmArgs a) {
  __shared__ float red[kFewWaves][CT][16][20];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  // blockIdx.z -> the z-th group that has a row: a lane per group (n_groups <= 64)
  int group = 0, row0 = 0, row_end = static_cast<int>(a.M);
  if (a.offsets) {
    const int e = lane < a.n_groups ? lane : a.n_groups - 1;
    const int lo = a.offsets[e], hi = a.offsets[e + 1];
    unsigned long long used = __ballot(lane < a.n_groups && hi > lo);
    for (unsigned skip = blockIdx.z; skip > 0 && used; --skip) used &= used - 1;
    if (used == 0) return;                                     // fewer such groups than the grid allows for
    group = __builtin_ctzll(used);
    row0 = __shfl(lo, group);
    row_end = __shfl(hi, group);
  }
  const int n0 = blockIdx.x * (16 * CT);
  const int k0 = blockIdx.y * a.k_per_split;
  const int k_end = k0 + a.k_per_split < a.K ? k0 + a.k_per_split : a.K;
  const int units = (k_end - k0) / 64;
  const int p_in = row0 + c < row_end ? row0 + c : row0;
  const bf16_t *Ap = static_cast<const bf16_t *>(a.A) + (a.a_rows ? a.a_rows[p_in] : p_in) * a.lda + k0 + 8 * g;
  const bf16_t *Wp[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int n = n0 + 16 * t + c < a.N ? n0 + 16 * t + c : a.N - 1;
    Wp[t] = static_cast<const bf16_t *>(a.W) + (static_cast<int64_t>(group) * a.N + n) * a.K + k0 + 8 * g;
  }
  f32x4_few_t acc[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) acc[t] = f32x4_few_t{0.0f, 0.0f, 0.0f, 0.0f};
  for (int u0 = wave; u0 < units; u0 += kFewWaves * UNITS) {
    bf16x8_t fw[UNITS][CT][2], fx[UNITS][2];
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
      const int u = u0 + i * kFewWaves < units ? u0 + i * kFewWaves : u0;      // past the end: re-read, not multiplied
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int t = 0; t < CT; ++t) fw[i][t][h] = *reinterpret_cast<const bf16x8_t *>(Wp[t] + u * 64 + h * 32);
        fx[i][h] = *reinterpret_cast<const bf16x8_t *>(Ap + u * 64 + h * 32);
      }
    }
    __builtin_amdgcn_sched_barrier(0);                         // all requests ahead of the first wait
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
      if (u0 + i * kFewWaves < units) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int t = 0; t < CT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i][t][h], fx[i][h], acc[t], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < CT; ++t) *reinterpret_cast<f32x4_few_t *>(&red[wave][t][c][4 * g]) = acc[t];
  __syncthreads();
  const int row = tid / (16 * CT), lc = tid % (16 * CT);
  if (row >= 16 || row0 + row >= row_end || n0 + lc >= a.N) return;
  const auto total = [&](int t, int q) __attribute__((always_inline)) {
    float v = red[0][t][row][q];
#pragma unroll
    for (int w = 1; w < kFewWaves; ++w) v += red[w][t][row][q];
    return v;
  };
  const int64_t crow = a.c_rows ? a.c_rows[row0 + row] : row0 + row;
  float v = total(lc >> 4, lc & 15);
  if constexpr (EPI == kEpiPlainF32) {
    static_cast<float *>(a.C)[blockIdx.y * a.c_split_stride + crow * a.ldc + n0 + lc] = v;
  } else if constexpr (EPI == kEpiSwiGLU) {                    // a block of 16 columns: 8 gate, then their 8 up features
    if ((lc & 15) >= 8) return;
    const float scale = a.row_scale ? a.row_scale[crow] : 1.0f;
    const float up = total(lc >> 4, (lc & 15) + 8);
    static_cast<bf16_t *>(a.C)[crow * a.ldc + (n0 + lc - (lc & 15)) / 2 + (lc & 15)] =
        f32_to_bf16(silu_f32(v * scale) * (up * scale));
  } else {
    if constexpr (EPI == kEpiRowScale || EPI == kEpiRowScaleResidual) v *= a.row_scale ? a.row_scale[crow] : 1.0f;
    bf16_t o = f32_to_bf16(v);
    if constexpr (EPI == kEpiRowScaleResidual)                 // added to the rounded branch output, as in mfma_epilogue
      o = f32_to_bf16(bf16_to_f32(o) + bf16_to_f32(static_cast<const bf16_t *>(a.residual)[crow * a.ldc + n0 + lc]));
    static_cast<bf16_t *>(a.C)[crow * a.ldc + n0 + lc] = o;
  }
}

// ------------------------------------------------------------------ bf16 MFMA kernel, one stream of slabs per CU
// The large routed projections: bound by the power the matrix pipe draws (a slab of random operands takes 1.5 us, of zeros
// 1.05; its MFMAs 0.85 us at 2.4 GHz, 1.0 at the 2.06 that the clock falls to), then by what stands between two tiles.  Of
// 16384 rows x 8192 x 2048 a launch without stores and epilogue takes 405 us.  With both, counted with the cycle counter per
// tile (32 slabs of 2420 cycles): a wavefront alone on its SIMD issues an instruction every five cycles, the L2 of an XCD
// takes about 16 bytes a cycle from each of its CUs when all store at once, and a wait for a register that came from memory
// drains the ring.  Hence: the stores spread over eight slabs, each covering 64 bytes of a row; everything else that a tile
// needs (row numbers, scales, the place of a later tile, offsets) between MFMAs; nothing spilled, but for one register with row
// scale and skip.  91.9 k cycles a tile (14.5 k more than its slabs) -> 84 k; the matrix pipe is busy for 65 % of a launch of
// 8192 columns x 2048 (56 % before) and 58 % of 2048 x 4096 (54 %).  16384 rows in 8 even groups, against the same kernel without this: 8192 x 512
// 167 -> 139 us, x 1024 276 -> 248, x 2048 467 -> 445, 2048 x 4096 217 -> 209; SwiGLU 4096 x 1024 144 -> 131; contraction-major
// 4096 x 2048 257 -> 245.
// One workgroup of four wavefronts per CU (2 x 2, 128 x 128 each: 256 accumulator
// registers, a third less LDS traffic per flop than eight 64 x 128 ones) walks its share of the 256 x 256 tiles; the ring
// of five half-slab slots above runs on across tile boundaries: the last two slabs of a tile already request the next
// tile's, so that between tiles only the epilogue (registers -> bf16 -> stores, no LDS) stops the matrix pipe.
//   * a 64-wide slab is four 16-wide steps of 16 MFMAs; between them, one by one and held there by scheduling fences,
//     the eight fragment reads of the next step and four DMA instructions.  All DMA issued at once behind the slab's
//     barrier (16 per wavefront) fills the L1's request queue and blocks the wavefront at issue.
//   * the workgroups that share an activation (weight) tile request its rows in rotated order: each line's first
//     request, the one that waits for HBM, comes from another CU, and the others find it in L2.
//   * tiles are dealt out from the device-side tile count, an equal contiguous run per XCD in patches of 4 x 8 tiles.
// Slab m's schedule, P = the one barrier per slab (slab m + 1 landed, slab m in registers):
//   step 0: W(m+1) second half | 1, 2: A(m+2) | P | 3: W(m+2) first half, first fragments of slab m + 1
// Rows past a group's end re-read the tile's first row and store that row's result over itself, so that every
// wavefront's requests for activations are whole.  Half of a tile's stores go out at once, the rest two a slab behind the
// barriers of the next slabs: loads and stores retire in order, and 128 KiB per CU at one time keep the L2 busy for longer
// than the ring lasts.
// An XCD's tiles rarely fill a whole number of rounds: its last, partial round is cut into 2, 4 or 8 pieces a tile, as
// many as give every CU one (dma_tile), and pieces without a row of their group do nothing.
struct StreamTile {
  int group, row0, row_end, n0;
};

template <int EPI, bool WT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_stream_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint4 smem[];
  constexpr int TM = 4, TN = 4, NI = 8;                       // NI: DMA instructions per wavefront and half slab
  constexpr unsigned kSlotBytes = 256 * kDmaBK * 2;           // 32 KiB
  constexpr int kPieces = EPI == kEpiSwiGLU ? TN : 2 * TN;    // 16-byte stores per lane and 32-row block

  // ---- this workgroup's tiles
  // Lane e keeps where group e's tiles end, and the group's rows: finding a tile's group is a ballot, not a walk over the
  // offsets in memory.
  const int n_tiles = (a.N + 255) / 256;
  static_assert(kMaxExperts <= 64, "a group a lane");
  int m_tiles, grp_end, grp_lo, grp_hi;
  {
    const int e = threadIdx.x & 63;
    const bool have = a.offsets != nullptr && e < a.n_groups;
    grp_lo = have ? a.offsets[e] : 0;
    grp_hi = have ? a.offsets[e + 1] : a.offsets == nullptr && e == 0 ? static_cast<int>(a.M) : 0;
    grp_end = (grp_hi - grp_lo + 255) / 256;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const int below = __shfl_up(grp_end, d);
      if (e >= d) grp_end += below;
    }
    m_tiles = __builtin_amdgcn_readlane(grp_end, 63);
  }
  const int pn = patch_n_for(n_tiles), pm = kPatchTiles / pn;
  const int xcd = blockIdx.x % 8, cu = blockIdx.x / 8, cus = gridDim.x / 8;
  const int64_t total = static_cast<int64_t>(m_tiles) * n_tiles;
  const int tile_lo = static_cast<int>(total * xcd / 8), tile_hi = static_cast<int>(total * (xcd + 1) / 8);
  // x / d for 0 <= x < 2^31 with inv = ceil(2^32 / d), d > 1: the product is less than half too large
  auto inverse = [](int d) { return d > 1 ? 0xFFFFFFFFu / static_cast<unsigned>(d) + 1u : 0u; };
  auto divide = [](int x, int d, unsigned inv) __attribute__((always_inline)) {
    if (d == 1) return x;
    const int q = static_cast<int>(__umulhi(static_cast<unsigned>(x), inv));
    return q * d > x ? q - 1 : q;
  };
  const int band_tiles = pm * n_tiles, last_rows = m_tiles % pm;
  const unsigned inv_band = inverse(band_tiles), inv_pm = inverse(pm), inv_last = inverse(last_rows);
  const int pn_log2 = __builtin_ctz(pn);
  // in stages short enough to stand between two MFMAs
  struct Finder {
    int t, band, rows, in, in_col, mt;
    StreamTile tl;
  };
  auto locate_stage = [&](Finder &f, int stage) __attribute__((always_inline)) {
    if (stage == 0) {
      f.band = divide(f.t, band_tiles, inv_band);             // pm tile rows (fewer in the last band) x all columns
      f.rows = m_tiles - f.band * pm >= pm ? pm : last_rows;
    } else if (stage == 1) {
      const int r = f.t - f.band * band_tiles, patch = divide(r >> pn_log2, f.rows, f.rows == pm ? inv_pm : inv_last);
      f.in = r - patch * (f.rows << pn_log2);
      f.tl.n0 = (patch << pn_log2) * 256;
    } else if (stage == 2) {
      f.in_col = divide(f.in, f.rows, f.rows == pm ? inv_pm : inv_last);
      f.mt = f.band * pm + f.in - f.in_col * f.rows;
      f.tl.n0 += f.in_col * 256;
    } else if (stage == 3) {
      f.tl.group = __builtin_popcountll(__ballot(grp_end <= f.mt));
    } else if (stage == 4) {
      f.tl.row0 = __builtin_amdgcn_readlane(grp_lo, f.tl.group);
      f.tl.row_end = __builtin_amdgcn_readlane(grp_hi, f.tl.group);
    } else if (stage == 5) {                                  // the group's first tile: its end less its tiles
      const int first = __builtin_amdgcn_readlane(grp_end, f.tl.group) - (f.tl.row_end - f.tl.row0 + 255) / 256;
      f.tl.row0 += (f.mt - first) * 256;
      if (f.tl.row_end > f.tl.row0 + 256) f.tl.row_end = f.tl.row0 + 256;
    }
  };
  auto locate = [&](int t) __attribute__((always_inline)) {
    Finder f;
    f.t = t;
#pragma unroll
    for (int stage = 0; stage < 6; ++stage) locate_stage(f, stage);
    return f.tl;
  };
  const int rounds = (tile_hi - tile_lo) / cus, rest = (tile_hi - tile_lo) % cus;
  // pieces per tile of the last round: 1 (then it is a round like the others), 2, 4 or 8
  const int cut = rest == 0 || rest * 2 > cus ? 1 : rest * 4 > cus ? 2 : rest * 8 > cus ? 4 : 8;
  const int tile_end = cut == 1 ? tile_hi : tile_lo + rounds * cus;
  int t = tile_lo + cu;
  if (t < tile_end) {

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int KT = a.K / kDmaBK;

  // ---- DMA side.  Instruction j of a half slab fills 1 KiB block (4 j + wave + rotation) mod 32 of its slot: eight rows
  // of 128 bytes (contraction-major W: two rows of 512)
  const int rot_a = (cu / pm % pn) * (32 / pn), rot_w = (cu % pm) * (32 / pm);
  const unsigned lds_base =
      static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void *)smem));
  unsigned a_lds[NI], w_lds[NI], a_voff[NI], w_voff[NI], a_next[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int ba = (4 * j + wave + rot_a) & 31, bw = (4 * j + wave + rot_w) & 31;
    a_lds[j] = __builtin_amdgcn_readfirstlane(lds_base + ba * 1024);
    w_lds[j] = __builtin_amdgcn_readfirstlane(lds_base + bw * 1024);
  }
  // tile row / weight row that this lane fetches with instruction j; the lane number passes through an empty asm so that
  // the compiler forms these (once a tile) anew instead of keeping them in registers.  (Spilling even a few costs the ring:
  // a reload waits for everything outstanding.  One epilogue for whole and for partial column tiles for the same reason:
  // with a branch between two, the compiler moved the work common to both, all 256 sums, ahead of the branch.)
  auto here = [&]() __attribute__((always_inline)) {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
  };
  auto a_row = [&](int j, int l) __attribute__((always_inline)) { return ((4 * j + wave + rot_a) & 31) * 8 + (l >> 3); };
  auto w_row = [&](int j, int l) __attribute__((always_inline)) {
    const int b = (4 * j + wave + rot_w) & 31;
    return WT ? b * 2 + (l >> 5) : b * 8 + (l >> 3);
  };
  const char *const a_base_g = static_cast<const char *>(a.A);
  auto a_offset = [&](int j, int l, int64_t row) __attribute__((always_inline)) {
    return static_cast<unsigned>((row * a.lda + ((l & 7) ^ ((a_row(j, l) >> 1) & 7)) * 8) * 2);
  };
  auto set_w = [&](const StreamTile &tl, int j, int l) __attribute__((always_inline)) {
    if constexpr (WT) {
      w_voff[j] = static_cast<unsigned>((static_cast<int64_t>(w_row(j, l)) * a.N + ((l & 31) ^ (4 * (w_row(j, l) & 3))) * 8) * 2);
    } else {
      const int r = w_row(j, l) < a.N - tl.n0 ? w_row(j, l) : a.N - tl.n0 - 1;       // rows past N: never stored
      w_voff[j] = static_cast<unsigned>((static_cast<int64_t>(r) * a.K + ((l & 7) ^ ((w_row(j, l) >> 1) & 7)) * 8) * 2);
    }
  };
  auto w_at = [&](const StreamTile &tl) __attribute__((always_inline)) {
    const int64_t at = WT ? static_cast<int64_t>(tl.group) * a.N * a.K + tl.n0
                          : (static_cast<int64_t>(tl.group) * a.N + tl.n0) * a.K;
    return static_cast<const char *>(a.W) + at * 2;
  };
  const int64_t a_step = kDmaBK * 2, w_step = WT ? static_cast<int64_t>(kDmaBK) * a.N * 2 : kDmaBK * 2;
  // A row number or scale word, asked for a slab before its use.  An ordinary load: the compiler waits for it wherever it
  // touches the register, be it to spill it.  Its count does not know the DMA requests, which only makes that wait
  // longer (it ends when the newest of them has landed).
  auto load_idx = [](const void *base, unsigned voff) __attribute__((always_inline)) {
    typedef const __attribute__((address_space(1))) char gbyte_t;
    return *reinterpret_cast<const __attribute__((address_space(1))) int *>(reinterpret_cast<gbyte_t *>(reinterpret_cast<uintptr_t>(base)) + voff);
  };

  // ---- MFMA side
  const int a_frag = (wm * 128 + frag_row) * kDmaRC, w_frag = (wn * 128 + frag_row) * kDmaRC;
  const int swz = (frag_row >> 1) & 7;
  unsigned wt_off[TN];
  if constexpr (WT) {
    const int i16 = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int chunk = (wn * 16 + j * 4 + 2 * (grp & 1) + ((i16 >> 1) & 1)) ^ (4 * (i16 >> 2));
      wt_off[j] = static_cast<unsigned>((8 * (grp >> 1) + (i16 >> 2)) * 512 + chunk * 16 + (i16 & 1) * 8);
    }
  }
  f32x16_t acc[TM][TN];
  bf16x8_t fa0[TM], fa1[TM], fb0[TN], fb1[TN];
  auto read_a = [&](unsigned slot, int kk, int i) __attribute__((always_inline)) {
    const uint4 v = smem[slot * (kSlotBytes / 16) + a_frag + i * 32 * kDmaRC + ((kk * 2 + frag_half) ^ swz)];
    return *reinterpret_cast<const bf16x8_t *>(&v);
  };
  auto read_w = [&](unsigned slot, int kk, int j) __attribute__((always_inline)) {
    if constexpr (WT) {
      typedef short i16x4_t __attribute__((ext_vector_type(4)));
      typedef short i16x8_t __attribute__((ext_vector_type(8)));
      typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
      const __attribute__((address_space(3))) unsigned char *pb =
          (const __attribute__((address_space(3))) unsigned char *)(smem + slot * (kSlotBytes / 16)) + kk * (16 * 512) + wt_off[j];
      const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)pb);
      const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(pb + 4 * 512));
      return __builtin_bit_cast(bf16x8_t, (i16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      const uint4 v = smem[slot * (kSlotBytes / 16) + w_frag + j * 32 * kDmaRC + ((kk * 2 + frag_half) ^ swz)];
      return *reinterpret_cast<const bf16x8_t *>(&v);
    }
  };
  // one 16-wide step on (fa, fb); (na, nb) receive the fragments of step kn of the slab in slots (sa, sw); dma(q) runs
  // behind MFMA q
  auto step = [&](auto zero, const bf16x8_t(&fa)[TM], const bf16x8_t(&fb)[TN], bf16x8_t(&na)[TM], bf16x8_t(&nb)[TN],
                  unsigned sa, unsigned sw, int kn, auto dma) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int q = i * TN + j;
        if constexpr (decltype(zero)::value) {
          f32x16_t z;
#pragma unroll
          for (int v = 0; v < 16; ++v) z[v] = 0.0f;
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], z, 0, 0, 0);
        } else {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
        }
        // in the order of first use by the next step
        if (q == 0) na[0] = read_a(sa, kn, 0);
        else if (q <= TN) nb[q - 1] = read_w(sw, kn, q - 1);
        else if (q < TN + TM) na[q - TN] = read_a(sa, kn, q - TN);
        dma(q);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  const auto mod5 = [](unsigned s) { return s >= 5 ? s - 5 : s; };
  using True = std::true_type;
  using False = std::false_type;
  const char *a_ptr = a_base_g, *w_ptr;
  auto dma_a = [&](unsigned slot, int j) __attribute__((always_inline)) { dma_load_16(a_lds[j] + slot * kSlotBytes, a_voff[j], a_ptr); };
  auto dma_w = [&](unsigned slot, int j) __attribute__((always_inline)) { dma_load_16(w_lds[j] + slot * kSlotBytes, w_voff[j], w_ptr); };
  const auto none = [](int) {};

  // ---- fill the ring for the first tile: A(0) W(0) A(1) W(1) A(2)
  StreamTile cur = locate(t), nxt = locate(t + cus < tile_end ? t + cus : t);
  w_ptr = w_at(cur);
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int l = here();
    set_w(cur, j, l);
    int p = cur.row0 + a_row(j, l);
    if (p >= cur.row_end) p = cur.row0;
    a_voff[j] = a_offset(j, l, a.a_rows ? a.a_rows[p] : p);
  }
  int c_pos[TM], c_next[TM];                                  // row of C that lane l & 31 has in each 32-row block
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    int p = cur.row0 + wm * 128 + i * 32 + (here() & 31);
    if (p >= cur.row_end) p = cur.row0;
    c_pos[i] = a.c_rows ? a.c_rows[p] : p;
  }
#pragma unroll
  for (unsigned h = 0; h < 5; ++h) {
    if (h & 1) {
#pragma unroll
      for (int j = 0; j < NI; ++j) dma_w(h, j);
      w_ptr += w_step;
    } else {
#pragma unroll
      for (int j = 0; j < NI; ++j) dma_a(h, j);
      a_ptr += a_step;
    }
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * NI) : "memory");
  unsigned ra = 0;                                            // slot of A(m); W(m) and the next slabs follow it in the ring
  fa0[0] = read_a(0, 0, 0);
#pragma unroll
  for (int j = 0; j < TN; ++j) fb0[j] = read_w(1, 0, j);
#pragma unroll
  for (int i = 1; i < TM; ++i) fa0[i] = read_a(0, 0, i);
  u32x4_t held[TM / 2][kPieces];                              // the previous tile's last two row blocks
  int held_pos[TM / 2];                                       // their rows of C, as lane l & 31 has them
  int held_col = 0, held_cols = 0;                            // their first column, and how many exist (0: nothing held)
  // a store instruction covers 16 rows x 32 columns: lane l has row (l & 15) + 16 h and eight columns from store_col on
  auto store_col = [&]() __attribute__((always_inline)) {
    const int l = here();
    return (l & 16) + (l >> 5) * 8;
  };
  auto out_at = [&](int pos, int h, int col) __attribute__((always_inline)) {
    const auto rows = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(pos), static_cast<unsigned>(pos), false, false);
    return static_cast<uint64_t>(rows[h]) * static_cast<uint64_t>(a.ldc) + static_cast<uint64_t>(col + store_col());
  };
  constexpr int kHeld = TM / 2 * kPieces, kHeldSlabs = kHeld / 2;
  auto store_held = [&](int k) __attribute__((always_inline)) {
    const int i = k / kPieces, pc = k % kPieces;
    const uint64_t at = out_at(held_pos[i], pc & 1, held_col);       // (trades between lanes: with all of them active)
    if (pc / 2 * 32 + store_col() < held_cols)
      *reinterpret_cast<u32x4_t *>(static_cast<bf16_t *>(a.C) + at + pc / 2 * 32) = held[i][pc];
  };

  // a slab of the steady state; at the tile's end the caller has pointed a_ptr / w_ptr at the next tile
  auto slab_head = [&](auto other) __attribute__((always_inline)) {
    const unsigned rw = mod5(ra + 1), rw1 = mod5(ra + 3);
    step(False{}, fa0, fb0, fa1, fb1, ra, rw, 1, [&](int q) __attribute__((always_inline)) {
      if (q % 4 == 3) dma_w(rw1, 4 + q / 4);
      other(q);
    });
    w_ptr += w_step;
  };
  auto slab_mid = [&](auto other) __attribute__((always_inline)) {
    const unsigned rw = mod5(ra + 1), ra2 = mod5(ra + 4);
    step(False{}, fa1, fb1, fa0, fb0, ra, rw, 2, [&](int q) __attribute__((always_inline)) {
      if (q % 4 == 3) dma_a(ra2, q / 4);
      other(q);
    });
    step(False{}, fa0, fb0, fa1, fb1, ra, rw, 3, [&](int q) __attribute__((always_inline)) { if (q % 4 == 3) dma_a(ra2, 4 + q / 4); });
    a_ptr += a_step;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NI) : "memory");
  };
  auto slab_tail = [&](auto other) __attribute__((always_inline)) {
    const unsigned r0 = ra;
    ra = mod5(ra + 2);
    step(False{}, fa1, fb1, fa0, fb0, ra, mod5(ra + 1), 0, [&](int q) __attribute__((always_inline)) {
      if (q % 4 == 3) dma_w(r0, q / 4);
      other(q);
    });
  };

  for (;;) {
    const bool last = t + cus >= tile_end;                    // after the last tile: its own first slabs again, unused
    // slab 0: its W(1) and A(2) were requested before the previous tile's stores, so that it requests nothing but the row
    // numbers of the next tile and this tile's row scales: the wait for these ends with everything landed in any case
    float scale[TM];
    {
      int idx_a[NI], idx_c[TM], sc[TM];
      const unsigned rw = mod5(ra + 1);
      step(True{}, fa0, fb0, fa1, fb1, ra, rw, 1, [&](int q) __attribute__((always_inline)) {
        if (q < NI) {
          int p = nxt.row0 + a_row(q, here());
          if (p >= nxt.row_end) p = nxt.row0;
          a_next[q] = static_cast<unsigned>(p);
          idx_a[q] = load_idx(a.a_rows ? static_cast<const void *>(a.a_rows) : a.A, a.a_rows ? static_cast<unsigned>(p) * 4u : 0u);
        } else if (q < NI + TM) {
          const int i = q - NI;
          int p = nxt.row0 + wm * 128 + i * 32 + (here() & 31);
          if (p >= nxt.row_end) p = nxt.row0;
          c_next[i] = p;
          idx_c[i] = load_idx(a.c_rows ? static_cast<const void *>(a.c_rows) : a.A, a.c_rows ? static_cast<unsigned>(p) * 4u : 0u);
        } else if constexpr (EPI != kEpiPlain) {
          const int i = q - NI - TM;
          sc[i] = load_idx(a.row_scale ? static_cast<const void *>(a.row_scale) : a.A, a.row_scale ? static_cast<unsigned>(c_pos[i]) * 4u : 0u);
        }
      });
      step(False{}, fa1, fb1, fa0, fb0, ra, rw, 2, none);
      step(False{}, fa0, fb0, fa1, fb1, ra, rw, 3, none);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        asm volatile("" : "+v"(idx_a[j]));
        if (a.a_rows) a_next[j] = static_cast<unsigned>(idx_a[j]);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        asm volatile("" : "+v"(idx_c[i]));
        if (a.c_rows) c_next[i] = idx_c[i];
        if constexpr (EPI != kEpiPlain) {
          asm volatile("" : "+v"(sc[i]));
          scale[i] = a.row_scale ? __int_as_float(sc[i]) : 1.0f;
        }
      }
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    // slabs 0 .. kHeldSlabs - 1 each with two of the stores that the previous tile has left
    auto held_pair = [&](int m, int q) __attribute__((always_inline)) {
      if (m < kHeldSlabs && (q == 5 || q == 13)) store_held(2 * m + q / 8);
    };
    slab_tail([&](int q) __attribute__((always_inline)) { held_pair(0, q); });
    // slab 1: row numbers of A into offsets
    slab_head([&](int q) __attribute__((always_inline)) {
      if (q < NI) a_next[q] = a_offset(q, here(), static_cast<int>(a_next[q]));
    });
    slab_mid(none);
    slab_tail([&](int q) __attribute__((always_inline)) { held_pair(1, q); });
    // slab 2: where the tile after the next lies
    Finder after;
    after.t = t + 2 * cus < tile_end ? t + 2 * cus : t;
    slab_head([&](int q) __attribute__((always_inline)) { if (q % 2 == 0) locate_stage(after, q / 2); });
    slab_mid(none);
    slab_tail([&](int q) __attribute__((always_inline)) { held_pair(2, q); });
    for (int m = 3; m < KT - 2; ++m) {
      slab_head(none);
      slab_mid(none);
      slab_tail([&](int q) __attribute__((always_inline)) {
        if (q == 5 || q == 13) {
#pragma unroll
          for (int h = 3; h < kHeldSlabs; ++h)
            if (m == h) held_pair(h, q);
        }
      });
    }
#pragma unroll
    for (int h = 3; h < kHeldSlabs; ++h)                      // a short K: what is left
      if (KT - 2 <= h) {
        held_pair(h, 5);
        held_pair(h, 13);
      }
    // slab KT - 2: A and W of the next tile from here on
    slab_head(none);
    a_ptr = a_base_g;
#pragma unroll
    for (int j = 0; j < NI; ++j) a_voff[j] = a_next[j];
    slab_mid([&](int q) __attribute__((always_inline)) { if (q % 2 == 0) set_w(nxt, q / 2, here()); });
    w_ptr = w_at(nxt);
    slab_tail(none);
    // slab KT - 1: everything that slab 0 of the next tile would request goes before the stores
    slab_head(none);
    slab_mid(none);
    {
      const unsigned r0 = ra, r1 = mod5(ra + 1);
      ra = mod5(ra + 2);
      step(False{}, fa1, fb1, fa0, fb0, ra, mod5(ra + 1), 0, [&](int q) __attribute__((always_inline)) {
        if (q < 8) dma_w(r0, q); else dma_a(r1, q - 8);
      });
      w_ptr += w_step;
      a_ptr += a_step;
    }

    // ---- epilogue: a lane holds, for row frag_row of each 32-row block, columns 8 q + 4 frag_half + (0..3) of each
    // 32-column block in elements 4 q ..; lanes l and l + 32 trade halves so that each has 8 neighbouring columns, then
    // lanes l and l + 16 trade rows between two neighbouring 16-column pieces, so that a store writes 64 bytes of each of
    // 16 rows and not 32 of 32 (an L2 channel takes a request a clock, whatever its width).
    // (held_cols counts output columns from this wavefront's first; there may be none)
    constexpr int kWaveCols = EPI == kEpiSwiGLU ? 64 : 128;
    const int col0 = (EPI == kEpiSwiGLU ? cur.n0 / 2 : cur.n0) + wn * kWaveCols;
    const int n_cols = (EPI == kEpiSwiGLU ? a.N / 2 : a.N) - col0;
    // The residual's rows are asked for kAhead pairs of pieces ahead, and the two blocks that are held go first: few loads
    // stand behind stores, whose acknowledgement they wait for.
    constexpr bool kRes = EPI == kEpiRowScaleResidual;
    constexpr int kPairs = kPieces / 2, kAhead = 3;
    u32x4_t res[kRes ? kAhead : 1][2];
    auto block = [](int ii) { return kRes ? (ii + TM / 2) % TM : ii; };
    auto load_res = [&](int u) __attribute__((always_inline)) {      // u: pair of pieces, in the order of the loops below
      const int pos = c_pos[block(u / kPairs)], pp = u % kPairs * 2, c = store_col();
      const int back = pp * 16 + c < n_cols ? 0 : -(col0 + c) - pp * 16;   // past the end: the row's first columns
#pragma unroll
      for (int h = 0; h < 2; ++h)
        res[u % kAhead][h] = *reinterpret_cast<const u32x4_t *>(static_cast<const bf16_t *>(a.residual) + out_at(pos, h, col0) + back + pp * 16);
    };
    if constexpr (kRes) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) load_res(u);
    }
#pragma unroll
    for (int ii = 0; ii < TM; ++ii) {
      const int i = block(ii);
      const uint64_t at[2] = {out_at(c_pos[i], 0, col0), out_at(c_pos[i], 1, col0)};
#pragma unroll
      for (int pp = 0; pp < kPieces; pp += 2) {
        u32x4_t o[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int pc = pp + e;
          unsigned x0, x1, y0, y1;
          if constexpr (EPI == kEpiSwiGLU) {
            float g[2][4];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                g[m][r] = silu_f32(acc[i][pc][8 * m + r] * scale[i]) * (acc[i][pc][8 * m + 4 + r] * scale[i]);
            x0 = pack_bf16x2(g[0][0], g[0][1]); x1 = pack_bf16x2(g[0][2], g[0][3]);
            y0 = pack_bf16x2(g[1][0], g[1][1]); y1 = pack_bf16x2(g[1][2], g[1][3]);
          } else {
            const int j = pc / 2, q = (pc % 2) * 8;
            float v[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) v[r] = EPI == kEpiPlain ? acc[i][j][q + r] : acc[i][j][q + r] * scale[i];
            x0 = pack_bf16x2(v[0], v[1]); x1 = pack_bf16x2(v[2], v[3]);
            y0 = pack_bf16x2(v[4], v[5]); y1 = pack_bf16x2(v[6], v[7]);
          }
          const auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
          o[e] = u32x4_t{s0[0], s1[0], s0[1], s1[1]};
          __builtin_amdgcn_sched_barrier(0);                  // (registers: one piece at a time)
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const auto rows = __builtin_amdgcn_permlane16_swap(o[0][w], o[1][w], false, false);
          o[0][w] = rows[0];
          o[1][w] = rows[1];
        }
        if constexpr (kRes) {
          const int u = ii * kPairs + pp / 2;
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int w = 0; w < 4; ++w)
              o[h][w] = pack_bf16x2(__uint_as_float(o[h][w] << 16) + __uint_as_float(res[u % kAhead][h][w] << 16),
                                    __uint_as_float(o[h][w] & 0xFFFF0000u) + __uint_as_float(res[u % kAhead][h][w] & 0xFFFF0000u));
          if (u + kAhead < TM * kPairs) load_res(u + kAhead);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (i >= TM / 2) held[i - TM / 2][pp + h] = o[h];
          else if (pp * 16 + store_col() < n_cols) *reinterpret_cast<u32x4_t *>(static_cast<bf16_t *>(a.C) + at[h] + pp * 16) = o[h];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (i >= TM / 2) held_pos[i - TM / 2] = c_pos[i];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) c_pos[i] = c_next[i];
    held_col = col0;
    held_cols = n_cols;
    if (last) break;
    cur = nxt;
    nxt = after.tl;
    t += cus;
  }
#pragma unroll
  for (int k = 0; k < kHeld; ++k) store_held(k);
  }

  // ---- the last, partial round in pieces
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the ring's last requests have landed
  if (cut == 1 || cu >= rest * cut) return;
  const StreamTile tl = locate(tile_end + cu / cut);
  TileCoord tc;
  const int piece = cu % cut;
  // rows x columns of a piece: 128 x 256, 128 x 128, 64 x 128; fewest lines of both operands per product, which bound a piece
  // (contraction-major weights in pieces of 64 x 256 and 32 x 256: 2000 x 768 x 3072 in 4 groups 36 us, so 33; 8192 x 2048 x 1024 in 8 49.5 / 47.7)
  const int col_cuts = cut == 2 ? 1 : 2, rows = 256 * col_cuts / cut;
  tc.group = tl.group;
  tc.n0 = tl.n0 + piece % col_cuts * 128;
  tc.row0 = tl.row0 + piece / col_cuts * rows;
  tc.row_end = tl.row_end < tc.row0 + rows ? tl.row_end : tc.row0 + rows;
  tc.valid = true;
  if (tc.row0 >= tc.row_end || tc.n0 >= a.N) return;
  if (cut == 2) dma_tile<256, 1, 4, EPI, WT, 128>(a, tc, smem);
  else if (cut == 4) dma_tile<128, 2, 2, EPI, WT, 128>(a, tc, smem);
  else dma_tile<128, 2, 2, EPI, WT, 64>(a, tc, smem);
}

// ------------------------------------------------------------------ bf16 MFMA kernel, narrow fp32 output
// At most 160 columns (the x projection, and what comes back through the dt projection): a workgroup of four wavefronts owns RB blocks of
// 32 rows and every column, and a quarter of each 64-wide slab's contraction belongs to each wavefront, so that a fragment is read once per
// workgroup; the four sums are added through LDS at the end.  Bound by what a CU brings in, a row's share of A and all of its group's W:
// rows straight into a ring of four slabs in LDS, three under way, and a row count that makes one workgroup per CU (thin_row_blocks); with
// many rows by memory: rows that the launch before wrote come in at 2.4 TB/s, whoever reads them, while that launch's lines are written back.
// In 8 experts, in place: 16384 x 160 x 4096 67 us and 10.6 to add two slices, now 62 and 8.7 for one; 16384 x 128 x 4096 62 -> 50; 16384 x
// 96 x 2048 30.3 + 6.6 -> 23.7 + 5.5; 8192 x 96 x 2048 19.6 -> 15.8, x 64 20.9 -> 18 (256- or 128-row tiles of eight or four wavefronts,
// of which 72 to 144 workgroups had work).  Requests ahead of the products instead of between them: 30.2 and 24.2 for the last two but one.
// A row's products are added in one order wherever it lies in its group: the other rows of a call don't show in its sums.  (Workgroups
// starting on different slabs are no faster than with W's lines asked for ahead: layer calls of 12000 x 1536 723 / 726 us, 8192 x 1024 322 / 322,
// 3063 x 1536 271.5 / 271.7; without either 733, 326 and 272.)
constexpr int kThinSlots = 4, kThinWShare = 4;
constexpr int thin_slab_bytes(int rb, int nb) { return (rb + nb) * 32 * kDmaBK * 2; }
template <int RB, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1))) void gemm_bf16_thin_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint4 thin_smem[];
  constexpr int BM = RB * 32, kSlab = thin_slab_bytes(RB, NB), kInstr = RB + NB;       // requests per wavefront and slab, 8 rows each
  constexpr int kPitch = NB * 32 + 4;                          // floats: sixteen rows' 16-byte pieces cover the banks
  static_assert(4 * 32 * kPitch * 4 <= kThinSlots * kSlab, "the sums of 32 rows fit the ring");
  const TileCoord tc = locate_tile(a, BM, kThinMaxCols);
  if (!tc.valid) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int split = blockIdx.y, k0 = split * a.k_per_split;
  const int k_len = (a.K - k0 < a.k_per_split ? a.K - k0 : a.k_per_split), slabs = k_len / kDmaBK;
  typedef __attribute__((address_space(3))) unsigned char lds_char_t;
  lds_char_t *lds = (lds_char_t *)thin_smem;
  const unsigned lds_base = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void *)thin_smem));

  const char *const a_base = static_cast<const char *>(a.A);
  const char *const w_base = static_cast<const char *>(a.W) + static_cast<int64_t>(tc.group) * a.N * a.K * 2;

  // An XCD's workgroups multiply the same slab of W at the same time, and each would wait for it to come from memory.  So each asks for
  // a share of its group's lines ahead of everything else, one access a line, into the slot that is requested last.
  {
    const int lines = a.N * slabs, neighbours = static_cast<int>(gridDim.x >> 3), share = neighbours < kThinWShare ? neighbours : kThinWShare;
    for (int l = (static_cast<int>(blockIdx.x >> 3) % share * 4 + wave) * 64; l < lines; l += share * 256) {
      const int line = l + lane < lines ? l + lane : lines - 1, n = line / slabs, slab = line - n * slabs;
      dma_load_16(lds_base + (kThinSlots - 1) * kSlab + wave * (kInstr * 1024),
                  static_cast<unsigned>((static_cast<int64_t>(n) * a.K + k0 + slab * kDmaBK) * 2), w_base);
    }
  }

  // lane l of an instruction brings 16-byte place l & 7 of row l >> 3 (of eight): chunk place ^ ((row >> 1) & 7)
  unsigned voff[kInstr];
#pragma unroll
  for (int j = 0; j < kInstr; ++j) {
    const int r = (wave * kInstr + j) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
    if (r < BM) {
      const int64_t pos = tc.row0 + r < tc.row_end ? tc.row0 + r : tc.row_end - 1;
      const int64_t row = a.a_rows ? a.a_rows[pos] : pos;
      voff[j] = static_cast<unsigned>((row * a.lda + k0 + chunk * 8) * 2);
    } else {
      const int n = r - BM < a.N ? r - BM : a.N - 1;
      voff[j] = static_cast<unsigned>((static_cast<int64_t>(n) * a.K + k0 + chunk * 8) * 2);
    }
  }
  auto request = [&](int t, int j) __attribute__((always_inline)) {
    const unsigned at = lds_base + (t & (kThinSlots - 1)) * kSlab + wave * (kInstr * 1024);
    const int slab = t < slabs ? t : slabs - 1;
    dma_load_16(at + j * 1024, voff[j], ((wave * kInstr + j) * 8 < BM ? a_base : w_base) + static_cast<int64_t>(slab) * (kDmaBK * 2));
  };

  const int frag_row = lane & 31, place = ((wave * 2 + (lane >> 5)) ^ ((frag_row >> 1) & 7)) * 16;      // this wavefront's 16 of 64
  const int frag = frag_row * (kDmaBK * 2) + place;
  f32x16_t acc[RB][NB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
#pragma unroll
  for (int t = 0; t < kThinSlots - 1; ++t)
#pragma unroll
    for (int j = 0; j < kInstr; ++j) request(t, j);
  for (int t = 0; t < slabs; ++t) {
    // this slab has landed (two more are under way), and every wavefront has multiplied the one before
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kThinSlots - 2) * kInstr) : "memory");
    typedef const __attribute__((address_space(3))) bf16x8_t lds_frag_t;
    const lds_char_t *sl = lds + (t & (kThinSlots - 1)) * kSlab + frag;
    bf16x8_t fa[RB], fw[NB];
#pragma unroll
    for (int i = 0; i < RB; ++i) fa[i] = *(lds_frag_t *)(sl + i * (32 * kDmaBK * 2));
#pragma unroll
    for (int j = 0; j < NB; ++j) fw[j] = *(lds_frag_t *)(sl + (RB + j) * (32 * kDmaBK * 2));
    // the requests go out between the products (past the end: the last slab once more, into a slot that nobody reads)
    const int ahead = t + kThinSlots - 1;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[j], fa[i], acc[i][j], 0, 0, 0);
        const int q = i * NB + j;
#pragma unroll
        for (int d = q * kInstr / (RB * NB); d < (q + 1) * kInstr / (RB * NB); ++d) request(ahead, d);
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (the slabs asked for past the end: the sums take their place)
  // lane: row frag_row of a block, columns 8 q + 4 (lane / 32) + 0 .. 3 of a block in elements 4 q ..
  float *const sums = reinterpret_cast<float *>(thin_smem);
  float *const C = static_cast<float *>(a.C) + split * a.c_split_stride;
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4 *>(sums + (wave * 32 + frag_row) * kPitch + j * 32 + q * 8 + (lane >> 5) * 4) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int item = k * 256 + threadIdx.x, r = item / (NB * 8), c = item % (NB * 8) * 4;
      const int64_t pos = tc.row0 + i * 32 + r;
      if (pos >= tc.row_end || c >= a.N) continue;
      float4 v[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const float4 *>(sums + (w * 32 + r) * kPitch + c);
      const int64_t row = a.c_rows ? a.c_rows[pos] : pos;
      *reinterpret_cast<float4 *>(C + row * a.ldc + c) =
          make_float4((v[0].x + v[1].x) + (v[2].x + v[3].x), (v[0].y + v[1].y) + (v[2].y + v[3].y),
                      (v[0].z + v[1].z) + (v[2].z + v[3].z), (v[0].w + v[1].w) + (v[2].w + v[3].w));
    }
  }
}

// ------------------------------------------------------------------ bf16 MFMA kernel, short inner dimension
// For a K of up to ten 16-wide steps (the dt projection, K = dt_rank, and its input gradient, dt_rank + 32) there is no K loop to
// pipeline: a tile of the general kernel is one load, a few MFMAs and a long epilogue in sequence, and the epilogue
// (bias + softplus, two transcendentals per element) is bound by plain ALU issue, which needs
// about four wavefronts per SIMD to run at full rate.  Here a workgroup of eight waves keeps its
// 128-column slice of W (all of K) and of the bias in LDS and the waves stream 32-row sub-tiles of
// A past it: A fragments come straight from global memory into registers, each 32x64 half of the
// result goes through bias + softplus into the wave's own LDS patch and leaves as whole 128-byte
// row segments.  No workgroup barrier after the W load; registers are capped at 128 so that two
// workgroups (16 waves) share a CU.  There are just two workgroups a CU, each with an equal run of the rows for its slice: with one per 512
// rows, two sub-tiles a wave paid for each load of W and the last of 2.5 rounds left the chip half empty (16384 x 4096 x 128 in 8
// groups 58 -> 50 us, without softplus 50 -> 37, 2048 x 64 32 -> 26).  RES reads whole row pieces ahead of the products (113 -> 67; eight
// bytes a lane where the sums lie had every line of the output asked for eight times).
// What a group costs a workgroup besides its rows (weights, a fresh start), in sub-tiles: 15 of 16 groups with 64 of 16384 rows, one
// with the rest, 16384 x 4096 x 128 in us at 0 / 1 / 3 / 8: 71 / 61 / 52 / 55; even groups 48 at each.
constexpr int kSkGroup = 3;
constexpr int kSkBN = 128, kSkWaves = 8, kSkWgs = 512;     // two workgroups a CU
__host__ __device__ inline int64_t smallk_most(int64_t rows, int groups) { return rows / 32 + (groups > 0 ? groups : 1); }   // sub-tiles, at most

// PLAIN: no bias, no softplus.  RES: the rows of a.residual (the output's layout and row map) are
// added to the sums before bias and activation: the passes of K > 1 accumulate into the output,
// the last one activates.
template <int KSTEPS, bool PLAIN, bool RES = false>
__global__ __launch_bounds__(kSkWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 8)))
void gemm_bf16_smallk_kernel(const GemmArgs a) {
  constexpr int KC = KSTEPS * 2;                       // 16-byte chunks per row of A / W
  static_assert(KSTEPS >= 2 && KSTEPS <= 10, "W and two workgroups' patches in 160 KiB, A in 128 registers");
  constexpr int kWPitch = KC + 1;                      // an odd number of chunks: 16 consecutive rows -> 16 distinct 16-byte banks
  constexpr int kHalf = kSkBN / 2;                     // columns per pass over the accumulators
  constexpr int kPitch = kHalf * 2 + 16;               // bytes per staged output row; the pad holds its C row index

  extern __shared__ __attribute__((aligned(16))) uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this workgroup's column slice and its run of the sub-tiles (32 rows of one group); an XCD has neighbouring runs for all slices
  const int n_slices = (a.N + kSkBN - 1) / kSkBN, runs = gridDim.x / n_slices;
  int t = blockIdx.x;
  if (gridDim.x % 8 == 0) t = (t % 8) * (gridDim.x / 8) + t / 8;
  const int n0 = t % n_slices * kSkBN, run = t / n_slices;
  const int per_group = runs < smallk_most(a.M, a.n_groups) ? kSkGroup : 0;         // (else each sub-tile has a workgroup)
  int grp_lo, grp_hi, grp_end;       // lane e: group e's rows, and where it ends in sub-tiles, per_group more for each group that has rows
  {
    const bool have = a.offsets != nullptr && lane < a.n_groups;
    grp_lo = have ? a.offsets[lane] : 0;
    grp_hi = have ? a.offsets[lane + 1] : a.offsets == nullptr && lane == 0 ? static_cast<int>(a.M) : 0;
    grp_end = grp_hi > grp_lo ? (grp_hi - grp_lo + 31) / 32 + per_group : 0;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const int below = __shfl_up(grp_end, d);
      if (lane >= d) grp_end += below;
    }
  }
  const int64_t total = __builtin_amdgcn_readlane(grp_end, 63);
  int at = static_cast<int>(total * run / runs);
  const int at_end = static_cast<int>(total * (run + 1) / runs);

  const bf16_t *Ap = static_cast<const bf16_t *>(a.A);
  uint4 *Ws = smem;                                                        // [128][KC], rows kWPitch apart
  float *bias_s = reinterpret_cast<float *>(smem + kSkBN * kWPitch);            // [128]
  char *stage = reinterpret_cast<char *>(bias_s + kSkBN) + wave * (32 * kPitch);
  if (tid < kSkBN) bias_s[tid] = PLAIN ? 0.0f : a.bias[(n0 + tid < a.N) ? n0 + tid : a.N - 1];

  const int frag_row = lane & 31, frag_half = lane >> 5;
  const int chunk = lane & 7, sub_row = lane >> 3;     // store phase: 8 rows x 128 bytes per instruction

  while (at < at_end) {                                // one group after the other
    const int group = __builtin_popcountll(__ballot(grp_end <= at));
    const int lo = __builtin_amdgcn_readlane(grp_lo, group), hi = __builtin_amdgcn_readlane(grp_hi, group);
    const int end = __builtin_amdgcn_readlane(grp_end, group), first = end - (hi - lo + 31) / 32;
    const int sub0 = at > first ? at - first : 0, stop = (end < at_end ? end : at_end) - first;
    at = end;
    if (sub0 >= stop) continue;
    const bf16_t *Wp = static_cast<const bf16_t *>(a.W) + static_cast<int64_t>(group) * a.N * a.K;
    for (int q = tid; q < kSkBN * KC; q += kSkWaves * 64) {
      const int r = q / KC, c = q % KC;
      const int n = (n0 + r < a.N) ? n0 + r : a.N - 1;
      const u32x4_t v = *reinterpret_cast<const u32x4_t *>(Wp + static_cast<int64_t>(n) * a.K + c * 8);
      Ws[r * kWPitch + c] = make_uint4(v.x, v.y, v.z, v.w);
    }
    // rows of A and C of this lane's position, a sub-tile ahead; positions past the group's end: computed, never stored
    auto position = [&](int sub) __attribute__((always_inline)) {
      const int p = lo + sub * 32 + frag_row;
      return sub < stop && p < hi ? p : lo;
    };
    int p_next = position(sub0 + wave);
    int ar_next = a.a_rows ? a.a_rows[p_next] : p_next, cr_next = a.c_rows ? a.c_rows[p_next] : p_next;
    __syncthreads();

  for (int sub = sub0 + wave; sub < stop; sub += kSkWaves) {
    const int ar = ar_next, crow = cr_next, row0 = lo + sub * 32;
    // A fragment: row frag_row of the sub-tile, 8 elements at K offset 16 kk + 8 frag_half
    const bf16_t *src = Ap + static_cast<int64_t>(ar) * a.lda + frag_half * 8;
    bf16x8_t af[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) af[kk] = *reinterpret_cast<const bf16x8_t *>(src + kk * 16);
    if (frag_half == 0) *reinterpret_cast<int *>(stage + frag_row * kPitch + kHalf * 2) = crow;
    p_next = position(sub + kSkWaves);
    ar_next = a.a_rows ? a.a_rows[p_next] : p_next;
    cr_next = a.c_rows ? a.c_rows[p_next] : p_next;

#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      // RES: whole row pieces, in the layout of the stores, ahead of the products; through the wave's patch to the lanes that add them
      const int col = n0 + h * kHalf + chunk * 8;
      u32x4_t res[RES ? 4 : 1];
      if constexpr (RES) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int cr = *reinterpret_cast<const int *>(stage + (i * 8 + sub_row) * kPitch + kHalf * 2);
          res[i] = *reinterpret_cast<const u32x4_t *>(static_cast<const bf16_t *>(a.residual) + static_cast<int64_t>(cr) * a.ldc +
                                                      (col < a.N ? col : 0));
        }
      }
      f32x16_t acc[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) {
        const int c = kk * 2 + frag_half;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint4 w = Ws[(h * kHalf + j * 32 + frag_row) * kWPitch + c];
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t *>(&w), af[kk], acc[j], 0, 0, 0);
        }
      }
      if constexpr (RES) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4_t *>(stage + (i * 8 + sub_row) * kPitch + chunk * 16) = res[i];
      }
      // W is the MFMA's row operand: this lane holds, for A row frag_row, the output columns
      // 32 j + 8 q + 4 frag_half + r of this half in acc[j][4 q + r]
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int lcol = j * 32 + q * 8 + frag_half * 4;
          const float4 b4 = *reinterpret_cast<const float4 *>(bias_s + h * kHalf + lcol);
          float v0 = acc[j][4 * q], v1 = acc[j][4 * q + 1], v2 = acc[j][4 * q + 2], v3 = acc[j][4 * q + 3];
          if constexpr (RES) {
            const u32x2_t o = *reinterpret_cast<const u32x2_t *>(stage + frag_row * kPitch + lcol * 2);
            v0 += __uint_as_float(o.x << 16); v1 += __uint_as_float(o.x & 0xFFFF0000u);
            v2 += __uint_as_float(o.y << 16); v3 += __uint_as_float(o.y & 0xFFFF0000u);
          }
          uint2 pk;
          if constexpr (PLAIN) {
            pk.x = pack_bf16x2(v0, v1);
            pk.y = pack_bf16x2(v2, v3);
          } else {
            pk.x = pack_bf16x2(softplus_fast(v0 + b4.x), softplus_fast(v1 + b4.y));
            pk.y = pack_bf16x2(softplus_fast(v2 + b4.z), softplus_fast(v3 + b4.w));
          }
          *reinterpret_cast<uint2 *>(stage + frag_row * kPitch + lcol * 2) = pk;
        }
      }
      // the wave's own patch: LDS serves one wave's accesses in program order, no barrier needed
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = i * 8 + sub_row;
        const uint4 v = *reinterpret_cast<const uint4 *>(stage + row * kPitch + chunk * 16);
        const int cr = *reinterpret_cast<const int *>(stage + row * kPitch + kHalf * 2);
        if (row0 + row < hi && col < a.N)
          *reinterpret_cast<uint4 *>(static_cast<bf16_t *>(a.C) + static_cast<int64_t>(cr) * a.ldc + col) = v;
      }
    }
  }
    if (at < at_end) __syncthreads();                  // the next group's weights go over these
  }
}

// ------------------------------------------------------------------ fp32 products on the matrix cores
// For fp32 operands (and the bf16 shapes that the kernels above do not take, widened as they are read).  What bounds the small
// calls that use it is latency, so nothing goes through LDS: a lane of v_mfma_f32_16x16x4_f32 takes one row and, of every four
// contraction indices, one.  Which four is free as long as both operands agree, so lane l reads 16 bytes, k = 4 (l / 16) .. + 3 of
// row l & 15 (8 in bf16), straight into the operand of four instructions; kDirectBlocks of these 16-wide blocks are requested
// together.  Small calls take 16 x 16 products a wavefront, side by side in a workgroup's four; calls that fill the CUs
// with 64 x 64 tiles take 32 x 32 ones, whose operands the four share in L1 (gemm_f32_tile).  A lane's sums are four neighbouring
// columns: one store.
// Sums are fp32 throughout; their error against 64 bits over ten layers of 22 ... 369 tokens, d_model 64 ... 256, is that of the
// fp32 FMA tiles it replaced (4.57e-7 both).  64 tokens, d_model 64, four experts, the call's four products: 61 -> 25 us (LDS
// tiles of 16 contraction indices waited for memory at each); the layer call 77 -> 41.  8192 rows in 8 experts, fp32 8192 x 2048
// 7817 -> 5094, 2048 x 4096 4331 -> 2575, 4096 x 128 with softplus 322 -> 204; bf16 1680 x 52 74 -> 74, 94 x 2000 (an output that the
// bf16 kernels' stores do not take) 177 -> 119.
constexpr int kDirectBlocks = 4;

// elements k .. k + 3 of a row, zero from k_stop on; VEC: rows aligned to four elements and k_stop a multiple of four
template <typename T, bool VEC>
__device__ __forceinline__ f32x4_t load_k4(const T *row, int k, int k_begin, int k_stop) {
  f32x4_t v;
  if constexpr (VEC) {
    typedef T t4_t __attribute__((ext_vector_type(4)));
    const bool in = k < k_stop;
    const t4_t x = *reinterpret_cast<const t4_t *>(row + (in ? k : k_begin));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = in ? to_f32(x[i]) : 0.0f;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = k + i < k_stop;
      const float x = to_f32(row[in ? k + i : k_begin]);
      v[i] = in ? x : 0.0f;
    }
  }
  return v;
}

// a workgroup of WM x WN wavefronts, each TM x TN tiles of 16 x 16; AHEAD: the next blocks' requests stand ahead of the products
template <typename T, bool VEC, bool AHEAD, int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64) void gemm_f32_direct_kernel(const GemmArgs a) {
  const TileCoord tc = locate_tile(a, WM * TM * 16, WN * TN * 16);
  if (!tc.valid) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, kq = (lane >> 4) * 4;
  const int64_t row0 = tc.row0 + wave / WN * (TM * 16);
  const int col0 = tc.n0 + wave % WN * (TN * 16);
  if (row0 >= tc.row_end || col0 >= a.N) return;
  const int k_begin = blockIdx.y * a.k_per_split;
  const int k_stop = (a.K - k_begin < a.k_per_split) ? a.K : k_begin + a.k_per_split;
  // rows and columns past the end re-read the tile's first ones; their products are not stored
  const T *a_row[TM], *w_row[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int c = col0 + j * 16 + r16;
    w_row[j] = static_cast<const T *>(a.W) + (static_cast<int64_t>(tc.group) * a.N + (c < a.N ? c : col0)) * a.K;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t p = row0 + i * 16 + r16 < tc.row_end ? row0 + i * 16 + r16 : row0;
    a_row[i] = static_cast<const T *>(a.A) + static_cast<int64_t>(a.a_rows ? a.a_rows[p] : p) * a.lda;
  }
  f32x4_t acc[TM][TN] = {};
  struct Blocks {
    f32x4_t a[kDirectBlocks][TM], w[kDirectBlocks][TN];
  };
  auto load = [&](int k0, Blocks &f) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < kDirectBlocks; ++b) {
#pragma unroll
      for (int j = 0; j < TN; ++j) f.w[b][j] = load_k4<T, VEC>(w_row[j], k0 + b * 16 + kq, k_begin, k_stop);
#pragma unroll
      for (int i = 0; i < TM; ++i) f.a[b][i] = load_k4<T, VEC>(a_row[i], k0 + b * 16 + kq, k_begin, k_stop);
    }
  };
  auto products = [&](int k0, const Blocks &f) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < kDirectBlocks; ++b) {
      if (k0 + b * 16 >= k_stop) break;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.w[b][j][s], f.a[b][i][s], acc[i][j], 0, 0, 0);
    }
  };
  constexpr int kStep = kDirectBlocks * 16;
  if constexpr (AHEAD) {
    Blocks f0, f1;
    load(k_begin, f0);
    for (int k0 = k_begin; k0 < k_stop; k0 += 2 * kStep) {
      if (k0 + kStep < k_stop) load(k0 + kStep, f1);
      products(k0, f0);
      if (k0 + kStep >= k_stop) break;
      if (k0 + 2 * kStep < k_stop) load(k0 + 2 * kStep, f0);
      products(k0 + kStep, f1);
    }
  } else {
    for (int k0 = k_begin; k0 < k_stop; k0 += kStep) {
      Blocks f;
      load(k0, f);
      products(k0, f);
    }
  }
  // the weight is the instruction's row operand: a lane holds row r16 of C, columns kq .. kq + 3
  const bool whole = out_in_fours(a);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t p = row0 + i * 16 + r16;
    if (p >= tc.row_end) continue;
    const int64_t crow = a.c_rows ? a.c_rows[p] : p;
#pragma unroll
    for (int j = 0; j < TN; ++j) store_out4(a, whole, crow, col0 + j * 16 + kq, acc[i][j]);
  }
}

// The same for many rows that cannot be read four elements at a time (an odd dt_rank): the 64 x 64 tile's operands go through LDS,
// in slabs of 16 contraction indices, so that each element is asked for once in a workgroup where the kernel above asks for it
// in two wavefronts.  Bound by these requests; 256 threads, 4 x 4 fp32 FMA sums each.
constexpr int kSB = 64, kSK = 16;

template <typename T>
__global__ __launch_bounds__(256) void gemm_f32_staged_kernel(const GemmArgs a) {
  __shared__ float As[kSK][kSB + 4];
  __shared__ float Bs[kSK][kSB + 4];
  const TileCoord tc = locate_tile(a, kSB, kSB);
  if (!tc.valid) return;
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  const T *Ap = static_cast<const T *>(a.A);
  const T *Wp = static_cast<const T *>(a.W) + static_cast<int64_t>(tc.group) * a.N * a.K;
  // staging: thread -> (row = tid / 4, 4 consecutive k = (tid % 4) * 4)
  const int s_r = tid / 4, s_k = (tid % 4) * 4;
  const int64_t pa = tc.row0 + s_r;
  const int64_t a_off = (pa < tc.row_end) ? static_cast<int64_t>(a.a_rows ? a.a_rows[pa] : pa) * a.lda : -1;
  const int64_t b_off = (tc.n0 + s_r < a.N) ? static_cast<int64_t>(tc.n0 + s_r) * a.K : -1;
  float acc[4][4] = {};
  const int k_begin = blockIdx.y * a.k_per_split;
  const int k_stop = (a.K - k_begin < a.k_per_split) ? a.K : k_begin + a.k_per_split;
  for (int k0 = k_begin; k0 < k_stop; k0 += kSK) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = k0 + s_k + i;
      As[s_k + i][s_r] = (a_off >= 0 && k < k_stop) ? to_f32(Ap[a_off + k]) : 0.0f;
      Bs[s_k + i][s_r] = (b_off >= 0 && k < k_stop) ? to_f32(Wp[b_off + k]) : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSK; ++k) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { av[i] = As[k][ty * 4 + i]; bv[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t p = tc.row0 + ty * 4 + i;
    const bool row_ok = p < tc.row_end;
    const int64_t crow = row_ok ? (a.c_rows ? a.c_rows[p] : p) : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = tc.n0 + tx * 4 + j;
      if (row_ok && col < a.N) store_out(a, crow, col, acc[i][j]);
    }
  }
}

// A kernel that asks for more than 64 KiB of dynamic LDS needs a function attribute, set once
// per device (the attribute belongs to the device's copy of the code object).  One instance per
// kernel instantiation; safe to call from several host threads.
constexpr int kAttrMaxDevices = 64;
struct LdsAttrOnce {
  std::mutex mu;
  std::atomic<bool> done[kAttrMaxDevices] = {};
  hipError_t ensure(const void *kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kAttrMaxDevices) return hipErrorInvalidDevice;
    if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
    std::lock_guard<std::mutex> lock(mu);
    if (done[dev].load(std::memory_order_relaxed)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done[dev].store(true, std::memory_order_release);
    return e;
  }
};

int grid_tiles(const GemmArgs &a, int BM, int BN) {
  const int64_t m_tiles = a.offsets ? (a.M / BM + a.n_groups) : ceil_div(a.M, BM);
  const int64_t n_tiles = ceil_div(a.N, BN);
  const int pn = patch_n_for(static_cast<int>(n_tiles)), pm = kPatchTiles / pn;
  const int64_t patches = ceil_div(m_tiles, pm) * ceil_div(n_tiles, pn);
  int64_t g = patches * kPatchTiles;
  g = ceil_div(g, 8) * 8;
  return static_cast<int>(g);
}

template <typename T, bool VEC>
hipError_t launch_f32_t(const GemmArgs &a, hipStream_t s) {
  const dim3 grid64(grid_tiles(a, 64, 64), a.k_splits);
  switch (gemm_f32_tile(a.M, a.offsets ? a.n_groups : 1, a.N, a.k_per_split < a.K ? a.k_per_split : a.K, a.k_splits, VEC)) {
    case GemmF32Tile::kStaged:
      if constexpr (!VEC) hipLaunchKernelGGL(gemm_f32_staged_kernel<T>, grid64, dim3(256), 0, s, a);
      break;
    case GemmF32Tile::kWide:
      if constexpr (VEC) hipLaunchKernelGGL((gemm_f32_direct_kernel<T, VEC, true, 2, 2, 2, 2>), grid64, dim3(256), 0, s, a);
      break;
    case GemmF32Tile::kWideShort:
      if constexpr (VEC) hipLaunchKernelGGL((gemm_f32_direct_kernel<T, VEC, false, 2, 2, 2, 2>), grid64, dim3(256), 0, s, a);
      break;
    case GemmF32Tile::kSmall:
      hipLaunchKernelGGL((gemm_f32_direct_kernel<T, VEC, true, 1, 1, 1, 4>), dim3(grid_tiles(a, 16, 64), a.k_splits), dim3(256), 0, s, a);
      break;
  }
  return hipGetLastError();
}
template <typename T>
hipError_t launch_f32(const GemmArgs &a, hipStream_t s) {
  // whole pieces of four elements in every row of both operands (a slice of K starts at a multiple of 64)
  const bool vec = a.K % 4 == 0 && a.lda % 4 == 0 && reinterpret_cast<uintptr_t>(a.A) % (4 * sizeof(T)) == 0 &&
                   reinterpret_cast<uintptr_t>(a.W) % (4 * sizeof(T)) == 0;
  return vec ? launch_f32_t<T, true>(a, s) : launch_f32_t<T, false>(a, s);
}

template <int BM, int BN, int WM, int WN, int EPI, bool KTAIL>
hipError_t launch_mfma_k(const GemmArgs &a, hipStream_t s) {
  constexpr int kLoopSmem = 2 * (BM + BN) * kRowChunks * 16;
  constexpr int kStageSmem = EPI == kEpiPlainF32 ? 0 : WM * WN * 32 * ((BN / WN) * 2 + 16);
  constexpr int kSmem = kLoopSmem > kStageSmem ? kLoopSmem : kStageSmem;
  static LdsAttrOnce attr;         // per instantiation
  const hipError_t e =
      attr.ensure(reinterpret_cast<const void *>(&gemm_bf16_mfma_kernel<BM, BN, WM, WN, EPI, KTAIL>), kSmem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_bf16_mfma_kernel<BM, BN, WM, WN, EPI, KTAIL>),
                     dim3(grid_tiles(a, BM, BN), a.k_splits), dim3(WM * WN * 64), kSmem, s, a);
  return hipGetLastError();
}
template <int BM, int BN, int WM, int WN, int EPI>
hipError_t launch_mfma(const GemmArgs &a, hipStream_t s) {
  if (a.K % kBK == 0 && a.k_per_split % kBK == 0) return launch_mfma_k<BM, BN, WM, WN, EPI, false>(a, s);
  return launch_mfma_k<BM, BN, WM, WN, EPI, true>(a, s);
}

template <int KSTEPS, bool PLAIN, bool RES>
hipError_t launch_smallk_t(const GemmArgs &a, hipStream_t s) {
  constexpr int kSmem = kSkBN * (KSTEPS * 2 + 1) * 16 + kSkBN * 4 + kSkWaves * 32 * (kSkBN + 16);
  static LdsAttrOnce attr;
  const hipError_t e = attr.ensure(reinterpret_cast<const void *>(&gemm_bf16_smallk_kernel<KSTEPS, PLAIN, RES>), kSmem);
  if (e != hipSuccess) return e;
  const int64_t slices = ceil_div(a.N, kSkBN), most = smallk_most(a.M, a.n_groups);
  const int64_t fill = kSkWgs / slices > 0 ? kSkWgs / slices : 1, runs = fill < most ? fill : most;
  hipLaunchKernelGGL((gemm_bf16_smallk_kernel<KSTEPS, PLAIN, RES>), dim3(static_cast<unsigned>(slices * runs)), dim3(kSkWaves * 64), kSmem,
                     s, a);
  return hipGetLastError();
}
// the accumulating form goes with the activation (the last pass of K > 1), the plain one without
template <bool PLAIN>
hipError_t launch_smallk(const GemmArgs &a, hipStream_t s) {
  const auto steps = [&](auto k) -> hipError_t {
    constexpr int KS = decltype(k)::value;
    if constexpr (!PLAIN && (KS == 2 || KS == 4 || KS == 8))
      if (a.residual) return launch_smallk_t<KS, false, true>(a, s);
    return launch_smallk_t<KS, PLAIN, false>(a, s);
  };
  switch (a.K / 16) {
#define ROM_STEPS(KS) \
  case KS: return steps(std::integral_constant<int, KS>{})
    ROM_STEPS(2);
    ROM_STEPS(3);
    ROM_STEPS(4);
    ROM_STEPS(5);
    ROM_STEPS(6);
    ROM_STEPS(7);
    ROM_STEPS(8);
    ROM_STEPS(9);
    ROM_STEPS(10);
#undef ROM_STEPS
  }
  return hipErrorInvalidValue;
}
// whether the streaming small-K kernel takes the call (dense rows of A)
bool smallk_takes(const GemmArgs &a, bool plain) {
  return kUseSmallK && a.lda >= a.K && a.M < (1ll << 31) && !a.row_scale && !a.c_is_f32 && !(plain && a.residual) &&
         gemm_smallk(a.M, a.n_groups, a.K, a.residual != nullptr);
}

template <int BN, int WM, int WN, int EPI>
hipError_t launch_dma(const GemmArgs &a, hipStream_t s) {
  constexpr int kSmem = kDmaSlots * 256 * kDmaRC * 16;     // 160 KiB
  static LdsAttrOnce attr;
  const hipError_t e = attr.ensure(reinterpret_cast<const void *>(&gemm_bf16_dma_kernel<BN, WM, WN, EPI>), kSmem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_bf16_dma_kernel<BN, WM, WN, EPI>), dim3(grid_tiles(a, 256, BN), a.k_splits),
                     dim3(WM * WN * 64), kSmem, s, a);
  return hipGetLastError();
}
template <int RB, int NB>
hipError_t launch_thin_t(const GemmArgs &a, hipStream_t s) {
  constexpr int kSmem = kThinSlots * thin_slab_bytes(RB, NB);
  static LdsAttrOnce attr;
  const hipError_t e = attr.ensure(reinterpret_cast<const void *>(&gemm_bf16_thin_kernel<RB, NB>), kSmem);
  if (e != hipSuccess) return e;
  const int64_t tiles = a.offsets ? a.M / (RB * 32) + a.n_groups : ceil_div(a.M, RB * 32);
  hipLaunchKernelGGL((gemm_bf16_thin_kernel<RB, NB>), dim3(static_cast<unsigned>(ceil_div(tiles, 8) * 8), a.k_splits), dim3(256), kSmem, s, a);
  return hipGetLastError();
}
template <int NB>
hipError_t launch_thin_nb(const GemmArgs &a, hipStream_t s) {
  switch (thin_row_blocks(a.M, a.offsets ? a.n_groups : 1, a.N, a.k_splits)) {
    case 1: return launch_thin_t<1, NB>(a, s);
    case 2: return launch_thin_t<2, NB>(a, s);
    case 3: return launch_thin_t<3, NB>(a, s);
    case 4: return launch_thin_t<4, NB>(a, s);
    default: return launch_thin_t<NB < 5 ? 5 : 4, NB>(a, s);
  }
}
hipError_t launch_thin(const GemmArgs &a, hipStream_t s) {
  switch ((a.N + 31) / 32) {
    case 1: return launch_thin_nb<1>(a, s);
    case 2: return launch_thin_nb<2>(a, s);
    case 3: return launch_thin_nb<3>(a, s);
    case 4: return launch_thin_nb<4>(a, s);
    default: return launch_thin_nb<5>(a, s);
  }
}
constexpr int kStreamWgs = 256;      // one workgroup per CU
template <int EPI, bool WT = false>
hipError_t launch_stream(const GemmArgs &a, hipStream_t s) {
  constexpr int kSmem = kDmaSlots * 256 * kDmaRC * 16;     // 160 KiB
  static LdsAttrOnce attr;
  const hipError_t e = attr.ensure(reinterpret_cast<const void *>(&gemm_bf16_stream_kernel<EPI, WT>), kSmem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_bf16_stream_kernel<EPI, WT>), dim3(kStreamWgs), dim3(256), kSmem, s, a);
  return hipGetLastError();
}
// the DMA kernel addresses both operands with unsigned 32-bit byte offsets and walks whole 64-wide slabs
inline bool dma_ok(const GemmArgs &a) {
  return kUseDma && a.K % kDmaBK == 0 && a.k_per_split % kDmaBK == 0 && a.lda >= a.K &&
         a.a_span < (1ll << 31) && static_cast<int64_t>(a.N) * a.K < (1ll << 31);
}

inline GemmShape shape_of(const GemmArgs &a, bool f32_or_softplus) {
  GemmArgs narrow = a;
  narrow.a_span = 0;
  const bool whole_k = a.k_splits == 1;
  return {a.M, a.n_groups, a.N, a.K, whole_k && dma_ok(a), whole_k && !dma_ok(a) && dma_ok(narrow), a.w_kmajor != 0,
          a.residual == a.C, f32_or_softplus};
}

inline bool few_rows_takes(const GemmArgs &a) {
  return !a.w_kmajor && gemm_few_rows(a.M, a.offsets ? a.n_groups : 1, a.N, a.K);
}

template <int CT, int EPI>
hipError_t launch_few_rows_cols(const GemmArgs &a, hipStream_t s) {
  const unsigned gz = static_cast<unsigned>(!a.offsets ? 1 : a.M < a.n_groups ? a.M : a.n_groups);
  const dim3 grid(static_cast<unsigned>(ceil_div(a.N, 16 * CT)), a.k_splits, gz), block(kFewWaves * 64);
  // a wavefront's whole share of K at once where that is up to eight units
  if (a.k_per_split > kFewWaves * 4 * 64) hipLaunchKernelGGL((gemm_bf16_few_rows_kernel<CT, EPI, 8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gemm_bf16_few_rows_kernel<CT, EPI, 4>), grid, block, 0, s, a);
  return hipGetLastError();
}
template <int EPI>
hipError_t launch_few_rows(const GemmArgs &a, hipStream_t s) {
  return a.N >= kFewWideCols ? launch_few_rows_cols<2, EPI>(a, s) : launch_few_rows_cols<1, EPI>(a, s);
}

template <int EPI>
hipError_t launch_mfma_tiles(const GemmArgs &a, hipStream_t s) {
  constexpr bool kNoStream = EPI == kEpiPlainF32 || EPI == kEpiBiasSoftplus;
  const GemmTile tile = gemm_tile(shape_of(a, kNoStream));
  if constexpr (kNoStream) {
    if (tile == GemmTile::kDma256) return launch_dma<256, 4, 2, EPI>(a, s);
  } else {
    if (tile == GemmTile::kStream) return launch_stream<EPI>(a, s);
    if (tile == GemmTile::kReg256) return launch_mfma_k<256, 256, 4, 2, EPI, false>(a, s);
  }
  if (tile == GemmTile::k128) return launch_mfma<128, 128, 2, 2, EPI>(a, s);
  // One row tile per group at most (the recurrent step): every weight tile is read by exactly one
  // workgroup, so there is no L2 sharing for the XCD runs to protect, while a run of logical tiles
  // is one expert's column tiles - with few active experts the runs would put all the work on a
  // few XCDs.  Deal the tiles round-robin instead.
  GemmArgs spread = a;
  spread.no_xcd_remap = 1;
  // a narrow output (the step's out projection: 8 experts x 16 column tiles) leaves half of the CUs
  // without a workgroup while the weights stream past once: halve the column tile.  The same helps while
  // there are only about two workgroups per CU (the step's in projection, 8 x 64 tiles: twice the
  // workgroups keep more of the weight stream in flight; 256 sequences: step 173 -> 161 us)
  const int64_t groups = a.n_groups > 0 ? a.n_groups : 1;
  const int64_t row_tiles = groups * ceil_div(a.M / groups > 0 ? a.M / groups : 1, 64);
  if (row_tiles * ceil_div(a.N, 128) < kSkinnyColsMaxWgs && a.N % 64 == 0) return launch_mfma<64, 64, 2, 2, EPI>(spread, s);
  return launch_mfma<64, 128, 2, 2, EPI>(spread, s);
}

}  // namespace

// whether a call with a contraction-major weight (GemmArgs::w_kmajor) is taken: the stream kernel with a
// plain epilogue only; the caller otherwise makes a transposed copy of the weight
bool grouped_gemm_takes_kmajor(const GemmArgs &args) {
  GemmArgs a = args;
  a.k_splits = 1;
  a.k_per_split = static_cast<int>(ceil_div(a.K, 64) * 64);
  return grouped_gemm_on_mfma(a) && !a.c_is_f32 && !a.bias && !a.row_scale && !a.residual && !a.swiglu &&
         a.N % 256 == 0 && gemm_tile(shape_of(a, false)) == GemmTile::kStream;
}

// whether the call takes the MFMA kernels (else the fp32 one, which has no fused SwiGLU)
bool grouped_gemm_on_mfma(const GemmArgs &a) {
  const int out_align = a.c_is_f32 ? 4 : 8;      // elements per output store
  return a.dtype == ROM_DTYPE_BF16 && a.K % 8 == 0 && a.lda % 8 == 0 &&
         a.N % out_align == 0 && a.ldc % out_align == 0 && (reinterpret_cast<uintptr_t>(a.A) % 16 == 0) &&
         (reinterpret_cast<uintptr_t>(a.W) % 16 == 0) &&
         (reinterpret_cast<uintptr_t>(a.C) % 16 == 0) && a.a_span < (1ll << 32) &&
         static_cast<int64_t>(a.N) * a.K < (1ll << 32) &&
         !(a.bias && !a.softplus) && !(a.softplus && !a.bias) &&
         !(a.row_scale && (a.bias || a.c_is_f32)) && !(a.bias && a.c_is_f32) &&
         !(a.residual && a.c_is_f32) && (reinterpret_cast<uintptr_t>(a.residual) % 16 == 0) &&
         !(a.swiglu && (a.bias || a.c_is_f32 || a.residual || a.N % 16 != 0));
}

hipError_t launch_grouped_gemm(const GemmArgs &args, hipStream_t s) {
  if (args.M <= 0) return hipSuccess;
  GemmArgs a = args;
  if (a.k_splits < 1 || !a.c_is_f32 || a.bias || a.row_scale || a.residual) a.k_splits = 1;   // partial sums need a plain fp32 output
  a.k_per_split = static_cast<int>(ceil_div(ceil_div(a.K, a.k_splits), 64) * 64);
  a.k_splits = static_cast<int>(ceil_div(a.K, a.k_per_split));
  const bool mfma_ok = grouped_gemm_on_mfma(a);
  if (a.w_kmajor) {                                           // the caller asks grouped_gemm_takes_kmajor first
    if (!grouped_gemm_takes_kmajor(args)) return hipErrorInvalidValue;
    return launch_stream<kEpiPlain, true>(a, s);
  }
  if (a.swiglu && !mfma_ok) return hipErrorInvalidValue;      // the caller asks grouped_gemm_on_mfma first
  const bool few = mfma_ok && few_rows_takes(a);
  if (a.swiglu) return few ? launch_few_rows<kEpiSwiGLU>(a, s) : launch_mfma_tiles<kEpiSwiGLU>(a, s);
  if (!mfma_ok) {
    return a.dtype == ROM_DTYPE_BF16 ? launch_f32<bf16_t>(a, s) : launch_f32<float>(a, s);
  }
  if (few && a.c_is_f32) return launch_few_rows<kEpiPlainF32>(a, s);
  if (a.c_is_f32) {
    // one column tile: every workgroup re-reads the whole weight slice of its group, so take the
    // tallest row tile (256 rows, 128 on four waves, 64 on two) that still puts a workgroup on
    // a good part of the CUs, counting the inner-dimension slices
    const auto wgs = [&](int rows) { return (a.M / rows + a.n_groups) * a.k_splits; };
    if (a.N <= kThinMaxCols && (a.M >= kThinMinRows || wgs(256) >= kSkinnyMinWgs) && dma_ok(a)) return launch_thin(a, s);
    if (a.N <= 192) {
      const int tile_rows = wgs(256) >= kSkinnyMinWgs ? 256 : (wgs(128) >= kSkinnyMinWgs ? 128 : 64);
      switch ((a.N + 31) / 32) {
#define ROM_SKINNY(NN)                                                               \
  return tile_rows == 256 ? launch_mfma<256, NN, 4, 1, kEpiPlainF32>(a, s)           \
       : tile_rows == 128 ? launch_mfma<128, NN, 4, 1, kEpiPlainF32>(a, s)           \
                          : launch_mfma<64, NN, 2, 1, kEpiPlainF32>(a, s)
        case 1: ROM_SKINNY(32);
        case 2: ROM_SKINNY(64);
        case 3: ROM_SKINNY(96);
        case 4: ROM_SKINNY(128);
        case 5: ROM_SKINNY(160);
        default:
          if (tile_rows == 256 && dma_ok(a)) return launch_dma<192, 8, 1, kEpiPlainF32>(a, s);
          ROM_SKINNY(192);
#undef ROM_SKINNY
      }
    }
    return launch_mfma_tiles<kEpiPlainF32>(a, s);
  }
  if (a.bias) {
    if (smallk_takes(a, false)) return launch_smallk<false>(a, s);
    if (a.residual) return hipErrorInvalidValue;       // bias + activation on top of an accumulated output: small-K kernel only
    return launch_mfma_tiles<kEpiBiasSoftplus>(a, s);
  }
  // short inner dimension, many rows, wide output: the streaming kernel without its activation
  if (smallk_takes(a, true) && a.M >= 4096 && a.N >= 1024) return launch_smallk<true>(a, s);
  if (few) return a.residual ? launch_few_rows<kEpiRowScaleResidual>(a, s)
                : a.row_scale ? launch_few_rows<kEpiRowScale>(a, s) : launch_few_rows<kEpiPlain>(a, s);
  if (a.residual) return launch_mfma_tiles<kEpiRowScaleResidual>(a, s);
  if (a.row_scale) return launch_mfma_tiles<kEpiRowScale>(a, s);
  return launch_mfma_tiles<kEpiPlain>(a, s);
}

}  // namespace rom
