// RoM on a Mamba2 layer (Sec. 5.2, Table 3): the sequence part between the routed input and output
// projections - Mamba2's recurrence per head
//     H_t = exp(dt_t A) H_{t-1} + dt_t x_t B_t^T   (H: P x N),     y_t = H_t C_t + D x_t
// followed by the SiLU(z) gate, and the RMS norm of the gated rows.  gfx950 only, bf16 activations.
//
// The recurrence runs in its chunked ("dual") form on the matrix cores: over a chunk of Q = 64 steps
// with cum_t = sum_{r <= t} dt_r A inside the chunk,
//     y_t   = exp(cum_t) C_t . H_prev + sum_{s <= t} (C_t . B_s) exp(cum_t - cum_s) dt_s x_s
//     H_new = exp(cum_Q) H_prev + sum_s exp(cum_Q - cum_s) dt_s B_s x_s^T
// which is four small matrix products per chunk (scores C B^T, scores x inputs, C x state, B^T x
// inputs); every exponent is <= 0, so nothing overflows however strong the decay.  A workgroup
// (4 wavefronts) owns one (sequence, head, segment of the sequence) and walks its chunks in order
// with the state H in MFMA accumulators (fp32): wavefront w holds H[:, 16w .. 16w+15] and produces
// the same 16 output channels, so the state never leaves its registers - as the B operand of
// C x state it is read straight from the accumulators (the contraction index is permuted the same
// way on the C side).  Sequences are cut into segments until there are two workgroups per CU; a
// first pass (the same kernel without its output part) leaves every segment's end state from a
// zero start and its total log decay, which the main pass folds in segment order.
#include "rom_chunk.h"

#include <atomic>
#include <mutex>

namespace rom {
namespace {

using namespace chunk;

constexpr int kP = 64;          // channels per head

// LDS of one workgroup.  Rows are padded by 8 halfs (16 bytes): the 16-byte fragment reads of 16
// consecutive rows then fall into different banks.
template <int NS>
struct SsdSmem {
  union {
    bf16_t b[kQ][NS + 8];       // B, step-major (operand of the scores)
    float y[kQ][kP + 4];        // later in the chunk: the output tile, for row-wise stores
  } u;
  bf16_t c[kQ][NS + 8];         // C, step-major
  bf16_t bw[kQ][NS + 16];       // exp(cum_Q - cum_s) dt_s B_s, step-major, columns as read_steps wants them
  bf16_t x[kQ][kP + 16];        // x, likewise
  bf16_t g[kQ][kQ + 8];         // masked, decayed, dt-weighted scores [t][s]
  float cum[kQ], ecum[kQ], dt[kQ];   // cum_t, exp(cum_t), dt_t
};

// The operands that are contracted over steps are step-major in LDS and come out of it through the transposing read: the 16 lanes
// of group g name four rows of 32 bytes, lane c receives column c of them.  Groups 1 and 3 read rows 8 and 24 behind those of groups 0 and
// 2: their columns are exchanged in blocks of `flip`, so that 32 lanes meet 64 different banks.
template <int NC>
__device__ __forceinline__ int flip_of(int row) { return ((row >> 3) & 1) * (NC == 128 ? 64 : 16); }
template <int NC>
__device__ __forceinline__ bf16x8_t read_steps(const bf16_t (*arr)[NC + 16], int k2, int block, int g, int c) {
  typedef short i16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  const int row = 32 * k2 + 8 * g + (c >> 2), col = ((16 * block) ^ flip_of<NC>(8 * g)) + 4 * (c & 3);
  const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)&arr[row][col]);
  const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)&arr[row + 4][col]);
  return frag_from_halves(__builtin_bit_cast(u32x2_t, lo), __builtin_bit_cast(u32x2_t, hi));
}

// Grid (n_heads, B * n_seg).  CARRY: the state-only pass (segments before the last one).
//   xbc   bf16 [B*L, ld_xbc]: x of head h at columns x_col + 64 h, B at b_col, C at c_col (after conv + SiLU)
//   dt_raw bf16 [B*L, ld_dt]: column dt_col + h, before bias and softplus;   z bf16 [B*L, ld_z]: column 64 h
//   carry_state f32 [B][n_seg][H][NS][64], carry_decay f32 [B][n_seg][H]
//   h_in / h_out f32 [B][H][NS][64] or NULL: the state before the first and after the last step
//   yz    bf16 [B*L, ld_y]: (y + D x) * SiLU(z)
template <int NS, bool CARRY>
__global__ __launch_bounds__(256, 2) void ssd_kernel(const bf16_t *__restrict__ xbc, int64_t ld_xbc, int x_col, int b_col,
                                                  int c_col, const bf16_t *__restrict__ dt_raw, int64_t ld_dt,
                                                  int dt_col, const bf16_t *__restrict__ z, int64_t ld_z,
                                                  const float *__restrict__ dt_bias, const float *__restrict__ A_log,
                                                  const float *__restrict__ Dp, int64_t L, int n_seg, int64_t seg_len,
                                                  float *__restrict__ carry_state, float *__restrict__ carry_decay,
                                                  const float *h_in, float *h_out, bf16_t *__restrict__ yz,
                                                  int64_t ld_y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  SsdSmem<NS> &sm = *reinterpret_cast<SsdSmem<NS> *>(smem_raw);
  constexpr int kNB = NS / 16;          // 16-row blocks of the state
  constexpr int kKS = NS / 32;          // 32-wide steps of a contraction over the state index
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int h = blockIdx.x, n_heads = gridDim.x;
  const int64_t b = blockIdx.y / n_seg;
  const int seg = static_cast<int>(blockIdx.y % n_seg);
  if (CARRY && seg == n_seg - 1) return;            // nobody needs the last segment's end state
  const int64_t ts = seg * seg_len, te = ts + seg_len < L ? ts + seg_len : L;
  const float a = -__expf(A_log[h]);
  const float bias = dt_bias[h];
  const bf16_t *xbc_b = xbc + b * L * ld_xbc;
  const bf16_t *dt_b = dt_raw + b * L * ld_dt + dt_col + h;
  const int xc = x_col + h * kP;

  // state: hacc[nb][r] = H[n = 16 nb + 4 g + r][p = 16 wave + c]
  f32x4_t hacc[kNB];
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb) hacc[nb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t carry_stride = static_cast<int64_t>(NS) * kP;
  if (!CARRY) {
    if (h_in) {
      const float *sp = h_in + (b * n_heads + h) * carry_stride + wave * 16 + c;
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) hacc[nb][r] = sp[(16 * nb + 4 * g + r) * kP];
    }
    // fold the earlier segments' (decay, end state from zero) in order
    for (int j = 0; j < seg; ++j) {
      const int64_t unit = (b * n_seg + j) * n_heads + h;
      const float dec = fast_exp2(carry_decay[unit] * kLog2e);
      const float *sp = carry_state + unit * carry_stride + wave * 16 + c;
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) hacc[nb][r] = fmaf(dec, hacc[nb][r], sp[(16 * nb + 4 * g + r) * kP]);
    }
  }
  float log_decay_total = 0.0f;

  // While a chunk is parked a thread has pieces of 16 bytes: NS / 32 of B and of C, in rows p_row + i 256 / (NS / 8), and two of x, in rows
  // x_row + 32 i.  (With two wavefronts for B, one for x, which transposed 8 x 8 blocks in registers, the fourth waited: 16384 steps,
  // 64 heads of 128 states: main pass 220 us, carry 78.)
  constexpr int kPer = NS / 32, kRows = 256 / (NS / 8);
  const int p_row = tid / (NS / 8), p_col = tid % (NS / 8) * 8;
  const int x_row = tid >> 3, x_piece = tid & 7;
  // output rows: a wavefront stores the 16 channels it computed, two 8-channel pieces per step
  const int e_row = lane >> 1, e_po = 2 * wave + (lane & 1);

  // A chunk's inputs are requested one chunk ahead (rows beyond the segment's end: the last valid
  // row, zeroed when parked - no branch around a load, so that the requests go out back to back):
  // what the parking needs right after the chunk before has been parked, what the output rows need
  // (z) after the chunk before has been stored.  A row is a uniform base and one lane offset.
  u32x4_t pb[kPer], pc[kPer], px[2], ez[2];
  unsigned short p_dt = 0;
  auto load16 = [](const bf16_t *base, unsigned off) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4_t *>(reinterpret_cast<const char *>(base) + off);
  };
  const auto bytes = [](int64_t row, int64_t ld, int col) { return static_cast<unsigned>((row * ld + col) * 2); };
  const unsigned b_off = bytes(p_row, ld_xbc, p_col), x_off = bytes(x_row, ld_xbc, 8 * x_piece), z_off = bytes(e_row, ld_z, 8 * e_po);
  const unsigned dt_off = bytes(lane, ld_dt, 0);
  auto fetch_main = [&](int64_t t0) {
    if (t0 >= te) return;
    const bf16_t *const rows = xbc_b + t0 * ld_xbc;
    const char *const dts = reinterpret_cast<const char *>(dt_b + t0 * ld_dt);
    if (t0 + kQ <= te) {
      p_dt = *reinterpret_cast<const unsigned short *>(dts + dt_off);
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        pb[i] = load16(rows + b_col + i * kRows * ld_xbc, b_off);
        if (!CARRY) pc[i] = load16(rows + c_col + i * kRows * ld_xbc, b_off);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) px[i] = load16(rows + xc + 32 * i * ld_xbc, x_off);
    } else {
      const int last = static_cast<int>(te - 1 - t0);               // last valid row of the chunk
      const auto upto = [&](int r) { return r <= last ? r : last; };
      p_dt = *reinterpret_cast<const unsigned short *>(dts + bytes(upto(lane), ld_dt, 0));
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const unsigned off = bytes(upto(p_row + i * kRows), ld_xbc, p_col);
        pb[i] = load16(rows + b_col, off);
        if (!CARRY) pc[i] = load16(rows + c_col, off);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) px[i] = load16(rows + xc, bytes(upto(x_row + 32 * i), ld_xbc, 8 * x_piece));
    }
  };
  auto fetch_out = [&](int64_t t0) {
    if (CARRY || t0 >= te) return;
    const bf16_t *const rows = z + (b * L + t0) * ld_z + h * kP;
    if (t0 + kQ <= te) {
#pragma unroll
      for (int i = 0; i < 2; ++i) ez[i] = load16(rows + 32 * i * ld_z, z_off);
    } else {
      const int last = static_cast<int>(te - 1 - t0);
#pragma unroll
      for (int i = 0; i < 2; ++i) ez[i] = load16(rows, bytes(e_row + 32 * i <= last ? e_row + 32 * i : last, ld_z, 8 * e_po));
    }
  };
  fetch_main(ts);
  fetch_out(ts);
  // Scores on and below the diagonal, in blocks of 16 x 16 (row block 4 t + column block s a nibble), three for wavefronts 0 and 1, two for 2
  // and 3.  Of the others the products read (0, 1) and (2, 3) only: zero for good.
  constexpr uint64_t kBlocks = 0x0FA098E54DC0ull;
  const int n_blocks = wave < 2 ? 3 : 2;
  if (!CARRY) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (wave < 2) sm.g[32 * wave + c][32 * wave + 16 + 4 * g + r] = 0;
  }

  for (int64_t t0 = ts; t0 < te; t0 += kQ) {
    // time steps of the chunk, one per lane (every wavefront computes them for itself)
    float dtv = 0.0f;
    if (t0 + lane < te) dtv = softplus_f32(bf16_to_f32(p_dt) + bias);
    const float cum = wave_inclusive_sum(dtv * a);
    const float cum_last = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cum), 63));
    log_decay_total += cum_last;

    __syncthreads();                // the chunk before this one is done with the LDS
    if (t0 + kQ > te) {
      const int live = static_cast<int>(te - t0);
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (p_row + i * kRows >= live) pb[i] = pc[i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (x_row + 32 * i >= live) px[i] = u32x4_t{0u, 0u, 0u, 0u};
    }
    {
      // weight w_s = exp(cum_Q - cum_s) dt_s of step `lane`; the pieces' steps come from their lanes
      const float w_lane = fast_exp2((cum_last - cum) * kLog2e) * dtv;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int row = p_row + i * kRows;
        *reinterpret_cast<u32x4_t *>(&sm.bw[row][p_col ^ flip_of<NS>(row)]) = scale8(pb[i], __shfl(w_lane, row));
        if (!CARRY) {
          *reinterpret_cast<u32x4_t *>(&sm.u.b[row][p_col]) = pb[i];
          *reinterpret_cast<u32x4_t *>(&sm.c[row][p_col]) = pc[i];
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = x_row + 32 * i;
        *reinterpret_cast<u32x4_t *>(&sm.x[row][(8 * x_piece) ^ flip_of<kP>(row)]) = px[i];
      }
    }
    if (!CARRY) {
      if (wave == 3) {
        sm.cum[lane] = cum;
        sm.ecum[lane] = fast_exp2(cum * kLog2e);
        sm.dt[lane] = dtv;
      }
    }
    __syncthreads();
    fetch_main(t0 + kQ);

    f32x4_t yacc[4];
    if (!CARRY) {
      // scores, steps t = 16 tb + c against s = 16 sb + 4 g ..: G^T[s][t] = B_s . C_t, then the
      // causal mask, the decay exp(cum_t - cum_s) and the step size dt_s; stored [t][s]
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (j >= n_blocks) break;
        const int block = static_cast<int>(kBlocks >> (4 * (3 * wave + j))) & 15, tb = block >> 2, sb = block & 3;
        f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
          const bf16x8_t fa = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.u.b[16 * sb + c][32 * ks + 8 * g]));
          const bf16x8_t fb = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.c[16 * tb + c][32 * ks + 8 * g]));
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc, 0, 0, 0);
        }
        const float cum_t = sm.cum[16 * tb + c];
        const f32x4_t cum_s = *reinterpret_cast<const f32x4_t *>(&sm.cum[16 * sb + 4 * g]);
        const f32x4_t dt_s = *reinterpret_cast<const f32x4_t *>(&sm.dt[16 * sb + 4 * g]);
        float val[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int s = 16 * sb + 4 * g + r, t = 16 * tb + c;
          const float dec = exp2_here(s <= t ? (cum_t - cum_s[r]) * kLog2e : 0.0f);
          val[r] = s <= t ? acc[r] * dt_s[r] * dec : 0.0f;
        }
        const u32x2_t packed = {pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
        *reinterpret_cast<u32x2_t *>(&sm.g[16 * tb + c][16 * sb + 4 * g]) = packed;
      }
      // contribution of the state the chunk starts from: Y[t][p] = exp(cum_t) sum_n C[t][n] H[n][p].
      // The accumulators are the B operand as they are: slot (g, e) of a 32-wide step holds
      // n = 32 ks + 4 g + e (e < 4) or 32 ks + 16 + 4 g + e - 4, and C is read in the same order.
      bf16x8_t hop[kKS];
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) {
        const u32x4_t hv = {pack_bf16x2(hacc[2 * ks][0], hacc[2 * ks][1]), pack_bf16x2(hacc[2 * ks][2], hacc[2 * ks][3]),
                            pack_bf16x2(hacc[2 * ks + 1][0], hacc[2 * ks + 1][1]),
                            pack_bf16x2(hacc[2 * ks + 1][2], hacc[2 * ks + 1][3])};
        hop[ks] = as_frag(hv);
      }
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) {
        yacc[tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) {
          const u32x2_t lo = *reinterpret_cast<const u32x2_t *>(&sm.c[16 * tb + c][32 * ks + 4 * g]);
          const u32x2_t hi = *reinterpret_cast<const u32x2_t *>(&sm.c[16 * tb + c][32 * ks + 16 + 4 * g]);
          yacc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_halves(lo, hi), hop[ks], yacc[tb], 0, 0, 0);
        }
        const f32x4_t e = *reinterpret_cast<const f32x4_t *>(&sm.ecum[16 * tb + 4 * g]);
#pragma unroll
        for (int r = 0; r < 4; ++r) yacc[tb][r] *= e[r];
      }
      __syncthreads();              // all scores are in LDS; nobody reads B's step-major copy any more
    }

    // x of this wavefront's 16 channels, all 64 steps: B operand of both remaining products
    bf16x8_t xop[2];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
      xop[k2] = read_steps<kP>(sm.x, k2, wave, g, c);
    if (!CARRY) {
      // inside the chunk: Y[t][p] += sum_{s <= t} G[t][s] x_s[p]; steps 32.. only reach t >= 32
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
          if (k2 == 0 || tb >= 2) {
            const bf16x8_t fa = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.g[16 * tb + c][32 * k2 + 8 * g]));
            yacc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, xop[k2], yacc[tb], 0, 0, 0);
          }
    }
    // state at the chunk's end: H = exp(cum_Q) H + sum_s (exp(cum_Q - cum_s) dt_s B_s) x_s^T
    {
      const float dec = fast_exp2(cum_last * kLog2e);
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) hacc[nb][r] *= dec;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
          const bf16x8_t fa = read_steps<NS>(sm.bw, k2, nb, g, c);
          hacc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, xop[k2], hacc[nb], 0, 0, 0);
        }
      }
    }
    if (!CARRY) {
      // output tile through LDS (over B's step-major copy) so that rows go out in 16-byte pieces, with
      // the D skip and the SiLU(z) gate applied on the way; a wavefront reads back only the 16
      // columns it wrote itself, so no barrier is needed between the two
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sm.u.y[16 * tb + 4 * g + r][16 * wave + c] = yacc[tb][r];
      const float d_skip = Dp[h];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = e_row + 32 * i;
        const int64_t t = t0 + row;
        const f32x4_t y0 = *reinterpret_cast<const f32x4_t *>(&sm.u.y[row][8 * e_po]);
        const f32x4_t y1 = *reinterpret_cast<const f32x4_t *>(&sm.u.y[row][8 * e_po + 4]);
        const u32x4_t xv = *reinterpret_cast<const u32x4_t *>(&sm.x[row][(8 * e_po) ^ flip_of<kP>(row)]);
        float o[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const float yv = (m < 4 ? y0[m & 3] : y1[m & 3]) + d_skip * bf16_elem(xv, m);
          o[m] = yv * silu_f32(bf16_elem(ez[i], m));
        }
        const u32x4_t ov = {pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                            pack_bf16x2(o[6], o[7])};
        if (t < te) *reinterpret_cast<u32x4_t *>(yz + (b * L + t) * ld_y + h * kP + 8 * e_po) = ov;
      }
      fetch_out(t0 + kQ);
    }
  }

  if (CARRY) {
    const int64_t unit = (b * n_seg + seg) * n_heads + h;
    float *sp = carry_state + unit * carry_stride + wave * 16 + c;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) sp[(16 * nb + 4 * g + r) * kP] = hacc[nb][r];
    if (tid == 0) carry_decay[unit] = log_decay_total;
  } else if (h_out && seg == n_seg - 1) {
    float *sp = h_out + (b * n_heads + h) * carry_stride + wave * 16 + c;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) sp[(16 * nb + 4 * g + r) * kP] = hacc[nb][r];
  }
}

// One step per sequence (L == 1): grid (n_heads, B); thread = (four channels, every sixteenth state).  Bound by reading and
// writing the state once: a wavefront's instruction moves four whole states of 64 channels (1 KiB), and all of a thread's
// states are asked for before anything is computed.  256 sequences, 64 heads of 128 states: 266 us a lane a channel (256 bytes
// an instruction, eight states ahead), the step 401 -> 341; one sequence 54 -> 42.
template <int NS>
__global__ __launch_bounds__(256) void ssd_step_kernel(const bf16_t *__restrict__ xbc, int64_t ld_xbc, int x_col, int b_col,
                                                       int c_col, const bf16_t *__restrict__ dt_raw, int64_t ld_dt,
                                                       int dt_col, const bf16_t *__restrict__ z, int64_t ld_z,
                                                       const float *__restrict__ dt_bias, const float *__restrict__ A_log,
                                                       const float *__restrict__ Dp, const float *h_in, float *h_out,
                                                       bf16_t *__restrict__ yz, int64_t ld_y) {
  constexpr int kSt = NS / 16;                       // states per thread
  __shared__ float part[4][kP], bcs[2][NS];
  const int tid = threadIdx.x, p = (tid & 15) * 4, n0 = tid >> 4;
  const int h = blockIdx.x, n_heads = gridDim.x;
  const int64_t b = blockIdx.y;
  const int64_t base = (b * n_heads + h) * static_cast<int64_t>(NS) * kP + p;
  f32x4_t hv[kSt];
#pragma unroll
  for (int j = 0; j < kSt; ++j)
    hv[j] = h_in ? *reinterpret_cast<const f32x4_t *>(h_in + base + (n0 + 16 * j) * kP) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  const bf16_t *row = xbc + b * ld_xbc;
  if (tid < NS) bcs[0][tid] = bf16_to_f32(row[b_col + tid]);
  else if (tid < 2 * NS) bcs[1][tid - NS] = bf16_to_f32(row[c_col + tid - NS]);
  const float dt = softplus_f32(bf16_to_f32(dt_raw[b * ld_dt + dt_col + h]) + dt_bias[h]);
  const float dec = fast_exp2(-__expf(A_log[h]) * dt * kLog2e);
  float dtx[4], acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i) dtx[i] = dt * bf16_to_f32(row[x_col + h * kP + p + i]);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSt; ++j) {
    const int n = n0 + 16 * j;
    const float bv = bcs[0][n], cv = bcs[1][n];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      hv[j][i] = fmaf(dec, hv[j][i], dtx[i] * bv);
      acc[i] = fmaf(cv, hv[j][i], acc[i]);
    }
    if (h_out) *reinterpret_cast<f32x4_t *>(h_out + base + n * kP) = hv[j];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[i] += __shfl_xor(acc[i], 16);
    acc[i] += __shfl_xor(acc[i], 32);
    if ((tid & 63) < 16) part[tid >> 6][p + i] = acc[i];
  }
  __syncthreads();
  if (tid < kP) {
    const float y = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid] + Dp[h] * bf16_to_f32(row[x_col + h * kP + tid]);
    yz[b * ld_y + h * kP + tid] = f32_to_bf16(y * silu_f32(bf16_to_f32(z[b * ld_z + h * kP + tid])));
  }
}

// g[n, :] = yz[n, :] / sqrt(mean(yz[n, :]^2) + eps) * w: one wavefront per row, fp32 sums
__global__ __launch_bounds__(256) void rms_rows_kernel(const bf16_t *__restrict__ yz, const float *__restrict__ w,
                                                       float eps, int64_t n_rows, int n_cols, bf16_t *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const bf16_t *src = yz + row * n_cols;
  float ss = 0.0f;
  for (int c0 = lane * 8; c0 < n_cols; c0 += 512) {
    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(src + c0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const float f = bf16_elem(v, m);
      ss = fmaf(f, f, ss);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
  const float rstd = rsqrtf(ss / static_cast<float>(n_cols) + eps);
  bf16_t *dst = out + row * n_cols;
  for (int c0 = lane * 8; c0 < n_cols; c0 += 512) {
    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(src + c0);
    const f32x4_t w0 = *reinterpret_cast<const f32x4_t *>(w + c0), w1 = *reinterpret_cast<const f32x4_t *>(w + c0 + 4);
    float o[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) o[m] = bf16_elem(v, m) * rstd * (m < 4 ? w0[m & 3] : w1[m & 3]);
    const u32x4_t ov = {pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7])};
    *reinterpret_cast<u32x4_t *>(dst + c0) = ov;
  }
}

struct SsdPlan {
  int n_seg;
  int64_t seg_len;
};
SsdPlan ssd_plan(int64_t B, int64_t L, int n_heads) {
  // two workgroups for each of the 256 CUs; a segment is whole chunks and at least four of them
  const int64_t chunks = ceil_div(L, kQ);
  int64_t n_seg = ceil_div(512, B * n_heads);
  const int64_t max_seg = chunks / 4 > 0 ? chunks / 4 : 1;
  n_seg = n_seg < 1 ? 1 : (n_seg > max_seg ? max_seg : n_seg);
  SsdPlan p;
  p.seg_len = ceil_div(chunks, n_seg) * kQ;
  p.n_seg = static_cast<int>(ceil_div(L, p.seg_len));
  return p;
}

template <int NS, bool CARRY>
hipError_t ssd_allow_lds() {
  // more than 64 KiB of dynamic LDS: a function attribute, set once per device
  static std::mutex mu;
  static std::atomic<bool> done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!done[dev].load(std::memory_order_acquire)) {
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev].load(std::memory_order_relaxed)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&ssd_kernel<NS, CARRY>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(sizeof(SsdSmem<NS>)));
      if (e != hipSuccess) return e;
      done[dev].store(true, std::memory_order_release);
    }
  }
  return hipSuccess;
}

template <int NS>
hipError_t ssd_dispatch(const bf16_t *xbc, int64_t ld_xbc, int x_col, int b_col, int c_col, const bf16_t *dt_raw,
                        int64_t ld_dt, int dt_col, const bf16_t *z, int64_t ld_z, const float *dt_bias,
                        const float *A_log, const float *D, const float *h_in, float *h_out, int64_t B, int64_t L,
                        int n_heads, float *carry, bf16_t *yz, int64_t ld_y, hipStream_t s) {
  if (L == 1) {
    hipLaunchKernelGGL((ssd_step_kernel<NS>), dim3(static_cast<unsigned>(n_heads), static_cast<unsigned>(B)), dim3(256), 0,
                       s, xbc, ld_xbc, x_col, b_col, c_col, dt_raw, ld_dt, dt_col, z, ld_z, dt_bias, A_log, D, h_in, h_out,
                       yz, ld_y);
    return hipGetLastError();
  }
  const SsdPlan p = ssd_plan(B, L, n_heads);
  float *carry_state = carry;
  float *carry_decay = carry + static_cast<size_t>(B) * p.n_seg * n_heads * NS * kP;
  const dim3 grid(static_cast<unsigned>(n_heads), static_cast<unsigned>(B * p.n_seg));
  const size_t lds = sizeof(SsdSmem<NS>);
  hipError_t e;
  if (p.n_seg > 1) {
    if ((e = ssd_allow_lds<NS, true>()) != hipSuccess) return e;
    hipLaunchKernelGGL((ssd_kernel<NS, true>), grid, dim3(256), lds, s, xbc, ld_xbc, x_col, b_col, c_col, dt_raw, ld_dt,
                       dt_col, z, ld_z, dt_bias, A_log, D, L, p.n_seg, p.seg_len, carry_state, carry_decay, h_in, h_out, yz,
                       ld_y);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = ssd_allow_lds<NS, false>()) != hipSuccess) return e;
  hipLaunchKernelGGL((ssd_kernel<NS, false>), grid, dim3(256), lds, s, xbc, ld_xbc, x_col, b_col, c_col, dt_raw, ld_dt,
                     dt_col, z, ld_z, dt_bias, A_log, D, L, p.n_seg, p.seg_len, carry_state, carry_decay, h_in, h_out, yz,
                     ld_y);
  return hipGetLastError();
}

}  // namespace

size_t ssd_carry_bytes(int64_t B, int64_t L, int n_heads, int d_state) {
  const SsdPlan p = ssd_plan(B, L, n_heads);
  if (p.n_seg <= 1) return 0;
  return static_cast<size_t>(B) * p.n_seg * n_heads * (static_cast<size_t>(d_state) * kP + 1) * sizeof(float);
}

bool ssd_supported(int d_state, int headdim) { return headdim == kP && (d_state == 64 || d_state == 128); }

hipError_t launch_ssd_scan(const void *xbc, int64_t ld_xbc, int x_col, int b_col, int c_col, const void *dt_raw,
                           int64_t ld_dt, int dt_col, const void *z, int64_t ld_z, const float *dt_bias,
                           const float *A_log, const float *D, const float *h_in, float *h_out, int64_t B, int64_t L,
                           int n_heads, int d_state, float *carry, void *yz, int64_t ld_y, hipStream_t s) {
  if (B * L <= 0) return hipSuccess;
  if (B * ssd_plan(B, L, n_heads).n_seg > 65535) return hipErrorInvalidValue;
  const bf16_t *xp = static_cast<const bf16_t *>(xbc), *dp = static_cast<const bf16_t *>(dt_raw);
  const bf16_t *zp = static_cast<const bf16_t *>(z);
  if (d_state == 128)
    return ssd_dispatch<128>(xp, ld_xbc, x_col, b_col, c_col, dp, ld_dt, dt_col, zp, ld_z, dt_bias, A_log, D, h_in, h_out, B,
                             L, n_heads, carry, static_cast<bf16_t *>(yz), ld_y, s);
  if (d_state == 64)
    return ssd_dispatch<64>(xp, ld_xbc, x_col, b_col, c_col, dp, ld_dt, dt_col, zp, ld_z, dt_bias, A_log, D, h_in, h_out, B,
                            L, n_heads, carry, static_cast<bf16_t *>(yz), ld_y, s);
  return hipErrorInvalidValue;
}

hipError_t launch_rms_rows(const void *yz, const float *w, float eps, int64_t n_rows, int n_cols, void *out,
                           hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(rms_rows_kernel, dim3(static_cast<unsigned>(ceil_div(n_rows, 4))), dim3(256), 0, s,
                     static_cast<const bf16_t *>(yz), w, eps, n_rows, n_cols, static_cast<bf16_t *>(out));
  return hipGetLastError();
}

}  // namespace rom
