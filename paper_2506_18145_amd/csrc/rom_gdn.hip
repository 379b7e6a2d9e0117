// RoM on a Gated DeltaNet layer (Sec. 5.2, Table 3): the sequence part between the routed input and
// output projections - per head the gated delta rule on the state S (d_v x d_k)
//     S_t = exp(g_t) S_{t-1} (I - beta_t k_t k_t^T) + beta_t v_t k_t^T,     o_t = S_t q_t
// with q, k L2-normalised per head, then the per-head RMS norm and the SiLU(z) gate.  gfx950 only,
// bf16 activations, d_v = 64, d_k = 64 or 128.
//
// Chunked form (chunks of 64 steps, cum_t = sum_{r <= t} g_r inside the chunk, gamma = exp(cum)): the
// rank-one updates u_t = beta_t (v_t - exp(g_t) S_{t-1} k_t) of a chunk obey the unit lower-triangular
// system
//     (I + A) U = diag(beta) (V - diag(gamma) K S_0^T),   A[t][s] = beta_t exp(cum_t - cum_s) (k_t . k_s), s < t,
// and then  O = diag(gamma) Q S_0^T + (Q K^T o exp(cum_t - cum_s), s <= t) U,
//           S_new = gamma_64 S_0 + sum_s exp(cum_64 - cum_s) u_s k_s^T.
// Everything but the inverse is a small matrix product on v_mfma_f32_16x16x32_bf16; T = (I + A)^-1 is
// computed in fp32: the four 16 x 16 diagonal blocks by forward substitution (one wavefront, a lane per
// column), the six blocks below them by block substitution on v_mfma_f32_16x16x4_f32.  T and the decayed
// scores Q K^T do not depend on the state: gdn_prep_kernel forms them for all chunks at once.
// In the recurrence a workgroup (4 wavefronts) owns one (sequence, head, segment of the sequence) and walks its chunks in
// order.  Few (sequence, head) pairs: the sequences are cut into segments.  A segment's effect on the
// state is S_end = S_start Phi + Z with Phi = prod_t exp(g_t)(I - beta_t k_t k_t^T) a d_k x d_k MATRIX, so
// the carry pass runs the same rule on the state augmented by d_k more "value" rows that start from the
// identity and see v = 0 (their end value is Phi), a small kernel folds (Phi, Z) along each sequence, and
// the main pass starts every segment from its folded state.  Wavefront w
// holds the state columns S^T[:, 16w .. 16w+15] (d_k x 16 values of d_v) in accumulators, as the
// Mamba2 kernel does, and the products that contract over steps or over d_k take their second
// operand straight from accumulators (the contraction index permuted alike on the other side).
#include "rom_chunk.h"

#include <atomic>
#include <mutex>

namespace rom {
namespace {

using namespace chunk;

constexpr int kV = 64;          // value channels per head
constexpr float kL2Eps = 1e-6f;

// The step-parallel part of a chunk needs no state: it runs over all chunks at once, ahead of the recurrence.
template <int NS>
struct GdnPrepSmem {
  union {
    struct {
      bf16_t kn[kQ][NS + 8];    // normalised keys, step-major
      bf16_t qr[kQ][NS + 8];    // raw queries, step-major
    } in;
    float tm[kQ][kQ + 4];       // after the scores: T = (I + A)^-1
  } u;
  float am[kQ][kQ + 4];         // A (strictly lower triangle)
  float cum[kQ], beta[kQ];
};

template <int NS, bool CARRY>
struct GdnSmem {
  bf16_t kn[kQ][NS + 8];                  // normalised keys, step-major
  bf16_t vt[kQ][kV + 16];                 // values, step-major
  bf16_t kw[kQ][NS + 16];                 // exp(cum_64 - cum_s) k_s, step-major
  bf16_t qr[CARRY ? 1 : kQ][NS + 8];      // raw queries, step-major
  float y[CARRY ? 1 : kQ][kV + 4];        // the output tile
  float ecum[kQ], beta[kQ], rq[kQ];
};

// Operand fragments of a chunk in HBM: T, then G = exp(cum_t - cum_s) (q_t . k_s), s <= t, both in bf16 and
// lower triangular.  Fragment (tb, k2) covers rows 16 tb .. +15 and columns 32 k2 .. +31; the two that lie
// above the diagonal do not exist.  Lane (g, c) owns row 16 tb + c, columns 32 k2 + 4 g .. +3 and 32 k2 + 16 + 4 g .. +3.
constexpr int kFrags = 6;
// Behind them cum_t and beta_t of its 64 steps, fp32.
constexpr int kChunkWords = 2 * kFrags * 64 + 2 * kQ / 4;  // of one chunk, in 16-byte words
constexpr size_t kFragFloats = kChunkWords * 4;
template <int NS>
struct GdnOneSmem {
  GdnSmem<NS, false> main;
  GdnPrepSmem<NS> prep;
  u32x4_t frags[kChunkWords];
};
// Four rows x 16 columns of a step-major array in LDS per 16 lanes: lane i names row i / 4, columns 4 (i % 4) .. +3, and receives column
// i of the four rows.  Rows of 32 bytes more than a multiple of 256 or 128 keep 32 lanes' pieces in different banks.
__device__ __forceinline__ u32x2_t read_transposed(const bf16_t *at) {
  typedef short i16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)at));
}
__device__ __forceinline__ constexpr int frag_id(int tb, int k2) { return k2 == 0 ? tb : 2 + tb; }

__device__ __forceinline__ float sum_sq8(const u32x4_t &v) {
  float s = 0.0f;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const float f = bf16_elem(v, m);
    s = fmaf(f, f, s);
  }
  return s;
}
// sum over the WIDTH (8 or 16) consecutive lanes that share a row
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int WIDTH>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(WIDTH == 8 || WIDTH == 16, "mirrors of 8 and of 16 lanes");
  v += dpp_of<0xB1>(v);                          // lane ^ 1
  v += dpp_of<0x4E>(v);                          // lane ^ 2
  v += dpp_of<0x141>(v);                         // lane 7 - i of its eight: from here on all of a half hold its sum
  if constexpr (WIDTH == 16) v += dpp_of<0x140>(v);       // lane 15 - i
  return v;
}

// T = (I + A)^-1 for the 64 x 64 unit lower-triangular I + A: am -> tm (blocks on and below the diagonal).  Called by the
// whole workgroup (it contains barriers): wavefront 0 solves the four diagonal blocks, then the blocks
// at distance 1, 2, 3 below the diagonal are computed level by level, one block per wavefront.
__device__ __forceinline__ void invert_unit_lower(const float (*am)[kQ + 4], float (*tm)[kQ + 4],
                                                  int lane, int wave) {
  const int g = lane >> 4, c = lane & 15;
  // diagonal blocks: lane (g, c) solves column c of block g by forward substitution
  if (wave == 0) {
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float acc = r == c ? 1.0f : 0.0f;
#pragma unroll
      for (int m = 0; m < r; ++m) acc = fmaf(-am[16 * g + r][16 * g + m], x[m], acc);
      x[r] = acc;
      asm volatile("" ::: "memory");         // row by row: hoisting all 120 LDS reads costs as many registers
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) tm[16 * g + r][16 * g + c] = x[r];
  }
  __syncthreads();
  // blocks below the diagonal, by distance d from it: T_ij = -T_ii sum_{m = j .. i-1} A_im T_mj, i = j + d
#pragma unroll
  for (int d = 1; d < 4; ++d) {
    const int j = wave, i = wave + d;
    if (i < 4) {
      f32x4_t m0 = {0.0f, 0.0f, 0.0f, 0.0f}, m1 = {0.0f, 0.0f, 0.0f, 0.0f};      // two chains of dependent MFMAs
      for (int m = j; m < i; ++m)
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          m0 = __builtin_amdgcn_mfma_f32_16x16x4f32(am[16 * i + c][16 * m + 4 * q + g], tm[16 * m + 4 * q + g][16 * j + c], m0, 0,
                                                     0, 0);
          m1 = __builtin_amdgcn_mfma_f32_16x16x4f32(am[16 * i + c][16 * m + 4 * q + 4 + g], tm[16 * m + 4 * q + 4 + g][16 * j + c],
                                                     m1, 0, 0, 0);
        }
      const f32x4_t macc = m0 + m1;
      // second product with the accumulators as the B operand: contraction slot (q, g) <-> k = 4 g + q
      f32x4_t res = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        res = __builtin_amdgcn_mfma_f32_16x16x4f32(tm[16 * i + c][16 * i + 4 * g + q], macc[q], res, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) tm[16 * i + 4 * g + r][16 * j + c] = -res[r];
    }
    __syncthreads();
  }
}

// What a chunk needs besides the state: T and the decayed scores G of every (sequence, chunk, head), one
// workgroup each (grid 1-D: heads fastest, then chunks, then sequences), written as operand fragments.
// The inverse is a serial chain (forward substitution, then three levels of small products); inside the
// recurrence, one workgroup per CU, it stood in every chunk's critical path and was done twice, in the carry
// and in the main pass.  Here three or four workgroups share a CU and cover one another's waits, and the
// recurrence has three barriers a chunk instead of eight.  1 x 16384 x 2048, 32 heads of 64: this launch, carry, fold and
// main pass 573 -> 408 us, the layer 1467 -> 1166 us.
// T and G of the chunk at step t0 of a sequence of L steps (qkv_b, proj_b: its first step), head h, as fragments: `out` is the
// calling lane's place in the first of them.
template <int NS>
__device__ __forceinline__ void gdn_prep_chunk(GdnPrepSmem<NS> &sm, const bf16_t *__restrict__ qkv_b, int64_t ld_qkv, int q_col,
                                               int k_col, const bf16_t *__restrict__ proj_b, int64_t ld_p, int b_col, int a_col,
                                               const float *__restrict__ dt_bias, const float *__restrict__ A_log, int64_t L,
                                               int64_t t0, int h, u32x4_t *out) {
  constexpr int kKS = NS / 32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;

  u32x4_t pk[NS / 32], pq[NS / 32];
#pragma unroll
  for (int i = 0; i < NS / 32; ++i) {
    const int piece = tid + 256 * i;
    const int64_t t = t0 + piece / (NS / 8);
    const bf16_t *row = qkv_b + (t < L ? t : L - 1) * ld_qkv + h * NS + 8 * (piece % (NS / 8));
    pk[i] = *reinterpret_cast<const u32x4_t *>(row + k_col);
    pq[i] = *reinterpret_cast<const u32x4_t *>(row + q_col);
  }
  if (wave == 3) {
    const bool live = t0 + lane < L;
    const bf16_t *row = proj_b + (live ? t0 + lane : L - 1) * ld_p;
    const float pb = bf16_to_f32(row[b_col + h]), pa = bf16_to_f32(row[a_col + h]);
    const float beta = live ? fast_rcp(1.0f + __expf(-pb)) : 0.0f;
    const float gl = live ? -__expf(A_log[h]) * softplus_f32(pa + dt_bias[h]) : 0.0f;
    const float cum = wave_inclusive_sum(gl);
    sm.cum[lane] = cum;
    sm.beta[lane] = beta;
  }
#pragma unroll
  for (int i = 0; i < NS / 32; ++i) {
    const int piece = tid + 256 * i;
    const int row = piece / (NS / 8), oc = piece % (NS / 8);
    if (t0 + row >= L) pk[i] = pq[i] = u32x4_t{0u, 0u, 0u, 0u};
    const float rk = rsqrtf(group_sum<NS / 8>(sum_sq8(pk[i])) + kL2Eps);
    *reinterpret_cast<u32x4_t *>(&sm.u.in.kn[row][8 * oc]) = scale8(pk[i], rk);
    *reinterpret_cast<u32x4_t *>(&sm.u.in.qr[row][8 * oc]) = pq[i];
  }
  __syncthreads();

  // scores of this wavefront's 16 steps t = 16 wave + c against all s <= t, computed transposed: a lane's
  // values of G are the row segment that its fragments hold
  u32x2_t gpk[4];
  {
    const float cum_t = sm.cum[16 * wave + c], beta_t = sm.beta[16 * wave + c];
#pragma unroll
    for (int sb = 0; sb < 4; ++sb) {
      f32x4_t kk = {0.0f, 0.0f, 0.0f, 0.0f}, qk = {0.0f, 0.0f, 0.0f, 0.0f};
      gpk[sb] = u32x2_t{0u, 0u};
      if (sb > wave) continue;
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) {
        const bf16x8_t fa = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.u.in.kn[16 * sb + c][32 * ks + 8 * g]));
        const bf16x8_t fk = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.u.in.kn[16 * wave + c][32 * ks + 8 * g]));
        const bf16x8_t fq = as_frag(*reinterpret_cast<const u32x4_t *>(&sm.u.in.qr[16 * wave + c][32 * ks + 8 * g]));
        kk = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fk, kk, 0, 0, 0);
        qk = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fq, qk, 0, 0, 0);
      }
      const f32x4_t cum_s = *reinterpret_cast<const f32x4_t *>(&sm.cum[16 * sb + 4 * g]);
      f32x4_t av;
      float gv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 16 * sb + 4 * g + r, t = 16 * wave + c;
        const float e = exp2_here(s <= t ? (cum_t - cum_s[r]) * kLog2e : 0.0f), dec = s <= t ? e : 0.0f;
        av[r] = s < t ? beta_t * dec * kk[r] : 0.0f;
        gv[r] = dec * qk[r];
      }
      *reinterpret_cast<f32x4_t *>(&sm.am[16 * wave + c][16 * sb + 4 * g]) = av;
      gpk[sb] = u32x2_t{pack_bf16x2(gv[0], gv[1]), pack_bf16x2(gv[2], gv[3])};
    }
  }
  __syncthreads();                // A is complete; the step-major keys and queries are no longer read
  invert_unit_lower(sm.am, sm.u.tm, lane, wave);

  out[(kFrags + frag_id(wave, 0)) * 64] = u32x4_t{gpk[0][0], gpk[0][1], gpk[1][0], gpk[1][1]};
  if (wave >= 2) out[(kFrags + frag_id(wave, 1)) * 64] = u32x4_t{gpk[2][0], gpk[2][1], gpk[3][0], gpk[3][1]};
  if (wave == 3) {
    float *const tail = reinterpret_cast<float *>(out - lane + 2 * kFrags * 64);
    tail[lane] = sm.cum[lane];
    tail[kQ + lane] = sm.beta[lane];
  }
#pragma unroll
  for (int k2 = 0; k2 < 2; ++k2) {
    if (k2 == 1 && wave < 2) break;
    const float *row = &sm.u.tm[16 * wave + c][32 * k2 + 4 * g];
    f32x4_t lo = *reinterpret_cast<const f32x4_t *>(row), hi = {0.0f, 0.0f, 0.0f, 0.0f};
    if (2 * k2 + 1 <= wave) hi = *reinterpret_cast<const f32x4_t *>(row + 16);       // blocks above the diagonal are zero
    out[frag_id(wave, k2) * 64] = u32x4_t{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]),
                                          pack_bf16x2(hi[2], hi[3])};
  }
}

template <int NS>
__global__ __launch_bounds__(256, NS == 64 ? 4 : 3) void gdn_prep_kernel(
    const bf16_t *__restrict__ qkv, int64_t ld_qkv, int q_col, int k_col, const bf16_t *__restrict__ proj, int64_t ld_p,
    int b_col, int a_col, const float *__restrict__ dt_bias, const float *__restrict__ A_log, int64_t L, int n_chunks,
    int n_heads, u32x4_t *__restrict__ frags) {
  __shared__ GdnPrepSmem<NS> sm;
  const int h = blockIdx.x % n_heads;
  const int64_t bc = blockIdx.x / n_heads;
  const int64_t b = bc / n_chunks, chunk = bc % n_chunks;
  gdn_prep_chunk<NS>(sm, qkv + b * L * ld_qkv, ld_qkv, q_col, k_col, proj + b * L * ld_p, ld_p, b_col, a_col, dt_bias, A_log, L,
                     chunk * kQ, h, frags + ((b * n_heads + h) * n_chunks + chunk) * kChunkWords + (threadIdx.x & 63));
}

//   qkv   bf16 [B*L, ld_qkv] after conv + SiLU: q of head h at q_col + NS h, k at k_col + NS h, v at v_col + 64 h
//   proj  bf16 [B*L, ld_p]: z of head h at columns 64 h, the beta logit at b_col + h, the decay logit at a_col + h
//   s_in / s_out f32 [B][H][NS][64] (S^T: [d_k][d_v]) or NULL;   y bf16 [B*L, ld_y]: RMSNorm_head(o) * norm_w * SiLU(z)
// Grid (n_heads, B * n_seg).  CARRY: the carry pass (no queries, no outputs; segments before the last):
//   carry_z f32 [B][H][n_seg][NS][64] <- Z^T, carry_m f32 [B][H][n_seg][NS][NS] <- [n][j] = Phi[j][n].
//   frags: gdn_prep_kernel's T and G of every chunk
// Main pass with n_seg > 1: segment `seg` starts from s_start f32 [B][H][n_seg][NS][64].
// ONE: the sequences are one chunk, whose T and G this workgroup forms itself and keeps in LDS (frags unused).
template <int NS, bool CARRY, bool ONE = false>
__global__ __launch_bounds__(256, CARRY && NS == 128 ? 1 : 2) void gdn_kernel(const bf16_t *__restrict__ qkv, int64_t ld_qkv, int q_col, int k_col,
                                                     int v_col, const bf16_t *__restrict__ proj, int64_t ld_p, int b_col,
                                                     int a_col, const float *__restrict__ dt_bias,
                                                     const float *__restrict__ A_log, const float *__restrict__ norm_w,
                                                     float eps, int64_t L, int n_seg, int64_t seg_len, int n_chunks,
                                                     const u32x4_t *__restrict__ frags,
                                                     float *__restrict__ carry_z, float *__restrict__ carry_m,
                                                     const float *__restrict__ s_start, const float *s_in, float *s_out,
                                                     bf16_t *__restrict__ y, int64_t ld_y) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  GdnSmem<NS, CARRY> &sm = *reinterpret_cast<GdnSmem<NS, CARRY> *>(smem_raw);
  constexpr int kNB = NS / 16, kKS = NS / 32;
  constexpr int kG = CARRY ? 1 + NS / 64 : 1;      // groups of 64 "value" columns: the state, and in the carry pass Phi
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int h = blockIdx.x, n_heads = gridDim.x;
  const int64_t b = blockIdx.y / n_seg;
  const int seg = static_cast<int>(blockIdx.y % n_seg);
  if (CARRY && seg == n_seg - 1) return;            // nobody needs the last segment's carry
  const int64_t ts = seg * seg_len, te = ts + seg_len < L ? ts + seg_len : L;
  const bf16_t *qkv_b = qkv + b * L * ld_qkv;
  const bf16_t *proj_b = proj + b * L * ld_p;
  const float q_scale = rsqrtf(static_cast<float>(NS));

  // state: sacc[0][nb][r] = S^T[d_k index 16 nb + 4 g + r][d_v index 16 wave + c]; carry pass: groups 1.. hold
  // the columns 64 (grp - 1) + 16 wave + c of the transition's transpose, starting from the identity
  f32x4_t sacc[kG][kNB];
  const int64_t s_stride = static_cast<int64_t>(NS) * kV;
  const int64_t unit = (b * n_heads + h) * n_seg + seg;
  GdnOneSmem<NS> &one = *reinterpret_cast<GdnOneSmem<NS> *>(smem_raw);
  if constexpr (ONE)
    gdn_prep_chunk<NS>(one.prep, qkv_b, ld_qkv, q_col, k_col, proj_b, ld_p, b_col, a_col, dt_bias, A_log, L, 0, h, one.frags + lane);
  if constexpr (ONE) __syncthreads();             // cum and beta are read before the loop's first barrier
#pragma unroll
  for (int grp = 0; grp < kG; ++grp)
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sacc[grp][nb][r] = (grp > 0 && 16 * nb + 4 * g + r == 64 * (grp - 1) + 16 * wave + c) ? 1.0f : 0.0f;
  if (!CARRY) {
    const float *sp = n_seg > 1 ? s_start + unit * s_stride : (s_in ? s_in + (b * n_heads + h) * s_stride : nullptr);
    if (sp) {
      sp += wave * 16 + c;
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sacc[0][nb][r] = sp[(16 * nb + 4 * g + r) * kV];
    }
  }

  const int e_row = tid >> 3, e_po = tid & 7;

  // A chunk's inputs are requested one chunk ahead (rows beyond the end: the last valid row, zeroed
  // when parked): what the parking needs right after the chunk before has been parked, the gate rows
  // after the chunk before has been stored.
  u32x4_t pk[NS / 32], pv[2], pq[NS / 32], ez[2];
  const u32x4_t *frag_ptr = ONE ? one.frags + lane : frags + ((b * n_heads + h) * n_chunks + ts / kQ) * kChunkWords + lane;
  float p_cum = 0.0f, p_beta = 0.0f;
  auto fetch_main = [&](int64_t t0) {
    if (t0 >= te) return;
    const float *const tail = reinterpret_cast<const float *>(frag_ptr - lane + 2 * kFrags * 64);     // frag_ptr: this chunk's
    p_cum = tail[lane];
    p_beta = tail[kQ + lane];
#pragma unroll
    for (int i = 0; i < NS / 32; ++i) {
      const int piece = tid + 256 * i;
      const int64_t t = t0 + piece / (NS / 8);
      const bf16_t *src = qkv_b + (t < te ? t : te - 1) * ld_qkv + h * NS + 8 * (piece % (NS / 8));
      pk[i] = *reinterpret_cast<const u32x4_t *>(src + k_col);
      if (!CARRY) pq[i] = *reinterpret_cast<const u32x4_t *>(src + q_col);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t t = t0 + e_row + 32 * i;
      pv[i] = *reinterpret_cast<const u32x4_t *>(qkv_b + (t < te ? t : te - 1) * ld_qkv + v_col + h * kV + 8 * e_po);
    }
  };
  auto fetch_out = [&](int64_t t0) {
    if (CARRY || t0 >= te) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t t = t0 + e_row + 32 * i;
      ez[i] = *reinterpret_cast<const u32x4_t *>(proj_b + (t < te ? t : te - 1) * ld_p + h * kV + 8 * e_po);
    }
  };
  fetch_main(ts);
  fetch_out(ts);

  for (int64_t t0 = ts; t0 < te; t0 += kQ) {
    // The lane's coordinates go through an opaque copy every chunk: with them loop-invariant the compiler
    // hoists some two hundred addresses and mask predicates out of the loop and spills them.
    const int gq = opaque(g), cq = opaque(c);
    const int tq = opaque(tid), erq = opaque(e_row), epq = opaque(e_po);
    // cumulative log decay and beta, one step per lane
    const float cum = p_cum, beta = p_beta;
    const float cum_last = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, cum), 63));

    // this chunk's T and G, wanted after the products with the state the chunk starts from: ahead of the next chunk's inputs, whose
    // arrival the wait for them would include
    u32x4_t tfr[kFrags], gfr[kFrags];
#pragma unroll
    for (int i = 0; i < kFrags; ++i) {
      tfr[i] = frag_ptr[i * 64];
      if (!CARRY) gfr[i] = frag_ptr[(kFrags + i) * 64];
    }
    frag_ptr += kChunkWords;
    __syncthreads();                // the chunk before this one is done with the LDS
    // Pieces of 16 bytes, NS / 32 (keys, queries) and two (values) a thread: the NS / 8 lanes that hold a row sum its squares.  With
    // a wavefront each for the keys and the values, a lane eight rows, this stood for half of a chunk's time.
    const float w_lane = fast_exp2((cum_last - cum) * kLog2e);
    if (t0 + kQ > te) {
      const int live = static_cast<int>(te - t0);
#pragma unroll
      for (int i = 0; i < NS / 32; ++i)
        if ((tq + 256 * i) / (NS / 8) >= live) pk[i] = pq[i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (erq + 32 * i >= live) pv[i] = u32x4_t{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < NS / 32; ++i) {
      const int piece = tq + 256 * i;
      const int row = piece / (NS / 8), oc = piece % (NS / 8);
      const u32x4_t v = pk[i];
      const float rk = rsqrtf(group_sum<NS / 8>(sum_sq8(v)) + kL2Eps);
      *reinterpret_cast<u32x4_t *>(&sm.kn[row][8 * oc]) = scale8(v, rk);
      *reinterpret_cast<u32x4_t *>(&sm.kw[row][8 * oc]) = scale8(v, rk * __shfl(w_lane, row));
      if (!CARRY) {                                 // queries: raw, and their norms
        const u32x4_t q = pq[i];
        *reinterpret_cast<u32x4_t *>(&sm.qr[row][8 * oc]) = q;
        const float ss = group_sum<NS / 8>(sum_sq8(q));
        if (oc == 0) sm.rq[row] = rsqrtf(ss + kL2Eps) * q_scale;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4_t *>(&sm.vt[erq + 32 * i][8 * epq]) = pv[i];
    if (wave == 3) {
      sm.ecum[lane] = fast_exp2(cum * kLog2e);
      sm.beta[lane] = beta;
    }
    __syncthreads();
    fetch_main(t0 + kQ);

    bf16x8_t sop[kG][kKS];
#pragma unroll
    for (int grp = 0; grp < kG; ++grp)
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) sop[grp][ks] = frag_from_acc(sacc[grp][2 * ks], sacc[grp][2 * ks + 1]);
    f32x4_t rhs[kG][4], oacc[4];
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      f32x4_t pacc[kG];
#pragma unroll
      for (int grp = 0; grp < kG; ++grp) pacc[grp] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      oacc[tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks) {
        const bf16x8_t fk = frag_perm<NS + 8>(sm.kn, 16 * tb + cq, 32 * ks, gq);
#pragma unroll
        for (int grp = 0; grp < kG; ++grp) pacc[grp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fk, sop[grp][ks], pacc[grp], 0, 0, 0);
        if (!CARRY)
          oacc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_perm<NS + 8>(sm.qr, 16 * tb + cq, 32 * ks, gq), sop[0][ks],
                                                             oacc[tb], 0, 0, 0);
      }
      const f32x4_t e = *reinterpret_cast<const f32x4_t *>(&sm.ecum[16 * tb + 4 * gq]);
      const f32x4_t bt = *reinterpret_cast<const f32x4_t *>(&sm.beta[16 * tb + 4 * gq]);
      const u32x2_t v4 = read_transposed(&sm.vt[16 * tb + 4 * gq + (cq >> 2)][16 * wave + 4 * (cq & 3)]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float vv = __uint_as_float(r & 1 ? v4[r / 2] & 0xFFFF0000u : v4[r / 2] << 16);
        rhs[0][tb][r] = bt[r] * (vv - e[r] * pacc[0][r]);    // beta_t (v_t - gamma_t S_0 k_t)
#pragma unroll
        for (int grp = 1; grp < kG; ++grp) rhs[grp][tb][r] = -bt[r] * e[r] * pacc[grp][r];      // the same with v = 0
        oacc[tb][r] *= e[r];                                  // gamma_t S_0 q_t
      }
    }
    // ---- U = T rhs (rows t, this wavefront's 16 value channels); the contraction runs over steps,
    //      with rhs taken from the accumulators
    f32x4_t uacc[kG][4];
    {
      bf16x8_t rop[kG][2];
#pragma unroll
      for (int grp = 0; grp < kG; ++grp)
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) rop[grp][k2] = frag_from_acc(rhs[grp][2 * k2], rhs[grp][2 * k2 + 1]);
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) {
#pragma unroll
        for (int grp = 0; grp < kG; ++grp) uacc[grp][tb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
          if (k2 == 0 || tb >= 2) {
            const bf16x8_t ft = as_frag(tfr[frag_id(tb, k2)]);
#pragma unroll
            for (int grp = 0; grp < kG; ++grp)
              uacc[grp][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ft, rop[grp][k2], uacc[grp][tb], 0, 0, 0);
          }
      }
    }
    bf16x8_t uop[kG][2];
#pragma unroll
    for (int grp = 0; grp < kG; ++grp)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) uop[grp][k2] = frag_from_acc(uacc[grp][2 * k2], uacc[grp][2 * k2 + 1]);
    if (!CARRY) {
      // inside the chunk: O[t] += sum_{s <= t} exp(cum_t - cum_s) (q_t . k_s) u_s
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
          if (k2 == 0 || tb >= 2)
            oacc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(gfr[frag_id(tb, k2)]), uop[0][k2], oacc[tb], 0, 0, 0);
    }
    // state at the chunk's end: S^T = gamma_64 S^T + sum_s (exp(cum_64 - cum_s) k_s) u_s^T
    {
      const float dec = fast_exp2(cum_last * kLog2e);
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb) {
#pragma unroll
        for (int grp = 0; grp < kG; ++grp)
#pragma unroll
          for (int r = 0; r < 4; ++r) sacc[grp][nb][r] *= dec;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
          // channel 16 nb + cq of steps 32 k2 + 4 gq .. +3 and 32 k2 + 16 + 4 gq .. +3
          const bf16_t *at = &sm.kw[32 * k2 + 4 * gq + (cq >> 2)][16 * nb + 4 * (cq & 3)];
          const u32x2_t lo = read_transposed(at), hi = read_transposed(at + 16 * (NS + 16));
          const bf16x8_t fw = frag_from_halves(lo, hi);
#pragma unroll
          for (int grp = 0; grp < kG; ++grp)
            sacc[grp][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw, uop[grp][k2], sacc[grp][nb], 0, 0, 0);
        }
      }
    }
    if (CARRY) continue;
    // ---- output rows: query norm and scale, RMS norm over the head's 64 channels, SiLU(z) gate
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      const f32x4_t rq = *reinterpret_cast<const f32x4_t *>(&sm.rq[16 * tb + 4 * gq]);
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.y[16 * tb + 4 * gq + r][16 * wave + cq] = oacc[tb][r] * rq[r];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = erq + 32 * i;
      const int64_t t = t0 + row;
      const f32x4_t y0 = *reinterpret_cast<const f32x4_t *>(&sm.y[row][8 * epq]);
      const f32x4_t y1 = *reinterpret_cast<const f32x4_t *>(&sm.y[row][8 * epq + 4]);
      float ss = 0.0f;
#pragma unroll
      for (int m = 0; m < 4; ++m) ss = fmaf(y0[m], y0[m], fmaf(y1[m], y1[m], ss));
      const float rstd = rsqrtf(group_sum<8>(ss) * (1.0f / kV) + eps);
      const u32x4_t zv = ez[i];
      const f32x4_t w0 = *reinterpret_cast<const f32x4_t *>(norm_w + 8 * epq);
      const f32x4_t w1 = *reinterpret_cast<const f32x4_t *>(norm_w + 8 * epq + 4);
      float o[8];
#pragma unroll
      for (int m = 0; m < 8; ++m)
        o[m] = (m < 4 ? y0[m & 3] * w0[m & 3] : y1[m & 3] * w1[m & 3]) * rstd * silu_f32(bf16_elem(zv, m));
      const u32x4_t ov = {pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7])};
      if (t < te) *reinterpret_cast<u32x4_t *>(y + (b * L + t) * ld_y + h * kV + 8 * epq) = ov;
    }
    fetch_out(t0 + kQ);
  }

  if (CARRY) {
    float *zp = carry_z + unit * s_stride + wave * 16 + c;
    float *mp = carry_m + unit * static_cast<int64_t>(NS) * NS + wave * 16 + c;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        zp[(16 * nb + 4 * g + r) * kV] = sacc[0][nb][r];
#pragma unroll
        for (int grp = 1; grp < kG; ++grp) mp[(16 * nb + 4 * g + r) * NS + 64 * (grp - 1)] = sacc[grp][nb][r];
      }
  } else if (s_out && seg == n_seg - 1) {
    float *sp = s_out + (b * n_heads + h) * s_stride + wave * 16 + c;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) sp[(16 * nb + 4 * g + r) * kV] = sacc[0][nb][r];
  }
}

// Workgroup barrier for data that travels through LDS only: __syncthreads() also waits for the wave's
// outstanding global accesses, a memory round trip behind every barrier
__device__ __forceinline__ void fold_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The state every segment starts from: start[0] = s_in (or 0), start[j + 1]^T = M_j start[j]^T + Z_j^T with the
// carry pass's arrays as stored (M_j[n][m] = Phi_j[m][n]).  The value channels are independent: grid
// (n_heads, B, 4), 16 of them per workgroup; a thread owns NS / 16 columns of one row and holds its row of M,
// requested a whole segment ahead.  The chain over the segments is latency: one workgroup per head that fetched M in
// batches took 7.5 us a segment.
template <int NS>
__global__ __launch_bounds__(256) void gdn_fold_kernel(const float *__restrict__ carry_z, const float *__restrict__ carry_m,
                                                       const float *__restrict__ s_in, float *__restrict__ s_start,
                                                       int n_seg) {
  constexpr int kCols = NS / 16, kPerRow = 16 / kCols;      // columns per thread, threads per row
  __shared__ float cur[2][NS][16];
  const int tid = threadIdx.x, n = tid / kPerRow, v0 = (tid % kPerRow) * kCols;
  const int h = blockIdx.x, n_heads = gridDim.x;
  const int64_t bh = static_cast<int64_t>(blockIdx.y) * n_heads + h;
  const int64_t s_stride = static_cast<int64_t>(NS) * kV;
  const int64_t at = n * kV + 16 * blockIdx.z + v0;         // this thread's columns within a state
  f32x4_t m_next[NS / 4], z_next[kCols / 4];
  auto fetch = [&](int j) {
    const int64_t unit = bh * n_seg + j;
    const float *mrow = carry_m + unit * static_cast<int64_t>(NS) * NS + static_cast<int64_t>(n) * NS;
#pragma unroll
    for (int q = 0; q < NS / 4; ++q) m_next[q] = *reinterpret_cast<const f32x4_t *>(mrow + 4 * q);
#pragma unroll
    for (int q = 0; q < kCols / 4; ++q) z_next[q] = *reinterpret_cast<const f32x4_t *>(carry_z + unit * s_stride + at + 4 * q);
  };
  f32x4_t acc[kCols / 4];
#pragma unroll
  for (int i = 0; i < kCols; ++i) acc[i / 4][i % 4] = s_in ? s_in[bh * s_stride + at + i] : 0.0f;
  fetch(0);                                                 // n_seg >= 2 here: segment 0 has a carry
  for (int j = 0; j < n_seg; ++j) {
#pragma unroll
    for (int q = 0; q < kCols / 4; ++q) {
      *reinterpret_cast<f32x4_t *>(s_start + (bh * n_seg + j) * s_stride + at + 4 * q) = acc[q];
      *reinterpret_cast<f32x4_t *>(&cur[j & 1][n][v0 + 4 * q]) = acc[q];
    }
    if (j == n_seg - 1) break;
    fold_barrier();                                         // two buffers: one barrier a segment
    f32x4_t m_cur[NS / 4];
#pragma unroll
    for (int q = 0; q < NS / 4; ++q) m_cur[q] = m_next[q];
#pragma unroll
    for (int q = 0; q < kCols / 4; ++q) acc[q] = z_next[q];
    if (j + 1 < n_seg - 1) fetch(j + 1);
#pragma unroll
    for (int m = 0; m < NS; ++m)
#pragma unroll
      for (int q = 0; q < kCols / 4; ++q) {
        const f32x4_t cv = *reinterpret_cast<const f32x4_t *>(&cur[j & 1][m][v0 + 4 * q]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[q][i] = fmaf(m_cur[m / 4][m % 4], cv[i], acc[q][i]);
      }
  }
}

// One step per sequence (L == 1): grid (n_heads, B); thread = (four value channels, every sixteenth key channel).  Bound by
// reading and writing the state once: a wavefront's instruction moves four whole rows of 64 value channels (1 KiB), and all of
// a thread's rows are asked for before the norms, sums and barriers that they wait for.  Step of 256 sequences, 12 heads of 128
// keys 98.6 -> 92.6 us, 32 heads 262 -> 258, of 64 keys 175 -> 171, one sequence 37.3 -> 34.9, against a lane a channel.
template <int NS>
__global__ __launch_bounds__(256) void gdn_step_kernel(const bf16_t *__restrict__ qkv, int64_t ld_qkv, int q_col, int k_col,
                                                       int v_col, const bf16_t *__restrict__ proj, int64_t ld_p, int b_col,
                                                       int a_col, const float *__restrict__ dt_bias,
                                                       const float *__restrict__ A_log, const float *__restrict__ norm_w,
                                                       float eps, const float *s_in, float *s_out, bf16_t *__restrict__ y,
                                                       int64_t ld_y) {
  constexpr int kPer = NS / 16;
  __shared__ float kq[2][NS];          // normalised key, normalised and scaled query
  __shared__ __attribute__((aligned(16))) float part[2][4][kV];
  __shared__ float red[2][4];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, v = (tid & 15) * 4, n0 = tid >> 4;
  const int h = blockIdx.x, n_heads = gridDim.x;
  const int64_t b = blockIdx.y;
  const bf16_t *row = qkv + b * ld_qkv;
  const bf16_t *prow = proj + b * ld_p;
  // this thread's state values: S^T[n][v .. v + 3]
  const int64_t base = (b * n_heads + h) * static_cast<int64_t>(NS) * kV + v;
  f32x4_t st[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    st[j] = s_in ? *reinterpret_cast<const f32x4_t *>(s_in + base + (n0 + 16 * j) * kV) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  // L2 norms of q and k: threads [0, NS) square a key element, threads [128, 128 + NS) a query element
  float kval = 0.0f, qval = 0.0f;
  if (tid < NS) kval = bf16_to_f32(row[k_col + h * NS + tid]);
  if (tid >= 128 && tid < 128 + NS) qval = bf16_to_f32(row[q_col + h * NS + tid - 128]);
  float sk = kval * kval, sq = qval * qval;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    sk += __shfl_xor(sk, off);
    sq += __shfl_xor(sq, off);
  }
  if (lane == 0) {
    red[0][wave] = sk;
    red[1][wave] = sq;
  }
  const float beta = fast_rcp(1.0f + __expf(-bf16_to_f32(prow[b_col + h])));
  const float alpha = __expf(-__expf(A_log[h]) * softplus_f32(bf16_to_f32(prow[a_col + h]) + dt_bias[h]));
  float val[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) val[i] = bf16_to_f32(row[v_col + h * kV + v + i]);
  __syncthreads();
  const float rk = rsqrtf(red[0][0] + red[0][1] + red[0][2] + red[0][3] + kL2Eps);
  const float rq = rsqrtf(red[1][0] + red[1][1] + red[1][2] + red[1][3] + kL2Eps) * rsqrtf(static_cast<float>(NS));
  if (tid < NS) kq[0][tid] = kval * rk;
  if (tid >= 128 && tid < 128 + NS) kq[1][tid - 128] = qval * rq;
  __syncthreads();
  // sums over the key channels: a wavefront's four rows of lanes, then the four wavefronts
  auto share = [&](float (&s)[4], float (&dst)[4][kV]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] += __shfl_xor(s[i], 16);
      s[i] += __shfl_xor(s[i], 32);
      if (lane < 16) dst[wave][v + i] = s[i];
    }
    __syncthreads();
  };
  float pred[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const float kn = kq[0][n0 + 16 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[j][i] = alpha * st[j][i];
      pred[i] = fmaf(st[j][i], kn, pred[i]);
    }
  }
  share(pred, part[0]);
  float u[4], o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = beta * (val[i] - (part[0][0][v + i] + part[0][1][v + i] + part[0][2][v + i] + part[0][3][v + i]));
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const float kn = kq[0][n0 + 16 * j], qn = kq[1][n0 + 16 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[j][i] = fmaf(u[i], kn, st[j][i]);
      o[i] = fmaf(st[j][i], qn, o[i]);
    }
    if (s_out) *reinterpret_cast<f32x4_t *>(s_out + base + (n0 + 16 * j) * kV) = st[j];
  }
  share(o, part[1]);
  if (wave == 0) {
    const float ov = part[1][0][lane] + part[1][1][lane] + part[1][2][lane] + part[1][3][lane];
    float ss = ov * ov;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    const float rstd = rsqrtf(ss * (1.0f / kV) + eps);
    y[b * ld_y + h * kV + lane] = f32_to_bf16(ov * rstd * norm_w[lane] * silu_f32(bf16_to_f32(prow[h * kV + lane])));
  }
}

constexpr int kGdnOneWgs = 256;
struct GdnPlanSeg {
  int n_seg;
  int64_t seg_len;
};
GdnPlanSeg gdn_plan(int64_t B, int64_t L, int n_heads) {
  // One workgroup for each of the 256 CUs; a segment is whole chunks and at least four of them.  The recurrence fits two
  // to a CU and twice the segments take less time (1 x 16384, 32 heads of 64: 308 against 408 us), but every segment's
  // start state is a product with the carry pass's bf16 operands, so their number shows in the outputs (2e-3, at an
  // unchanged error against 64 bits of 3.7e-3): it stays.
  const int64_t chunks = ceil_div(L, kQ);
  int64_t n_seg = ceil_div(256, B * n_heads);
  const int64_t max_seg = chunks / 4 > 0 ? chunks / 4 : 1;
  n_seg = n_seg < 1 ? 1 : (n_seg > max_seg ? max_seg : n_seg);
  GdnPlanSeg p;
  p.seg_len = ceil_div(chunks, n_seg) * kQ;
  p.n_seg = static_cast<int>(ceil_div(L, p.seg_len));
  return p;
}

template <int NS, bool CARRY, bool ONE = false>
hipError_t gdn_allow_lds() {
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
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gdn_kernel<NS, CARRY, ONE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(ONE ? sizeof(GdnOneSmem<NS>) : sizeof(GdnSmem<NS, CARRY>)));
      if (e != hipSuccess) return e;
      done[dev].store(true, std::memory_order_release);
    }
  }
  return hipSuccess;
}

template <int NS>
hipError_t gdn_dispatch(const bf16_t *qkv, int64_t ld_qkv, int q_col, int k_col, int v_col, const bf16_t *proj, int64_t ld_p,
                        int b_col, int a_col, const float *dt_bias, const float *A_log, const float *norm_w, float eps,
                        int64_t B, int64_t L, int n_heads, const float *s_in, float *s_out, float *carry, bf16_t *y,
                        int64_t ld_y, hipStream_t s) {
  if (L == 1) {
    hipLaunchKernelGGL((gdn_step_kernel<NS>), dim3(static_cast<unsigned>(n_heads), static_cast<unsigned>(B)), dim3(256), 0,
                       s, qkv, ld_qkv, q_col, k_col, v_col, proj, ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, s_in, s_out,
                       y, ld_y);
    return hipGetLastError();
  }
  const GdnPlanSeg p = gdn_plan(B, L, n_heads);
  const int64_t n_chunks = ceil_div(L, kQ);
  const size_t units = static_cast<size_t>(B) * n_heads * p.n_seg;
  u32x4_t *frags = reinterpret_cast<u32x4_t *>(carry);
  carry += static_cast<size_t>(B) * n_heads * n_chunks * kFragFloats;
  float *carry_z = carry, *carry_m = carry + units * NS * kV, *s_start = carry_m + units * NS * NS;
  const dim3 grid(static_cast<unsigned>(n_heads), static_cast<unsigned>(B * p.n_seg));
  hipError_t e;
  // One chunk and no more workgroups than CUs: the preparation has nothing to share a CU with, and the launch costs 2 us
  // (four sequences of 64 steps, 32 heads of 64: 14.1 us in two launches, 11.2 in one; 12 sequences 18.0 / 22.2).
  if (n_chunks == 1 && B * n_heads <= kGdnOneWgs) {
    if ((e = gdn_allow_lds<NS, false, true>()) != hipSuccess) return e;
    hipLaunchKernelGGL((gdn_kernel<NS, false, true>), grid, dim3(256), sizeof(GdnOneSmem<NS>), s, qkv, ld_qkv, q_col, k_col, v_col, proj,
                       ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, L, p.n_seg, p.seg_len, 1, static_cast<const u32x4_t *>(nullptr),
                       carry_z, carry_m, s_start, s_in, s_out, y, ld_y);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((gdn_prep_kernel<NS>), dim3(static_cast<unsigned>(B * n_chunks * n_heads)), dim3(256), 0, s, qkv, ld_qkv,
                     q_col, k_col, proj, ld_p, b_col, a_col, dt_bias, A_log, L, static_cast<int>(n_chunks), n_heads, frags);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (p.n_seg > 1) {
    if ((e = gdn_allow_lds<NS, true>()) != hipSuccess) return e;
    hipLaunchKernelGGL((gdn_kernel<NS, true>), grid, dim3(256), sizeof(GdnSmem<NS, true>), s, qkv, ld_qkv, q_col, k_col, v_col, proj,
                       ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, L, p.n_seg, p.seg_len, static_cast<int>(n_chunks),
                       frags, carry_z, carry_m, s_start, s_in,
                       s_out, y, ld_y);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((gdn_fold_kernel<NS>), dim3(static_cast<unsigned>(n_heads), static_cast<unsigned>(B), 4), dim3(256), 0, s,
                       carry_z, carry_m, s_in, s_start, p.n_seg);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = gdn_allow_lds<NS, false>()) != hipSuccess) return e;
  hipLaunchKernelGGL((gdn_kernel<NS, false>), grid, dim3(256), sizeof(GdnSmem<NS, false>), s, qkv, ld_qkv, q_col, k_col, v_col, proj,
                     ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, L, p.n_seg, p.seg_len, static_cast<int>(n_chunks),
                       frags, carry_z, carry_m, s_start, s_in,
                     s_out, y, ld_y);
  return hipGetLastError();
}

}  // namespace

bool gdn_supported(int d_k, int d_v) { return d_v == kV && (d_k == 64 || d_k == 128); }

size_t gdn_carry_bytes(int64_t B, int64_t L, int n_heads, int d_k) {
  const GdnPlanSeg p = gdn_plan(B, L, n_heads);
  if (L <= 1) return 0;
  const size_t frag_bytes = static_cast<size_t>(B) * n_heads * ceil_div(L, kQ) * kFragFloats * sizeof(float);
  if (p.n_seg <= 1) return frag_bytes;
  return frag_bytes + static_cast<size_t>(B) * n_heads * p.n_seg * (2 * static_cast<size_t>(d_k) * kV + static_cast<size_t>(d_k) * d_k) *
         sizeof(float);
}

hipError_t launch_gdn_scan(const void *qkv, int64_t ld_qkv, int q_col, int k_col, int v_col, const void *proj, int64_t ld_p,
                           int b_col, int a_col, const float *dt_bias, const float *A_log, const float *norm_w, float eps,
                           int64_t B, int64_t L, int n_heads, int d_k, const float *s_in, float *s_out, float *carry,
                           void *y, int64_t ld_y, hipStream_t s) {
  if (B * L <= 0) return hipSuccess;
  if (B * gdn_plan(B, L, n_heads).n_seg > 65535) return hipErrorInvalidValue;
  const bf16_t *qp = static_cast<const bf16_t *>(qkv), *pp = static_cast<const bf16_t *>(proj);
  if (d_k == 128)
    return gdn_dispatch<128>(qp, ld_qkv, q_col, k_col, v_col, pp, ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, B, L,
                             n_heads, s_in, s_out, carry, static_cast<bf16_t *>(y), ld_y, s);
  if (d_k == 64)
    return gdn_dispatch<64>(qp, ld_qkv, q_col, k_col, v_col, pp, ld_p, b_col, a_col, dt_bias, A_log, norm_w, eps, B, L, n_heads,
                            s_in, s_out, carry, static_cast<bf16_t *>(y), ld_y, s);
  return hipErrorInvalidValue;
}

}  // namespace rom
