// Backward pass of the RoM layer's sequence part and the small gradient kernels around the
// grouped GEMMs (training, Sec. 5.1): adjoint of the selective scan of Eq. (5) with the gate of
// Eq. (6)/(13) and the softplus of the time step folded in, adjoint of the causal conv + SiLU of
// Eq. (2), gradient of the gate weights of Eq. (9)/(12), and the gather / transpose kernels that
// bring activations into the layout the weight-gradient GEMMs contract over.
// Correct-first: plain ALU kernels, deterministic (fixed summation orders, no atomics).
#include <atomic>
#include <mutex>
#include <type_traits>
#include "rom_dpp.h"
#include "rom_internal.h"
#include "rom_scan_rule.h"

namespace rom {

namespace {

__device__ __forceinline__ float sigmoid_f32(float v) { return fast_rcp(1.0f + fast_exp2(-1.44269504088896341f * v)); }

inline dim3 grid1d(int64_t work, int block) { return dim3(static_cast<unsigned>(ceil_div(work, block))); }

// Workgroup barrier for data that travels through LDS only.  __syncthreads() also waits for the
// wavefront's outstanding global stores (its fence covers global memory), which puts a memory round
// trip behind every barrier that follows a store; threads of these kernels never read what another
// thread wrote to global memory, so waiting for the LDS counter is enough.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ------------------------------------------------------------------ adjoint of the selective scan
// Sequences are cut into chunks (of 128 steps where there are enough, see scan_bwd_chunk), so that the chip is full whatever
// the batch.  Three kernels:
//   scan_bwd_carry_kernel: a lane owns a channel with its 16 states (B and C through the scalar cache, as in the
//           forward's lane = channel scan) and walks one chunk forwards once, leaving its end state Q from a zero start,
//           the adjoint state R that leaves its start from a zero adjoint at its end (sum over t of the decay from the
//           start to t times C_t d y_t), and its sum of dt;
//   scan_bwd_fold_kernel: every chunk's start state and incoming adjoint state from those, in chunk order;
//   scan_bwd_kernel: the chunk itself.  A wavefront owns 16 channels; lane (q, c) = (lane / 16, lane % 16) holds states
//           4 q .. 4 q + 3 of channel c.  Pass 1 (forward in time) leaves the state at the start of every group of 16
//           steps in LDS; pass 2 (backward, group by group) recomputes the group's states into registers and walks the
//           adjoint recurrence d_h[t-1] = exp(dt_t a) d_h[t] back over it.
// With four states a lane, three quarters of the sums over a channel's states need no other lane; the rest (y, the
// input term, d dt: four rows of lanes) are three swap-and-add per four steps that leave step 4 i + q with row q, whose
// lanes own that step's loads, activation derivatives and stores.  The sums over channels (d B, d C) go over the 16
// lanes of a row by a transposing butterfly, over the block's four wavefronts through LDS (the only barrier, one per
// group), over the channel blocks in bwd_reduce_bc_kernel; parameter gradients go to per-unit partials that
// scan_bwd_finish_kernel sums in unit order.  All sums in fixed order, no atomics.
// Bound by ALU issue: 115 vector instructions, 10 of them transcendental, per step of 256 (channel, state) pairs, issue busy for
// 98 % of the cycles.  16384 x 4096, launches alone: 1.27 ms (a lane per (channel, state) pair with row sums over the states
// and channel sums through LDS: 2.27); within a training step carries 0.29, fold 0.04, main 1.02, sums 0.04 ms.
constexpr int kBwdMaxChunk = 128, kBwdGroup = 16, kBwdCh = 64, kBwdHalf = 8, kBwdGroups = kBwdMaxChunk / kBwdGroup;
constexpr int kBwdStPitch = kBwdGroup + 4;   // floats per channel row: 16 rows of four-step reads or writes cover the banks

// Scratch of the adjoint scan, all f32.  Units are numbered (sequence * n_chunks + chunk) * n_cb + channel block.
struct ScanBwdLayout {
  int n_cb, n_chunks, chunk;   // channel blocks; chunks per sequence; steps per chunk (whole groups)
  int64_t n_units;
  size_t carry_q, carry_r, carry_s, part_a, part_d, part_bias, total;   // offsets in floats
};
inline ScanBwdLayout scan_bwd_layout(int64_t B, int64_t L, int d_inner) {
  ScanBwdLayout l;
  l.n_cb = static_cast<int>(ceil_div(d_inner, kBwdCh));
  l.chunk = scan_bwd_chunk(B, L, d_inner);
  l.n_chunks = static_cast<int>(ceil_div(L, l.chunk));
  l.n_units = B * l.n_chunks * l.n_cb;
  size_t off = 0;
  auto take = [&](size_t n) { size_t o = off; off += (n + 63) / 64 * 64; return o; };
  const size_t carries = l.n_chunks > 1 ? static_cast<size_t>(B) * l.n_chunks * d_inner : 0;
  l.carry_q = take(carries * 16);
  l.carry_r = take(carries * 16);
  l.carry_s = take(carries);
  l.part_a = take(static_cast<size_t>(l.n_units) * kBwdCh * 16);
  l.part_d = take(static_cast<size_t>(l.n_units) * kBwdCh);
  l.part_bias = take(static_cast<size_t>(l.n_units) * kBwdCh);
  l.total = off;
  return l;
}

typedef unsigned int bwd_u32x2 __attribute__((ext_vector_type(2)));
typedef float bwd_f32x4 __attribute__((ext_vector_type(4)));
typedef float bwd_f32x16 __attribute__((ext_vector_type(16)));
// four consecutive elements as floats, one 8-byte (bf16) or 16-byte (f32) load
__device__ __forceinline__ void bwd_load4(const bf16_t *p, float *f) {
  const bwd_u32x2 w = *reinterpret_cast<const bwd_u32x2 *>(p);
  f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xFFFF0000u);
  f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xFFFF0000u);
}
__device__ __forceinline__ void bwd_load4(const float *p, float *f) {
  const bwd_f32x4 w = *reinterpret_cast<const bwd_f32x4 *>(p);
  f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w;
}

__device__ __forceinline__ void bwd_store4(bf16_t *p, const float *f) {
  bwd_u32x2 w;
  w.x = pack_bf16x2(f[0], f[1]);
  w.y = pack_bf16x2(f[2], f[3]);
  *reinterpret_cast<bwd_u32x2 *>(p) = w;
}
__device__ __forceinline__ void bwd_store4(float *p, const float *f) {
  bwd_f32x4 w;
  w.x = f[0]; w.y = f[1]; w.z = f[2]; w.w = f[3];
  *reinterpret_cast<bwd_f32x4 *>(p) = w;
}

// grid.x: (sequence * n_chunks + chunk) * gx + block of 256 channels.  carry_q, carry_r: f32 [B][n_chunks][16][d_inner],
// carry_s [B][n_chunks][d_inner]
template <typename T>
__global__ __launch_bounds__(256) void scan_bwd_carry_kernel(
    const T *__restrict__ u, const T *__restrict__ dt, const float *__restrict__ bc, const T *__restrict__ z,
    int64_t ld_z, const T *__restrict__ dg, const float *__restrict__ gate, const float *__restrict__ A_log, int64_t L,
    int d_inner, int gx, int n_chunks, int chunk, float *__restrict__ carry_q, float *__restrict__ carry_r,
    float *__restrict__ carry_s) {
  typedef const __attribute__((address_space(4))) bwd_f32x16 const_f32x16_t;
  typedef const __attribute__((address_space(4))) float const_f32_t;
  typedef __attribute__((address_space(1))) char global_char_t;
  typedef __attribute__((address_space(1))) T global_t;
  const int lane = threadIdx.x & 63;
  const int64_t bk = blockIdx.x / gx;                          // sequence * n_chunks + chunk
  const int ch0 = (blockIdx.x % gx * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 64;
  if (ch0 >= d_inner) return;
  const int cl = ch0 + lane < d_inner ? lane : d_inner - 1 - ch0;      // idle lanes repeat the last channel, stores included
  const int ch = ch0 + cl;
  const int64_t b = bk / n_chunks, ts = bk % n_chunks * chunk, row0 = b * L + ts;
  const int len = static_cast<int>(L - ts < chunk ? L - ts : chunk);

  float a2[16], h[16], e[16], r[16], sum = 0.0f;
#pragma unroll
  for (int n = 0; n < 16; n += 4) bwd_load4(A_log + static_cast<int64_t>(ch) * 16 + n, a2 + n);
#pragma unroll
  for (int n = 0; n < 16; ++n) {
    a2[n] = -__expf(a2[n]) * 1.44269504088896341f;
    h[n] = r[n] = 0.0f;
    e[n] = 1.0f;
  }
  // uniform row address plus one 32-bit lane offset (see scan_lane_kernel for the empty asm)
  const uintptr_t u_p = reinterpret_cast<uintptr_t>(u + row0 * d_inner + ch0), dt_p = reinterpret_cast<uintptr_t>(dt + row0 * d_inner + ch0);
  const uintptr_t dg_p = reinterpret_cast<uintptr_t>(dg + row0 * d_inner + ch0), z_p = reinterpret_cast<uintptr_t>(z + row0 * ld_z + ch0);
  const uintptr_t bc_p = reinterpret_cast<uintptr_t>(bc + row0 * 32), gate_p = gate ? reinterpret_cast<uintptr_t>(gate + row0) : bc_p;
  const uint32_t pitch = static_cast<uint32_t>(d_inner * sizeof(T)), pitch_z = static_cast<uint32_t>(ld_z * sizeof(T));
  auto at = [](uintptr_t base, uint32_t off, uint32_t lo) __attribute__((always_inline)) {
    uintptr_t p = base + off;
    asm("" : "+s"(p));
    return *reinterpret_cast<global_t *>(reinterpret_cast<global_char_t *>(p) + lo);
  };
  // ring of the next kRun rows: a slot is requested anew as soon as its step has taken the values out
  constexpr int kRun = 4;
  T rdt[kRun], ru[kRun], rz[kRun], rg[kRun];
  auto fetch = [&](int t, int j, uint32_t lo) __attribute__((always_inline)) {
    const uint32_t rr = static_cast<uint32_t>(t < len ? t : len - 1);    // past the chunk's end: its last row again
    rdt[j] = at(dt_p, rr * pitch, lo);
    ru[j] = at(u_p, rr * pitch, lo);
    rz[j] = at(z_p, rr * pitch_z, lo);
    rg[j] = at(dg_p, rr * pitch, lo);
  };
  const uint32_t loff = static_cast<uint32_t>(cl) * sizeof(T);
#pragma unroll
  for (int j = 0; j < kRun; ++j) fetch(j, j, loff);
  // B and the gate weight of Eq. (12) one step ahead, C within the step
  bwd_f32x16 bv = *reinterpret_cast<const_f32x16_t *>(bc_p);
  // (no gate: any readable word, replaced by 1 - a branch here would part the step's loads from its arithmetic)
  const uint32_t gate_step = gate ? 4 : 0;
  float gw = *reinterpret_cast<const_f32_t *>(gate_p);
  auto step = [&](int t, int j) __attribute__((always_inline)) {
    const int tn = t + 1 < len ? t + 1 : t;
    const float d = to_f32(rdt[j]), du = d * to_f32(ru[j]), dy = to_f32(rg[j]) * (gate ? gw : 1.0f) * silu_f32(to_f32(rz[j]));
    const bwd_f32x16 cv = *reinterpret_cast<const_f32x16_t *>(bc_p + t * 128 + 64);
    const bwd_f32x16 bn = *reinterpret_cast<const_f32x16_t *>(bc_p + tn * 128);
    gw = *reinterpret_cast<const_f32_t *>(gate_p + static_cast<uint32_t>(tn) * gate_step);
    uint32_t lo = loff;
    asm volatile("" : "+v"(lo));
    fetch(t + kRun, j, lo);
    sum += d;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      const float da = fast_exp2(d * a2[n]);
      h[n] = fmaf(da, h[n], du * bv[n]);
      e[n] *= da;
    }
#pragma unroll
    for (int n = 0; n < 16; ++n) r[n] = fmaf(e[n] * dy, cv[n], r[n]);
    bv = bn;
    __builtin_amdgcn_sched_barrier(0);
  };
  int t = 0;
  const int p2 = len / 2, p1 = p2 + len / 4, p0 = p1 + len / 8;          // (priorities: see scan_lane_kernel)
  __builtin_amdgcn_s_setprio(3);
  for (; t + kRun <= len; t += kRun) {
    if (t >= p0) __builtin_amdgcn_s_setprio(0);
    else if (t >= p1) __builtin_amdgcn_s_setprio(1);
    else if (t >= p2) __builtin_amdgcn_s_setprio(2);
    // brings the B / C rows of the run after the next into L2, ahead of the scalar loads
    const int wr = t + 2 * kRun + (lane >> 4) < len ? t + 2 * kRun + (lane >> 4) : len - 1;
    const bwd_u32x2 warm = *reinterpret_cast<const bwd_u32x2 *>(bc + (row0 + wr) * 32 + (lane & 15) * 2);
#pragma unroll
    for (int j = 0; j < kRun; ++j) step(t + j, j);
    asm volatile("" ::"v"(warm));
  }
#pragma unroll
  for (int j = 0; j < kRun - 1; ++j)
    if (t + j < len) step(t + j, j);
  float *q_out = carry_q + bk * 16 * d_inner + ch, *r_out = carry_r + bk * 16 * d_inner + ch;
#pragma unroll
  for (int n = 0; n < 16; ++n) {
    q_out[static_cast<int64_t>(n) * d_inner] = h[n];
    r_out[static_cast<int64_t>(n) * d_inner] = r[n];
  }
  carry_s[bk * d_inner + ch] = sum;
}

// thread = (sequence, state, channel); blockIdx.y 0: q_k <- state at the start of chunk k (zero before the first),
// 1: r_k <- adjoint state flowing into the end of chunk k (zero behind the last)
__global__ __launch_bounds__(256) void scan_bwd_fold_kernel(const float *__restrict__ A_log, int64_t n_seq, int d_inner,
                                                            int n_chunks, float *__restrict__ carry_q,
                                                            float *__restrict__ carry_r, const float *__restrict__ carry_s) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t per_seq = static_cast<int64_t>(d_inner) * 16;
  if (idx >= n_seq * per_seq) return;
  const int64_t b = idx / per_seq;
  const int w = static_cast<int>(idx % per_seq), n = w / d_inner, ch = w % d_inner;
  const float a2 = -__expf(A_log[static_cast<int64_t>(ch) * 16 + n]) * 1.44269504088896341f;
  const bool rev = blockIdx.y == 1;
  float *x = (rev ? carry_r : carry_q) + b * n_chunks * per_seq + w;
  const float *s = carry_s + b * n_chunks * d_inner + ch;
  float v = 0.0f;
  constexpr int kAhead = 16;
  float xv[kAhead], sv[kAhead];
  for (int k0 = 0; k0 < n_chunks; k0 += kAhead) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      int k = k0 + j < n_chunks ? k0 + j : n_chunks - 1;
      if (rev) k = n_chunks - 1 - k;
      xv[j] = x[k * per_seq];
      sv[j] = s[static_cast<int64_t>(k) * d_inner];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      if (k0 + j < n_chunks) {
        const int k = rev ? n_chunks - 1 - k0 - j : k0 + j;
        x[k * per_seq] = v;
        v = fmaf(fast_exp2(a2 * sv[j]), v, xv[j]);
      }
    }
  }
}

// v_s (s = 0 .. 3): partial sums of four steps, one part per row of 16 lanes; row q receives the total of step q
__device__ __forceinline__ float sum_rows4(const float (&v)[4]) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[2]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[1]), __float_as_uint(v[3]), false, false);
  const float s02 = __uint_as_float(a[0]) + __uint_as_float(a[1]), s13 = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(s02), __float_as_uint(s13), false, false);
  return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

struct BwdSmem {
  float ck[4][kBwdGroups][256];                        // [wave][group][lane * 4 + j]: state at the group's start
  float dt[4][16 * kBwdStPitch], dtu[4][16 * kBwdStPitch], dy[4][16 * kBwdStPitch];     // [wave][channel][step of the group]
  float bc[4][kBwdGroup * 32];                         // [wave][step][B_0..15, C_0..15]
  float o_bc[2][4][kBwdGroup * 32];                    // each wavefront's share of d_B, d_C of a group, two groups in turn
};

// grid.x: units.  start_h / start_dh: f32 [B][n_chunks][16][d_inner] or NULL (one chunk: zeros).  d_bc_part: f32
// [n_cb][N][32].  Outputs d_pre (w.r.t. the softplus argument), d_u, d_z have type T.
template <typename T>
__global__ __launch_bounds__(256, 2) void scan_bwd_kernel(
    const T *__restrict__ u, const T *__restrict__ dt, const float *__restrict__ bc, const T *__restrict__ z,
    int64_t ld_z, const T *__restrict__ dg, const float *__restrict__ gate, const float *__restrict__ A_log,
    const float *__restrict__ D, int64_t n_tok, int64_t L, int d_inner, int n_cb, int n_chunks, int chunk,
    const float *__restrict__ start_h, const float *__restrict__ start_dh, T *__restrict__ d_pre, T *__restrict__ d_u,
    T *__restrict__ d_z, int64_t ld_dz, float *__restrict__ d_bc_part, float *__restrict__ part_a,
    float *__restrict__ part_d, float *__restrict__ part_bias) {
  extern __shared__ __attribute__((aligned(16))) unsigned char bwd_smem[];
  BwdSmem &sm = *reinterpret_cast<BwdSmem *>(bwd_smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4;
  const int64_t unit = blockIdx.x;
  const int cb = static_cast<int>(unit % n_cb);
  const int64_t bk = unit / n_cb, b = bk / n_chunks, ts = bk % n_chunks * chunk, row0 = b * L + ts;
  const int len = static_cast<int>(L - ts < chunk ? L - ts : chunk);
  const int n_grp = (len + kBwdGroup - 1) / kBwdGroup;
  const int c0 = cb * kBwdCh + wave * 16;
  const bool active = c0 < d_inner;                     // (d_inner is a multiple of 16)
  const int ch = active ? c0 + c : c;
  float a_nat[4], a2[4], h[4] = {0.f, 0.f, 0.f, 0.f}, dh[4] = {0.f, 0.f, 0.f, 0.f};
  bwd_load4(A_log + static_cast<int64_t>(ch) * 16 + q * 4, a_nat);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a_nat[j] = -__expf(a_nat[j]);                       // A = -exp(A_log)
    a2[j] = a_nat[j] * 1.44269504088896341f;
    if (start_h) {
      const int64_t at = (bk * 16 + q * 4 + j) * d_inner + ch;
      h[j] = start_h[at];
      dh[j] = start_dh[at];
    }
  }
  const float d_skip = D[ch];
  float acc_a[4] = {0.f, 0.f, 0.f, 0.f}, acc_d = 0.0f, acc_bias = 0.0f;

  // what lane (q, c) brings of a group: steps 4 i + q of channel c, and 2 x 16 bytes of the B / C rows.  Addresses are a
  // uniform base and a 32-bit byte offset (the launcher keeps a chunk's rows within 2 GiB).
  struct Raw {
    T dt[4], u[4], z[4], dg[4];
    float gate[4];
    bwd_f32x4 bc0, bc1;
  } raw;
  // (rows are whole 32-byte pieces: a 24-bit product and a shift that goes with the addition)
  const unsigned pitch = static_cast<unsigned>(d_inner * sizeof(T) / 32), pitch_z = static_cast<unsigned>(ld_z * sizeof(T) / 32);
  const unsigned pitch_dz = static_cast<unsigned>(ld_dz * sizeof(T) / 32), ch_off = static_cast<unsigned>(ch * sizeof(T));
  auto row_at = [&](unsigned t, unsigned p) __attribute__((always_inline)) { return (__umul24(t, p) << 5) + ch_off; };
  const char *const dt_p = reinterpret_cast<const char *>(dt + row0 * d_inner), *const u_p = reinterpret_cast<const char *>(u + row0 * d_inner);
  const char *const dg_p = reinterpret_cast<const char *>(dg + row0 * d_inner), *const z_p = reinterpret_cast<const char *>(z + row0 * ld_z);
  const char *const bc_p = reinterpret_cast<const char *>(bc + row0 * 32);
  auto fetch = [&](int g, bool full) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tt = g * kBwdGroup + 4 * i + q;
      const unsigned t = static_cast<unsigned>(tt < len ? tt : len - 1), at = row_at(t, pitch);
      raw.dt[i] = *reinterpret_cast<const T *>(dt_p + at);
      raw.u[i] = *reinterpret_cast<const T *>(u_p + at);
      if (full) {
        raw.z[i] = *reinterpret_cast<const T *>(z_p + row_at(t, pitch_z));
        raw.dg[i] = *reinterpret_cast<const T *>(dg_p + at);
        raw.gate[i] = gate ? *reinterpret_cast<const float *>(reinterpret_cast<const char *>(gate + row0) + t * 4u) : 1.0f;
      }
    }
    const int r0 = g * kBwdGroup + (lane >> 3), r1 = r0 + 8;
    const unsigned o0 = static_cast<unsigned>(r0 < len ? r0 : len - 1) * 128u, o1 = static_cast<unsigned>(r1 < len ? r1 : len - 1) * 128u;
    raw.bc0 = *reinterpret_cast<const bwd_f32x4 *>(bc_p + (o0 + (lane & 7) * 16u));
    raw.bc1 = *reinterpret_cast<const bwd_f32x4 *>(bc_p + (o1 + (lane & 7) * 16u));
  };
  // steps past the end (and wavefronts past the last channel): dt = dt u = d y = 0, which leaves states and sums alone
  float dt_o[4], u_o[4], dy_o[4], dzf_o[4];
  auto park = [&](int g, bool full) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool ok = active && g * kBwdGroup + 4 * i + q < len;
      const float dv = ok ? to_f32(raw.dt[i]) : 0.0f, uv = ok ? to_f32(raw.u[i]) : 0.0f;
      sm.dt[wave][c * kBwdStPitch + 4 * i + q] = dv;
      sm.dtu[wave][c * kBwdStPitch + 4 * i + q] = dv * uv;
      if (full) {
        const float zs = to_f32(raw.z[i]), dgs = ok ? to_f32(raw.dg[i]) * raw.gate[i] : 0.0f;
        const float sig = sigmoid_f32(zs);
        dt_o[i] = dv;
        u_o[i] = uv;
        dy_o[i] = dgs * zs * sig;                       // g = y * SiLU(z)
        dzf_o[i] = dgs * sig * (1.0f + zs * (1.0f - sig));
        sm.dy[wave][c * kBwdStPitch + 4 * i + q] = dy_o[i];
      }
    }
    const int r0 = g * kBwdGroup + (lane >> 3);
    const bwd_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<bwd_f32x4 *>(&sm.bc[wave][lane * 4]) = r0 < len ? raw.bc0 : zero;
    *reinterpret_cast<bwd_f32x4 *>(&sm.bc[wave][256 + lane * 4]) = r0 + 8 < len ? raw.bc1 : zero;
    // (a wavefront's own LDS accesses are served in program order: its lanes may read what the others wrote)
    asm volatile("" ::: "memory");
  };
  auto ld4 = [](const float *p) __attribute__((always_inline)) { return *reinterpret_cast<const bwd_f32x4 *>(p); };

  // the states of steps 4 i .. 4 i + 3 of the parked group
  auto walk = [&](int i, float(&x)[4]) __attribute__((always_inline)) {
    const bwd_f32x4 d4 = ld4(&sm.dt[wave][c * kBwdStPitch + 4 * i]), x4 = ld4(&sm.dtu[wave][c * kBwdStPitch + 4 * i]);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bwd_f32x4 b4 = ld4(&sm.bc[wave][(4 * i + s) * 32 + q * 4]);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = fmaf(fast_exp2(d4[s] * a2[j]), x[j], x4[s] * b4[j]);
    }
  };

  // ---- pass 1: the state at the start of every group
  fetch(0, n_grp == 1);
  for (int g = 0; g < n_grp; ++g) {
    *reinterpret_cast<bwd_f32x4 *>(&sm.ck[wave][g][lane * 4]) = bwd_f32x4{h[0], h[1], h[2], h[3]};
    if (g + 1 == n_grp) break;
    park(g, false);
    fetch(g + 1, g + 2 == n_grp);                       // pass 2 starts with the last group
#pragma unroll
    for (int i = 0; i < 4; ++i) walk(i, h);
    asm volatile("" ::: "memory");
  }

  // ---- pass 2: groups in reverse
  char *const dpre_p = reinterpret_cast<char *>(d_pre + row0 * d_inner), *const du_p = reinterpret_cast<char *>(d_u + row0 * d_inner);
  char *const dz_p = reinterpret_cast<char *>(d_z + row0 * ld_dz);
  // (all: every step of the group and every channel of the wavefront exists - no branch around the stores, which would
  // cut the group into pieces too short to schedule)
  auto group = [&](int g, auto all) __attribute__((always_inline)) {
    // the group in two halves of eight steps, the later one first, so that its states and decays (68 registers) fit with two
    // wavefronts per SIMD (253 registers; the 71 KiB of LDS allow no third workgroup either); the state between the
    // halves is walked to once more
    float mid[4];
    {
      const bwd_f32x4 k4 = ld4(&sm.ck[wave][g][lane * 4]);
#pragma unroll
      for (int j = 0; j < 4; ++j) mid[j] = k4[j];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) walk(i, mid);
    float *o_bc = sm.o_bc[g & 1][wave];
#pragma unroll
    for (int half = 1; half >= 0; --half) {
      __builtin_amdgcn_sched_barrier(0);
      float hs[kBwdHalf + 1][4], da[kBwdHalf][4];
      if (half == 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) hs[0][j] = mid[j];
      } else {
        const bwd_f32x4 k4 = ld4(&sm.ck[wave][g][lane * 4]);
#pragma unroll
        for (int j = 0; j < 4; ++j) hs[0][j] = k4[j];
      }
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2) {
        const int i = 2 * half + i2;
        const bwd_f32x4 d4 = ld4(&sm.dt[wave][c * kBwdStPitch + 4 * i]), x4 = ld4(&sm.dtu[wave][c * kBwdStPitch + 4 * i]);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int t = 4 * i2 + s;
          const bwd_f32x4 b4 = ld4(&sm.bc[wave][(4 * i + s) * 32 + q * 4]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            da[t][j] = fast_exp2(d4[s] * a2[j]);
            hs[t + 1][j] = fmaf(da[t][j], hs[t][j], x4[s] * b4[j]);
          }
        }
      }
#pragma unroll
      for (int i2 = 1; i2 >= 0; --i2) {
        const int i = 2 * half + i2;
        const bwd_f32x4 d4 = ld4(&sm.dt[wave][c * kBwdStPitch + 4 * i]), x4 = ld4(&sm.dtu[wave][c * kBwdStPitch + 4 * i]);
        const bwd_f32x4 y4 = ld4(&sm.dy[wave][c * kBwdStPitch + 4 * i]);
        float v_y[4], v_in[4], v_dt[4];                 // this lane's part of C.h, of the input term and of d (dt A) A
#pragma unroll
        for (int pair = 1; pair >= 0; --pair) {
          float p16[16];                                // [step of the pair][d_B of four states, d_C]
#pragma unroll
          for (int s1 = 1; s1 >= 0; --s1) {
            const int s = 2 * pair + s1, t = 4 * i2 + s;
            const bwd_f32x4 b4 = ld4(&sm.bc[wave][(4 * i + s) * 32 + q * 4]), c4 = ld4(&sm.bc[wave][(4 * i + s) * 32 + 16 + q * 4]);
            float y = 0.0f, in = 0.0f, ddt = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              dh[j] = fmaf(c4[j], y4[s], dh[j]);        // y_t = C_t . h_t
              y = j == 0 ? c4[j] * hs[t + 1][j] : fmaf(c4[j], hs[t + 1][j], y);
              in = j == 0 ? dh[j] * b4[j] : fmaf(dh[j], b4[j], in);           // input term dt * B * u
              p16[8 * s1 + j] = dh[j] * x4[s];
              p16[8 * s1 + 4 + j] = y4[s] * hs[t + 1][j];
              dh[j] *= da[t][j];
              const float darg = dh[j] * hs[t][j];      // d / d (dt_t * A)
              ddt = j == 0 ? darg * a_nat[j] : fmaf(darg, a_nat[j], ddt);
              acc_a[j] = fmaf(darg, d4[s], acc_a[j]);
            }
            v_y[s] = y;
            v_in[s] = in;
            v_dt[s] = ddt;
          }
          o_bc[(4 * i + 2 * pair + (c >> 3)) * 32 + ((c >> 2) & 1) * 16 + q * 4 + (c & 3)] = transpose_sum16(p16, c);
        }
        // step 4 i + q belongs to this lane from here on
        const float y = sum_rows4(v_y), in = sum_rows4(v_in), ddt = fmaf(in, u_o[i], sum_rows4(v_dt));
        const float o_z = dzf_o[i] * fmaf(d_skip, u_o[i], y);
        // dt = softplus(pre): d pre = d dt * sigmoid(pre) = d dt * (1 - exp(-dt))
        const float o_pre = ddt * (1.0f - fast_exp2(-1.44269504088896341f * dt_o[i]));
        const float o_u = fmaf(in, dt_o[i], d_skip * dy_o[i]);
        acc_bias += o_pre;
        acc_d = fmaf(dy_o[i], u_o[i], acc_d);
        const int t = g * kBwdGroup + 4 * i + q;
        if (decltype(all)::value || (active && t < len)) {
          const unsigned at = row_at(static_cast<unsigned>(t), pitch);
          *reinterpret_cast<T *>(dpre_p + at) = from_f32<T>(o_pre);
          *reinterpret_cast<T *>(du_p + at) = from_f32<T>(o_u);
          *reinterpret_cast<T *>(dz_p + row_at(static_cast<unsigned>(t), pitch_dz)) = from_f32<T>(o_z);
        }
        __builtin_amdgcn_sched_barrier(0);              // (registers: no more than four steps in flight)
      }
    }
  };
  for (int g = n_grp - 1; g >= 0; --g) {
    park(g, true);
    if (g > 0) fetch(g - 1, true);
    if (active && (g + 1) * kBwdGroup <= len) group(g, std::true_type{});
    else group(g, std::false_type{});
    lds_barrier();
    // d_B, d_C of the group: the four wavefronts' shares in wavefront order, two values per thread.  (The next group
    // writes the other copy; this one is written again only behind the next barrier.)
    {
      const int row = tid / 16;
      float v0 = 0.0f, v1 = 0.0f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        v0 += sm.o_bc[g & 1][w][2 * tid];
        v1 += sm.o_bc[g & 1][w][2 * tid + 1];
      }
      if (g * kBwdGroup + row < len) {
        float *dst = d_bc_part + (static_cast<int64_t>(cb) * n_tok + row0 + g * kBwdGroup) * 32 + 2 * tid;
        dst[0] = v0;
        dst[1] = v1;
      }
    }
  }
  // d A_log = d A * A; the rows' shares of d_D, d_dt_bias added in row order
  float *pa = part_a + (unit * kBwdCh + wave * 16 + c) * 16 + q * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) pa[j] = acc_a[j] * a_nat[j];
  acc_d += __shfl_xor(acc_d, 16, 64);
  acc_d += __shfl_xor(acc_d, 32, 64);
  acc_bias += __shfl_xor(acc_bias, 16, 64);
  acc_bias += __shfl_xor(acc_bias, 32, 64);
  if (q == 0) {
    part_d[unit * kBwdCh + wave * 16 + c] = acc_d;
    part_bias[unit * kBwdCh + wave * 16 + c] = acc_bias;
  }
}

// d_A_log, d_D, d_dt_bias: the units' partials summed in unit order.  One thread per (channel, state).
__global__ __launch_bounds__(256) void scan_bwd_finish_kernel(const float *__restrict__ part_a,
                                                              const float *__restrict__ part_d,
                                                              const float *__restrict__ part_bias, int n_cb, int d_inner,
                                                              int64_t n_rep, float *__restrict__ d_A_log,
                                                              float *__restrict__ d_D, float *__restrict__ d_dt_bias) {
  const int idx = blockIdx.x * 256 + threadIdx.x, ch = idx / 16, n = idx % 16;
  if (ch >= d_inner) return;
  const int64_t stride = static_cast<int64_t>(n_cb) * kBwdCh;
  float a = 0.0f;
#pragma unroll 8
  for (int64_t r = 0; r < n_rep; ++r) a += part_a[r * stride * 16 + idx];
  d_A_log[idx] = a;
  if (n < 2) {
    const float *src = (n == 0 ? part_d : part_bias) + ch;
    float v = 0.0f;
#pragma unroll 8
    for (int64_t r = 0; r < n_rep; ++r) v += src[r * stride];
    (n == 0 ? d_D : d_dt_bias)[ch] = v;
  }
}

// d_bc[t, :] = sum over the channel-block partials, in block order
__global__ __launch_bounds__(256) void bwd_reduce_bc_kernel(const float *__restrict__ part, int n_parts, int64_t n_tok,
                                                            float *__restrict__ d_bc) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n_tok * 32) return;
  float tot = 0.0f;
#pragma unroll 8
  for (int p = 0; p < n_parts; ++p) tot += part[static_cast<int64_t>(p) * n_tok * 32 + i];
  d_bc[i] = tot;
}

// ------------------------------------------------------------------ gate weights, Eq. (9)/(12)
// d_gate[r] = a[ia(r), :] . b[ib(r), :], one wavefront per row r.
// top-1: d_gate[n] = d_out[n, :] . (W_out[e_n] g[n, :]) = (W_out[e_n]^T d_out[n, :]) . g[n, :] = dg_raw[n, :] . g[n, :]
// (both in token order, no maps).  top-K: r is a slot, a = d_out by the slot's token (r / K), b = the
// expert output W_out[e] g that the forward pass left per sorted position (row inv_perm[r]).
template <typename T>
__global__ __launch_bounds__(256) void gate_bwd_kernel(const T *__restrict__ a, const T *__restrict__ b,
                                                       const int32_t *__restrict__ b_rows, int a_div, int64_t n_rows,
                                                       int n_cols, float *__restrict__ d_gate) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  if (r >= n_rows) return;
  const int64_t ra = r / a_div, rb = b_rows ? b_rows[r] : r;
  float acc = 0.0f;
  if (n_cols % 8 == 0) {            // rows are 16-byte aligned: eight (bf16) or two times four (fp32) columns per lane and trip
    for (int c = lane * 8; c < n_cols; c += 512) {
      float va[8], vb[8];
      bwd_load4(a + ra * n_cols + c, va);
      bwd_load4(a + ra * n_cols + c + 4, va + 4);
      bwd_load4(b + rb * n_cols + c, vb);
      bwd_load4(b + rb * n_cols + c + 4, vb + 4);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc = fmaf(va[q], vb[q], acc);
    }
  } else {
    for (int c = lane; c < n_cols; c += 64) acc = fmaf(to_f32(a[ra * n_cols + c]), to_f32(b[rb * n_cols + c]), acc);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) d_gate[r] = acc;
}

// d_logits [N, E] from d_gate [N, K]: softmax over all E experts, gate = P of the selected
// (gate_mode 1: divided by their sum).  One thread per token, which asks for all of its logits at once (EMAX of them, those past
// the last expert its copies): an expert at a time is a chain of memory round trips (8192 tokens, 8 experts 8.5-9 us, now 4.9).
template <int EMAX>
__global__ __launch_bounds__(64) void router_bwd_kernel(const float *__restrict__ logits,
                                                        const int32_t *__restrict__ expert_idx,
                                                        const float *__restrict__ d_gate, int64_t n_tok, int n_experts,
                                                        int top_k, int gate_mode, float *__restrict__ d_logits) {
  const int64_t n = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= n_tok) return;
  const float *lp = logits + n * n_experts;
  float p[EMAX], dp[EMAX];
#pragma unroll
  for (int e = 0; e < EMAX; ++e) p[e] = lp[e < n_experts ? e : n_experts - 1], dp[e] = 0.0f;
  float m = p[0];
#pragma unroll
  for (int e = 1; e < EMAX; ++e) m = fmaxf(m, p[e]);
  float den = 0.0f;
#pragma unroll
  for (int e = 0; e < EMAX; ++e) {
    p[e] = __expf(p[e] - m);
    if (e < n_experts) den += p[e];
  }
  const float inv = 1.0f / den;
  // d P of the selected experts
  float s_sel = 0.0f, dot = 0.0f;
  for (int k = 0; k < top_k; ++k) {
    const float pk = __expf(lp[expert_idx[n * top_k + k]] - m) * inv;
    s_sel += pk;
    dot = fmaf(d_gate[n * top_k + k], pk, dot);              // sum_k d_gate_k P_k
  }
  // mode 1: gate_k = P_k / S  ->  dP_k = (d_gate_k - sum_j d_gate_j gate_j) / S ;  mode 0: dP_k = d_gate_k
  // (a single renormalised pick is the constant 1: its gradient is exactly zero, not rounding noise)
  const float shift = gate_mode == 1 ? (top_k == 1 ? d_gate[n] : dot / s_sel) : 0.0f;
  const float scale = gate_mode == 1 ? 1.0f / s_sel : 1.0f;
  float pdp = 0.0f;                                          // sum_e P_e dP_e
  for (int k = 0; k < top_k; ++k) {
    const int idx = expert_idx[n * top_k + k];
    const float pk = __expf(lp[idx] - m) * inv, dk = (d_gate[n * top_k + k] - shift) * scale;
    pdp = fmaf(pk, dk, pdp);
#pragma unroll
    for (int e = 0; e < EMAX; ++e) dp[e] = e == idx ? dk : dp[e];
  }
#pragma unroll
  for (int e = 0; e < EMAX; ++e)
    if (e < n_experts) d_logits[n * n_experts + e] = p[e] * inv * (dp[e] - pdp);
}

// two consecutive channels of a row (4- or 8-byte accesses)
__device__ __forceinline__ void conv_ld2(const bf16_t *p, float (&f)[2]) {
  const unsigned u = *reinterpret_cast<const unsigned *>(p);
  f[0] = bf16_to_f32(static_cast<bf16_t>(u & 0xffffu));
  f[1] = bf16_to_f32(static_cast<bf16_t>(u >> 16));
}
__device__ __forceinline__ void conv_ld2(const float *p, float (&f)[2]) {
  const float2 v = *reinterpret_cast<const float2 *>(p);
  f[0] = v.x; f[1] = v.y;
}
__device__ __forceinline__ void conv_st2(bf16_t *p, const float (&f)[2]) {
  *reinterpret_cast<unsigned *>(p) = static_cast<unsigned>(f32_to_bf16(f[0])) | (static_cast<unsigned>(f32_to_bf16(f[1])) << 16);
}
__device__ __forceinline__ void conv_st2(float *p, const float (&f)[2]) { *reinterpret_cast<float2 *>(p) = make_float2(f[0], f[1]); }

// partial[chunk][e][d] = sum over the chunk's tokens of d_logits[n, e] * x[n, d]  (d = d_model is the
// bias column: x = 1).  grid (ceil((d_model + 1) / 512), n_chunks); a thread owns two columns (d_model is even) and asks for
// kRouterAhead rows together: a row at a time it is a chain of memory round trips.
constexpr int kRouterAhead = 16;
// 8192 tokens x 1024 with 8 experts 48 -> 11 us, 16384 x 2048 52 -> 27 (a column and a row at a time; sixteen rows of one column with
// their ends checked one by one 51 and 76).  Tokens per chunk: workgroups count, down to one round of 64 tokens.
inline int router_chunk(int64_t n_tok) { return n_tok > 8192 ? 128 : 64; }
template <typename T, int EMAX>
__global__ __launch_bounds__(256) void router_wgrad_partial_kernel(const float *__restrict__ d_logits,
                                                                   const T *__restrict__ x, int64_t n_tok, int d_model,
                                                                   int n_experts, int chunk, float *__restrict__ partial) {
  __shared__ float dl[64][EMAX];                    // [token in round][expert]
  const int d = (blockIdx.x * 256 + threadIdx.x) * 2;
  const int64_t n0 = static_cast<int64_t>(blockIdx.y) * chunk;
  const int64_t n1 = n0 + chunk < n_tok ? n0 + chunk : n_tok;
  float acc[2][EMAX];
#pragma unroll
  for (int e = 0; e < EMAX; ++e) acc[0][e] = acc[1][e] = 0.0f;
  for (int64_t r0 = n0; r0 < n1; r0 += 64) {
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * EMAX; i += 256) {
      const int64_t n = r0 + i / EMAX;
      const int e = i % EMAX;
      dl[i / EMAX][e] = (n < n1 && e < n_experts) ? d_logits[n * n_experts + e] : 0.0f;
    }
    __syncthreads();
    const int rows = static_cast<int>(n1 - r0 < 64 ? n1 - r0 : 64);
    const T *xr = x + r0 * d_model + (d < d_model ? d : 0);
    const auto add = [&](int i, float x0, float x1) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < EMAX; ++e) {
        acc[0][e] = fmaf(dl[i][e], x0, acc[0][e]);
        acc[1][e] = fmaf(dl[i][e], x1, acc[1][e]);
      }
    };
    if (d < d_model) {
      int i = 0;
      for (; i + kRouterAhead <= rows; i += kRouterAhead) {
        float xv[kRouterAhead][2];
#pragma unroll
        for (int k = 0; k < kRouterAhead; ++k) conv_ld2(xr + static_cast<int64_t>(k) * d_model, xv[k]);
        xr += static_cast<int64_t>(kRouterAhead) * d_model;
#pragma unroll
        for (int k = 0; k < kRouterAhead; ++k) add(i + k, xv[k][0], xv[k][1]);
      }
      for (; i < rows; ++i, xr += d_model) {
        float xv[2];
        conv_ld2(xr, xv);
        add(i, xv[0], xv[1]);
      }
    } else if (d == d_model) {
      for (int i = 0; i < rows; ++i) add(i, 1.0f, 0.0f);
    }
  }
#pragma unroll
  for (int v = 0; v < 2; ++v)
    if (d + v <= d_model)
#pragma unroll
      for (int e = 0; e < EMAX; ++e)
        if (e < n_experts) partial[(static_cast<int64_t>(blockIdx.y) * n_experts + e) * (d_model + 1) + d + v] = acc[v][e];
}

// Waves per 64 outputs of the two kernels that add partial sums: each adds every sixteenth, then the wave sums are added in
// wave order (one thread walking all partials is a chain of memory round trips).
constexpr int kFinishWaves = 16;
__device__ __forceinline__ float finish_total(float acc, float (&sums)[kFinishWaves][64], int lane, int wave) {
  sums[wave][lane] = acc;
  __syncthreads();
  float tot = sums[0][lane];
#pragma unroll
  for (int w = 1; w < kFinishWaves; ++w) tot += sums[w][lane];
  return tot;
}

__global__ __launch_bounds__(kFinishWaves * 64) void router_wgrad_finish_kernel(const float *__restrict__ partial, int n_chunks,
                                                                  int d_model, int n_experts,
                                                                  float *__restrict__ d_w_router,
                                                                  float *__restrict__ d_b_router) {
  __shared__ float sums[kFinishWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const bool live = i < n_experts * (d_model + 1);
  float acc = 0.0f;
  if (live)
    for (int c = q; c < n_chunks; c += kFinishWaves) acc += partial[static_cast<int64_t>(c) * n_experts * (d_model + 1) + i];
  const float tot = finish_total(acc, sums, lane, q);
  if (q != 0 || !live) return;
  const int e = i / (d_model + 1), d = i % (d_model + 1);
  if (d < d_model) d_w_router[e * d_model + d] = tot;
  else if (d_b_router) d_b_router[e] = tot;
}

// Row passes: 16 bytes of a row a lane, so a wavefront has 512 columns of it (fp32 256), or, NARROW, as many lanes as a shorter row fills
// (2^lanes_log2) and several rows.
template <typename T> constexpr int kRowCols = 16 / static_cast<int>(sizeof(T));
template <typename T>
inline int row_lanes_log2(int n_cols) {
  int lg = 0;
  while (lg < 6 && (kRowCols<T> << lg) < n_cols) ++lg;
  return lg;
}
template <typename T>
inline dim3 row_grid(int64_t n_rows, int n_cols) {
  return grid1d(ceil_div(n_rows, 64 >> row_lanes_log2<T>(n_cols)) * ceil_div(n_cols, 64 * kRowCols<T>), 4);
}
// this lane's row and first column
template <typename T, bool NARROW>
__device__ __forceinline__ void row_place(int n_cols, int lanes_log2, int64_t &row, int &col) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (NARROW) {
    row = wave * (64 >> lanes_log2) + (lane >> lanes_log2);
    col = (lane & ((1 << lanes_log2) - 1)) * kRowCols<T>;
  } else {
    const int col_waves = (n_cols + 64 * kRowCols<T> - 1) / (64 * kRowCols<T>);
    row = wave / col_waves;
    col = (static_cast<int>(wave % col_waves) * 64 + lane) * kRowCols<T>;
  }
}

// d_x[n, d] = dx_in[n, d] + sum_e d_logits[n, e] * W_r[e, d].  A lane has kDxRows tokens: the router weights are loaded once for all of them,
// and d_logits, uniform, through the scalar cache; in short rows one (four leave 8192 x 128 too few wavefronts, 5.9 us, one 4.2).
// Bound by memory: 16384 x 2048 with 8 experts 47 us a token at a time and an index division per thread, now 31; 8192 x 1024 12.2 -> 9.8,
// fp32 21.7 -> 15.6; 32768 x 64 5.5 -> 5.0, fp32 7.8 -> 6.2 (10.0 and 19.9 with a row a wavefront).
template <bool NARROW> constexpr int kDxRows = NARROW ? 1 : 4;
template <typename T, bool NARROW>
__global__ __launch_bounds__(256) void dx_finish_kernel(const T *__restrict__ dx_in, const float *__restrict__ d_logits,
                                                        const T *__restrict__ w_router, int64_t n_tok, int d_model, int n_experts,
                                                        int lanes_log2, T *__restrict__ d_x) {
  constexpr int kCols = kRowCols<T>, kRows = kDxRows<NARROW>;
  int64_t n0;
  int d;
  row_place<T, NARROW>(d_model, lanes_log2, n0, d);
  n0 *= kRows;
  if (n0 >= n_tok || d >= d_model) return;
  const int rows = static_cast<int>(n_tok - n0 < kRows ? n_tok - n0 : kRows);
  typedef const __attribute__((address_space(4))) float const_f32_t;
  const uintptr_t dl = reinterpret_cast<uintptr_t>(d_logits + n0 * n_experts);
  float v[kRows][kCols];
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int q = 0; q < kCols; q += 4) bwd_load4(dx_in + (n0 + (r < rows ? r : rows - 1)) * d_model + d + q, v[r] + q);
#pragma unroll 4
  for (int e = 0; e < n_experts; ++e) {
    float wv[kCols];
#pragma unroll
    for (int q = 0; q < kCols; q += 4) bwd_load4(w_router + static_cast<int64_t>(e) * d_model + d + q, wv + q);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int at = (r < rows ? r : rows - 1) * n_experts + e;
      float g;
      if constexpr (NARROW) g = d_logits[n0 * n_experts + at];
      else g = *reinterpret_cast<const_f32_t *>(dl + static_cast<uint32_t>(at) * 4u);
#pragma unroll
      for (int q = 0; q < kCols; ++q) v[r][q] = fmaf(g, wv[q], v[r][q]);
    }
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    if (r >= rows) break;
#pragma unroll
    for (int q = 0; q < kCols; q += 4) bwd_store4(d_x + (n0 + r) * d_model + d + q, v[r] + q);
  }
}

// ------------------------------------------------------------------ adjoint of conv + SiLU, Eq. (2)
// A thread owns one channel (or two) and a run of steps of one sequence (conv_bwd_run).  c_t = b + sum_j w_j x_{t-3+j}
// is recomputed, d_c_t = (du_a + du_b)_t * SiLU'(c_t); d_x_{t} = sum_j w_j d_c_{t+3-j} needs d_c of three
// later steps (zero past the sequence end), so the thread runs three steps into the next run.
// Per-run partial sums of d_w[i, j] = sum_t d_c_t x_{t-3+j} and d_b = sum_t d_c_t go to
// partial[run][5][channel] and are added in run order by conv_bwd_finish_kernel.
// Steps per run: 128, and half of that as long as there are fewer than 4096 wavefronts (16 a CU).  A run reads six rows more than
// its steps, and its partial sums are five rows.  4 x 2048 steps x 2048 channels: runs of 64 29 us, 32 30, 16 33; 16384 x 4096 (4096 wavefronts of
// 128) 114, of 64 118.  Bound by memory (three rows in, one out: 537 MB, 4.7 TB/s); with the rows of eight steps requested in one go
// and converted where they were requested, 8192 x 2048 took 41 and 16384 x 4096 139.
inline int conv_bwd_run(int64_t B, int64_t L, int d_inner) {
  int run = 128;
  while (run > 16 && B * ceil_div(L, run) * ceil_div(d_inner, 128) < 4096) run /= 2;
  return run;
}
constexpr int kConvBwdAhead = 8;     // steps whose rows are requested together
// V = 2: a thread owns two neighbouring channels (half the memory instructions, twice their width)
template <typename T, int V>
__global__ __launch_bounds__(256) void conv_bwd_kernel(const T *__restrict__ xz, int64_t ld_xz,
                                                       const float *__restrict__ conv_w,
                                                       const float *__restrict__ conv_b, const T *__restrict__ du_a,
                                                       const T *__restrict__ du_b, int64_t L, int d_inner,
                                                       T *__restrict__ d_xpre, int64_t ld_dx, int run_steps,
                                                       float *__restrict__ partial) {
  static_assert(V == 1 || V == 2, "one or two channels per thread");
  const int ch = (blockIdx.x * blockDim.x + threadIdx.x) * V;
  if (ch >= d_inner) return;
  const int64_t b = blockIdx.z, run = blockIdx.y;
  const int64_t t0 = run * run_steps;
  const int64_t t1 = t0 + run_steps < L ? t0 + run_steps : L;
  float w[V][4], bias[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const float4 wv = *reinterpret_cast<const float4 *>(conv_w + static_cast<int64_t>(ch + v) * 4);
    w[v][0] = wv.x; w[v][1] = wv.y; w[v][2] = wv.z; w[v][3] = wv.w;
    bias[v] = conv_b ? conv_b[ch + v] : 0.0f;
  }
  const T *xr = xz + b * L * ld_xz + ch;
  const int64_t tok0 = b * L;
  // the rows a step needs from memory, as they lie there: x_{t+3} and the two d u rows of step t+3 (zeros outside the sequence,
  // put in place of the values of its ends - the same number of requests for every step, and none that waits for a conversion)
  using Raw = std::conditional_t<V == 1, T, std::conditional_t<sizeof(T) == 2, uint32_t, float2>>;
  struct Rows {
    Raw x, ua, ub;
  };
  auto fetch = [&](int64_t t) __attribute__((always_inline)) {
    const int64_t tc = t < 0 ? 0 : t < L ? t : L - 1;
    Rows r;
    r.x = *reinterpret_cast<const Raw *>(xr + tc * ld_xz);
    r.ua = *reinterpret_cast<const Raw *>(du_a + (tok0 + tc) * d_inner + ch);
    r.ub = *reinterpret_cast<const Raw *>(du_b + (tok0 + tc) * d_inner + ch);
    return r;
  };
  auto value = [&](int64_t t, const Raw &raw, float (&f)[V]) __attribute__((always_inline)) {
    const bool in = t >= 0 && t < L;
    if constexpr (V == 1) {
      f[0] = in ? to_f32(raw) : 0.0f;
    } else if constexpr (sizeof(T) == 2) {
      const uint32_t w2 = in ? raw : 0u;
      f[0] = __uint_as_float(w2 << 16);
      f[1] = __uint_as_float(w2 & 0xFFFF0000u);
    } else {
      f[0] = in ? raw.x : 0.0f;
      f[1] = in ? raw.y : 0.0f;
    }
  };
  // d loss / d c_t from the four inputs x_{t-3..t} of c_t and d u_t (d u = 0 outside the sequence gives 0)
  auto dc_of = [&](const float (&x0)[V], const float (&x1)[V], const float (&x2)[V], const float (&x3)[V],
                   const float (&ua)[V], const float (&ub)[V], float (&d)[V]) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const float c = bias[v] + w[v][0] * x0[v] + w[v][1] * x1[v] + w[v][2] * x2[v] + w[v][3] * x3[v];
      const float sig = sigmoid_f32(c);
      d[v] = (ua[v] + ub[v]) * sig * (1.0f + c * (1.0f - sig));
    }
  };
  float acc_w[V][4], acc_b[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc_b[v] = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) acc_w[v][j] = 0.0f;
  }
  // the inputs x_{t-3} .. x_{t+3} and d_c of t .. t+3 slide along the run: one new x row, one new pair
  // of d u rows and one output row per step.  The rows of kConvBwdAhead steps are under way at any time: a thread's loop
  // is otherwise one memory round trip per step.
  float xs[7][V], d0[V], d1[V], d2[V], d3[V];
  Rows ring[kConvBwdAhead];
  {
    Rows first[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) first[k] = fetch(t0 - 3 + k);
#pragma unroll
    for (int k = 0; k < kConvBwdAhead; ++k) ring[k] = fetch(t0 + 3 + k);
    float ua[3][V], ub[3][V];
#pragma unroll
    for (int k = 0; k < 6; ++k) value(t0 - 3 + k, first[k].x, xs[k]);
#pragma unroll
    for (int k = 0; k < 3; ++k) value(t0 + k, first[3 + k].ua, ua[k]), value(t0 + k, first[3 + k].ub, ub[k]);
    dc_of(xs[0], xs[1], xs[2], xs[3], ua[0], ub[0], d0);
    dc_of(xs[1], xs[2], xs[3], xs[4], ua[1], ub[1], d1);
    dc_of(xs[2], xs[3], xs[4], xs[5], ua[2], ub[2], d2);
  }
  auto step = [&](int64_t t, int k) __attribute__((always_inline)) {
    float una[V], unb[V];
    value(t + 3, ring[k].x, xs[6]);
    value(t + 3, ring[k].ua, una);
    value(t + 3, ring[k].ub, unb);
    ring[k] = fetch(t + kConvBwdAhead < t1 ? t + 3 + kConvBwdAhead : t1 + 2);          // (past the run's end: its last rows again)
    dc_of(xs[3], xs[4], xs[5], xs[6], una, unb, d3);
    // x_t feeds c_t (tap 3), c_{t+1} (tap 2), c_{t+2} (tap 1), c_{t+3} (tap 0)
    float o[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      o[v] = w[v][3] * d0[v] + w[v][2] * d1[v] + w[v][1] * d2[v] + w[v][0] * d3[v];
      {
#pragma clang fp contract(off)                                // (the rounded d_c, as everywhere else)
        acc_b[v] += d0[v];
      }
      acc_w[v][0] = fmaf(d0[v], xs[0][v], acc_w[v][0]);
      acc_w[v][1] = fmaf(d0[v], xs[1][v], acc_w[v][1]);
      acc_w[v][2] = fmaf(d0[v], xs[2][v], acc_w[v][2]);
      acc_w[v][3] = fmaf(d0[v], xs[3][v], acc_w[v][3]);
      d0[v] = d1[v]; d1[v] = d2[v]; d2[v] = d3[v];
    }
    if constexpr (V == 2) conv_st2(d_xpre + (tok0 + t) * ld_dx + ch, o);
    else d_xpre[(tok0 + t) * ld_dx + ch] = from_f32<T>(o[0]);
#pragma unroll
    for (int j = 0; j < 6; ++j)
#pragma unroll
      for (int v = 0; v < V; ++v) xs[j][v] = xs[j + 1][v];
  };
  int64_t t = t0;
  for (; t + kConvBwdAhead <= t1; t += kConvBwdAhead) {
#pragma unroll
    for (int k = 0; k < kConvBwdAhead; ++k) step(t + k, k);
  }
#pragma unroll
  for (int k = 0; k < kConvBwdAhead - 1; ++k)
    if (t + k < t1) step(t + k, k);
  const int64_t n_runs = gridDim.y;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    float *dst = partial + ((b * n_runs + run) * 5) * d_inner + ch + v;
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[j * d_inner] = acc_w[v][j];
    dst[4 * d_inner] = acc_b[v];
  }
}

__global__ __launch_bounds__(kFinishWaves * 64) void conv_bwd_finish_kernel(const float *__restrict__ partial, int64_t n_parts,
                                                              int d_inner, float *__restrict__ d_conv_w,
                                                              float *__restrict__ d_conv_b) {
  __shared__ float sums[kFinishWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane;
  const bool live = i < 5 * d_inner;
  const int j = live ? i / d_inner : 0, ch = live ? i % d_inner : 0;
  float acc = 0.0f;
  if (live)
    for (int64_t p = q; p < n_parts; p += kFinishWaves) acc += partial[(p * 5 + j) * d_inner + ch];
  const float tot = finish_total(acc, sums, lane, q);
  if (q != 0 || !live) return;
  if (j < 4) d_conv_w[ch * 4 + j] = tot;
  else if (d_conv_b) d_conv_b[ch] = tot;
}

// ------------------------------------------------------------------ weight transposes for the input gradients
// dst[e][c][r] = src[e][r][c]: the grouped GEMM contracts over the contiguous index of both operands,
// and d_inp = d_out W contracts over W's row index.  64 x 64 tiles through LDS; when rows and cols
// are multiples of 4, both the global reads and the global writes move four consecutive elements.
// Two weights in one launch (the second may have no blocks): 1024 x 2048, 8 experts, W_dt and W_x 5.2 + 5.3 -> 5.5 us.
template <typename T>
struct TransposeJob {
  const T *src;
  T *dst;
  int rows, cols, vec, tiles_r, tiles_c, blocks;
};
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const TransposeJob<T> first, const TransposeJob<T> second) {
  __shared__ float tile[64][65];
  const bool is_first = static_cast<int>(blockIdx.x) < first.blocks;
  const TransposeJob<T> job = is_first ? first : second;
  const int id = blockIdx.x - (is_first ? 0 : first.blocks), rows = job.rows, cols = job.cols, vec = job.vec;
  const T *const src = job.src;
  T *const dst = job.dst;
  const int64_t base = static_cast<int64_t>(id / (job.tiles_r * job.tiles_c)) * rows * cols;
  const int r0 = id / job.tiles_c % job.tiles_r * 64, c0 = id % job.tiles_c * 64;
  if (vec) {
    // thread -> (row i = tid / 16 + 16 q, columns 4 (tid % 16) .. + 3)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = (threadIdx.x >> 4) + 16 * q, j = (threadIdx.x & 15) * 4;
      float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (r0 + i < rows && c0 + j < cols) bwd_load4(src + base + static_cast<int64_t>(r0 + i) * cols + c0 + j, v);
#pragma unroll
      for (int e = 0; e < 4; ++e) tile[i][j + e] = v[e];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = (threadIdx.x >> 4) + 16 * q, j = (threadIdx.x & 15) * 4;     // output row c0 + i, columns r0 + j ..
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = tile[j + e][i];
      if (c0 + i < cols && r0 + j < rows) bwd_store4(dst + base + static_cast<int64_t>(c0 + i) * rows + r0 + j, v);
    }
  } else {
    for (int k = threadIdx.x; k < 64 * 64; k += 256) {
      const int i = k / 64, j = k % 64;
      if (r0 + i < rows && c0 + j < cols) tile[i][j] = to_f32(src[base + static_cast<int64_t>(r0 + i) * cols + c0 + j]);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < 64 * 64; k += 256) {
      const int i = k / 64, j = k % 64;
      if (c0 + i < cols && r0 + j < rows) dst[base + static_cast<int64_t>(c0 + i) * rows + r0 + j] = from_f32<T>(tile[j][i]);
    }
  }
}

// d_xdbl [N, R + 32] (type T) = [ d_dt_low (f32 [N, R]) | d_bc (f32 [N, 32]) ]
template <typename T>
__global__ __launch_bounds__(256) void pack_dxdbl_kernel(const float *__restrict__ d_dt_low,
                                                         const float *__restrict__ d_bc, int64_t n_tok, int dt_rank,
                                                         T *__restrict__ d_xdbl) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int cols = dt_rank + 32;
  if (i >= n_tok * cols) return;
  const int64_t n = i / cols;
  const int c = static_cast<int>(i % cols);
  d_xdbl[i] = from_f32<T>(c < dt_rank ? d_dt_low[n * dt_rank + c] : d_bc[n * 32 + (c - dt_rank)]);
}

// ------------------------------------------------------------------ weight gradients
//   d_W[e][m][n] = sum over the sorted positions p of expert e of s_p * A[a_row(p)][m] * B[b_row(p)][n]
// (A = the gradient of the projection's output, B = its input, s = gate weight for the out projection).
// Both operands are stored position-major, so the contraction index is the slow one: a 128 x 128
// output tile walks the expert's positions in slabs of 32, each thread fetches 16-byte pieces
// (eight consecutive m or n of one position) and scatters them transposed into LDS, from where the
// MFMA fragments (eight consecutive positions of one m / n) are read.  fp32 result, fixed order.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// 64 x 64 tiles where 128 x 128 ones would not give every CU a workgroup (8192 rows in 8 experts, 128 workgroups of 96 x 2048: 41 us, 28;
// 16384 rows, 512 of 160 x 4096: 78, 102).  Operands of at most 160 columns have a kernel of their own further down.
constexpr int kWgTileMinWgs = 256;
constexpr int kWgTile = 128, kWgSlab = 64, kWgPitch = kWgSlab + 8;     // halfs per LDS row (144 bytes: 16-byte aligned rows)

// eight 16-byte pieces (eight consecutive columns of eight consecutive positions) -> for each of the
// eight columns the eight positions as one 16-byte LDS row segment: word a of column m's segment
// holds positions 2a, 2a+1, which v_perm_b32 picks out of word m/2 of the two position rows
__device__ __forceinline__ void wgrad_park8x8(const u32x4_t (&v)[8], bf16_t (*dst)[kWgPitch], int col0, int pos0) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {          // word w of a piece = columns 2w, 2w+1
    u32x4_t lo, hi;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const unsigned int p0 = v[2 * a][w], p1 = v[2 * a + 1][w];
      lo[a] = __builtin_amdgcn_perm(p1, p0, 0x05040100u);      // (p0.lo16, p1.lo16)
      hi[a] = __builtin_amdgcn_perm(p1, p0, 0x07060302u);      // (p0.hi16, p1.hi16)
    }
    *reinterpret_cast<u32x4_t *>(&dst[col0 + 2 * w][pos0]) = lo;
    *reinterpret_cast<u32x4_t *>(&dst[col0 + 2 * w + 1][pos0]) = hi;
  }
}

// TILE x TILE on TILE / 32 wavefronts (128: 2 x 2 of 64 x 64; 64: two of 32 x 64)
template <int TILE>
__global__ __launch_bounds__(2 * TILE) void wgrad_bf16_kernel(const bf16_t *__restrict__ A, int64_t lda, int M,
                                                         const bf16_t *__restrict__ Bm, int64_t ldb, int N,
                                                         const int32_t *__restrict__ rows_a,
                                                         const int32_t *__restrict__ rows_b,
                                                         const int32_t *__restrict__ offsets, int64_t n_pos,
                                                         float *__restrict__ C) {
  constexpr int MB = TILE / 64;                                  // 32-row blocks of a wavefront
  __shared__ __attribute__((aligned(16))) bf16_t As[TILE][kWgPitch];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[TILE][kWgPitch];
  const int e = blockIdx.z;
  const int64_t p_lo = offsets ? offsets[e] : 0, p_hi = offsets ? offsets[e + 1] : n_pos;
  const int m0 = blockIdx.y * TILE, n0 = blockIdx.x * TILE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  f32x16_t acc[MB][2];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  // staging: a slab is 64 positions; the first half of the threads brings the A operand, the second the B operand, each an
  // 8-position x 8-column block: (position group pg = 0..7, column piece)
  const bool is_a = __builtin_amdgcn_readfirstlane(tid < TILE ? 1 : 0) != 0;     // wave-uniform
  const int t2 = tid & (TILE - 1), pg = t2 & 7, piece = t2 >> 3;       // 16 consecutive lanes park into 64 distinct banks
  const bf16_t *src = is_a ? A : Bm;
  const int32_t *rows = is_a ? rows_a : rows_b;      // position -> row of this operand (NULL: the position itself)
  const int64_t ld = is_a ? lda : ldb;
  const int col = (is_a ? m0 : n0) + piece * 8;
  const bool col_ok = col < (is_a ? M : N);
  bf16_t(*dst)[kWgPitch] = is_a ? As : Bs;
  // Row numbers are asked for two slabs ahead of their use and rows one slab ahead: with one or two workgroups on a CU nothing
  // else hides the two round trips (a tenth of the kernel at 16384 rows).  (Branch-free, indices first: see the 256 x 256
  // kernel.)
  const auto numbers = [&](int64_t p0, int(&r)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t p = p0 + pg * 8 + i;
      r[i] = static_cast<int>(p < p_hi ? p : p_hi - 1);
    }
    if (rows) {
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = rows[r[i]];
    }
  };
  u32x4_t v[8];
  int r[8];
  const auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const u32x4_t *>(src + r[i] * ld + (col_ok ? col : 0));
  };
  if (p_lo < p_hi) {
    numbers(p_lo, r);
    fetch();
    numbers(p_lo + kWgSlab, r);
  }
  for (int64_t p0 = p_lo; p0 < p_hi; p0 += kWgSlab) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (p0 + pg * 8 + i >= p_hi || !col_ok) v[i] = u32x4_t{0u, 0u, 0u, 0u};
    __syncthreads();                       // the slab before this one has been multiplied
    wgrad_park8x8(v, dst, piece * 8, pg * 8);
    __syncthreads();
    if (p0 + kWgSlab < p_hi) {
      fetch();
      numbers(p0 + 2 * kWgSlab, r);
      __builtin_amdgcn_sched_barrier(0);                         // the requests go out ahead of the products
    }
#pragma unroll
    for (int kk = 0; kk < kWgSlab / 16; ++kk) {
      bf16x8_t fa[MB], fb[2];
#pragma unroll
      for (int i = 0; i < MB; ++i)
        fa[i] = *reinterpret_cast<const bf16x8_t *>(&As[(wm * MB + i) * 32 + frag_row][kk * 16 + frag_half * 8]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        fb[i] = *reinterpret_cast<const bf16x8_t *>(&Bs[wn * 64 + i * 32 + frag_row][kk * 16 + frag_half * 8]);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  }
  // the B fragment is the MFMA's row operand: this lane holds, for output row m = frag_row, the
  // columns 8 q + 4 frag_half + r of each 32-wide tile in accumulator element 4 q + r
  float *Ce = C + static_cast<int64_t>(e) * M * N;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int m = m0 + (wm * MB + i) * 32 + frag_row;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = n0 + wn * 64 + j * 32 + q * 8 + frag_half * 4;
        if (m < M && cc + 3 < N)
          *reinterpret_cast<float4 *>(Ce + static_cast<int64_t>(m) * N + cc) =
              make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        else
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (m < M && cc + r < N) Ce[static_cast<int64_t>(m) * N + cc + r] = acc[i][j][4 * q + r];
      }
  }
}

// The same contraction for outputs of at least 256 x 256 per expert (the in and out projections):
// a 256 x 256 tile on eight waves (4 x 2, 64 x 128 each: 2 x 4 MFMA accumulators, six fragment
// reads per eight MFMAs instead of four per four, because the fragment reads out of LDS are what
// bounds the small tile), two LDS buffers so that the next slab is fetched into registers while
// this one is multiplied and parked into the other buffer afterwards: one barrier per slab.
constexpr int kWgBig = 256;
constexpr int kWgBigSmem = 2 * 2 * kWgBig * kWgPitch * 2;      // two buffers x (A, B) x 256 rows x 144 bytes
__global__ __launch_bounds__(512) void wgrad_bf16_big_kernel(const bf16_t *__restrict__ A, int64_t lda, int M,
                                                             const bf16_t *__restrict__ Bm, int64_t ldb, int N,
                                                             const int32_t *__restrict__ rows_a,
                                                             const int32_t *__restrict__ rows_b,
                                                             const int32_t *__restrict__ offsets, int64_t n_pos,
                                                             int n_groups, float *__restrict__ C) {
  extern __shared__ __attribute__((aligned(16))) unsigned char wg_smem[];
  typedef bf16_t (*Tile)[kWgPitch];
  // Workgroup ids go round the eight XCDs; logical tiles (column tile fastest, then row tile, then
  // expert) are dealt so that an XCD works on a contiguous run of them: the 32 tiles its CUs hold at
  // a time share their A and B column blocks in that XCD's L2 instead of each fetching its own.
  const int tn = (N + kWgBig - 1) / kWgBig, tm = (M + kWgBig - 1) / kWgBig;
  const int per_xcd = gridDim.x / 8;                             // the grid is padded to a multiple of 8
  const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= tn * tm * n_groups) return;
  const int e = t / (tn * tm);
  const int64_t p_lo = offsets ? offsets[e] : 0, p_hi = offsets ? offsets[e + 1] : n_pos;
  const int m0 = ((t / tn) % tm) * kWgBig, n0 = (t % tn) * kWgBig;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 3, wn = wave >> 2;                       // 4 x 2 waves, 64 x 128 each
  f32x16_t acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const int frag_row = lane & 31, frag_half = lane >> 5;
  // staging: threads 0..255 bring the A operand, 256..511 the B operand, each an 8-position x 8-column
  // block of the slab's 64 positions x 256 columns: (position group pg = 0..7, column piece = 0..31)
  // (wave-uniform, and said so: with a per-lane operand choice the row map's NULL test is a divergent
  // branch around every index load, each followed by its own wait)
  const bool is_a = __builtin_amdgcn_readfirstlane(tid < 256 ? 1 : 0) != 0;
  const int t2 = tid & 255, pg = t2 & 7, piece = t2 >> 3;
  const bf16_t *src = is_a ? A : Bm;
  const int32_t *rows = is_a ? rows_a : rows_b;
  const int64_t ld = is_a ? lda : ldb;
  const int col = (is_a ? m0 : n0) + piece * 8;
  const bool col_ok = col < (is_a ? M : N);
  auto tile_of = [&](int buf, bool a_side) {
    return reinterpret_cast<Tile>(wg_smem + (static_cast<size_t>(buf) * 2 + (a_side ? 0 : 1)) * kWgBig * kWgPitch * 2);
  };
  u32x4_t v[8];
  // Branch-free: the eight row indices first, then the eight rows (positions past the group's end
  // re-read its last row, columns past the matrix re-read column 0, and are zeroed afterwards) - with
  // a branch per row the compiler waits for each index and each row in turn, sixteen dependent
  // memory round trips per slab.
  const int col_c = col_ok ? col : 0;
  // (requesting the row indices a further slab ahead, so that their round trip is hidden too,
  // measured slower: 0.78 -> 0.94 ms)
  auto fetch = [&](int64_t p0) __attribute__((always_inline)) {
    int64_t r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t p = p0 + pg * 8 + i;
      r[i] = p < p_hi ? p : p_hi - 1;
    }
    if (rows) {
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = rows[r[i]];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const u32x4_t *>(src + r[i] * ld + col_c);
  };
  // zeroes what fetch(p0) read past the group's end or past the matrix; called where the rows are
  // parked, not where they are requested, so that the wait for them comes after the MFMAs
  auto mask = [&](int64_t p0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (p0 + pg * 8 + i >= p_hi || !col_ok) v[i] = u32x4_t{0u, 0u, 0u, 0u};
  };
  if (p_lo < p_hi) {
    fetch(p_lo);
    mask(p_lo);
    wgrad_park8x8(v, tile_of(0, is_a), piece * 8, pg * 8);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t p0 = p_lo; p0 < p_hi; p0 += kWgSlab, buf ^= 1) {
    const bool has_next = p0 + kWgSlab < p_hi;
    if (has_next) fetch(p0 + kWgSlab);                 // in flight while this slab is multiplied
    const Tile As = tile_of(buf, true), Bs = tile_of(buf, false);
#pragma unroll
    for (int kk = 0; kk < kWgSlab / 16; ++kk) {
      bf16x8_t fa[2], fb[4];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        fa[i] = *reinterpret_cast<const bf16x8_t *>(&As[wm * 64 + i * 32 + frag_row][kk * 16 + frag_half * 8]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        fb[j] = *reinterpret_cast<const bf16x8_t *>(&Bs[wn * 128 + j * 32 + frag_row][kk * 16 + frag_half * 8]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    // the other buffer was last read in the iteration before this one, which every wave has left
    if (has_next) {
      mask(p0 + kWgSlab);
      wgrad_park8x8(v, tile_of(buf ^ 1, is_a), piece * 8, pg * 8);
    }
    __syncthreads();
  }
  // the B fragment is the MFMA's row operand: this lane holds, for output row m = frag_row, the
  // columns 8 q + 4 frag_half + r of each 32-wide tile in accumulator element 4 q + r
  float *Ce = C + static_cast<int64_t>(e) * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + wm * 64 + i * 32 + frag_row;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = n0 + wn * 128 + j * 32 + q * 8 + frag_half * 4;
        if (m < M && cc + 3 < N)
          *reinterpret_cast<float4 *>(Ce + static_cast<int64_t>(m) * N + cc) =
              make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        else
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (m < M && cc + r < N) Ce[static_cast<int64_t>(m) * N + cc + r] = acc[i][j][4 * q + r];
      }
  }
}

// The 256 x 256 contraction once more, for outputs that are whole multiples of the tile: the operand
// rows go from global memory straight into LDS exactly as they lie in memory - position-major, 256
// columns = 512 bytes per position (global_load_lds_dwordx4: lane l of a wave deposits its 16 bytes
// at M0 + 16 l) - and the MFMA fragments, which want eight consecutive POSITIONS of one column per
// lane, are read with the transposing LDS read (ds_read_b64_tr_b16: the 16 lanes of a group name four
// rows of 16 columns, lane i receives column i of the four rows).  No register transposes, no LDS
// writes and no load -> park dependency are left in the loop.  A slab is 64 positions; LDS is a
// ring of five half-slab slots of 32 KiB (A rows of slab m, B rows of slab m, A rows of slab m + 1, ...)
// filled in ring order, eight DMA instructions per wave and half slab, so that "vmcnt(8)" means
// "everything but the newest half slab I asked for has landed".  The 16-byte chunk c of row r lies
// at position c ^ 4 (r & 3) of its row (the swizzle is applied where the global address is formed):
// the four rows x 64 bytes that 32 lanes read at a time then cover all 64 banks once.
//
// One workgroup of four wavefronts per CU (128 x 128 each: a third less LDS traffic per product than
// eight of 64 x 128, which kept the LDS port busy all the time) walks its share of the tiles, and the ring runs
// on across tile boundaries.  Every XCD has an eighth of every expert's tiles, so that experts of uneven
// size load all of them alike; consecutive tiles form patches four tile rows high, whose operands meet in
// the XCD's L2.  A tile of 256 KiB of sums is dear to store, all CUs at once and nothing multiplied meanwhile:
// half of it goes out at once behind requests for the next two slabs (loads and stores retire in order; the
// first wait that includes these stores is the one at the end of the next tile's second slab), the other
// half is kept in registers and goes out four stores a slab.  A store covers 64 bytes of each of 16 rows.
// Row indices (positions -> rows of the operand) are uniform per wave and instruction half: they are read
// sixteen at a time through the scalar cache, a 16-wide step of MFMAs ahead of the DMA that uses them.  Where a
// wavefront's 16 positions would reach past the last one they are moved down to end there; what a slab
// holds of positions that are not its own is zeroed in LDS before it is multiplied.
// Bound by the power that the matrix pipe draws: without its stores a launch of 16384 rows x 8192 x 2048 in 8 experts takes
// 450-470 us, with them 507-519 (601-574 with a tile per workgroup of eight wavefronts and both operands' stores at the
// end); 2048 x 4096 329 -> 271 through row maps, 272 -> 263 without; 8192 rows, 4096 x 1024 100 -> 88, 1024 x 2048 53 -> 47.  Stores past
// the caches: 549 us.  One held block instead of two makes no difference beyond 2 %.  Matrix pipe busy 48-51 % (38-47 % before).
// With half of 16384 rows on one of 8 experts 8192 x 2048 takes 510 us (even 525, a tile per workgroup 1966 and 672), but
// 2048 x 4096 329 (even 275, 1047 and 355): its 128 tiles an expert are dealt to half of each XCD's CUs, and the large expert's
// stay there.  With half of the slots on one of 16 experts 629 and 377 us (2453 and 1113).
constexpr int kWdSlots = 5;
constexpr int kWdSlotBytes = kWgSlab * kWgBig * 2;         // 64 positions x 256 columns x 2 bytes
constexpr int kWdSmem = kWdSlots * kWdSlotBytes;           // 160 KiB
constexpr int kWdInstr = 8;                                // DMA instructions per wave and half slab (2 rows each)
constexpr int kWdRows = 2 * kWdInstr;                      // positions that a wave brings per half slab
constexpr int kWdWgs = 256;                                // one workgroup per CU
constexpr int kWdBand = 4;                                 // tile rows of a patch
constexpr int kWdHeld = 2;                                 // 32-row blocks (of four) whose stores wait for the next tile
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef short i16x8_t __attribute__((ext_vector_type(8)));
typedef int i32x16_t __attribute__((ext_vector_type(16)));
typedef i32x16_t i32x16_word_t __attribute__((aligned(4)));
typedef float f32x4_wd_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_byte_t;

__device__ __forceinline__ void wd_dma_16(unsigned lds_addr, unsigned voff, const void *base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n"
               :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}

__device__ __forceinline__ void wt_dma_4(unsigned lds_addr, unsigned voff, const void *base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2\n"
               :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}

// eight consecutive positions of this lane's column: two transposing reads four rows apart
__device__ __forceinline__ bf16x8_t wd_frag(const lds_byte_t *p) {
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(p));
  const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(p + 4 * kWgBig * 2));
  const i16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, v);
}

// an output tile; a place in the list of this workgroup's tiles (e == n_groups: behind the last one)
struct WdTile {
  int e, i;                       // expert, and place among the XCD's tiles of that expert
  int m0, n0;
  int p_lo, p_hi, slabs;          // positions; an expert without any has one slab of zeros
};

// MAP_A / MAP_B: the operand's rows are rows_x[position] (else the position itself)
template <bool MAP_A, bool MAP_B>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void wgrad_bf16_dma_kernel(
    const bf16_t *__restrict__ A, int64_t lda, int M, const bf16_t *__restrict__ Bm, int64_t ldb, int N,
    const int32_t *__restrict__ rows_a, const int32_t *__restrict__ rows_b, const int32_t *__restrict__ offsets,
    int n_pos, int n_groups, float *__restrict__ C) {
  extern __shared__ __attribute__((aligned(16))) unsigned char wd_smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;                       // 2 x 2 waves, 128 x 128 each
  const int xcd = blockIdx.x % 8, cu = blockIdx.x / 8, cus = gridDim.x / 8;

  // ---- this workgroup's tiles (the launcher checks divisibility, and that the numbers fit)
  const int tn = N / kWgBig, tm = M / kWgBig, per_group = tn * tm;
  // x / d for 0 <= x < 2^31 with inv = ceil(2^32 / d), d > 1: the product is less than half too large
  auto inverse = [](int d) { return d > 1 ? 0xFFFFFFFFu / static_cast<unsigned>(d) + 1u : 0u; };
  auto divide = [](int x, int d, unsigned inv) __attribute__((always_inline)) {
    if (d == 1) return x;
    const int q = static_cast<int>(__umulhi(static_cast<unsigned>(x), inv));
    return q * d > x ? q - 1 : q;
  };
  const int band_tiles = kWdBand * tn, last_rows = tm % kWdBand;
  const unsigned inv_band = inverse(band_tiles), inv_last = inverse(last_rows);
  // an XCD's part of an expert's tiles: the eighths are dealt in turn, since they differ by a tile
  auto share_lo = [&](int e) __attribute__((always_inline)) { return per_group * ((xcd + e) & 7) / 8; };
  auto share = [&](int e) __attribute__((always_inline)) { return per_group * (((xcd + e) & 7) + 1) / 8 - share_lo(e); };
  typedef const __attribute__((address_space(4))) int32_t const_i32_t;
  auto tile_at = [&](int e, int i) __attribute__((always_inline)) {
    while (e < n_groups && i >= share(e)) {
      i -= share(e);
      ++e;
    }
    WdTile t;
    t.e = e;
    t.i = i;
    t.m0 = t.n0 = t.p_lo = t.p_hi = 0;
    t.slabs = 1;
    if (e < n_groups) {
      const int at = share_lo(e) + i, band = divide(at, band_tiles, inv_band), in = at - band * band_tiles;
      const int rows = tm - band * kWdBand >= kWdBand ? kWdBand : last_rows;
      const int col = rows == kWdBand ? in / kWdBand : divide(in, rows, inv_last);
      t.m0 = (band * kWdBand + in - col * rows) * kWgBig;
      t.n0 = col * kWgBig;
      const_i32_t *off = (const_i32_t *)(reinterpret_cast<uintptr_t>(offsets));
      t.p_lo = offsets ? off[e] : 0;
      t.p_hi = offsets ? off[e + 1] : n_pos;
      t.slabs = t.p_hi > t.p_lo ? (t.p_hi - t.p_lo + kWgSlab - 1) / kWgSlab : 1;
    }
    return t;
  };
  auto behind = [&](const WdTile &t) __attribute__((always_inline)) { return tile_at(t.e, t.i + cus); };
  WdTile cur = tile_at(0, cu);
  if (cur.e >= n_groups) return;
  WdTile nxt = behind(cur);

  // ---- DMA side: instruction j of a half slab fills rows 16 wave + 2 j and + 1 of the slot; this lane brings 16 bytes
  // lane & 31 of row 2 j + (lane >> 5), i.e. the chunk that belongs there
  const lds_byte_t *lds = (const lds_byte_t *)wd_smem;
  const unsigned lds_base =
      static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void *)wd_smem));
  const unsigned half_mask = lane >> 5 ? 0xFFFFFFFFu : 0u;
  unsigned lane_col[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    lane_col[j] = static_cast<unsigned>(((lane & 31) ^ (4 * ((2 * j + (lane >> 5)) & 3))) * 16);
  const unsigned lda2 = static_cast<unsigned>(lda) * 2, ldb2 = static_cast<unsigned>(ldb) * 2;
  // workgroups that share an operand tile start on different rows of it
  const int wave_a = (wave + cu / kWdBand) & 3, wave_b = (wave + cu) & 3;
  const unsigned lds_a = lds_base + wave_a * (kWdInstr * 1024), lds_b = lds_base + wave_b * (kWdInstr * 1024);

  // where the requests are: a slab of a tile, and the tile behind it
  WdTile rq = cur, rq_next = nxt;
  int rq_slab = 0;
  auto request_next = [&]() __attribute__((always_inline)) {
    if (rq_slab + 1 < rq.slabs) {
      ++rq_slab;
    } else if (rq_next.e < n_groups) {
      rq = rq_next;
      rq_slab = 0;
      rq_next = behind(rq);
    }                                                          // behind the last tile: its last slab again, unused
  };
  // first of the 16 positions that a wave brings of a slab: moved down where they would reach past the last one
  auto first_pos = [&](const WdTile &t, int slab, int w) __attribute__((always_inline)) {
    const int p = t.p_lo + slab * kWgSlab + w * kWdRows;
    return p < n_pos - kWdRows ? p : n_pos - kWdRows;
  };
  auto row_numbers = [](const int32_t *rows, int p) __attribute__((always_inline)) {
    typedef const __attribute__((address_space(4))) i32x16_word_t const_i32x16_t;
    return static_cast<i32x16_t>(*(const_i32x16_t *)(reinterpret_cast<uintptr_t>(rows + p)));
  };
  i32x16_t idx_a, idx_b;                                       // rows of the half slab under way
  int pos_a = 0, pos_b = 0, col_a = 0, col_b = 0;
  auto fetch_a = [&]() __attribute__((always_inline)) {
    pos_a = first_pos(rq, rq_slab, wave_a);
    col_a = rq.m0 * 2;
    if constexpr (MAP_A) idx_a = row_numbers(rows_a, pos_a);
  };
  auto fetch_b = [&]() __attribute__((always_inline)) {
    pos_b = first_pos(rq, rq_slab, wave_b);
    col_b = rq.n0 * 2;
    if constexpr (MAP_B) idx_b = row_numbers(rows_b, pos_b);
  };
  // (the launcher checks that row * ld2 fits 32 bits)
  auto dma_a = [&](unsigned slot, int j) __attribute__((always_inline)) {
    const unsigned s0 = (MAP_A ? static_cast<unsigned>(idx_a[2 * j]) : static_cast<unsigned>(pos_a + 2 * j)) * lda2;
    const unsigned d = MAP_A ? static_cast<unsigned>(idx_a[2 * j + 1]) * lda2 - s0 : lda2;
    wd_dma_16(lds_a + slot * kWdSlotBytes + j * 1024, (half_mask & d) + (s0 + col_a) + lane_col[j & 1], A);
  };
  auto dma_b = [&](unsigned slot, int j) __attribute__((always_inline)) {
    const unsigned s0 = (MAP_B ? static_cast<unsigned>(idx_b[2 * j]) : static_cast<unsigned>(pos_b + 2 * j)) * ldb2;
    const unsigned d = MAP_B ? static_cast<unsigned>(idx_b[2 * j + 1]) * ldb2 - s0 : ldb2;
    wd_dma_16(lds_b + slot * kWdSlotBytes + j * 1024, (half_mask & d) + (s0 + col_b) + lane_col[j & 1], Bm);
  };

  // ---- MFMA side: lane i of a 16-lane group names row i >> 2 (of four), columns 4 (i & 3) .. + 3 of
  // its group's 16 columns and receives column i; groups 0/1 hold tile rows 0-15 / 16-31 of
  // positions 0-7, groups 2/3 the same of positions 8-15
  unsigned frag_off[4];
  {
    const int i16 = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int chunk = (i * 4 + 2 * (grp & 1) + ((i16 >> 1) & 1)) ^ (4 * (i16 >> 2));
      frag_off[i] = static_cast<unsigned>((8 * (grp >> 1) + (i16 >> 2)) * (kWgBig * 2) + chunk * 16 + (i16 & 1) * 8);
    }
  }
  f32x16_t acc[4][4];
  bf16x8_t fa0[4], fa1[4], fb0[4], fb1[4];
  auto read_a = [&](unsigned slot, int kk, int i) __attribute__((always_inline)) {
    return wd_frag(lds + (slot * kWdSlotBytes + wm * 256) + frag_off[i] + kk * (16 * kWgBig * 2));
  };
  auto read_b = [&](unsigned slot, int kk, int j) __attribute__((always_inline)) {
    return wd_frag(lds + (slot * kWdSlotBytes + wn * 256) + frag_off[j] + kk * (16 * kWgBig * 2));
  };
  // one 16-wide step on (fa, fb); (na, nb) receive the fragments of step kn of the slab in slots (sa, sb); dma(q) runs
  // behind MFMA q
  auto step = [&](auto zero, const bf16x8_t(&fa)[4], const bf16x8_t(&fb)[4], bf16x8_t(&na)[4], bf16x8_t(&nb)[4],
                  unsigned sa, unsigned sb, int kn, auto dma) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = i * 4 + j;
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
        else if (q <= 4) nb[q - 1] = read_b(sb, kn, q - 1);
        else if (q < 8) na[q - 4] = read_a(sa, kn, q - 4);
        dma(q);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  const auto mod5 = [](unsigned s) { return s >= 5 ? s - 5 : s; };
  using True = std::true_type;
  using False = std::false_type;
  const auto none = [](int) {};

  // what slab `slab` of tile t holds of positions that are not its own, both operands; ends in a barrier
  auto zero_rest = [&](const WdTile &t, int slab, unsigned sa, unsigned sb) __attribute__((always_inline)) {
    if (t.p_hi - t.p_lo - slab * kWgSlab >= kWgSlab) return;   // (whole slabs end before p_hi <= n_pos: nothing was moved)
    typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
    __attribute__((address_space(3))) unsigned char *smem = (__attribute__((address_space(3))) unsigned char *)wd_smem;
    for (int r = threadIdx.x >> 5; r < kWgSlab; r += 8) {
      const int w = r / kWdRows, p = first_pos(t, slab, w) + r % kWdRows;
      if (p < t.p_lo + slab * kWgSlab + w * kWdRows || p >= t.p_hi) {
        const unsigned at = r * (kWgBig * 2) + (threadIdx.x & 31) * 16;
        *(lds_u32x4_t *)(smem + sa * kWdSlotBytes + at) = u32x4_t{0u, 0u, 0u, 0u};
        *(lds_u32x4_t *)(smem + sb * kWdSlotBytes + at) = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  // ---- stores: a lane holds, for row lane & 31 of each 32-row block, columns 8 q + 4 (lane >> 5) + (0..3) of each
  // 32-column block in elements 4 q ..; lanes l and l + 16 trade rows between two neighbouring q, so that a store covers
  // 64 bytes of each of 16 rows
  constexpr int kBlockStores = 16;                             // per 32-row block
  const unsigned lane_out = ((wm * 128 + (lane & 15)) * static_cast<unsigned>(N) + wn * 128 + ((lane >> 4) & 1) * 8 + (lane >> 5) * 4) * 4;
  f32x4_wd_t held[kWdHeld][kBlockStores];
  float *held_at = nullptr;                                    // where the held blocks' tile starts (NULL: nothing held)
  auto piece = [&](int i, int k) __attribute__((always_inline)) {   // k: column block k / 4, 16 columns k / 2 % 2, rows k % 2
    const int j = k / 4, q = k / 2 % 2 * 2;
    f32x4_wd_t o;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][j][4 * q + r]),
                                                         __float_as_uint(acc[i][j][4 * q + 4 + r]), false, false);
      o[r] = __uint_as_float(rows[k % 2]);
    }
    return o;
  };
  auto store = [&](float *tile, int i, int k, f32x4_wd_t v) __attribute__((always_inline)) {
    char *at = reinterpret_cast<char *>(tile + static_cast<int64_t>(i * 32 + k % 2 * 16) * N + k / 4 * 32 + k / 2 % 2 * 16);
    unsigned l = lane_out;
    asm volatile("" : "+v"(l));                                // (an address per block and tile in registers otherwise: they spill)
    *reinterpret_cast<f32x4_wd_t *>(at + l) = v;
  };
  constexpr int kHeldStores = kWdHeld * kBlockStores, kHeldSlabs = kHeldStores / 4;
  auto store_held = [&](int k) __attribute__((always_inline)) {
    store(held_at, 4 - kWdHeld + k / kBlockStores, k % kBlockStores, held[k / kBlockStores][k % kBlockStores]);
  };

  // Scalar loads answer in any order: while one is on its way, every wait for a fragment is a wait for everything.  So they
  // go out behind a step's fragment reads, once these have arrived, and are used behind the fragment reads of the next step.
  auto lds_landed = []() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0xC07F); };   // lgkmcnt(0)

  // ---- fill the ring: A(0) B(0) A(1) B(1) A(2)
  fetch_a();
  fetch_b();
#pragma unroll
  for (unsigned m = 0; m < 3; ++m) {
#pragma unroll
    for (int j = 0; j < kWdInstr; ++j) dma_a(2 * m, j);
    if (m < 2) {
#pragma unroll
      for (int j = 0; j < kWdInstr; ++j) dma_b(2 * m + 1, j);
      request_next();
      fetch_a();
      if (m == 0) fetch_b();
    }
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * kWdInstr) : "memory");
  unsigned ra = 0;                                            // slot of A(m); B(m) and the next slabs follow it in the ring
  zero_rest(cur, 0, 0, 1);
  fa0[0] = read_a(0, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) fb0[j] = read_b(1, 0, j);
#pragma unroll
  for (int i = 1; i < 4; ++i) fa0[i] = read_a(0, 0, i);

  bool stored = false;                                        // the wait below has a tile's stores to let pass
  for (;;) {
    // slab 0: what it would request went out ahead of the previous tile's stores
    {
      const unsigned rb = mod5(ra + 1);
      step(True{}, fa0, fb0, fa1, fb1, ra, rb, 1, none);
      step(False{}, fa1, fb1, fa0, fb0, ra, rb, 2, none);
      step(False{}, fa0, fb0, fa1, fb1, ra, rb, 3, [&](int q) __attribute__((always_inline)) {
        if (q == 11) {
          lds_landed();
          fetch_b();
        }
      });
      lds_landed();
      // slab 1 has landed once only A(2), and the stores behind it, are outstanding
      if (stored)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kWdInstr + (4 - kWdHeld) * kBlockStores) : "memory");
      else
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kWdInstr) : "memory");
      asm volatile("s_barrier" ::: "memory");
    }
    const int slabs = cur.slabs;
    for (int m = 0; m < slabs - 1; ++m) {
      // slab m is in registers, slab m + 1 in LDS: the last step of m, then the first three of m + 1
      zero_rest(cur, m + 1, mod5(ra + 2), mod5(ra + 3));
      if (held_at != nullptr && m < kHeldSlabs) {
#pragma unroll
        for (int h = 0; h < kHeldSlabs; ++h)
          if (m == h) {
#pragma unroll
            for (int k = 0; k < 4; ++k) store_held(4 * h + k);
          }
      }
      {
        const unsigned r0 = ra;
        ra = mod5(ra + 2);
        step(False{}, fa1, fb1, fa0, fb0, ra, mod5(ra + 1), 0, [&](int q) __attribute__((always_inline)) {
          if (q % 4 == 3) dma_b(r0, q / 4);                   // B(m+2) into the slot of A(m)
        });
      }
      const unsigned rb = mod5(ra + 1);
      {
        const unsigned r0 = mod5(ra + 3);
        step(False{}, fa0, fb0, fa1, fb1, ra, rb, 1, [&](int q) __attribute__((always_inline)) {
          if (q % 4 == 3) dma_b(r0, 4 + q / 4);
          if (q == 11) {
            lds_landed();
            request_next();
            fetch_a();
          }
        });
      }
      {
        const unsigned r0 = mod5(ra + 4);
        step(False{}, fa1, fb1, fa0, fb0, ra, rb, 2, [&](int q) __attribute__((always_inline)) {
          if (q > 8 && q % 2 == 1) dma_a(r0, (q - 9) / 2);    // A(m+3) into the slot of B(m)
        });
        step(False{}, fa0, fb0, fa1, fb1, ra, rb, 3, [&](int q) __attribute__((always_inline)) {
          if (q % 4 == 3) dma_a(r0, 4 + q / 4);
          if (q == 11) {
            lds_landed();
            fetch_b();
          }
        });
      }
      lds_landed();
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kWdInstr) : "memory");
    }
    // the tile's last step: everything that slab 0 of the next tile would request goes before the stores
    if (held_at != nullptr) {
#pragma unroll
      for (int h = 0; h < kHeldSlabs; ++h)                     // few slabs: what is left
        if (slabs - 1 <= h) {
#pragma unroll
          for (int k = 0; k < 4; ++k) store_held(4 * h + k);
        }
    }
    const bool last = nxt.e >= n_groups;
    if (!last) zero_rest(nxt, 0, mod5(ra + 2), mod5(ra + 3));
    request_next();
    {
      const unsigned r0 = ra, r1 = mod5(ra + 1);
      ra = mod5(ra + 2);
      step(False{}, fa1, fb1, fa0, fb0, ra, mod5(ra + 1), 0, [&](int q) __attribute__((always_inline)) {
        if (q == 0) fetch_a();
        if (q < 8) dma_b(r0, q); else dma_a(r1, q - 8);
      });
    }
    float *tile = C + (static_cast<int64_t>(cur.e) * M + cur.m0) * N + cur.n0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < kBlockStores; ++k) {
        const f32x4_wd_t v = piece(i, k);
        if (i < 4 - kWdHeld) store(tile, i, k, v);
        else held[i - (4 - kWdHeld)][k] = v;
        if (k % 2) __builtin_amdgcn_sched_barrier(0);         // (registers: two pieces at a time)
      }
    held_at = tile;
    stored = true;
    if (last) break;
    cur = nxt;
    nxt = behind(cur);
  }
#pragma unroll
  for (int k = 0; k < kHeldStores; ++k) store_held(k);
  // no DMA may be in flight into LDS that the next workgroup on this CU owns
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// The contraction where one operand has at most 160 columns (the routed x and dt projections: dt_rank + 32 and dt_rank): all of
// them and TW columns of the wide one to a workgroup of TW / 32 wavefronts, which hold 32 wide columns each and every column of the
// thin operand, so that the wide operand is read once.  Bound by what a CU brings in.  Rows go into LDS as in the 256 x 256 kernel,
// three slabs of 64 positions under way and one being multiplied; the row numbers of a slab are on their way three slabs earlier still, into a
// copy per wavefront (its own count of requests covers them).  A row's chunks are permuted where its length would put four consecutive
// rows on the same banks (lengths of an odd number of 64 bytes need none).  The products are summed in the order of the kernels above.
// 16384 rows in 8 experts, 160 x 4096 80 -> 43 us and 4096 x 128 105 -> 36 (128 x 128 tiles, rows through registers); 8192 rows, 80 x 1536 29 -> 17.5
// and 1536 x 48 29 -> 14 (64 x 64 tiles).
constexpr int kWtSlots = 4, kWtMaxBlocks = 5;                // slabs in LDS; 32-column blocks of the thin operand
template <int CHUNKS>
__device__ __forceinline__ int wt_swizzle(int chunk, int row) {
  return CHUNKS % 16 == 0 ? chunk ^ (4 * (row & 3)) : CHUNKS % 8 == 0 ? chunk ^ (4 * ((row >> 1) & 1)) : chunk;
}
template <int PITCH>
__device__ __forceinline__ bf16x8_t wt_frag(const lds_byte_t *p) {
  typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
  const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(p));
  const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(p + 4 * PITCH));
  const i16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, v);
}
constexpr int wt_slab_bytes(int tw, int nb) { return kWgSlab * (tw + 32 * nb) * 2; }
constexpr int wt_smem(int tw, int nb) { return kWtSlots * (wt_slab_bytes(tw, nb) + tw / 32 * 2 * kWgSlab * 4); }

// grid: x tiles of TW wide columns, y groups.  THIN_A: C [n_groups][T][W], else [n_groups][W][T].
template <int TW, int NB, bool THIN_A>
__global__ __launch_bounds__(2 * TW) void wgrad_bf16_thin_kernel(
    const bf16_t *__restrict__ wide, int64_t ldw, int W, const int32_t *__restrict__ rows_w, const bf16_t *__restrict__ thin,
    int64_t ldt, int T, const int32_t *__restrict__ rows_t, const int32_t *__restrict__ offsets, int n_pos, float *__restrict__ C) {
  constexpr int NW = TW / 32, kThin = 32 * NB;
  constexpr int kWideInstr = 4, kThinInstr = 4 * NB / NW, kInstr = kWideInstr + kThinInstr;      // per wavefront and slab
  constexpr int kWidePitch = TW * 2, kThinPitch = kThin * 2, kWideBytes = kWgSlab * kWidePitch, kSlab = wt_slab_bytes(TW, NB);
  static_assert(4 * NB % NW == 0 && (kWtSlots & (kWtSlots - 1)) == 0, "whole instructions; slots are masked");
  extern __shared__ __attribute__((aligned(16))) unsigned char wt_smem_bytes[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = blockIdx.y, w0 = blockIdx.x * TW;
  const int p_lo = offsets ? offsets[e] : 0, p_hi = offsets ? offsets[e + 1] : n_pos;
  const int slabs = (p_hi - p_lo + kWgSlab - 1) / kWgSlab;
  lds_byte_t *lds = (lds_byte_t *)wt_smem_bytes;
  const unsigned lds_base = static_cast<unsigned>(reinterpret_cast<size_t>((__attribute__((address_space(3))) void *)wt_smem_bytes));
  constexpr int kNumbers = kWtSlots * kSlab;                   // then [wave][slot][operand][64] row numbers
  auto numbers_at = [&](int slab, int op) __attribute__((always_inline)) {
    return kNumbers + ((wave * kWtSlots + (slab & (kWtSlots - 1))) * 2 + op) * (kWgSlab * 4);
  };

  // ---- requests: lane l of instruction k of an operand brings chunk 64 k + l of its slab in LDS
  unsigned col_w[kWideInstr], col_t[kThinInstr];
  int row_w[kWideInstr], row_t[kThinInstr];
#pragma unroll
  for (int k = 0; k < kWideInstr; ++k) {
    const int g = (wave * kWideInstr + k) * 64 + lane, r = g / (TW / 8), c = w0 + wt_swizzle<TW / 8>(g % (TW / 8), r) * 8;
    row_w[k] = r;
    col_w[k] = static_cast<unsigned>(c < W ? c : 0) * 2;       // (columns past the end: some others, not stored)
  }
#pragma unroll
  for (int k = 0; k < kThinInstr; ++k) {
    const int g = (wave * kThinInstr + k) * 64 + lane, r = g / (kThin / 8), c = wt_swizzle<kThin / 8>(g % (kThin / 8), r) * 8;
    row_t[k] = r;
    col_t[k] = static_cast<unsigned>(c < T ? c : 0) * 2;
  }
  const unsigned ldw2 = static_cast<unsigned>(ldw) * 2, ldt2 = static_cast<unsigned>(ldt) * 2;
  auto position = [&](int slab, int r) __attribute__((always_inline)) {
    const int p = p_lo + slab * kWgSlab + r;
    return p < p_hi ? p : p_hi - 1;
  };
  auto request_numbers = [&](int slab) __attribute__((always_inline)) {
    const unsigned off = static_cast<unsigned>(position(slab, lane)) * 4;
    if (rows_w) wt_dma_4(lds_base + numbers_at(slab, 0), off, rows_w);
    if (rows_t) wt_dma_4(lds_base + numbers_at(slab, 1), off, rows_t);
  };
  typedef const __attribute__((address_space(3))) int lds_int_t;
  auto rows_of = [&](const int32_t *rows, int slab, int op, const auto &r, auto &out) __attribute__((always_inline)) {
    constexpr int kN = sizeof(out) / sizeof(out[0]);
    if (rows) {
#pragma unroll
      for (int k = 0; k < kN; ++k) out[k] = static_cast<unsigned>(*(lds_int_t *)(lds + numbers_at(slab, op) + r[k] * 4));
    } else {
#pragma unroll
      for (int k = 0; k < kN; ++k) out[k] = static_cast<unsigned>(position(slab, r[k]));
    }
  };
  // (the launcher checks that row * ld2 fits 32 bits)
  auto request = [&](int slab) __attribute__((always_inline)) {
    const unsigned at = lds_base + (slab & (kWtSlots - 1)) * kSlab;
    unsigned rw[kWideInstr], rt[kThinInstr];
    rows_of(rows_w, slab, 0, row_w, rw);
    rows_of(rows_t, slab, 1, row_t, rt);
#pragma unroll
    for (int k = 0; k < kWideInstr; ++k) wd_dma_16(at + (wave * kWideInstr + k) * 1024, rw[k] * ldw2 + col_w[k], wide);
#pragma unroll
    for (int k = 0; k < kThinInstr; ++k) wd_dma_16(at + kWideBytes + (wave * kThinInstr + k) * 1024, rt[k] * ldt2 + col_t[k], thin);
  };

  // ---- products: fragments as in the 256 x 256 kernel
  const int i16 = lane & 15, grp = lane >> 4, frow = 8 * (grp >> 1) + (i16 >> 2);
  const int fchunk = 2 * (grp & 1) + ((i16 >> 1) & 1), fbyte = (i16 & 1) * 8;
  const int off_w = frow * kWidePitch + wt_swizzle<TW / 8>(wave * 4 + fchunk, frow) * 16 + fbyte;
  int off_t[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) off_t[i] = kWideBytes + frow * kThinPitch + wt_swizzle<kThin / 8>(i * 4 + fchunk, frow) * 16 + fbyte;
  f32x16_t acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;

  if (slabs > 0) {
#pragma unroll
    for (int t = 0; t < kWtSlots; ++t) request_numbers(t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int t = 0; t < kWtSlots - 1; ++t) {
      if (t < slabs) request(t);
      if (t < kWtSlots - 2) request_numbers(t + kWtSlots);
    }
  }
  for (int t = 0; t < slabs; ++t) {
    // this slab has landed (requested two slabs and their row numbers ago), and with it the row numbers of slab t + 3;
    // every wavefront has multiplied the one before
    if (t + kWtSlots - 2 < slabs) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kWtSlots - 2) * kInstr) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int slot = (t & (kWtSlots - 1)) * kSlab;
    if (t == slabs - 1) {                                      // positions that are another group's, or nobody's
      const int valid = p_hi - p_lo - t * kWgSlab;
      typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
      for (int at = valid * kWidePitch + threadIdx.x * 16; at < kWideBytes; at += 2 * TW * 16)
        *(lds_u32x4_t *)(lds + slot + at) = u32x4_t{0u, 0u, 0u, 0u};
      for (int at = kWideBytes + valid * kThinPitch + threadIdx.x * 16; at < kSlab; at += 2 * TW * 16)
        *(lds_u32x4_t *)(lds + slot + at) = u32x4_t{0u, 0u, 0u, 0u};
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (t + kWtSlots - 1 < slabs) {
      request_numbers(t + 2 * kWtSlots - 2);
      request(t + kWtSlots - 1);
    }
#pragma unroll
    for (int kk = 0; kk < kWgSlab / 16; ++kk) {
      const bf16x8_t fw = wt_frag<kWidePitch>(lds + slot + off_w + kk * (16 * kWidePitch));
      bf16x8_t ft[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) ft[i] = wt_frag<kThinPitch>(lds + slot + off_t[i] + kk * (16 * kThinPitch));
#pragma unroll
      for (int i = 0; i < NB; ++i)
        acc[i] = THIN_A ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw, ft[i], acc[i], 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_32x32x16_bf16(ft[i], fw, acc[i], 0, 0, 0);
    }
  }
  // this lane holds, of output row lane & 31 of a block, the columns 8 q + 4 (lane / 32) + 0 .. 3 in elements 4 q ..
  // (both operands are whole pieces of eight columns)
  const int M = THIN_A ? T : W, N = THIN_A ? W : T;
  float *Ce = C + static_cast<int64_t>(e) * M * N;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int m = (THIN_A ? i * 32 : w0 + wave * 32) + (lane & 31);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cc = (THIN_A ? w0 + wave * 32 : i * 32) + q * 8 + (lane >> 5) * 4;
      if (m < M && cc < N)
        *reinterpret_cast<float4 *>(Ce + static_cast<int64_t>(m) * N + cc) =
            make_float4(acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]);
    }
  }
}

// rows scaled by a per-row factor (the gate weight of Eq. (12) on d_out):
// dst[r, :] = scale[scale_idx ? scale_idx[r] : r] * src[src_idx ? src_idx[r] : r, :]
// (top-K: r is a sorted position, src_idx its token, scale_idx its slot)
// (A row pass, row_place.)  16384 x 2048 30-36 us with four columns a thread and two index divisions, now 22-23; 8192 x 1024 7.9 -> 6.6;
// 32768 x 64 4.8 -> 4.7 (6.7 with a row a wavefront); fp32 32768 x 512 22.1 both (25 with 32 bytes a lane).
template <typename T, bool NARROW>
__global__ __launch_bounds__(256) void scale_rows_kernel(const T *__restrict__ src, const float *__restrict__ scale,
                                                         const int32_t *__restrict__ src_idx, const int32_t *__restrict__ scale_idx,
                                                         int64_t n_rows, int n_cols, int lanes_log2, T *__restrict__ dst) {
  constexpr int kCols = kRowCols<T>;
  int64_t r;
  int c;
  row_place<T, NARROW>(n_cols, lanes_log2, r, c);
  if (r >= n_rows || c >= n_cols) return;
  const int64_t rs = src_idx ? src_idx[r] : r, rg = scale_idx ? scale_idx[r] : r;
  const float g = scale[rg];
  float v[kCols];
#pragma unroll
  for (int q = 0; q < kCols; q += 4) bwd_load4(src + rs * n_cols + c + q, v + q);
#pragma unroll
  for (int q = 0; q < kCols; ++q) v[q] *= g;
#pragma unroll
  for (int q = 0; q < kCols; q += 4) bwd_store4(dst + r * n_cols + c + q, v + q);
}

// the same contraction on the plain ALUs (fp32, or bf16 shapes the MFMA kernel does not take): 64 x 64 tiles
template <typename T>
__global__ __launch_bounds__(256) void wgrad_simple_kernel(const T *__restrict__ A, int64_t lda, int M,
                                                           const T *__restrict__ Bm, int64_t ldb, int N,
                                                           const int32_t *__restrict__ rows_a,
                                                           const int32_t *__restrict__ rows_b,
                                                           const float *__restrict__ row_scale,
                                                           const int32_t *__restrict__ offsets, int64_t n_pos,
                                                           float *__restrict__ C) {
  __shared__ float As[16][64 + 4], Bs[16][64 + 4];
  const int e = blockIdx.z;
  const int64_t p_lo = offsets ? offsets[e] : 0, p_hi = offsets ? offsets[e + 1] : n_pos;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  float acc[4][4] = {};
  for (int64_t p0 = p_lo; p0 < p_hi; p0 += 16) {
    __syncthreads();
    for (int i = tid; i < 16 * 64; i += 256) {
      const int pp = i / 64, c = i % 64;
      const int64_t p = p0 + pp;
      float va = 0.0f, vb = 0.0f;
      if (p < p_hi) {
        const int64_t ra = rows_a ? rows_a[p] : p, rb = rows_b ? rows_b[p] : p;
        const float sc = row_scale ? row_scale[ra] : 1.0f;
        if (m0 + c < M) va = to_f32(A[ra * lda + m0 + c]) * sc;
        if (n0 + c < N) vb = to_f32(Bm[rb * ldb + n0 + c]);
      }
      As[pp][c] = va;
      Bs[pp][c] = vb;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { av[i] = As[k][ty * 4 + i]; bv[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
  }
  float *Ce = C + static_cast<int64_t>(e) * M * N;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty * 4 + i, col = n0 + tx * 4 + j;
      if (m < M && col < N) Ce[static_cast<int64_t>(m) * N + col] = acc[i][j];
    }
}

}  // namespace

size_t scan_bwd_ckpt_bytes(int64_t B, int64_t L, int d_inner) {
  return scan_bwd_layout(B, L, d_inner).total * sizeof(float);
}
size_t scan_bwd_part_bytes(int64_t n_tok, int d_inner) {
  return static_cast<size_t>(ceil_div(d_inner, kBwdCh)) * static_cast<size_t>(n_tok) * 32 * sizeof(float);
}

template <typename T>
static hipError_t launch_scan_backward_t(const void *u, const void *dt, const float *bc, const void *z, int64_t ld_z,
                                         const void *dg, const float *gate, const float *A_log, const float *D, int64_t B,
                                         int64_t L, int d_inner, float *ws, float *d_bc_part, void *d_pre, void *d_u,
                                         void *d_z, int64_t ld_dz, float *d_A_log, float *d_D, float *d_dt_bias,
                                         hipStream_t s) {
  const ScanBwdLayout l = scan_bwd_layout(B, L, d_inner);
  const bool chunked = l.n_chunks > 1;
  if (chunked) {
    const int gx = static_cast<int>(ceil_div(d_inner, 256));
    hipLaunchKernelGGL((scan_bwd_carry_kernel<T>), dim3(static_cast<unsigned>(B * l.n_chunks * gx)), dim3(256), 0, s,
                       static_cast<const T *>(u), static_cast<const T *>(dt), bc, static_cast<const T *>(z), ld_z,
                       static_cast<const T *>(dg), gate, A_log, L, d_inner, gx, l.n_chunks, l.chunk, ws + l.carry_q, ws + l.carry_r,
                       ws + l.carry_s);
    hipLaunchKernelGGL(scan_bwd_fold_kernel, dim3(static_cast<unsigned>(ceil_div(B * d_inner * 16, 256)), 2), dim3(256), 0, s,
                       A_log, B, d_inner, l.n_chunks, ws + l.carry_q, ws + l.carry_r, ws + l.carry_s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // more than 64 KiB of LDS: a function attribute, set once per device
  static std::mutex mu;
  static std::atomic<bool> done[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!done[dev].load(std::memory_order_acquire)) {
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev].load(std::memory_order_relaxed)) {
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&scan_bwd_kernel<T>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(sizeof(BwdSmem)));
      if (e != hipSuccess) return e;
      done[dev].store(true, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL((scan_bwd_kernel<T>), dim3(static_cast<unsigned>(l.n_units)), dim3(256), sizeof(BwdSmem), s,
                     static_cast<const T *>(u), static_cast<const T *>(dt), bc, static_cast<const T *>(z), ld_z,
                     static_cast<const T *>(dg), gate, A_log, D, B * L, L, d_inner, l.n_cb, l.n_chunks, l.chunk,
                     chunked ? ws + l.carry_q : nullptr, chunked ? ws + l.carry_r : nullptr, static_cast<T *>(d_pre),
                     static_cast<T *>(d_u), static_cast<T *>(d_z), ld_dz, d_bc_part, ws + l.part_a, ws + l.part_d,
                     ws + l.part_bias);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(scan_bwd_finish_kernel, dim3(static_cast<unsigned>(ceil_div(d_inner * 16, 256))), dim3(256), 0, s,
                     ws + l.part_a, ws + l.part_d, ws + l.part_bias, l.n_cb, d_inner, B * l.n_chunks, d_A_log, d_D, d_dt_bias);
  return hipGetLastError();
}

hipError_t launch_scan_backward(int dtype, const void *u, const void *dt, const float *bc, const void *z, int64_t ld_z,
                                const void *dg, const float *gate, const float *A_log, const float *D, int64_t B,
                                int64_t L, int d_inner, float *ckpt, float *d_bc_part, void *d_pre, void *d_u, void *d_z,
                                int64_t ld_dz, float *d_bc, float *d_A_log, float *d_D, float *d_dt_bias,
                                hipStream_t s) {
  const ScanBwdLayout l = scan_bwd_layout(B, L, d_inner);
  // 32-bit row offsets inside a chunk, rows of whole 32-byte pieces
  const int64_t widest = (ld_z > ld_dz ? ld_z : ld_dz) > d_inner ? (ld_z > ld_dz ? ld_z : ld_dz) : d_inner;
  if (l.n_units >= (1ll << 31) || widest * 4 * l.chunk >= (1ll << 32) || ld_z % 16 || ld_dz % 16) return hipErrorInvalidValue;
  hipError_t e = dtype == ROM_DTYPE_BF16
                     ? launch_scan_backward_t<bf16_t>(u, dt, bc, z, ld_z, dg, gate, A_log, D, B, L, d_inner, ckpt, d_bc_part,
                                                      d_pre, d_u, d_z, ld_dz, d_A_log, d_D, d_dt_bias, s)
                     : launch_scan_backward_t<float>(u, dt, bc, z, ld_z, dg, gate, A_log, D, B, L, d_inner, ckpt, d_bc_part,
                                                     d_pre, d_u, d_z, ld_dz, d_A_log, d_D, d_dt_bias, s);
  if (e != hipSuccess) return e;
  const int64_t n_tok = B * L;
  hipLaunchKernelGGL(bwd_reduce_bc_kernel, grid1d(n_tok * 32, 256), dim3(256), 0, s, d_bc_part, l.n_cb, n_tok, d_bc);
  return hipGetLastError();
}

hipError_t launch_gate_backward(int dtype, const void *a, const void *b, const int32_t *b_rows, int a_div,
                                int64_t n_rows, int n_cols, float *d_gate, hipStream_t s) {
  const dim3 grid = grid1d(n_rows * 64, 256);
  if (dtype == ROM_DTYPE_BF16)
    hipLaunchKernelGGL((gate_bwd_kernel<bf16_t>), grid, dim3(256), 0, s, static_cast<const bf16_t *>(a),
                       static_cast<const bf16_t *>(b), b_rows, a_div, n_rows, n_cols, d_gate);
  else
    hipLaunchKernelGGL((gate_bwd_kernel<float>), grid, dim3(256), 0, s, static_cast<const float *>(a),
                       static_cast<const float *>(b), b_rows, a_div, n_rows, n_cols, d_gate);
  return hipGetLastError();
}

// (no less for fewer tokens: a workspace of the largest call serves the smaller ones)
size_t router_bwd_partial_bytes(int64_t n_tok, int d_model, int n_experts) {
  const int64_t at_line = 8192 / router_chunk(8192), chunks = ceil_div(n_tok, router_chunk(n_tok));
  return static_cast<size_t>(chunks > at_line || n_tok <= 8192 ? chunks : at_line) * n_experts * (d_model + 1) * sizeof(float);
}

hipError_t launch_router_backward(int dtype, const float *logits, const int32_t *expert_idx, const float *d_gate,
                                  const void *x, int64_t n_tok, int d_model, int n_experts, int top_k, int gate_mode,
                                  float *d_logits, float *partial, float *d_w_router, float *d_b_router, hipStream_t s) {
#define ROM_ROUTER_BWD(EMAX) \
  hipLaunchKernelGGL(router_bwd_kernel<EMAX>, grid1d(n_tok, 64), dim3(64), 0, s, logits, expert_idx, d_gate, n_tok, n_experts, \
                     top_k, gate_mode, d_logits)
  if (n_experts <= 8) ROM_ROUTER_BWD(8);
  else if (n_experts <= 16) ROM_ROUTER_BWD(16);
  else ROM_ROUTER_BWD(64);
#undef ROM_ROUTER_BWD
  const int chunk = router_chunk(n_tok), n_chunks = static_cast<int>(ceil_div(n_tok, chunk));
  const dim3 grid(static_cast<unsigned>(ceil_div(d_model + 1, 512)), static_cast<unsigned>(n_chunks));
#define ROM_RW(T, EMAX)                                                                                       \
  hipLaunchKernelGGL((router_wgrad_partial_kernel<T, EMAX>), grid, dim3(256), 0, s, d_logits, static_cast<const T *>(x), \
                     n_tok, d_model, n_experts, chunk, partial)
  if (dtype == ROM_DTYPE_BF16) {
    if (n_experts <= 8) ROM_RW(bf16_t, 8); else if (n_experts <= 16) ROM_RW(bf16_t, 16); else ROM_RW(bf16_t, 64);
  } else {
    if (n_experts <= 8) ROM_RW(float, 8); else if (n_experts <= 16) ROM_RW(float, 16); else ROM_RW(float, 64);
  }
#undef ROM_RW
  hipLaunchKernelGGL(router_wgrad_finish_kernel, grid1d(static_cast<int64_t>(n_experts) * (d_model + 1), 64), dim3(kFinishWaves * 64), 0,
                     s, partial, n_chunks, d_model, n_experts, d_w_router, d_b_router);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_dx_finish_t(const T *dx_in, const float *d_logits, const T *w_router, int64_t n_tok, int d_model, int n_experts,
                                     T *d_x, hipStream_t s) {
  const int lg = row_lanes_log2<T>(d_model);
  const dim3 grid = row_grid<T>(ceil_div(n_tok, lg < 6 ? kDxRows<true> : kDxRows<false>), d_model);
  const auto kernel = lg < 6 ? &dx_finish_kernel<T, true> : &dx_finish_kernel<T, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, dx_in, d_logits, w_router, n_tok, d_model, n_experts, lg, d_x);
  return hipGetLastError();
}
hipError_t launch_dx_finish(int dtype, const void *dx_in, const float *d_logits, const void *w_router, int64_t n_tok,
                            int d_model, int n_experts, void *d_x, hipStream_t s) {
  if (dtype == ROM_DTYPE_BF16)
    return launch_dx_finish_t(static_cast<const bf16_t *>(dx_in), d_logits, static_cast<const bf16_t *>(w_router), n_tok, d_model, n_experts,
                              static_cast<bf16_t *>(d_x), s);
  return launch_dx_finish_t(static_cast<const float *>(dx_in), d_logits, static_cast<const float *>(w_router), n_tok, d_model, n_experts,
                            static_cast<float *>(d_x), s);
}

size_t conv_bwd_partial_bytes(int64_t B, int64_t L, int d_inner) {
  // a run is halved only while there are fewer than 4096 wavefronts, which leaves fewer than 8192: that bound grows with B and L
  // where the runs themselves do not, so that a workspace of the largest call serves the smaller ones
  const int64_t most = B * ceil_div(L, 16), cut = 8191 / ceil_div(d_inner, 128), whole = B * ceil_div(L, 128);
  const int64_t parts = whole > cut ? whole : most < cut ? most : cut;
  return static_cast<size_t>(parts) * 5 * d_inner * sizeof(float);
}

hipError_t launch_conv_backward(int dtype, const void *xz, int64_t ld_xz, const float *conv_w, const float *conv_b,
                                const void *du_a, const void *du_b, int64_t B, int64_t L, int d_inner, void *d_xpre,
                                int64_t ld_dx, float *partial, float *d_conv_w, float *d_conv_b, hipStream_t s) {
  const int run_steps = conv_bwd_run(B, L, d_inner);
  const int64_t n_runs = ceil_div(L, run_steps);
  const size_t eb = dtype == ROM_DTYPE_BF16 ? 2 : 4;
  const auto al = [&](const void *p) { return reinterpret_cast<uintptr_t>(p) % (2 * eb) == 0; };
  const bool two = d_inner % 2 == 0 && ld_xz % 2 == 0 && ld_dx % 2 == 0 && al(xz) && al(du_a) && al(du_b) && al(d_xpre);
  const dim3 grid(static_cast<unsigned>(ceil_div(d_inner, two ? 512 : 256)), static_cast<unsigned>(n_runs),
                  static_cast<unsigned>(B));
#define ROM_CONV_BWD(T, V)                                                                                          \
  hipLaunchKernelGGL((conv_bwd_kernel<T, V>), grid, dim3(256), 0, s, static_cast<const T *>(xz), ld_xz, conv_w, conv_b, \
                     static_cast<const T *>(du_a), static_cast<const T *>(du_b), L, d_inner, static_cast<T *>(d_xpre),  \
                     ld_dx, run_steps, partial)
  if (dtype == ROM_DTYPE_BF16) {
    if (two) ROM_CONV_BWD(bf16_t, 2); else ROM_CONV_BWD(bf16_t, 1);
  } else {
    if (two) ROM_CONV_BWD(float, 2); else ROM_CONV_BWD(float, 1);
  }
#undef ROM_CONV_BWD
  hipLaunchKernelGGL(conv_bwd_finish_kernel, grid1d(5 * d_inner, 64), dim3(kFinishWaves * 64), 0, s, partial, B * n_runs, d_inner,
                     d_conv_w, d_conv_b);
  return hipGetLastError();
}

namespace {
template <typename T>
TransposeJob<T> transpose_job(const void *src, void *dst, int n_mats, int rows, int cols) {
  const int vec = rows % 4 == 0 && cols % 4 == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0 &&
                  reinterpret_cast<uintptr_t>(dst) % 16 == 0;
  const int tr = static_cast<int>(ceil_div(rows, 64)), tc = static_cast<int>(ceil_div(cols, 64));
  return {static_cast<const T *>(src), static_cast<T *>(dst), rows, cols, vec, tr, tc, tr * tc * n_mats};
}
template <typename T>
hipError_t launch_transposes(const TransposeJob<T> &a, const TransposeJob<T> &b, hipStream_t s) {
  hipLaunchKernelGGL((transpose_kernel<T>), dim3(static_cast<unsigned>(a.blocks + b.blocks)), dim3(256), 0, s, a, b);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_transpose(int dtype, const void *src, void *dst, int n_mats, int rows, int cols, hipStream_t s) {
  if (dtype == ROM_DTYPE_BF16) return launch_transposes(transpose_job<bf16_t>(src, dst, n_mats, rows, cols), TransposeJob<bf16_t>{}, s);
  return launch_transposes(transpose_job<float>(src, dst, n_mats, rows, cols), TransposeJob<float>{}, s);
}

hipError_t launch_transpose2(int dtype, const void *src0, void *dst0, int rows0, int cols0, const void *src1, void *dst1, int rows1,
                             int cols1, int n_mats, hipStream_t s) {
  if (dtype == ROM_DTYPE_BF16)
    return launch_transposes(transpose_job<bf16_t>(src0, dst0, n_mats, rows0, cols0), transpose_job<bf16_t>(src1, dst1, n_mats, rows1, cols1), s);
  return launch_transposes(transpose_job<float>(src0, dst0, n_mats, rows0, cols0), transpose_job<float>(src1, dst1, n_mats, rows1, cols1), s);
}

hipError_t launch_pack_dxdbl(int dtype, const float *d_dt_low, const float *d_bc, int64_t n_tok, int dt_rank,
                             void *d_xdbl, hipStream_t s) {
  const dim3 grid = grid1d(n_tok * (dt_rank + 32), 256);
  if (dtype == ROM_DTYPE_BF16)
    hipLaunchKernelGGL((pack_dxdbl_kernel<bf16_t>), grid, dim3(256), 0, s, d_dt_low, d_bc, n_tok, dt_rank,
                       static_cast<bf16_t *>(d_xdbl));
  else
    hipLaunchKernelGGL((pack_dxdbl_kernel<float>), grid, dim3(256), 0, s, d_dt_low, d_bc, n_tok, dt_rank,
                       static_cast<float *>(d_xdbl));
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_scale_rows_t(const T *src, const float *scale, const int32_t *src_idx, const int32_t *scale_idx, int64_t n_rows,
                                      int n_cols, T *dst, hipStream_t s) {
  const int lg = row_lanes_log2<T>(n_cols);
  const auto kernel = lg < 6 ? &scale_rows_kernel<T, true> : &scale_rows_kernel<T, false>;
  hipLaunchKernelGGL(kernel, row_grid<T>(n_rows, n_cols), dim3(256), 0, s, src, scale, src_idx, scale_idx, n_rows, n_cols, lg, dst);
  return hipGetLastError();
}
hipError_t launch_scale_rows(int dtype, const void *src, const float *scale, const int32_t *src_idx,
                             const int32_t *scale_idx, int64_t n_rows, int n_cols, void *dst, hipStream_t s) {
  if (n_cols % 8 != 0) return hipErrorInvalidValue;       // (d_model is a multiple of 8)
  if (dtype == ROM_DTYPE_BF16)
    return launch_scale_rows_t(static_cast<const bf16_t *>(src), scale, src_idx, scale_idx, n_rows, n_cols, static_cast<bf16_t *>(dst), s);
  return launch_scale_rows_t(static_cast<const float *>(src), scale, src_idx, scale_idx, n_rows, n_cols, static_cast<float *>(dst), s);
}

namespace {
// ---- RMS norm of the pre-norm block, forward (materialised for the backward pass) and adjoint
// One wavefront per token row.  xn = x r norm_w, r = 1 / sqrt(mean(x^2) + eps), r kept per token.
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const T *__restrict__ x, const float *__restrict__ norm_w,
                                                          float eps, int64_t n_rows, int d_model, T *__restrict__ xn,
                                                          float *__restrict__ rstd) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const T *xr = x + row * d_model;
  float ss = 0.0f;
  for (int c = lane * 4; c < d_model; c += 256) {
    float v[4];
    bwd_load4(xr + c, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) ss = fmaf(v[q], v[q], ss);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  const float r = 1.0f / sqrtf(ss / static_cast<float>(d_model) + eps);
  if (lane == 0) rstd[row] = r;
  for (int c = lane * 4; c < d_model; c += 256) {
    float v[4];
    bwd_load4(xr + c, v);
    const float4 g = *reinterpret_cast<const float4 *>(norm_w + c);
    v[0] *= r * g.x; v[1] *= r * g.y; v[2] *= r * g.z; v[3] *= r * g.w;
    bwd_store4(xn + row * d_model + c, v);
  }
}

// d_x = d_skip + r (d_xn norm_w - x^ mean_d(d_xn norm_w x^)),  x^ = x r   (d_skip may be NULL: no skip connection)
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const T *__restrict__ x, const float *__restrict__ norm_w,
                                                          const float *__restrict__ rstd, const T *__restrict__ d_xn,
                                                          const T *__restrict__ d_skip, int64_t n_rows, int d_model,
                                                          T *__restrict__ d_x) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const T *xr = x + row * d_model, *dr = d_xn + row * d_model;
  const float r = rstd[row];
  float dot = 0.0f;
  for (int c = lane * 4; c < d_model; c += 256) {
    float v[4], dv[4];
    bwd_load4(xr + c, v);
    bwd_load4(dr + c, dv);
    const float4 g = *reinterpret_cast<const float4 *>(norm_w + c);
    dot = fmaf(dv[0] * g.x, v[0] * r, dot);
    dot = fmaf(dv[1] * g.y, v[1] * r, dot);
    dot = fmaf(dv[2] * g.z, v[2] * r, dot);
    dot = fmaf(dv[3] * g.w, v[3] * r, dot);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
  const float m = dot / static_cast<float>(d_model);
  for (int c = lane * 4; c < d_model; c += 256) {
    float v[4], dv[4], sk[4], o[4];
    bwd_load4(xr + c, v);
    bwd_load4(dr + c, dv);
    if (d_skip) bwd_load4(d_skip + row * d_model + c, sk);
    else sk[0] = sk[1] = sk[2] = sk[3] = 0.0f;
    const float4 g = *reinterpret_cast<const float4 *>(norm_w + c);
    o[0] = sk[0] + r * (dv[0] * g.x - v[0] * r * m);
    o[1] = sk[1] + r * (dv[1] * g.y - v[1] * r * m);
    o[2] = sk[2] + r * (dv[2] * g.z - v[2] * r * m);
    o[3] = sk[3] + r * (dv[3] * g.w - v[3] * r * m);
    bwd_store4(d_x + row * d_model + c, o);
  }
}

// d_norm_w partials: part[blockIdx.y][c] = sum over the block's rows of d_xn[n, c] x[n, c] r[n]; thread = column
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_wgrad_partial_kernel(const T *__restrict__ x,
                                                                    const float *__restrict__ rstd,
                                                                    const T *__restrict__ d_xn, int64_t n_rows,
                                                                    int d_model, int rows_per_block,
                                                                    float *__restrict__ part) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d_model) return;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n_rows ? r0 + rows_per_block : n_rows;
  float acc = 0.0f;
  for (int64_t n = r0; n < r1; ++n)
    acc = fmaf(to_f32(d_xn[n * d_model + c]) * to_f32(x[n * d_model + c]), rstd[n], acc);
  part[static_cast<int64_t>(blockIdx.y) * d_model + c] = acc;
}

// Both in one pass over x, d_xn and d_skip, for rows of up to 256 NP columns: a wavefront keeps a row in registers, with the next one on its
// way, and its columns' sums for d_norm_w over its rows (every fourth of the block's).  Bound by memory (268 MB, 5 TB/s): 16384 x 2048 51-54 us
// and 5 to add the parts up, in two passes 65-68, 26-31 and 21 (256 parts, four wavefronts for 64 columns).
template <typename T, int NP>
__global__ __launch_bounds__(256) void rmsnorm_bwd_rows_kernel(const T *__restrict__ x, const float *__restrict__ norm_w,
                                                               const float *__restrict__ rstd, const T *__restrict__ d_xn,
                                                               const T *__restrict__ d_skip, int64_t n_rows, int d_model,
                                                               int rows_per_block, T *__restrict__ d_x, float *__restrict__ part) {
  __shared__ float sums[4][NP * 256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < n_rows ? r0 + rows_per_block : n_rows;
  using Raw = std::conditional_t<sizeof(T) == 2, bwd_u32x2, bwd_f32x4>;
  struct Row {
    Raw x[NP], d[NP], s[NP];
    float r;
  };
  bool in[NP];
  float g[NP][4], acc[NP][4];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int c = p * 256 + lane * 4;
    in[p] = c < d_model;
    const float4 w = *reinterpret_cast<const float4 *>(norm_w + (in[p] ? c : 0));
    g[p][0] = w.x; g[p][1] = w.y; g[p][2] = w.z; g[p][3] = w.w;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[p][q] = 0.0f;
  }
  auto fetch = [&](int64_t row) __attribute__((always_inline)) {
    Row v;
    const int64_t at = (row < r1 ? row : r1 - 1) * d_model;
    v.r = rstd[row < r1 ? row : r1 - 1];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int64_t c = at + (in[p] ? p * 256 + lane * 4 : 0);
      v.x[p] = *reinterpret_cast<const Raw *>(x + c);
      v.d[p] = *reinterpret_cast<const Raw *>(d_xn + c);
      if (d_skip) v.s[p] = *reinterpret_cast<const Raw *>(d_skip + c);
    }
    return v;
  };
  auto unpack = [](const Raw &w, float (&f)[4]) __attribute__((always_inline)) {
    if constexpr (sizeof(T) == 2) {
      f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xFFFF0000u);
      f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xFFFF0000u);
    } else {
      f[0] = w.x; f[1] = w.y; f[2] = w.z; f[3] = w.w;
    }
  };
  Row next = fetch(r0 + wave);
  for (int64_t row = r0 + wave; row < r1; row += 4) {
    const Row cur = next;
    next = fetch(row + 4);
    const float r = cur.r;
    float dot = 0.0f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      float v[4], dv[4];
      unpack(cur.x[p], v);
      unpack(cur.d[p], dv);
      if (in[p]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          dot = fmaf(dv[q] * g[p][q], v[q] * r, dot);
          acc[p][q] = fmaf(dv[q] * v[q], r, acc[p][q]);
        }
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
    const float m = dot / static_cast<float>(d_model);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (!in[p]) continue;
      float v[4], dv[4], sk[4] = {0.f, 0.f, 0.f, 0.f}, o[4];
      unpack(cur.x[p], v);
      unpack(cur.d[p], dv);
      if (d_skip) unpack(cur.s[p], sk);
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = sk[q] + r * (dv[q] * g[p][q] - v[q] * r * m);
      bwd_store4(d_x + row * d_model + p * 256 + lane * 4, o);
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p)
    *reinterpret_cast<float4 *>(&sums[wave][p * 256 + lane * 4]) = make_float4(acc[p][0], acc[p][1], acc[p][2], acc[p][3]);
  __syncthreads();
  for (int c = threadIdx.x; c < d_model; c += 256)
    part[static_cast<int64_t>(blockIdx.x) * d_model + c] = (sums[0][c] + sums[1][c]) + (sums[2][c] + sums[3][c]);
}

// out[c] = sum over parts, 64 columns a workgroup (see kFinishWaves); a fixed order
__global__ __launch_bounds__(kFinishWaves * 64) void colsum_kernel(const float *__restrict__ part, int n_parts, int n_cols,
                                                                   float *__restrict__ out) {
  __shared__ float sums[kFinishWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane;
  float acc = 0.0f;
  if (c < n_cols) {
#pragma unroll 8
    for (int p = q; p < n_parts; p += kFinishWaves) acc += part[static_cast<int64_t>(p) * n_cols + c];
  }
  const float tot = finish_total(acc, sums, lane, q);
  if (q == 0 && c < n_cols) out[c] = tot;
}
}  // namespace

// at least 16 rows a part; two workgroups of the one-pass kernel per CU
int rmsnorm_wgrad_parts(int64_t n_rows) {
  const int64_t parts = (n_rows + 15) / 16;
  return static_cast<int>(parts < 512 ? (parts < 1 ? 1 : parts) : 512);
}

hipError_t launch_rmsnorm_forward(int dtype, const void *x, const float *norm_w, float eps, int64_t n_rows, int d_model,
                                  void *xn, float *rstd, hipStream_t s) {
  if (d_model % 4 != 0) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(ceil_div(n_rows, 4)));
  if (dtype == ROM_DTYPE_BF16)
    hipLaunchKernelGGL((rmsnorm_fwd_kernel<bf16_t>), grid, dim3(256), 0, s, static_cast<const bf16_t *>(x), norm_w, eps,
                       n_rows, d_model, static_cast<bf16_t *>(xn), rstd);
  else
    hipLaunchKernelGGL((rmsnorm_fwd_kernel<float>), grid, dim3(256), 0, s, static_cast<const float *>(x), norm_w, eps,
                       n_rows, d_model, static_cast<float *>(xn), rstd);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_rmsnorm_backward_t(const T *x, const float *norm_w, const float *rstd, const T *d_xn, const T *d_skip, int64_t n_rows,
                                     int d_model, T *d_x, float *part, float *d_norm_w, hipStream_t s) {
  const int parts = rmsnorm_wgrad_parts(n_rows);
  const int rows_per_block = static_cast<int>(ceil_div(n_rows, parts));
#define ROM_RMS_ROWS(NP)                                                                                                               \
  hipLaunchKernelGGL((rmsnorm_bwd_rows_kernel<T, NP>), dim3(static_cast<unsigned>(parts)), dim3(256), 0, s, x, norm_w, rstd, d_xn, d_skip, \
                     n_rows, d_model, rows_per_block, d_x, part)
  if (d_model <= 512) ROM_RMS_ROWS(2);
  else if (d_model <= 1024) ROM_RMS_ROWS(4);
  else if (d_model <= 1536) ROM_RMS_ROWS(6);
  else if (d_model <= 2048) ROM_RMS_ROWS(8);
#undef ROM_RMS_ROWS
  else {                                                       // a row does not fit the registers: two passes
    hipLaunchKernelGGL((rmsnorm_bwd_kernel<T>), dim3(static_cast<unsigned>(ceil_div(n_rows, 4))), dim3(256), 0, s, x, norm_w, rstd, d_xn,
                       d_skip, n_rows, d_model, d_x);
    hipLaunchKernelGGL((rmsnorm_wgrad_partial_kernel<T>), dim3(static_cast<unsigned>(ceil_div(d_model, 256)), static_cast<unsigned>(parts)),
                       dim3(256), 0, s, x, rstd, d_xn, n_rows, d_model, rows_per_block, part);
  }
  hipLaunchKernelGGL(colsum_kernel, dim3(static_cast<unsigned>(ceil_div(d_model, 64))), dim3(kFinishWaves * 64), 0, s, part, parts,
                     d_model, d_norm_w);
  return hipGetLastError();
}

hipError_t launch_rmsnorm_backward(int dtype, const void *x, const float *norm_w, const float *rstd, const void *d_xn,
                                   const void *d_skip, int64_t n_rows, int d_model, void *d_x, float *part,
                                   float *d_norm_w, hipStream_t s) {
  if (d_model % 4 != 0) return hipErrorInvalidValue;
  if (dtype == ROM_DTYPE_BF16)
    return launch_rmsnorm_backward_t(static_cast<const bf16_t *>(x), norm_w, rstd, static_cast<const bf16_t *>(d_xn),
                                     static_cast<const bf16_t *>(d_skip), n_rows, d_model, static_cast<bf16_t *>(d_x), part, d_norm_w, s);
  return launch_rmsnorm_backward_t(static_cast<const float *>(x), norm_w, rstd, static_cast<const float *>(d_xn),
                                   static_cast<const float *>(d_skip), n_rows, d_model, static_cast<float *>(d_x), part, d_norm_w, s);
}

template <int TW, int NB, bool THIN_A>
hipError_t launch_wgrad_thin(const bf16_t *wide, int64_t ldw, int W, const int32_t *rows_w, const bf16_t *thin, int64_t ldt, int T,
                             const int32_t *rows_t, const int32_t *offsets, int n_groups, int n_pos, float *C, hipStream_t s) {
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
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_bf16_thin_kernel<TW, NB, THIN_A>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, wt_smem(TW, NB));
      if (e != hipSuccess) return e;
      done[dev].store(true, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL((wgrad_bf16_thin_kernel<TW, NB, THIN_A>), dim3(static_cast<unsigned>(ceil_div(W, TW)), static_cast<unsigned>(n_groups)),
                     dim3(2 * TW), wt_smem(TW, NB), s, wide, ldw, W, rows_w, thin, ldt, T, rows_t, offsets, n_pos, C);
  return hipGetLastError();
}

hipError_t launch_wgrad(int dtype, const void *A, int64_t lda, int M, const void *Bm, int64_t ldb, int N,
                        const int32_t *rows_a, const int32_t *rows_b, const float *row_scale, const int32_t *offsets,
                        int n_groups, int64_t n_pos, float *C, hipStream_t s) {
  const bool mfma = dtype == ROM_DTYPE_BF16 && M % 8 == 0 && N % 8 == 0 && lda % 8 == 0 && ldb % 8 == 0 &&
                    reinterpret_cast<uintptr_t>(A) % 16 == 0 && reinterpret_cast<uintptr_t>(Bm) % 16 == 0;
  if (mfma && !row_scale && M % kWgBig == 0 && N % kWgBig == 0 && M > 0 && N > 0 && n_pos >= kWdRows &&
      n_pos < (1 << 30) && N <= (1 << 21) && ceil_div(M, kWgBig) * ceil_div(N, kWgBig) < (1 << 24) &&
      static_cast<uint64_t>(n_pos) * static_cast<uint64_t>(lda) * 2 < (1ull << 32) &&
      static_cast<uint64_t>(n_pos) * static_cast<uint64_t>(ldb) * 2 < (1ull << 32)) {
    // (operand rows are rows_x[p] < n_pos or p itself: 32-bit byte offsets reach every one of them)
    static std::mutex mu;
    static std::atomic<bool> done[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!done[dev].load(std::memory_order_acquire)) {
      std::lock_guard<std::mutex> lock(mu);
      if (!done[dev].load(std::memory_order_relaxed)) {
        const void *fns[4] = {reinterpret_cast<const void *>(&wgrad_bf16_dma_kernel<false, false>),
                              reinterpret_cast<const void *>(&wgrad_bf16_dma_kernel<false, true>),
                              reinterpret_cast<const void *>(&wgrad_bf16_dma_kernel<true, false>),
                              reinterpret_cast<const void *>(&wgrad_bf16_dma_kernel<true, true>)};
        for (const void *fn : fns) {
          e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kWdSmem);
          if (e != hipSuccess) return e;
        }
        done[dev].store(true, std::memory_order_release);
      }
    }
    auto kernel = rows_a ? (rows_b ? &wgrad_bf16_dma_kernel<true, true> : &wgrad_bf16_dma_kernel<true, false>)
                         : (rows_b ? &wgrad_bf16_dma_kernel<false, true> : &wgrad_bf16_dma_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(kWdWgs), dim3(256), kWdSmem, s, static_cast<const bf16_t *>(A), lda, M,
                       static_cast<const bf16_t *>(Bm), ldb, N, rows_a, rows_b, offsets, static_cast<int>(n_pos), n_groups, C);
    return hipGetLastError();
  }
  const bool thin_a = M <= N;
  const int T = thin_a ? M : N, W = thin_a ? N : M;
  if (mfma && !row_scale && T > 0 && T <= 32 * kWtMaxBlocks && n_pos > 0 && n_pos < (1 << 30) &&
      static_cast<uint64_t>(n_pos) * static_cast<uint64_t>(lda) * 2 < (1ull << 32) &&
      static_cast<uint64_t>(n_pos) * static_cast<uint64_t>(ldb) * 2 < (1ull << 32)) {
    const bf16_t *const a = static_cast<const bf16_t *>(A), *const b = static_cast<const bf16_t *>(Bm);
    const bool half = ceil_div(W, 128) * n_groups < kWgTileMinWgs;       // 64 wide columns where 128 would leave CUs without a workgroup
#define ROM_WT(TW, NB)                                                                                                                     \
  return thin_a ? launch_wgrad_thin<TW, NB, true>(b, ldb, W, rows_b, a, lda, T, rows_a, offsets, n_groups, static_cast<int>(n_pos), C, s)   \
                : launch_wgrad_thin<TW, NB, false>(a, lda, W, rows_a, b, ldb, T, rows_b, offsets, n_groups, static_cast<int>(n_pos), C, s)
#define ROM_WT_BLOCKS(NB)     \
  do {                        \
    if (half) ROM_WT(64, NB); \
    ROM_WT(128, NB);          \
  } while (0)
    if (T <= 64) ROM_WT_BLOCKS(2);
    if (T <= 96) ROM_WT_BLOCKS(3);
    if (T <= 128) ROM_WT_BLOCKS(4);
    ROM_WT_BLOCKS(5);
#undef ROM_WT_BLOCKS
#undef ROM_WT
  }
  if (mfma && !row_scale && M >= kWgBig && N >= kWgBig) {
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
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_bf16_big_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kWgBigSmem);
        if (e != hipSuccess) return e;
        done[dev].store(true, std::memory_order_release);
      }
    }
    const int64_t tiles = ceil_div(N, kWgBig) * ceil_div(M, kWgBig) * n_groups;
    const dim3 grid(static_cast<unsigned>(ceil_div(tiles, 8) * 8));
    hipLaunchKernelGGL(wgrad_bf16_big_kernel, grid, dim3(512), kWgBigSmem, s, static_cast<const bf16_t *>(A), lda, M,
                       static_cast<const bf16_t *>(Bm), ldb, N, rows_a, rows_b, offsets, n_pos, n_groups, C);
    return hipGetLastError();
  }
  if (mfma && !row_scale) {
    const bool small = ceil_div(N, kWgTile) * ceil_div(M, kWgTile) * n_groups < kWgTileMinWgs;
    const int tile = small ? kWgTile / 2 : kWgTile;
    const dim3 grid(static_cast<unsigned>(ceil_div(N, tile)), static_cast<unsigned>(ceil_div(M, tile)),
                    static_cast<unsigned>(n_groups));
    hipLaunchKernelGGL(small ? &wgrad_bf16_kernel<kWgTile / 2> : &wgrad_bf16_kernel<kWgTile>, grid, dim3(2 * tile), 0, s,
                       static_cast<const bf16_t *>(A), lda, M, static_cast<const bf16_t *>(Bm), ldb, N, rows_a, rows_b, offsets,
                       n_pos, C);
    return hipGetLastError();
  }
  const dim3 grid(static_cast<unsigned>(ceil_div(N, 64)), static_cast<unsigned>(ceil_div(M, 64)),
                  static_cast<unsigned>(n_groups));
  if (dtype == ROM_DTYPE_BF16)
    hipLaunchKernelGGL((wgrad_simple_kernel<bf16_t>), grid, dim3(256), 0, s, static_cast<const bf16_t *>(A), lda, M,
                       static_cast<const bf16_t *>(Bm), ldb, N, rows_a, rows_b, row_scale, offsets, n_pos, C);
  else
    hipLaunchKernelGGL((wgrad_simple_kernel<float>), grid, dim3(256), 0, s, static_cast<const float *>(A), lda, M,
                       static_cast<const float *>(Bm), ldb, N, rows_a, rows_b, row_scale, offsets, n_pos, C);
  return hipGetLastError();
}

}  // namespace rom
