// cx_kernels.hip -- gfx950 kernels of the batched EV charging-station step.
//
// One station occupies L lanes of a 64-wide wavefront and each lane holds P
// adjacent slots (L * P = the station's padded slot count); a wave carries 64 / L
// stations.  Slot s of a station lives in lane s / P, register s % P: blocks of up
// to P slots are summed inside a lane, and a lane's values of one feature are
// one 8- or 16-byte store (with slots L apart, P stores of 4 bytes).  A wave
// runs its stations for T steps with the whole state in registers and writes
// the per-step records out; the plain one-step form is the same kernel with
// T = 1.  Per step (App. A.2 order):
//   exogenous draws  (arrivals, price noise; computed L steps ahead, one step
//                     per lane, and broadcast -- they do not depend on the agent)
//   actions          (Philox levels / max / external)
//   apply actions    (clip by port max, charge curve, battery room)
//   projection       (Eq. ArchConst, deepest level first, butterfly sums over
//                     aligned power-of-two slot blocks: DPP inside a row,
//                     permlane swaps across rows, adds across registers; in the
//                     dense layout, one station-wide sum per node of a level)
//   charge, departures, arrivals (ballot + popcount ranks), reward, day end,
//   records (observations lane by lane, or, in the staged SIMPLE kernels,
//   through the block's LDS stage as 16-byte runs).
// Extended classes run their own kernels: V2G ports (signed levels, the
// mirrored discharge curve, two-sided limits, the split of the grid energy),
// a station battery (one FP64 scalar per station that every lane of the station
// updates alike), charge-sensitive users, per-episode price days and car
// models with AC / DC rates.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cx_device.h"
#include "cx_mlp.h"
#include "cx_internal.h"

namespace cx {
namespace {

// Arrivals of one step: thresholds exceeded by w in a row of 24 (and 8 of
// 0xFFFFFFFF).  The first four come in one 16-byte load, from the block's LDS
// copy of them where there is one; the rest are read only when w exceeds all
// four, from device memory and together: the wait for them is also one for the
// records in flight, and a bisection has five of them.
__device__ __forceinline__ int arrivals_after4(const uint32_t *row, uint32_t w) {
  const u32x4 *r = reinterpret_cast<const u32x4 *>(row);
  const u32x4 a = gld(r, 1), b = gld(r, 2);
  int m = 4 + (int)(w > a.x) + (int)(w > a.y) + (int)(w > a.z) + (int)(w > a.w) + (int)(w > b.x) + (int)(w > b.y) +
          (int)(w > b.z) + (int)(w > b.w);
  if (m == 12)
    for (int i = 12; i < kPoisK; ++i) m += (int)(w > gld(row, i));
  return m;
}
__device__ __forceinline__ int arrivals(const __attribute__((address_space(3))) u32x4 *first4, const uint32_t *row,
                                        uint32_t w) {
  u32x4 t;
  if (first4) t = *first4;
  else t = gld(reinterpret_cast<const u32x4 *>(row), 0);
  const int m = (int)(w > t.x) + (int)(w > t.y) + (int)(w > t.z) + (int)(w > t.w);
  return m < 4 ? m : arrivals_after4(row, w);
}

// Stay length of an arriving car: 1 + #{thresholds below w}, bisecting the
// table in LDS (staged by the block).
__device__ __forceinline__ int stay_len(const __attribute__((address_space(3))) uint32_t *t, int log2n, uint32_t w) {
  int pos = 0;
  for (int s = 1 << (log2n - 1); s >= 1; s >>= 1)
    if (t[pos + s - 1] < w) pos += s;
  return 1 + pos;
}

// Exchange with the lane whose index differs in bit K (K = 0..5), for use in
// butterfly all-reductions.  K = 0, 1: DPP quad permutes.  K = 2, 3: DPP
// mirrors of the half-row / row -- after the steps below K every lane of an
// aligned 2^K group holds the same value, so the mirror lane is as good as the
// XOR partner.  K = 4, 5: the gfx950 row-swap instructions (v_permlane16_swap /
// v_permlane32_swap, plain VALU, no LDS round trip) followed by a select of the
// half that came from the partner.
template <int K>
__device__ __forceinline__ float xlane(float v) {
  const int iv = __float_as_int(v);
  if constexpr (K == 0) return __int_as_float(__builtin_amdgcn_update_dpp(0, iv, 0xB1, 0xF, 0xF, false));
  if constexpr (K == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, iv, 0x4E, 0xF, 0xF, false));
  if constexpr (K == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, false));
  if constexpr (K == 3) return __int_as_float(__builtin_amdgcn_update_dpp(0, iv, 0x140, 0xF, 0xF, false));
  if constexpr (K == 4) {
    // rows (0,1,2,3): first result = (r0, r0, r2, r2), second = (r1, r1, r3, r3)
    const auto r = __builtin_amdgcn_permlane16_swap(iv, iv, false, false);
    return __int_as_float((__lane_id() & 16) ? r[0] : r[1]);
  }
  if constexpr (K == 5) {
    // halves (0,1): first result = (h0, h0), second = (h1, h1)
    const auto r = __builtin_amdgcn_permlane32_swap(iv, iv, false, false);
    return __int_as_float((__lane_id() & 32) ? r[0] : r[1]);
  }
  return v;
}

// The value of the lane whose index differs in bit K, whatever the lanes in
// between hold (xlane<2> and <3> take the mirrored lane, which holds the same
// only after the steps below K).
template <int K>
__device__ __forceinline__ float xor_lane(float v) {
  const int iv = __float_as_int(v);
  if constexpr (K == 2) {  // l ^ 7, then l ^ 3
    const int m = __builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, true);
    return __int_as_float(__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, true));
  } else if constexpr (K == 3) {  // rotate the row of 16 by 8
    return __int_as_float(__builtin_amdgcn_update_dpp(0, iv, 0x128, 0xF, 0xF, true));
  } else {
    return xlane<K>(v);
  }
}

// Exchange between lanes whose index differs in bit K: the lane with the bit clear
// gives its b for its partner's a, so that a then holds the lower lane's value and
// b the upper lane's, of a in the lower lane and of b in the upper one.
template <int K>
__device__ __forceinline__ void pair_swap(float &a, float &b) {
  if constexpr (K >= 4) {  // what the gfx950 row-swap instructions do
    const auto r = K == 4 ? __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false)
                          : __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float(r[0]);
    b = __int_as_float(r[1]);
  } else {
    const bool up = (__lane_id() >> K) & 1;
    const float got = xor_lane<K>(up ? a : b);
    a = up ? got : a;
    b = up ? b : got;
  }
}

// One butterfly step of a sum: v plus the value of the lane whose index
// differs in bit K.  K = 4, 5: the two halves the row-swap instruction leaves
// are exactly the pair to add (for a lane and its partner alike), so no select.
template <int K>
__device__ __forceinline__ float xsum(float v) {
  if constexpr (K == 4) {
    const int iv = __float_as_int(v);
    const auto r = __builtin_amdgcn_permlane16_swap(iv, iv, false, false);
    return __int_as_float(r[0]) + __int_as_float(r[1]);
  } else if constexpr (K == 5) {
    const int iv = __float_as_int(v);
    const auto r = __builtin_amdgcn_permlane32_swap(iv, iv, false, false);
    return __int_as_float(r[0]) + __int_as_float(r[1]);
  } else {
    return v + xlane<K>(v);
  }
}

// Sum over aligned groups of L lanes (every lane receives its group's sum).
template <int L>
__device__ __forceinline__ float station_sum(float v) {
  if constexpr (L > 1) v = xsum<0>(v);
  if constexpr (L > 2) v = xsum<1>(v);
  if constexpr (L > 4) v = xsum<2>(v);
  if constexpr (L > 8) v = xsum<3>(v);
  if constexpr (L > 16) v = xsum<4>(v);
  if constexpr (L > 32) v = xsum<5>(v);
  return v;
}

// xsum<K> for a K known only as a loop index of an unrolled loop.
template <int L>
__device__ __forceinline__ float xsum_k(float v, int K) {
  if (K == 0) return xsum<0>(v);
  if (K == 1) return xsum<1>(v);
  if (K == 2) return xsum<2>(v);
  if (K == 3) return xsum<3>(v);
  if (K == 4) return xsum<4>(v);
  return xsum<5>(v);
}

// Masked butterfly step: lanes whose block is smaller than 2^(K+1) send 0
// (a select, no branch; lb may vary per lane or be wave-uniform).
template <int K>
__device__ __forceinline__ float masked_step(float v, int lb) {
  const float u = (K < lb) ? v : 0.0f;
  return v + xlane<K>(u);
}

// Sums over aligned blocks of 2^lb lanes (a lane's block: lanes sharing the bits above lb).
template <int L>
__device__ __forceinline__ float block_sum_lanes(float v, int lb) {
  if constexpr (L > 1) v = masked_step<0>(v, lb);
  if constexpr (L > 2) v = masked_step<1>(v, lb);
  if constexpr (L > 4) v = masked_step<2>(v, lb);
  if constexpr (L > 8) v = masked_step<3>(v, lb);
  if constexpr (L > 16) v = masked_step<4>(v, lb);
  if constexpr (L > 32) v = masked_step<5>(v, lb);
  return v;
}

// The lanes of the wave in which b holds (a comparison's own result mask).
__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Four random action bytes from two Philox words: each 16-bit half h (low
// half first) gives (h n) >> 16, uniform over 0..n-1 up to 1 / 65536.
__device__ __forceinline__ uint32_t act_bytes(uint32_t wa, uint32_t wb, uint32_t n) {
  const uint32_t b0 = __umul24(wa & 0xFFFFu, n) >> 16, b1 = __umul24(wa >> 16, n) >> 16;
  const uint32_t b2 = __umul24(wb & 0xFFFFu, n) >> 16, b3 = __umul24(wb >> 16, n) >> 16;
  return b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
}

template <int L>
__device__ __forceinline__ int bcast(int v, int src) {
  if constexpr (L == 64) return __builtin_amdgcn_readlane(v, src);
  const int lane = __lane_id();
  return __builtin_amdgcn_ds_bpermute(((lane & ~(L - 1)) + src) << 2, v);
}
template <int L>
__device__ __forceinline__ float bcastf(float v, int src) {
  return __int_as_float(bcast<L>(__float_as_int(v), src));
}

struct Dyn {
  int32_t T, t_day0;
  uint32_t g0;
  int32_t mode, out_mode;
  float *obs;
  uint8_t *act;
  float *reward;
  uint8_t *done;
  const uint8_t *act_in;
  int64_t obs_stride, act_stride, env_stride;
  int32_t pace;         // 1: a step's records leave before the next step
};

// Store / load at a wave-uniform base plus a per-lane 32-bit byte offset
// (the global "saddr" form: no 64-bit address per lane).
template <class T>
__device__ __forceinline__ void st_at(T *base, uint32_t byte_off, T v) {
  typedef __attribute__((address_space(1))) T gT;
  typedef __attribute__((address_space(1))) char gchar;
  *(gT *)((gchar *)(char *)base + byte_off) = v;
}
template <class T>
__device__ __forceinline__ T gl_at(const T *base, uint32_t byte_off) {
  typedef const __attribute__((address_space(1))) T gT;
  typedef const __attribute__((address_space(1))) char gchar;
  return *(gT *)((gchar *)(const char *)base + byte_off);
}

// Observation records staged in LDS (SIMPLE classes).  Per step
// every lane puts its values in the block's stage (the adjacent envs of the
// block's waves, in record order); after the step barrier the block's running
// waves write the stage out as one contiguous run of 16-byte non-temporal
// stores.  HBM takes such whole-line streams much faster than the 4-byte
// stores of every lane, which leave lines partly written (for stations of 8
// lanes, 32 bytes per station and store).
typedef __attribute__((address_space(3))) float lds_float;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // at any float's address
typedef __attribute__((address_space(3))) f32x4u lds_f32x4u;
// P floats at any float's address
template <int P>
struct FVec;
template <>
struct FVec<1> { typedef float type; };
template <>
struct FVec<2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <>
struct FVec<4> { typedef f32x4u type; };
template <int P>
using fvec = typename FVec<P>::type;
template <class V>
__device__ __forceinline__ void set_at(V &x, int j, float v) {
  if constexpr (sizeof(V) == 4) x = v;
  else x[j] = v;
}

// Write n staged floats to dst (4-byte aligned).  The stage holds them from
// float pad = (dst / 4) mod 4 on, so that LDS and HBM agree on 16-byte chunks:
// the whole chunks go out as one 16-byte buffer store each (a resource over the
// 16-byte-aligned address dst - pad, offset 16 c for chunk c, non-temporal),
// the at most 3 floats before the first and after the last whole chunk one by
// one.  Lane 0 starts at the 128-byte line that holds dst (the chunks before
// dst, at most 7, are skipped), so that every wave's store covers whole lines:
// starting at dst itself, each 1 KiB store begins and ends inside a line, and
// HBM takes the two halves of a line from two non-temporal stores as two partial
// writes.  The mixture's record stream alone (five classes of 6.2-12.4 KB runs, 13.7 GB):
// 3.25 ms from dst, 2.86 from the line's start, 2.60 if every run were whole lines.
// tid / nthreads: this lane among the block's running lanes.
__device__ __forceinline__ void flush_stage(const lds_float *sb, float *dst, int pad, int n, int tid,
                                            int nthreads) {
  // chunk k counts from that line; [k_beg, k_end) are the whole chunks of the run
  const int phase = (int)((reinterpret_cast<uintptr_t>(dst) >> 4) & 7u);
  const int k_beg = phase + (pad ? 1 : 0), k_end = phase + ((pad + n) >> 2);
  // raw buffer: stride 0, range 2^31 - 1 bytes (offsets stay below 16 n + 192),
  // format word of a plain 32-bit buffer on gfx9-family GPUs
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<char *>(dst) - 4 * pad - 16 * phase, (short)0, 0x7fffffff, 0x00020000);
  const lds_float *line = sb - 4 * phase;  // (chunks below k_beg are not read)
  for (int k = tid; k < k_end; k += nthreads) {
    if (k < k_beg) continue;
    const f32x4 v = *reinterpret_cast<const lds_f32x4 *>(line + 4 * k);
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, 16 * k, 0, 2 /* nt */);
  }
  if (pad != 0 || ((pad + n) & 3) != 0) {  // the same in every lane
    const int head = (4 - pad) & 3;         // floats before the first whole chunk
    if (tid < head && tid < n) st_at(dst, 4u * (uint32_t)tid, (float)sb[pad + tid]);
    const int i = 4 * (k_end - phase) - pad + (tid - 4);  // lanes 4..7: the floats after the last whole chunk
    if (tid >= 4 && tid < 8 && i >= head && i < n) st_at(dst, 4u * (uint32_t)i, (float)sb[pad + i]);
  }
}

// SIMPLE: the class has no padding slots (slot s holds port s, N = L * P), one
// port maximum and efficiency, and per tree level one block size and one limit.
// Port indices and record offsets are then compile-time constants and every
// per-slot constant is wave-uniform (scalar registers).
// EXT: V2G ports, a station battery, charge-sensitive users, price days and / or
// car models (never SIMPLE); each switched on per class by a uniform flag.
// STAGE: observations through the block's LDS stage (SIMPLE classes): stage is the first
// buffer, the second stage_step floats on (0: one buffer, enough for a block of
// one wave), g_blk0 the block's first group and n_run the number of its waves
// that run.
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

// The fused policy rollout: after every step the block's staged observations
// (E = 32 envs, row stride obs_dim floats) go through the MLP on the matrix
// cores and each port gets its level for the next step, in LDS.  The products
// are those of the standalone policy kernel, K-step by K-step in the same
// order, so logits and levels are the same: the block's 4 waves split the
// hidden units (first product) and the port groups (second) among them, and
// each wave reads its weight fragments from device memory (L2) straight into
// the matrix-core operands.  K1 (K-steps of 32 features) and HP (K-steps of 32
// hidden units: 2, 4 or 8) are the class's and the policy's sizes rounded up;
// the second product's weights of the padding are zeros, so it adds exact zeros.
// LDS: hb (HP x 2 hidden-unit fragments, over the stage once it has been
// read), xb (the observations in BF16, 256 features per env, zero past in_dim,
// rows 33 fragments apart so that the 16 envs of a tile fall in different
// banks) and act (a level byte per port and env).  wv: this wave in the block;
// convert: the step left its observations in the FP32 stage; hid: the first
// product, its first fragments already asked for.  HELD (launches of at most one
// block per CU): both products' fragments and biases stay in registers for the
// whole rollout, those of the second in `held` (NG port groups a wave; HELD2) or
// a group's K-steps ahead in its ring, which then goes round over the steps.
template <int K1, int HP, int NT, bool HELD, bool HELD2, int DEPTH, int NG>
__device__ __forceinline__ void policy_phase(const LaunchArgs::Pol &pl, const lds_float *stage, lds_char *lds,
                                             int obs_dim, int N, int blk_envs, int wv, uint32_t env_id0,
                                             uint32_t g, uint32_t k0, uint32_t k1, bool convert,
                                             HiddenLayer<kPolRolloutWaves, NT, K1, HP, HELD> &hid,
                                             LogitLayer<NT, HP, HELD2, DEPTH> (&held)[NG]) {
  constexpr int W = kPolRolloutWaves, E = 16 * NT, CPR = 4 * K1;  // E envs; chunks of 8 per row
  const int lane = __lane_id(), col = lane & 15, lg = lane >> 4, tid = wv * 64 + lane;
  const int in_dim = pl.in_dim, G = pl.G, L1 = pl.L1;
  lds_u32x4 *xb = reinterpret_cast<lds_u32x4 *>(lds + pl.xb_off);
  lds_u32x4 *hb = reinterpret_cast<lds_u32x4 *>(lds + pl.hb_off);
  lds_u8 *act = reinterpret_cast<lds_u8 *>(lds + pl.act_off);
  // observations -> BF16 (features past in_dim and envs past the block's: 0).
  // Without observation records the step wrote its values straight into xb
  // (convert = false), whose padding the first conversion zeroed.
  if (convert) {
    for (int c = tid; c < E * CPR; c += 64 * W) {
      const int e = c / CPR, k = c % CPR, f = 8 * k;
      const lds_float *row = stage + e * obs_dim + f;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (e < blk_envs) {
        if (f + 8 <= in_dim) {
          const f32x4u x = *reinterpret_cast<const lds_f32x4u *>(row);
          const f32x4u y = *reinterpret_cast<const lds_f32x4u *>(row + 4);
          v = u32x4{pack2(x.x, x.y), pack2(x.z, x.w), pack2(y.x, y.y), pack2(y.z, y.w)};
        } else if (f < in_dim) {
          float x[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) x[j] = f + j < in_dim ? row[j] : 0.f;
          v = u32x4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
        }
      }
      xb[e * kPolXbRow + k] = v;
    }
    __syncthreads();
  }
  hid.run(frag_rsrc(pl.w1f, 2 * kPolHP * kPolK1), pl.b1, xb, kPolXbRow, hb, wv);
  const __amdgpu_buffer_rsrc_t w2 = frag_rsrc(pl.w2f, G * kPolR * kPolHP);
  LogitLayer<NT, HP, HELD2, DEPTH> &logit = held[0];
  if constexpr (!HELD) logit.start(w2, pl.b2f, min(wv, G - 1));
  // the lane's ports are 4 wv + lg + 16 i (group wv + 4 i): one Philox call per
  // env serves them all
  U4 dw[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
    dw[n] = philox(env_id0 + (uint32_t)(16 * n + col), g, draw_index(4 * wv + lg), kDomGum, k0, k1);
  __syncthreads();
  const auto draw_group = [&](int grp, LogitLayer<NT, HP, HELD2, DEPTH> &layer) {
    const int port = 4 * grp + lg;
    f32x4 c[kPolR][NT];
    layer.run(w2, pl.b2f, hb, grp, grp + W < G ? grp + W : HELD ? wv : -1, c);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int e = 16 * n + col;
      const f32x4 cn[kPolR] = {c[0][n], c[1][n], c[2][n]};
      const int lev = sample_level(cn, L1, draw_uniform(draw_word(dw[n], port)));
      if (port < N && e < blk_envs) act[e * N + port] = (uint8_t)lev;
    }
  };
  if constexpr (HELD2) {
#pragma unroll
    for (int i = 0; i < NG; ++i)
      if (wv + W * i < G) draw_group(wv + W * i, held[i]);
  } else {
    for (int grp = wv; grp < G; grp += W) draw_group(grp, logit);
  }
  __syncthreads();
}

// sg: the segment's descriptor; seg_args: take the horizon, clock, modes and
// record pointers from it (serving) instead of from the launch arguments.
// tdw: the block's LDS copy of the stay thresholds; exo_tp: its LDS
// copies of the first four arrival thresholds and the base price of every step
// of the day (NULL: read device memory); car_tab: of the car models' 8 thresholds
// and 8 x {capacity, AC rate, DC rate} (extended classes).
// HPOL: 0, or the fused policy rollout with HPOL K-steps of 32 hidden units; HELD:
// its weights stay in registers.
// MODE: what a kernel knows of the call: nothing, that it records no observations,
// or that it is one step (the loop, the draws ahead and the barrier fold away).
// One kernel for all held the registers of the longest: one step of a SIMPLE class
// needs 44-54 VGPRs (eight waves per SIMD), a rollout without observations 60-80.
// One step of 65,536 uneven stations 48.8 -> 44.5 us (46.3 -> 38.0 where state and
// records stay in the caches), of 64 stations 5.53 -> 5.22; of V2G ones, in the
// caches, 36.8 -> 32.0.  144 steps, rewards only: uneven 933 -> 833 us, V2G 820 -> 663,
// table-driven 768 -> 611; 288 steps of 20,011 uneven 526 -> 472.
enum { kModeAny = 0, kModeNoObs = 1, kModeStep = 2 };
template <int L, int P, bool SIMPLE, bool EXT, bool STAGE, int HPOL, bool HELD, int MODE, class Fill>
__device__ __forceinline__ void run_group(Fill &&fill_tables, CX_KONST SegDev *sgp, const Dyn &dy, int group,
                                          const lds_u32 *tdw,
                                          const lds_u32x4 *exo_tp,
                                          const lds_u32 *car_tab, lds_float *stage,
                                          int stage_step, int g_blk0, int n_run,
                                          const LaunchArgs::Pol *pol, lds_char *lds) {
  constexpr int SPW = 64 / L;
  constexpr int LOGP = P == 1 ? 0 : P == 2 ? 1 : 2;
  constexpr int LOGL = (L == 4) ? 2 : (L == 8) ? 3 : (L == 16) ? 4 : (L == 32) ? 5 : 6;
  constexpr bool NOPAD = SIMPLE;  // every slot holds a port: slot s = port s
  constexpr bool POL = HPOL > 0;
  CX_KONST SegDev &sg = *sgp;
  CX_KONST ClassDev *const cls = konst((const ClassDev *)sg.cls);
  CX_KONST ClassDev &C = *cls;
  const int lane = __lane_id();
  const int l = lane & (L - 1);
  const int sbase = lane & ~(L - 1);
  const int env = group * SPW + (lane >> LOGL);     // env index inside the segment
  const int n_envs = (int)sg.n_envs;
  const bool active = env < n_envs;
  const int S = NOPAD ? L * P : C.S;
  const int D = C.D;
  const int N = NOPAD ? L * P : C.n_ports;
  const int obs_dim = EXT ? C.obs_dim : 6 * N + 4;
  const int n_act = EXT ? C.n_act : N;      // action bytes per env
  const int n_neg = EXT ? C.n_neg : 0;      // discharge levels of a port
  const bool batt = EXT && C.has_batt != 0;
  const bool users = EXT && C.has_users != 0;  // some users are charge-sensitive
  const int n_days = EXT ? C.n_days : 0;       // exploring starts: price days
  const bool days = n_days > 0;
  const int n_models = EXT ? C.n_models : 0;   // car models (AC / DC rates)
  const bool models = n_models > 0;

  // Station sums of classes that are not SIMPLE, with several slots per lane, add
  // slots L apart first (see station_total): in the spread layout, register k of
  // lane l is slot k L + (l P mod L) + l P / L, the k-th of P such slots.
  constexpr bool SPREAD = !SIMPLE && !POL && P > 1;

  // ---- per-slot constants (the efficiencies in the spread layout where there is one)
  int port[P];
  float pmax[P], inv_pmax[P], inv_eta[P], lcap[kMaxLevels][P];
  float pdis[P], eta[P];  // EXT only
  uint32_t lbp[P];
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int s = l * P + j;
    [[maybe_unused]] const int spread_slot = SPREAD ? j * L + ((l * P) & (L - 1)) + (l * P) / L : s;
    port[j] = NOPAD ? s : gld(C.slot_port, s);
    if constexpr (SIMPLE) {
      pmax[j] = C.pmax_u;
      inv_pmax[j] = C.inv_pmax_u;
      inv_eta[j] = C.inv_eta_uniform;
      lbp[j] = C.lvl_lb_uniform;
#pragma unroll
      for (int d = 0; d < kMaxLevels; ++d) lcap[d][j] = C.lvl_cap_u[d];
    } else {
      pmax[j] = gld(C.slot_pmax, s);
      inv_pmax[j] = gld(C.slot_inv_pmax, s);
      inv_eta[j] = gld(C.slot_inv_eta, spread_slot);
      lbp[j] = gld(C.slot_lb, s);
#pragma unroll
      for (int d = 0; d < kMaxLevels; ++d) lcap[d][j] = d < D ? gld(C.slot_cap, d * S + s) : __builtin_inff();
    }
    if constexpr (EXT) {
      pdis[j] = gld(C.slot_pdis, s);
      eta[j] = gld(C.slot_eta, spread_slot);
    }
  }

  // ---- state
  double q[P];
  float qf[P];  // (float) q, kept in step with q: the FP32 work reads it
  float u[P], cap[P], icap[P], plast[P];
  int dw[P];
  int cs[P];  // EXT: 1 = a charge-sensitive user holds the slot (its dw may be <= 0)
  float rb[P];  // EXT: the car's maximum rate at this port (the port maximum without car models)
  int dc[P];    // EXT with car models: 1 = DC charger
  const int64_t sofs = (int64_t)env * S;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int64_t i = sofs + l * P + j;
    q[j] = active ? gld(sg.q, i) : 0.0;
    u[j] = active ? gld(sg.u, i) : 0.f;
    cap[j] = active ? gld(sg.cap, i) : 0.f;
    plast[j] = active ? gld(sg.p_last, i) : 0.f;
    dw[j] = active ? (int)gld(sg.dwell, i) : 0;
    cs[j] = (users && active) ? (int)gld(sg.utype, i) : 0;
    rb[j] = models ? (active ? gld(sg.rbar, i) : 0.f) : pmax[j];
    dc[j] = models ? gld(C.slot_dc, l * P + j) : 0;
  }
  double ret = active ? gld(sg.ret, env) : 0.0;
  // station battery (EXT): SoC in FP64 and last power, alike in every lane of the station
  double bsoc = 0.0;
  float bpw = 0.f;
  if constexpr (EXT) {
    if (batt && active) {
      bsoc = gld(sg.bsoc, env);
      bpw = gld(sg.bp, env);
    }
  }
  // the block's tables while the state is on its way
  fill_tables();
#pragma unroll
  for (int j = 0; j < P; ++j) {
    qf[j] = (float)q[j];
    icap[j] = cap[j] > 0.f ? frcp(cap[j]) : 0.f;
  }
  // The state is in registers before the first step: a load still pending when
  // the loop is entered would be waited for in every step, and with it the
  // records in flight.
#pragma unroll
  for (int j = 0; j < P; ++j) asm volatile("" ::"v"(u[j]), "v"(plast[j]), "v"(dw[j]), "v"(cs[j]), "v"(rb[j]), "v"(dc[j]));
  // the constants of every step, in scalar registers (the others are read where
  // they are used)
  const float dt = C.dt, inv_dt = C.inv_dt, inv_1mtau = C.inv_1mtau, inv_n_levels = C.inv_n_levels;
  const float p_sell = C.p_sell, p_sell_grid = C.p_sell_grid, fixed_cost = C.fixed_cost, alpha_dec = C.alpha_dec;
  const float inv_steps_ep = C.inv_steps_ep, inv_eta_u = C.inv_eta_uniform, alpha_sat = C.alpha_sat;
  const f32x4 *const glob = reinterpret_cast<const f32x4 *>(C.glob);
  // a slot is occupied while its car's stay runs, or while a charge-sensitive
  // user waits to be charged
#define CX_OCCUPIED(j) (EXT ? (dw[j] > 0 || cs[j] != 0) : dw[j] > 0)
  uint32_t bkp = 0u, bkq = 0u;  // EXT: the battery's action bytes of the current group of 8 steps
  // the levels of a SIMPLE class by block size (as a copy in scalar registers)
  constexpr int kBlk = LOGL + LOGP;
  [[maybe_unused]] float blk_cap[kBlk + 1];
  [[maybe_unused]] const uint32_t blk_mask = SIMPLE ? C.blk_mask : 0u;
  if constexpr (SIMPLE) {
#pragma unroll
    for (int k = 0; k < kBlk; ++k) blk_cap[k] = C.blk_cap[k];
  }
  // limit of the root (the whole station)
  const float c_root = D == 1 ? lcap[0][0] : D == 2 ? lcap[1][0] : D == 3 ? lcap[2][0] : lcap[3][0];

  const uint64_t seed = sg.seed;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const uint32_t env_id = (uint32_t)(sg.env0 + env);
  // the day clock is the same in every lane: kept in scalar registers, the
  // end-of-day reset is a branch, not selects in every step
  const int steps_ep = C.steps_ep;
  const int n_levels = C.n_levels;
  int t_day = uni(dy.t_day0);
  uint32_t g = dy.g0;
  int dday = 0;  // EXT: price day of the current episode (drawn at its first step)
  if constexpr (EXT) {
    if (days) dday = episode_day(env_id, g - (uint32_t)t_day, k0, k1, n_days);
  }
  int bM = 0, bdw = 1, bus = 0, bmod = 0;
  float bpb = 0.f, bcp = 0.f, bs0 = 0.f, btg = 0.f;
  [[maybe_unused]] float bpn = 0.f;  // price days: the base price after the step
  // SIMPLE stations of 64 ports and more, which often take two cars in a step:
  // the second car (rank 1) drawn ahead as well
  constexpr bool AHEAD2 = SIMPLE && L * P >= 64;
  int bdw1 = 1;

  float bcp1 = 0.f, bs01 = 0.f, btg1 = 0.f;
  // RANDOM: each slot's action bytes of the current group of 8 steps, one per
  // byte (steps 0-3 of the group in kp, 4-7 in kq)
  uint32_t kp[P], kq[P];
#pragma unroll
  for (int j = 0; j < P; ++j) kp[j] = kq[j] = 0u;
  const uint64_t smask = (L == 64) ? ~0ull : (((1ull << (L & 63)) - 1ull) << sbase);
  const uint64_t below_mask = (1ull << lane) - 1ull;

  // per-lane byte offsets of this env's records inside a step's segment block
  const uint32_t obs_bo = STAGE ? 0u : (uint32_t)env * (uint32_t)obs_dim * 4u;
  const uint32_t act_bo = (uint32_t)env * (uint32_t)n_act;
  const uint32_t env_bo = (uint32_t)env;
  // wave-uniform record pointers of the current step, advanced every step
  const bool w_obs = MODE != kModeNoObs && dy.out_mode == CX_OUT_FULL && dy.obs != nullptr;
  const bool w_act = (dy.out_mode == CX_OUT_FULL || dy.out_mode == CX_OUT_ACT_REWARD) && dy.act != nullptr;
  float *ob_t = w_obs ? dy.obs + sg.obs_off : nullptr;
  uint8_t *ab_t = w_act ? dy.act + sg.act_off : nullptr;
  const uint8_t *ai_t = dy.act_in ? dy.act_in + sg.act_off : nullptr;
  float *rw_t = dy.reward ? dy.reward + sg.env_off : nullptr;
  uint8_t *dn_t = dy.done ? dy.done + sg.env_off : nullptr;
  const int64_t obs_step = w_obs ? dy.obs_stride : 0;
  const int64_t act_step = (w_act || ai_t) ? dy.act_stride : 0;
  const int64_t env_step = (rw_t || dn_t) ? dy.env_stride : 0;
  // What the steps branch on, as bits of one scalar register that is read
  // afresh every step (a bit test and a scalar branch each).  Rewards and done
  // flags share their step: each is written under its own flag (with one of
  // them NULL, its advanced pointer is no address).
  enum : uint32_t { kWObs = 1, kWAct = 2, kWRew = 4, kWDone = 8, kActQuads = 16, kSat = 32, kRandom = 64, kMax = 128,
                    kDayTabs = 256, kBatt = 512, kUsers = 1024, kDays = 2048, kModels = 4096, kEtaU = 8192,
                    kPace = 16384 };
  const uint32_t flags0 =
      (uint32_t)uni((w_obs ? kWObs : 0) | (w_act ? kWAct : 0) | (rw_t ? kWRew : 0) | (dn_t ? kWDone : 0) |
                    // every step's action row is 4-byte aligned
                    (((reinterpret_cast<uintptr_t>(ab_t) | (uint64_t)act_step) & 3u) == 0 ? kActQuads : 0) |
                    (alpha_sat != 0.0f ? kSat : 0) | (dy.mode == CX_ACT_RANDOM ? kRandom : 0) |
                    (exo_tp ? kDayTabs : 0) | (w_obs && dy.pace ? kPace : 0) |
                    (batt ? kBatt : 0) | (users ? kUsers : 0) | (days ? kDays : 0) | (models ? kModels : 0) |
                    (!SIMPLE && !EXT && C.uniform_eta ? kEtaU : 0) |
                    (dy.mode == CX_ACT_MAX ? kMax : 0));
  // the block's LDS observation stage (staging packings, whenever observations
  // are written): the block's first env, the floats the block writes per step
  // and this lane's env in the stage
  const int env_blk0 = g_blk0 * SPW;
  const int blk_envs = min(n_envs - env_blk0, n_run * SPW);
  const int n_blk = blk_envs * obs_dim;
  const uint32_t stage_bo = (uint32_t)(env - env_blk0) * (uint32_t)obs_dim * 4u;
  // the fused policy: every wave of the block takes part (waves past the last
  // env too, their lanes inactive); the first step's levels come from the
  // observation the rollout starts from, put in the stage
  [[maybe_unused]] const int wv = group - g_blk0;
  [[maybe_unused]] const uint32_t env_id0 = (uint32_t)(sg.env0 + env_blk0);
  // K-steps of 32 features of the first product (a class of L P slots has at most
  // 6 L P + 4 features)
  constexpr int kPolSteps1 = (6 * L * P + 4 + 31) / 32;
  [[maybe_unused]] const auto w1_rsrc = [&] { return frag_rsrc(pol->w1f, 2 * kPolHP * kPolK1); };
  constexpr int NT = POL ? kPolRolloutWaves * SPW / 16 : 1, HP = POL ? HPOL : 2;  // 16-env tiles of the block
  // port groups of a wave, and whether the second product's fragments of all of
  // them fit in the registers beside the step (96 of them; at 32 slots and 256
  // hidden units they would take 192, and spill)
  constexpr bool DUAL = POL && policy_dual(L * P, HELD);
  constexpr int kGroups = L * P > 16 ? L * P / 16 : 1;
  constexpr bool HELD2 = HELD && kGroups * HP <= 8;
  constexpr int NG = HELD2 ? kGroups : 1;
  [[maybe_unused]] HiddenLayer<kPolRolloutWaves, NT, kPolSteps1, HP, HELD> held1;
  [[maybe_unused]] LogitLayer<NT, HP, HELD2, HELD ? HP : kRing> held2[NG];
  if constexpr (POL) {
    const float *src = pol->obs0 + sg.obs_off + (int64_t)env_blk0 * obs_dim;
    for (int i = wv * 64 + lane; i < n_blk; i += kPolRolloutWaves * 64) stage[i] = gld(src, i);
    held1.start(w1_rsrc(), pol->b1, wv);
    if constexpr (HELD) {
#pragma unroll
      for (int i = 0; i < NG; ++i)
        held2[i].start(frag_rsrc(pol->w2f, pol->G * kPolR * kPolHP), pol->b2f,
                       min(wv + kPolRolloutWaves * i, pol->G - 1));
    }
    __syncthreads();
    policy_phase(*pol, stage, lds, obs_dim, N, blk_envs, wv, env_id0, g, k0, k1, true, held1, held2);
  }

  // every lane's P slots hold P adjacent ports (no padding slots)
  [[maybe_unused]] const bool adjacent = NOPAD || S == N;
  // With four slots per lane a class with padding slots stores the observations of
  // the lanes whose ports are adjacent at once too, the others' one by one: stored one
  // by one from all lanes, 16 bytes apart, 96 steps of 20,000 31-port stations at 8
  // lanes took 734 us, so 546 (583 with slots L apart).  (With two slots, 8 bytes
  // apart, the test costs what it saves.)
  constexpr bool SOME = P == 4 && !NOPAD && !POL;
  [[maybe_unused]] bool whole = SOME && !adjacent;
  if constexpr (SOME) {
#pragma unroll
    for (int j = 0; j < P; ++j) whole = whole && port[j] >= 0 && port[j] == port[0] + j;
  }
  // (from LDS: a load from device memory would wait for the records in flight)
  [[maybe_unused]] auto car_model = [&](uint32_t w) {
    int m = 0;
    for (int i = 0; i < n_models; ++i) m += w > car_tab[i] ? 1 : 0;
    return m;
  };
  [[maybe_unused]] auto car_data = [&](int i) { return __uint_as_float(car_tab[8 + i]); };
  [[maybe_unused]] int k_in[P] = {};   // EXTERNAL: the next step's action bytes
  [[maybe_unused]] int kb_in = 0;
  const int T = MODE == kModeStep ? 1 : uni(dy.T);
  [[maybe_unused]] const uint32_t lvl_lb0 = C.lvl_lb_uniform, dense0 = C.dense_nodes;
  [[maybe_unused]] const int D0 = D;
  for (int t = 0; t < T; ++t, ++g) {
    uint32_t flags = flags0;
    asm volatile("" : "+s"(flags));
    // what the step tests, by bits and by slots: a test made ahead of the loop
    // holds a mask of two scalar registers, and the masks spilled to vector lanes
    [[maybe_unused]] uint32_t levels = blk_mask, lvl_lb = lvl_lb0, dense = dense0;
    [[maybe_unused]] int D = D0;
    if constexpr (SIMPLE) {
      // (at 8 lanes and fewer the masks fit: 0.266 ms a day of 400 stations so, 0.285
      // bit by bit; at 16 0.288 against 0.275, at 64 with two slots 0.50 / 0.46)
      if constexpr (L > 8) asm volatile("" : "+s"(levels));
    } else {
      asm volatile("" : "+s"(lvl_lb), "+s"(dense), "+s"(D));
#pragma unroll
      for (int j = 0; j < P; ++j) asm volatile("" : "+v"(lbp[j]));
    }
    [[maybe_unused]] const bool batt = EXT && (flags & kBatt), users = EXT && (flags & kUsers),
                                days = EXT && (flags & kDays), models = EXT && (flags & kModels);
    // ---- exogenous draws for the next L steps, lane l -> step t + l: the
    // arrival count, the price noise and the first arriving car's profile
    if ((t & (L - 1)) == 0) {
      CX_KONST ClassDev &C = *reload(cls);  // (constants of the draws: not held across the steps)
      int td = t_day + l;
      while (td >= steps_ep) td -= steps_ep;
      const uint32_t gl = g + (uint32_t)l;
      const U4 w = philox(env_id, gl, 0u, kDomEnv, k0, k1);
      bM = active ? arrivals(flags & kDayTabs ? exo_tp + td : nullptr, C.tpois + td * kPoisStride, w.x) : 0;
      const float u1 = (float)((w.y >> 8) + 1u) * 0x1p-24f;
      const float u2 = u24(w.z);
      const float z = __builtin_amdgcn_sqrtf(-2.0f * __logf(u1)) * __builtin_amdgcn_cosf(u2);
      float base;
      if (flags & kDayTabs) {
        base = reinterpret_cast<const lds_float *>(exo_tp + steps_ep)[td];
      } else {
        // wait for the load here, where it is issued: a load still pending
        // where the two paths join would make every step wait for all the
        // records in flight
        base = gld(C.glob, td * 4 + 2);
        asm volatile("" ::"v"(base));
      }
      if constexpr (EXT) {
        if (days) {
          // the price of this step and of the one after it (its observation's),
          // which is the first of the next day's when this is the day's last
          const int day = episode_day(env_id, gl - (uint32_t)td, k0, k1, n_days);
          int day1 = day, td1 = td + 1;
          if (ballot(td1 == steps_ep)) {
            const int next = episode_day(env_id, gl + 1u, k0, k1, n_days);
            day1 = td1 == steps_ep ? next : day;
            td1 = td1 == steps_ep ? 0 : td1;
          }
          base = gld(C.price_days, day * steps_ep + td);
          bpn = gld(C.price_days, day1 * steps_ep + td1);
          asm volatile("" ::"v"(base), "v"(bpn));  // (waited for here, not in every step)
        }
      }
      bpb = base + C.price_sigma * z;
      const U4 b = philox(env_id, gl, 0u, kDomCar, k0, k1);
      bcp = C.cap_lo + C.cap_span * u24(b.x);
      if constexpr (EXT) {
        if (models) {  // the car's model fixes its capacity
          bmod = car_model(b.x);
          bcp = car_data(3 * bmod);
        }
      }
      bs0 = C.soc_lo + C.soc_span * u24(b.y);
      btg = C.tgt_lo + C.tgt_span * u24(b.z);
      bdw = stay_len(tdw, C.dwell_log2, b.w);
      if constexpr (EXT) {
        if (users) bus = philox(env_id, gl, 0u, kDomUser, k0, k1).x <= C.cs_thresh ? 1 : 0;
      }
      if constexpr (AHEAD2) {
        if (ballot(bM >= 2)) {  // some step ahead brings a second car
          const U4 b1 = philox(env_id, gl, 1u, kDomCar, k0, k1);
          bcp1 = C.cap_lo + C.cap_span * u24(b1.x);
          bs01 = C.soc_lo + C.soc_span * u24(b1.y);
          btg1 = C.tgt_lo + C.tgt_span * u24(b1.z);
          bdw1 = stay_len(tdw, C.dwell_log2, b1.w);
        }
      }
    }
    const int tb = t & (L - 1);
    const int M = bcast<L>(bM, tb);
    const float pbuy = bcastf<L>(bpb, tb);
    [[maybe_unused]] float p_next = 0.f;
    if constexpr (EXT) {
      if (days) p_next = bcastf<L>(bpn, tb);
    }
    // the observation's time features of the step after this one (a scalar
    // load, issued early; it does not wait for the records in flight)
    const int t_obs = t_day + 1 == steps_ep ? 0 : t_day + 1;
    const f32x4 gl = sld(glob, t_obs);

    // ---- actions: action bytes k (level + n_neg)
    int k[P];
    int kb = 0;  // the battery's action byte (level + n_levels)
    if constexpr (POL) {  // the levels the policy drew after the last step
      const lds_u8 *lv = reinterpret_cast<const lds_u8 *>(lds + pol->act_off) + (env - env_blk0) * N;
#pragma unroll
      for (int j = 0; j < P; ++j) k[j] = active && (NOPAD || port[j] >= 0) ? (int)lv[port[j]] : 0;
    } else if (flags & kRandom) {
      if (t == 0 || (g & 7u) == 0) {
        // one Philox call gives the 8 steps' bytes: its 16-bit halves (low
        // half first) scaled to the n byte values, (h n) >> 16; n <= 255, so
        // the product is exact in a 24-bit multiply.  Action bytes are at most
        // 254 (n_levels <= 254; 127 with discharging).
        const uint32_t nk = (uint32_t)(n_levels + n_neg + 1);
#pragma unroll
        for (int j = 0; j < P; ++j) {
          const U4 w = philox(env_id, g >> 3, (uint32_t)port[j], kDomAct, k0, k1);
          kp[j] = act_bytes(w.x, w.y, nk);
          kq[j] = act_bytes(w.z, w.w, nk);
        }
        if constexpr (EXT) {
          if (batt) {
            const U4 w = philox(env_id, g >> 3, (uint32_t)N, kDomAct, k0, k1);
            const uint32_t nb = (uint32_t)(2 * n_levels + 1);
            bkp = act_bytes(w.x, w.y, nb);
            bkq = act_bytes(w.z, w.w, nb);
          }
        }
      }
      // the step's byte (wave-uniform selection of register and byte)
      const bool hi4 = (g & 4u) != 0;
      const uint32_t sh = 8u * (g & 3u);
#pragma unroll
      for (int j = 0; j < P; ++j) k[j] = (int)__builtin_amdgcn_ubfe(hi4 ? kq[j] : kp[j], sh, 8);
      if constexpr (EXT) kb = (int)__builtin_amdgcn_ubfe(hi4 ? bkq : bkp, sh, 8);
    } else if (flags & kMax) {
#pragma unroll
      for (int j = 0; j < P; ++j) k[j] = n_levels + n_neg;
      kb = 2 * n_levels;
    } else {
      // this step's bytes were asked for a step ago (the wait for them is then
      // no wait for the records of this step); the next step's are asked for now
      // (SIMPLE classes: a lane's bytes at once, at any address)
      typedef uint16_t __attribute__((aligned(1))) u16a1;
      typedef uint32_t __attribute__((aligned(1))) u32a1;
#define CX_ASK(row)                                                                                    \
  do {                                                                                                 \
    if constexpr (NOPAD && P == 2) {                                                                   \
      k_in[0] = active ? (int)gl_at((const u16a1 *)(row), act_bo + (uint32_t)port[0]) : 0;             \
    } else if constexpr (NOPAD && P == 4) {                                                            \
      k_in[0] = active ? (int)gl_at((const u32a1 *)(row), act_bo + (uint32_t)port[0]) : 0;             \
    } else {                                                                                           \
      _Pragma("unroll") for (int j = 0; j < P; ++j)                                                    \
          k_in[j] = active && port[j] >= 0 ? (int)gl_at(row, act_bo + (uint32_t)port[j]) : 0;          \
    }                                                                                                  \
    if constexpr (EXT) kb_in = batt && active ? (int)gl_at(row, act_bo + (uint32_t)N) : 0;             \
  } while (0)
      if (t == 0) CX_ASK(ai_t);
#pragma unroll
      for (int j = 0; j < P; ++j)
        k[j] = min(NOPAD && P > 1 ? (int)__builtin_amdgcn_ubfe((uint32_t)k_in[0], 8 * j, 8) : k_in[j], n_levels + n_neg);
      if constexpr (EXT) kb = min(kb_in, 2 * n_levels);
      if (t + 1 < T) CX_ASK(ai_t + act_step);
#undef CX_ASK
    }

    // ---- apply actions: clip by request, charge curve, battery room; a
    // discharging port (EXT) by its discharge maximum, the charging curve
    // mirrored about SoC 1/2 and the energy stored
    float pw[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const float req = (float)k[j] * inv_n_levels * pmax[j];
      const float rhat = pmax[j] * fminf(1.0f, qf[j] * inv_1mtau);
      const float room = qf[j] * cap[j] * inv_dt;
      if constexpr (EXT) {
        const float crate = rb[j] * fminf(1.0f, qf[j] * inv_1mtau);   // the car's curve
        float p;
        if (n_neg != 0) {
          const int lev = k[j] - n_neg;
          const float soc = (float)(1.0 - q[j]);
          const float creq = (float)lev * inv_n_levels * pmax[j];
          const float dreq = (float)(-lev) * inv_n_levels * pdis[j];
          const float drate = rb[j] * fminf(1.0f, soc * inv_1mtau);
          const float stored = soc * cap[j] * inv_dt;
          p = lev >= 0 ? fminf(fminf(creq, crate), room) : -fminf(fminf(dreq, drate), stored);
        } else {
          p = fminf(fminf(req, crate), room);
        }
        pw[j] = CX_OCCUPIED(j) ? p : 0.0f;
      } else {
        pw[j] = dw[j] > 0 ? fminf(fminf(req, rhat), room) : 0.0f;
      }
    }

    // Sum over the station of one value per slot.  With one slot per lane, in
    // SIMPLE classes and in the fused policy: adjacent slots first (slot bits from
    // the lowest up, the order of one slot per lane in every packing).  The general
    // and extended kinds with two or four slots per lane add the slots L apart
    // first, in order, then the L sums from the lowest bit up: the order they have
    // always summed in, on which a charge-sensitive user's departure at a near-tie,
    // and with it every later record, can depend.
    [[maybe_unused]] auto spread = [&](const float (&v)[P], float (&w)[P]) {
#pragma unroll
      for (int j = 0; j < P; ++j) w[j] = v[j];
      if constexpr (P == 2) {
        pair_swap<LOGL - 1>(w[0], w[1]);
      } else if constexpr (P == 4) {
        pair_swap<LOGL - 1>(w[0], w[2]);
        pair_swap<LOGL - 1>(w[1], w[3]);
        pair_swap<LOGL - 2>(w[0], w[1]);
        pair_swap<LOGL - 2>(w[2], w[3]);
      }
    };
    // ... of the L sums, one per lane in the spread layout
    [[maybe_unused]] auto spread_sum = [&](float v) {
      if constexpr (P == 4) v += xor_lane<LOGL - 2>(v);
      if constexpr (P > 1) v += xor_lane<LOGL - 1>(v);
      return station_sum<L / P>(v);
    };
    auto station_total = [&](const float (&v)[P]) {
      if constexpr (P == 1) {
        return station_sum<L>(v[0]);
      } else if constexpr (P == 2 && SPREAD) {
        const float a = v[0] + xor_lane<LOGL - 1>(v[0]), b = v[1] + xor_lane<LOGL - 1>(v[1]);
        return station_sum<L / 2>(a + b);
      } else if constexpr (SPREAD) {
        float w[P];
        spread(v, w);
        return spread_sum(((w[0] + w[1]) + w[2]) + w[3]);
      } else if constexpr (P == 2) {
        return station_sum<L>(v[0] + v[1]);
      } else {
        return station_sum<L>((v[0] + v[1]) + (v[2] + v[3]));
      }
    };

    // ---- projection onto the capacity tree (Eq. ArchConst), deepest level
    // first; the root (level D-1) holds the whole station
    float e_net, e_grid, e_out = 0.f;
    if constexpr (SIMPLE) {
      // Every node of a level owns an aligned block of 2^k slots, k the same for
      // the whole level.  One butterfly over the station's slots holds, after k
      // exchange steps, the load of each block of 2^k slots, already scaled by
      // the levels below (a scaled block contributes its limit); so each level
      // is checked when its block size is reached.  A slot's final factor is
      // the product of the factors of the nodes on its path.
      // Blocks smaller than a lane's P slots (rare: such trees take a path of
      // their own) have a factor per slot, which the larger ones' then multiply, as
      // with one slot per lane (a slot's factors from the deepest node up); without
      // them all factors are the lane's.
      float F[P], r;
      auto limit = [&](float &load, float &f, float c) {
        const bool over = load > c;
        f = over ? f * (c * frcp(load)) : f;
        load = over ? c : load;
      };
      // the levels of blocks of P slots and more; factor(c): one of them, of limit c
      auto climb = [&](auto factor) {
#pragma unroll
        for (int k = 0; k < LOGL; ++k) {
          if ((levels >> (k + LOGP)) & 1u) {  // a level of blocks of P 2^k slots (wave-uniform)
            // a real (scalar) branch: most sizes have no level, and computing the
            // check for every one and selecting would cost more than it saves
            asm volatile("");
            factor(blk_cap[k + LOGP]);
          }
          r = xsum_k<L>(r, k);
        }
      };
      if (P > 1 && (levels & ((1u << LOGP) - 1u))) {
        float v[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
          v[j] = pw[j];
          F[j] = 1.0f;
          if (levels & 1u) limit(v[j], F[j], blk_cap[0]);
        }
        if constexpr (P == 2) {
          r = v[0] + v[1];
        } else if constexpr (P == 4) {
          float lo = v[0] + v[1], hi = v[2] + v[3];
          if (levels & 2u) {
            float fl = 1.0f, fh = 1.0f;
            limit(lo, fl, blk_cap[1]);
            limit(hi, fh, blk_cap[1]);
            F[0] *= fl; F[1] *= fl; F[2] *= fh; F[3] *= fh;
          }
          r = lo + hi;
        } else {
          r = v[0];
        }
        climb([&](float c) {
          float g = 1.0f;
          limit(r, g, c);
#pragma unroll
          for (int j = 0; j < P; ++j) F[j] *= g;
        });
      } else {
        if constexpr (P == 1) r = pw[0];
        if constexpr (P == 2) r = pw[0] + pw[1];
        if constexpr (P == 4) r = (pw[0] + pw[1]) + (pw[2] + pw[3]);
        float f = 1.0f;
        climb([&](float c) { limit(r, f, c); });
#pragma unroll
        for (int j = 0; j < P; ++j) F[j] = f;
      }
      // the root: the whole station, delivered energy its scaled load (App. A.3)
      const float tot = r;
      const bool over = tot > c_root;
      const float fr = over ? c_root * frcp(tot) : 1.0f;
#pragma unroll
      for (int j = 0; j < P; ++j) pw[j] *= F[j] * fr;
      e_net = dt * (over ? c_root : tot);
      e_grid = e_net * inv_eta_u;
    } else {
#pragma unroll
    for (int d = 0; d < kMaxLevels - 1; ++d) {
      if (d < D - 1) {
        float s[P];
        const int lbu = (int)((lvl_lb >> (8 * d)) & 0xFF);
        const int nd = (int)((dense >> (8 * d)) & 0xFF);
        if (nd != 0) {
          // dense layout: at most 4 nodes on this level, each summed over the
          // whole station from the slots it covers
#pragma unroll
          for (int j = 0; j < P; ++j) s[j] = 0.f;
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            if (m < nd) {
              const uint32_t code = 0x80u | (uint32_t)m;
              float in[P];
#pragma unroll
              for (int j = 0; j < P; ++j) in[j] = ((lbp[j] >> (8 * d)) & 0xFFu) == code ? pw[j] : 0.f;
              const float acc = station_total(in);
#pragma unroll
              for (int j = 0; j < P; ++j) s[j] = ((lbp[j] >> (8 * d)) & 0xFFu) == code ? acc : s[j];
            }
          }
        } else if (lbu != 0xFF && lbu >= LOGP) {  // every slot of the level sits in a block of 2^lbu slots
          float v = pw[0];
          if constexpr (P == 2) v = pw[0] + pw[1];
          if constexpr (P == 4) v = (pw[0] + pw[1]) + (pw[2] + pw[3]);
          v = block_sum_lanes<L>(v, lbu - LOGP);
#pragma unroll
          for (int j = 0; j < P; ++j) s[j] = v;
        } else {
          // block sizes differ from slot to slot (a block's own slots agree):
          // first inside the lane, then over the lanes of blocks wider than it
          int lb[P];
#pragma unroll
          for (int j = 0; j < P; ++j) {
            lb[j] = (int)((lbp[j] >> (8 * d)) & 0xFF);
            s[j] = pw[j];
          }
          if constexpr (P >= 2) {
            const float a = s[0] + s[1];
            s[0] = lb[0] > 0 ? a : s[0];
            s[1] = lb[1] > 0 ? a : s[1];
          }
          if constexpr (P == 4) {
            const float b = s[2] + s[3];
            s[2] = lb[2] > 0 ? b : s[2];
            s[3] = lb[3] > 0 ? b : s[3];
            const float a = s[0] + s[2];
            const bool quad = lb[0] > 1;
#pragma unroll
            for (int j = 0; j < P; ++j) s[j] = quad ? a : s[j];
          }
#pragma unroll
          for (int j = 0; j < P; ++j) s[j] = block_sum_lanes<L>(s[j], lb[j] - LOGP);
        }
#pragma unroll
        for (int j = 0; j < P; ++j) {
          const float c = lcap[d][j];
          if constexpr (EXT) {
            const float a = fabsf(s[j]);   // the limit bounds the magnitude of the net power
            pw[j] = a > c ? pw[j] * (c * frcp(a)) : pw[j];
          } else {
            pw[j] = s[j] > c ? pw[j] * (c * frcp(s[j])) : pw[j];
          }
        }
      }
    }
    // root: the station total before root scaling; the delivered energy is its
    // scaled value (App. A.3, charging only)
    // The grid energy (a product per slot) and the root's sum before it are taken
    // in the spread layout: a lane adds its products by fused multiply-adds, one
    // rounding a slot, and every lane of the station then adds the same sums.
    // (Products left to be added across lanes would be fused into the exchange's sum
    // on one side only; each rounded first, the energy's root-mean-square error against
    // 64 bits, in a simulation of both sums, is 1.5 % larger at 16 ports and two
    // slots per lane, 0.3-0.8 % at 64-256 ports.)
    [[maybe_unused]] float w[P];
    float tot;
    if constexpr (SPREAD) {
      spread(pw, w);
      tot = w[0] + w[1];
      if constexpr (P == 4) tot = (tot + w[2]) + w[3];
      tot = spread_sum(tot);
    } else {
      tot = station_total(pw);
    }
    const float mag = EXT ? fabsf(tot) : tot;
    const bool over = mag > c_root;
    const float f = over ? c_root * frcp(mag) : 1.0f;
#pragma unroll
    for (int j = 0; j < P; ++j) pw[j] *= f;
    e_net = dt * (over ? (EXT ? copysignf(c_root, tot) : c_root) : tot);
    // station sum of c(k, w) w over the slots' powers w; c(k, .) the factor of the
    // lane's k-th slot in the layout of w; fused: false adds rounded products
    [[maybe_unused]] auto weighted = [&](auto c, [[maybe_unused]] bool fused) {
#pragma clang fp contract(off)
      if constexpr (SPREAD) {
        float v = w[0] * c(0, w[0]);
#pragma unroll
        for (int k = 1; k < P; ++k) v = fused ? __builtin_fmaf(w[k], c(k, w[k]), v) : v + w[k] * c(k, w[k]);
        return spread_sum(v);
      } else {
        float v[P];
#pragma unroll
        for (int j = 0; j < P; ++j) v[j] = pw[j] * c(j, pw[j]);
        return station_total(v);
      }
    };
    if constexpr (SPREAD) {
#pragma unroll
      for (int k = 0; k < P; ++k) w[k] *= f;
    }
    if constexpr (EXT) {
      // grid energy: charging ports draw e / eta, discharging ports return eta e
      e_grid = dt * weighted([&](int k, float p) { return p > 0.f ? inv_eta[k] : eta[k]; }, true);
      if (C.alpha_dc != 0.0f) e_out = dt * weighted([&](int k, float p) { return p < 0.f ? eta[k] : 0.f; }, false);
    } else if (flags & kEtaU) {
      e_grid = e_net * inv_eta_u;
    } else {
      e_grid = dt * weighted([&](int k, float) { return inv_eta[k]; }, true);
    }
    }  // projection of classes that are not SIMPLE

    // ---- the station battery (EXT): the (N+1)-th pole at the grid
    // connection, same curves, FP64 like the cars' q
    float e_b = 0.f;
    if constexpr (EXT) {
      if (batt) {
        const int lev = kb - n_levels;
        const double sb = bsoc;
        double pb;
        if (lev >= 0) {
          const double req = (double)lev * C.inv_n_d * C.b_rate;
          const double rhat = C.b_rate * fmin(1.0, (1.0 - sb) * C.b_inv_1mtau);
          const double room = (1.0 - sb) * C.b_cap * C.inv_dt_d;
          pb = fmin(fmin(req, rhat), room);
        } else {
          const double req = (double)(-lev) * C.inv_n_d * C.b_rate;
          const double rhat = C.b_rate * fmin(1.0, sb * C.b_inv_1mtau);
          const double stored = sb * C.b_cap * C.inv_dt_d;
          pb = -fmin(fmin(req, rhat), stored);
        }
        const double eb = C.dt_d * pb;
        const double ns = sb + eb * C.b_inv_cap;
        bsoc = ns > 1.0 ? 1.0 : (ns < 0.0 ? 0.0 : ns);
        bpw = (float)pb;
        e_b = (float)eb;
      }
    }

    // ---- charge, departures (selects: no branches): a time-sensitive user
    // leaves when its stay ends (c_satisfaction,0: energy still wanted), a
    // charge-sensitive one (EXT) when no energy is wanted any more
    // (c_satisfaction,1: hours overstayed - beta x hours left early)
    float csat = 0.f, csat1 = 0.f;
    float missed[P] = {}, moved[P] = {};
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const bool occ = CX_OCCUPIED(j);              // (pw = 0 on empty slots)
      const float e = dt * pw[j];
      const double nq = q[j] - (double)(e * icap[j]);
      q[j] = nq > 0.0 ? nq : 0.0;
      if constexpr (EXT) q[j] = q[j] < 1.0 ? q[j] : 1.0;  // discharging never below SoC 0
      qf[j] = (float)q[j];
      plast[j] = pw[j];
      dw[j] -= occ ? 1 : 0;
      bool dep = occ && dw[j] == 0;
      bool dep0 = dep;  // a time-sensitive user leaves
      if constexpr (EXT) {
        if (users) {
          const bool csu = cs[j] != 0;
          dep = occ && (csu ? q[j] <= (double)u[j] : dw[j] == 0);
          dep0 = dep && !csu;
          const float tl = (float)dw[j] * dt;
          moved[j] = (dep && csu) ? fmaxf(0.0f, -tl) - C.beta_sat1 * fmaxf(0.0f, tl) : 0.0f;
          cs[j] = dep ? 0 : cs[j];
          dw[j] = dep ? 0 : dw[j];   // a charged user may leave with steps of its stay left
        }
      }
      if (flags & kSat) {  // energy still wanted by a departing car (c_satisfaction,0)
        const float miss = fmaxf(0.0f, (qf[j] - u[j]) * cap[j]);
        missed[j] = dep0 ? miss : 0.0f;
      }
      // (an empty slot keeps its last car's values: its power and every feature
      // are masked by its being empty, an arrival overwrites them, and the state
      // goes back to HBM as zeros)
    }
    if (flags & kSat) csat = station_total(missed);
    if constexpr (EXT) {
      if (users && C.alpha_sat1 != 0.0f) csat1 = station_total(moved);
    }

    // ---- arrivals: first free ports in port order take the accepted cars
    int rej = 0;
    if (ballot(M > 0)) {
      bool fr[P];
      int n_free = 0, below = 0;   // free slots of the station, and of its lanes before this one
#pragma unroll
      for (int j = 0; j < P; ++j) {
        fr[j] = (EXT ? !CX_OCCUPIED(j) : dw[j] == 0) && (NOPAD || port[j] >= 0);
        const uint64_t m = ballot(fr[j]) & smask;
        n_free += __popcll(m);
        below += __popcll(m & below_mask);
      }
      const int acc = M < n_free ? M : n_free;
      rej = M - acc;
      // the first car's profile was drawn ahead by lane tb of the station
      const float f_cp = bcastf<L>(bcp, tb), f_s0 = bcastf<L>(bs0, tb), f_tg = bcastf<L>(btg, tb);
      const int f_dw = bcast<L>(bdw, tb);
      const int f_us = EXT ? bcast<L>(bus, tb) : 0;
      const int f_mod = EXT ? bcast<L>(bmod, tb) : 0;
      // (AHEAD2) the second car's, when the station takes two
      float f_cp1 = 0.f, f_s01 = 0.f, f_tg1 = 0.f;
      int f_dw1 = 1;
      if constexpr (AHEAD2) {
        if (ballot(acc > 1)) {
          f_cp1 = bcastf<L>(bcp1, tb);
          f_s01 = bcastf<L>(bs01, tb);
          f_tg1 = bcastf<L>(btg1, tb);
          f_dw1 = bcast<L>(bdw1, tb);
        }
      }
      int run = below;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const int rank = run;
        if (fr[j] && rank < acc) {
          float cp = f_cp, s0 = f_s0, tg = f_tg;
          int dd = f_dw;
          int us = f_us, md = f_mod;
          if (AHEAD2 && rank == 1) {
            cp = f_cp1;
            s0 = f_s01;
            tg = f_tg1;
            dd = f_dw1;
          } else if (rank > 0) {
            const U4 b = philox(env_id, g, (uint32_t)rank, kDomCar, k0, k1);
            cp = C.cap_lo + C.cap_span * u24(b.x);
            if constexpr (EXT) {
              if (models) {
                md = car_model(b.x);
                cp = car_data(3 * md);
              }
            }
            s0 = C.soc_lo + C.soc_span * u24(b.y);
            tg = C.tgt_lo + C.tgt_span * u24(b.z);
            dd = stay_len(tdw, C.dwell_log2, b.w);
            if constexpr (EXT) {
              if (users) us = philox(env_id, g, (uint32_t)rank, kDomUser, k0, k1).x <= C.cs_thresh ? 1 : 0;
            }
          }
          dw[j] = dd;
          if constexpr (EXT) {
            cs[j] = us;
            if (models) rb[j] = car_data(3 * md + (dc[j] ? 2 : 1));
          }
          cap[j] = cp;
          icap[j] = frcp(cp);
          q[j] = 1.0 - (double)s0;
          qf[j] = 1.0f - s0;  // the same rounding as (float) q
          u[j] = 1.0f - tg;
          plast[j] = 0.f;
        }
        run += fr[j] ? 1 : 0;
      }
    }

    // ---- reward (App. A.3)
    float r;
    if constexpr (EXT) {
      const float e_gn = e_grid + e_b;
      const float price = e_gn > 0.0f ? pbuy : p_sell_grid;
      r = p_sell * e_net - price * e_gn - fixed_cost - alpha_sat * csat - alpha_dec * (float)rej -
          C.alpha_db * fmaxf(0.0f, -e_b) + C.alpha_dc * e_out - C.alpha_sat1 * csat1;
    } else {
      const float price = e_grid > 0.0f ? pbuy : p_sell_grid;
      r = p_sell * e_net - price * e_grid - fixed_cost - alpha_sat * csat - alpha_dec * (float)rej;
    }
    ret += (double)r;

    // ---- end of day
    t_day += 1;
    const bool done = t_day == steps_ep;
    if (done) {
      t_day = 0;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        dw[j] = 0;
        if constexpr (EXT) cs[j] = 0;
      }
      if constexpr (EXT) {
        if (days) dday = episode_day(env_id, g + 1u, k0, k1, n_days);  // the next episode begins
      }
      if constexpr (EXT) {
        if (batt) {
          bsoc = C.b_soc0;
          bpw = 0.f;
        }
      }
    }

    // ---- records: an env's observation (byte offsets o inside its record)
    // goes to the block's LDS stage, or (wide stations) straight to HBM
    float *const ob_now = ob_t;  // this step's observation block of the segment
    // per-lane offsets, re-read every step: with the 32-bit offset visible at
    // each store the compiler emits the scalar-base form (no 64-bit lane address)
    uint32_t obs_bo_t = obs_bo, act_bo_t = act_bo, env_bo_t = env_bo;
    asm volatile("" : "+v"(obs_bo_t), "+v"(act_bo_t), "+v"(env_bo_t));
    // (the fused policy's records of a SIMPLE class are always 16-byte aligned)
    const int pad = !(POL && SIMPLE) && STAGE && (flags & kWObs)
                        ? (int)((reinterpret_cast<uintptr_t>(ob_now + (int64_t)env_blk0 * obs_dim) >> 2) & 3u)
                        : 0;
    if (active) {
      if (MODE != kModeNoObs && (POL || (flags & kWObs))) {
        // put(feature offset, port's offset, value) writes one value; put_lane the
        // P values of a feature of a lane whose ports are adjacent at once
        int n_occ = 0;
        if constexpr (P == 1) {
          n_occ = __popcll(ballot(CX_OCCUPIED(0) && (NOPAD || port[0] >= 0)) & smask);
        } else {
          float on = 0.f;   // (small whole numbers: exact)
#pragma unroll
          for (int j = 0; j < P; ++j) on += CX_OCCUPIED(j) && (NOPAD || port[j] >= 0) ? 1.0f : 0.0f;
          n_occ = (int)station_sum<L>(on);
        }
        auto obs_record = [&](auto put, auto put_lane, auto put4) {
          float f[6][P];
#pragma unroll
          for (int j = 0; j < P; ++j) {
            const bool occ = CX_OCCUPIED(j);
            f[0][j] = occ ? 1.0f : 0.0f;
            f[1][j] = occ ? 1.0f - qf[j] : 0.0f;
            f[2][j] = occ ? qf[j] - u[j] : 0.0f;
            f[3][j] = (float)dw[j] * inv_steps_ep;
            float rh = fminf(1.0f, qf[j] * inv_1mtau);
            if constexpr (EXT) {
              if (models) rh *= rb[j] * inv_pmax[j];  // the car's curve, as a share of the port maximum
            }
            f[4][j] = occ ? rh : 0.0f;
            f[5][j] = occ ? plast[j] * inv_pmax[j] : 0.0f;
          }
          const uint32_t Nb = 4u * (uint32_t)N;
          const auto put_at_once = [&] {
#pragma unroll
            for (int i = 0; i < 6; ++i) put_lane((uint32_t)i * Nb, 4u * (uint32_t)port[0], f[i]);
            if constexpr (EXT) {
              if (users) {
                float c[P];
#pragma unroll
                for (int j = 0; j < P; ++j) c[j] = cs[j] ? 1.0f : 0.0f;
                put_lane(4u * (uint32_t)C.user_obs, 4u * (uint32_t)port[0], c);
              }
            }
          };
          if (P > 1 && adjacent) {
            put_at_once();
          } else if (SOME && whole) {
            put_at_once();
          } else {
#pragma unroll
            for (int j = 0; j < P; ++j) {
              if (NOPAD || port[j] >= 0) {
                const uint32_t o = 4u * (uint32_t)port[j];
#pragma unroll
                for (int i = 0; i < 6; ++i) put((uint32_t)i * Nb, o, f[i][j]);
                if constexpr (EXT) {
                  if (users) put(4u * (uint32_t)C.user_obs, o, cs[j] ? 1.0f : 0.0f);
                }
              }
            }
          }
          if (l == 0) {  // the station's four: its first lane
            float price = gl.z;
            if constexpr (EXT) {
              if (days) price = p_next;
            }
            put4(4u * (uint32_t)(6 * N), gl.x, gl.y, price, (float)n_occ * (1.0f / (float)N));
          }
          if constexpr (EXT) {
            if (batt && l < 2) put(4u * (uint32_t)(6 * N + 4), 4u * (uint32_t)l, l == 0 ? (float)bsoc : bpw * C.b_inv_rate);
            if (days && l < 2)
              put(4u * (uint32_t)C.day_obs, 4u * (uint32_t)l, l == 0 ? (float)dday * C.inv_n_days : (dday % 7 >= 5 ? 1.0f : 0.0f));
          }
        };
        // the fused policy: the values go to the MLP's BF16 rows directly (their
        // padding was zeroed by the first conversion), unless they are converted
        // from the stage
        [[maybe_unused]] lds_char *const sb =
            STAGE ? reinterpret_cast<lds_char *>(stage + (POL ? 0 : (t & 1) * stage_step) + pad) + stage_bo : nullptr;
        const bool to_stage = flags & kWObs;
        if (POL && (DUAL || !to_stage)) {
          typedef __attribute__((address_space(3))) uint16_t lds_u16;
          lds_u16 *xr = reinterpret_cast<lds_u16 *>(lds + pol->xb_off) + (env - env_blk0) * (kPolXbRow * 8);
          obs_record([&](uint32_t fo, uint32_t lo, float v) {
                       xr[(fo + lo) >> 2] = (uint16_t)pack2(v, 0.f);
                       if (DUAL && to_stage) *reinterpret_cast<lds_float *>(sb + fo + lo) = v;
                     },
                     [&](uint32_t fo, uint32_t lo, const float (&v)[P]) {
                       // (P even and N a multiple of P: a whole number of words)
                       lds_u32 *x2 = reinterpret_cast<lds_u32 *>(xr) + ((fo + lo) >> 3);
#pragma unroll
                       for (int j = 0; j + 1 < P; j += 2) x2[j / 2] = pack2(v[j], v[j + 1]);
                       if (DUAL && to_stage) {
                         fvec<P> x;
#pragma unroll
                         for (int j = 0; j < P; ++j) set_at(x, j, v[j]);
                         *reinterpret_cast<__attribute__((address_space(3))) fvec<P> *>(sb + fo + lo) = x;
                       }
                     },
                     [&](uint32_t fo, float a, float b, float c, float d) {
                       lds_u32 *x2 = reinterpret_cast<lds_u32 *>(xr) + (fo >> 3);  // (6 N is even)
                       x2[0] = pack2(a, b);
                       x2[1] = pack2(c, d);
                       if (DUAL && to_stage) *reinterpret_cast<lds_f32x4u *>(sb + fo) = f32x4{a, b, c, d};
                     });
        } else if constexpr (STAGE) {
          obs_record([&](uint32_t fo, uint32_t lo, float v) { *reinterpret_cast<lds_float *>(sb + fo + lo) = v; },
                     [&](uint32_t fo, uint32_t lo, const float (&v)[P]) {
                       fvec<P> x;
#pragma unroll
                       for (int j = 0; j < P; ++j) set_at(x, j, v[j]);
                       *reinterpret_cast<__attribute__((address_space(3))) fvec<P> *>(sb + fo + lo) = x;
                     },
                     [&](uint32_t fo, float a, float b, float c, float d) {
                       *reinterpret_cast<lds_f32x4u *>(sb + fo) = f32x4{a, b, c, d};
                     });
        } else {
          // the feature's offset goes on the wave-uniform base, the lane's on its
          // 32-bit offset
          obs_record([&](uint32_t fo, uint32_t lo, float v) { st_at((float *)((char *)ob_now + fo), obs_bo_t + lo, v); },
                     [&](uint32_t fo, uint32_t lo, const float (&v)[P]) {
                       fvec<P> x;
#pragma unroll
                       for (int j = 0; j < P; ++j) set_at(x, j, v[j]);
                       st_at((fvec<P> *)((char *)ob_now + fo), obs_bo_t + lo, x);
                     },
                     [&](uint32_t fo, float a, float b, float c, float d) {
                       st_at((f32x4u *)((char *)ob_now + fo), obs_bo_t, (f32x4u){a, b, c, d});
                     });
        }
      }
      if (flags & kWAct) {
        if (NOPAD && (flags & kActQuads)) {
          // four consecutive ports' bytes gathered into the lane of the first
          // (moved from the neighbours and shifted by one 24-bit multiply a pair)
          // and stored as one dword (an env's bytes start at a multiple of 4, N
          // being one; every step's row too)
          uint32_t w = (uint32_t)k[0];   // the lane's own bytes
#pragma unroll
          for (int j = 1; j < P; ++j) w |= (uint32_t)k[j] << (8 * j);
          if constexpr (P == 1) {  // lanes 1, 1, 3, 3 of the quad
            const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xF5, 0xF, 0xF, true);
            w |= __umul24(b, 1u << 8);
          }
          if constexpr (P <= 2) {  // lane 2 (P = 1), lanes 1, 1, 3, 3 (P = 2)
            const uint32_t b =
                (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, P == 1 ? 0xAA : 0xF5, 0xF, 0xF, true);
            w |= __umul24(b, 1u << 16);
          }
          if ((l & (4 / P - 1)) == 0) st_at((uint32_t *)ab_t, act_bo_t + (uint32_t)port[0], w);
        } else if (P > 1 && adjacent) {  // the lane's bytes at once, at any address
          uint32_t w = (uint32_t)k[0];
#pragma unroll
          for (int j = 1; j < P; ++j) w |= (uint32_t)k[j] << (8 * j);
          typedef uint16_t __attribute__((aligned(1))) u16a1;
          typedef uint32_t __attribute__((aligned(1))) u32a1;
          if constexpr (P == 2) st_at((u16a1 *)ab_t, act_bo_t + (uint32_t)port[0], (u16a1)w);
          else st_at((u32a1 *)ab_t, act_bo_t + (uint32_t)port[0], (u32a1)w);
        } else {
#pragma unroll
          for (int j = 0; j < P; ++j)
            if (NOPAD || port[j] >= 0) st_at(ab_t, act_bo_t + (uint32_t)port[j], (uint8_t)k[j]);
        }
        if constexpr (EXT) {
          if (batt && l == 0) st_at(ab_t, act_bo_t + (uint32_t)N, (uint8_t)kb);
        }
      }
      if (l == 0) {
        if (flags & kWRew) st_at(rw_t, 4u * env_bo_t, r);
        if (flags & kWDone) st_at(dn_t, env_bo_t, (uint8_t)(done ? 1 : 0));
      }
    }
    ob_t += obs_step;
    ab_t += act_step;
    ai_t += act_step;
    rw_t += env_step;
    dn_t += env_step;
    // Keep the block's waves on the same step: their records for the step
    // are then adjacent envs' blocks written together, which HBM takes
    // noticeably faster (better row locality) than the same bytes spread over
    // many steps.  Waves that left early (past the last env) do not count.
    // (Rewards and done flags alone are too few bytes for that.)
    if (MODE != kModeStep && (POL || (flags & (kWObs | kWAct)))) __syncthreads();
    // (the host's rule stands at paced())
    if constexpr (!POL && !EXT && !STAGE && MODE == kModeAny) {
      if (flags & kPace) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt 0, the other counters as they are
    }
    // the stage of this step is complete: out to HBM (the next step fills the
    // other buffer; the barrier of that step keeps this one until it is read)
    if (STAGE && (flags & kWObs) && (!POL || wv < n_run))
      flush_stage(stage + (POL ? 0 : (t & 1) * stage_step), ob_now + (int64_t)env_blk0 * obs_dim, pad, n_blk,
                  (group - g_blk0) * 64 + lane, n_run * 64);
    if constexpr (POL) {
      // the next step's levels (the phase's barriers keep the stage until the
      // flush above has read it)
      if (t + 1 < T) {
        if constexpr (!HELD) held1.start(w1_rsrc(), pol->b1, wv);
        policy_phase(*pol, stage + pad, lds, obs_dim, N, blk_envs, wv, env_id0, g + 1u, k0, k1,
                     w_obs && !DUAL, held1, held2);
      }
    }
  }

  // ---- state back to HBM (its addresses read again, not held over the steps)
  CX_KONST SegDev &so = *reload(sgp);
  if (active) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int64_t i = sofs + l * P + j;
      const bool occ = CX_OCCUPIED(j);
      gst(so.q, i, occ ? q[j] : 0.0);
      gst(so.u, i, occ ? u[j] : 0.f);
      gst(so.cap, i, occ ? cap[j] : 0.f);
      gst(so.p_last, i, occ ? plast[j] : 0.f);
      gst(so.dwell, i, (int16_t)dw[j]);
      if constexpr (EXT) {
        if (users) gst(so.utype, i, (uint8_t)cs[j]);
        if (models) gst(so.rbar, i, occ ? rb[j] : 0.f);
      }
    }
    if (l == 0) gst(so.ret, env, ret);
    if constexpr (EXT) {
      if (batt && l == 0) {
        gst(so.bsoc, env, bsoc);
        gst(so.bp, env, bpw);
      }
    }
  }
}

#undef CX_OCCUPIED

// A launch's blocks are dealt to the chip's 8 XCDs in turn (block i to XCD
// i mod 8).  Numbered so that each XCD's blocks are consecutive, blocks of
// adjacent envs, whose small records (actions, rewards, done flags) share
// 128-byte lines, write those lines through the same L2 (V2G at 8 lanes and one
// wave per block: 2.57 -> 2.41 ms).
__device__ __forceinline__ int xcd_block(int i, int n) {
  const int x = i & 7, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + (i >> 3);
}

// One kernel per packing (lanes per station L, slots per lane P) and class
// kind (general, SIMPLE, bidirectional), so that each keeps its own register
// budget; the entry points below add the launch bounds of each kind.
template <int L, int P, bool SIMPLE, bool EXT, bool STAGE, int HPOL, bool HELD = false, int MODE = kModeAny>
__device__ __forceinline__ void rollout_body(const LaunchArgs &a, const SegDev *segs, int n_segs, int b) {
  constexpr bool POL = HPOL > 0;
  extern __shared__ uint32_t block_lds[];
  CX_KONST SegDev *const seg0 = konst(segs);
  int lo = 0, hi = n_segs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg0[mid].block_begin <= b) lo = mid;
    else hi = mid - 1;
  }
  // the segment is block-uniform: say so, so its fields come in scalar loads
  lo = uni(lo);
  CX_KONST SegDev *const sgp = seg0 + lo;
  CX_KONST SegDev &sg = *sgp;
  CX_KONST ClassDev &C = *konst((const ClassDev *)sg.cls);
  Dyn dy;
  if (a.per_segment) {
    dy = Dyn{sg.T, sg.t_day0, sg.g0, sg.mode, sg.out_mode, sg.obs, sg.act, sg.reward, sg.done, sg.act_in,
             sg.obs_stride, sg.act_stride, sg.env_stride, 0};
  } else {
    dy = Dyn{a.T, a.t_day0, a.g0, a.mode, a.out_mode, a.obs, a.act, a.reward, a.done, a.act_in,
             a.obs_stride, a.act_stride, a.env_stride, a.pace};
  }
  // stay-length thresholds in LDS; the day's per-step tables too, for launches
  // long enough to repay copying them (short ones read them from device memory)
  const lds_u32x4 *exo_tp = nullptr;
  const int steps = C.steps_ep;
  if (MODE != kModeStep && (HELD ? a.day_off > 0 : !POL) && steps <= kLdsExoSteps && dy.T >= kLdsExoMinT) {
    exo_tp = (const lds_u32x4 *)((lds_char *)block_lds + a.day_off);
  }
  lds_u32 *const car_tab = EXT ? (lds_u32 *)((lds_char *)block_lds + a.car_off) : nullptr;
  // every wave of the block helps load them, those past the last env too; the
  // others ask for their state first, so that a short launch waits once (one step
  // of 65,536 uneven stations 54.4 -> 48.8 us) and nothing is still on its way
  // when the steps begin (a step had waited for its records at the first use of
  // the return's load: a day of 64 16-port stations 226 -> 210 us)
  const auto fill_tables = [&] {
    const int n_stay = 1 << C.dwell_log2;
    for (int i = threadIdx.x; i < n_stay; i += blockDim.x) block_lds[i] = gld(C.tdwell, i);
    if (exo_tp) {
      lds_u32x4 *tp = const_cast<lds_u32x4 *>(exo_tp);
      lds_float *pr = reinterpret_cast<lds_float *>(tp + steps);
      for (int i = threadIdx.x; i < steps; i += blockDim.x) {
        tp[i] = gld(reinterpret_cast<const u32x4 *>(C.tpois + (int64_t)i * kPoisStride), 0);
        pr[i] = gld(C.glob, 4 * i + 2);
      }
    }
    if constexpr (EXT) {
      const int i = threadIdx.x;
      if (i < 8) car_tab[i] = gld(C.model_thresh, i);
      else if (i < 32) car_tab[i] = __float_as_uint(gld(C.model_data, i - 8));
    }
    __syncthreads();
  };
  const int W = blockDim.x >> 6;
  const int g_blk0 = (b - sg.block_begin) * W;  // the block's first group
  const int group = uni(g_blk0 + (int)(threadIdx.x >> 6));
  // (the fused policy keeps every wave: all take part in the MLP)
  const int n_groups = sg.n_groups;
  if (!POL && group >= n_groups) {
    fill_tables();
    return;
  }
  const int n_run = min(W, n_groups - g_blk0);  // waves of the block that run
  lds_float *stage = a.stage_floats > 0 ? (lds_float *)((lds_char *)block_lds + a.stage_off) : nullptr;
  run_group<L, P, SIMPLE, EXT, STAGE, HPOL, HELD, MODE>(
      fill_tables, sgp, dy, group, (const lds_u32 *)block_lds, exo_tp, car_tab, stage, W == 1 ? 0 : a.stage_floats,
      g_blk0, n_run, &a.pol, (lds_char *)block_lds);
}

// Waves per SIMD extended classes are held to.  One slot per lane: five, 96
// registers of the 102 they would take (at 16 lanes V2G 2.71 -> 2.56 ms).  Two, without
// observation records: four, 128 registers of 135 (V2G, 144 steps, 768 -> 663
// us; with the records four cost more than they give: 288 steps 2.52 -> 2.80 ms).
constexpr int ext_waves(int P, int mode) {
  return mode == kModeStep ? 1 : P == 1 ? 5 : P == 2 && mode == kModeNoObs ? 4 : 1;
}
template <int L, int P, bool SIMPLE, bool EXT, bool STAGE, int MODE>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(EXT ? ext_waves(P, MODE) : 1))) void k_rollout(LaunchArgs a) {
  rollout_body<L, P, SIMPLE, EXT, STAGE, 0, false, MODE>(a, a.segs, a.n_segs, xcd_block(blockIdx.x, gridDim.x));
}

// SIMPLE classes of 1 or 2 slots per lane, with observation records: 64-75 VGPRs at
// one slot per lane (six to eight waves per SIMD), 80-91 at two (five or six), with
// their constants in scalar registers and no vector register spilled (of the scalar
// ones, to lanes of a vector register: 2-6 with the stage, 14 at 64 lanes and two
// slots, 2 there without it); the bound keeps every one at five waves at
// least.  Every record, 65,536 uneven stations x 288 steps: 3.74
// ms with the constants in vector registers (96, some spilled), 3.48 now; rewards
// only 2.25 and 1.60.
#ifndef CX_SIMPLE_WAVES
#define CX_SIMPLE_WAVES 5
#endif
template <int L, int P, bool STAGE, int MODE>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(MODE == kModeNoObs ? 6 : CX_SIMPLE_WAVES))) void k_rollout_simple(LaunchArgs a) {
  rollout_body<L, P, true, false, STAGE, 0, false, MODE>(a, a.segs, a.n_segs, xcd_block(blockIdx.x, gridDim.x));
}

// The fused policy rollout (4 waves per block): three blocks per CU, so that
// one block's matrix-core work and memory waits overlap the others' steps, and
// the weights' way from L2 bounds it (304 KB a block and step at 32 ports and 256
// hidden units: 16 of the 31 us a step of 65,536 stations takes).  HELD: one
// block per CU with the weights in registers and the day's tables in LDS, so
// that a step loads nothing from device memory (but the second product's weights at
// 32 slots and 256 hidden units, which come round a ring, and the tables of a day
// of more than 512 steps, of a call of fewer than 32 or where LDS is short); it is
// bound by the length of one step's chain (10 DC + 6 AC ports, 256 hidden units,
// every record, 4,096 x 288 steps: 1,770 -> 766 us, 2.65 us a step).
template <int L, int P, int HP, bool HELD>
__global__ __launch_bounds__(64 * kPolRolloutWaves)
__attribute__((amdgpu_waves_per_eu(HELD ? 1 : 3))) void k_rollout_policy(LaunchArgs a) {
  rollout_body<L, P, true, false, true, HP, HELD>(a, a.segs, a.n_segs, xcd_block(blockIdx.x, gridDim.x));
}
// ... of classes that are not SIMPLE (padding slots, port maxima or limits that
// differ, the dense layout): a policy rollout of the 10 DC + 6 AC station used to
// take two launches a step.
template <int L, int P, int HP, bool HELD>
__global__ __launch_bounds__(64 * kPolRolloutWaves)
__attribute__((amdgpu_waves_per_eu(HELD ? 1 : P == 4 ? 2 : 3))) void k_rollout_policy_general(LaunchArgs a) {
  rollout_body<L, P, false, false, true, HP, HELD>(a, a.segs, a.n_segs, xcd_block(blockIdx.x, gridDim.x));
}

// Several groups of SIMPLE classes in one launch (a.part: each group's blocks, at
// a multiple of 8 so that they are dealt to the XCDs as in a launch of their
// own).  For launches too short to fill the chip one group at a time: one step
// of 65,536 uneven stations takes 68.4 us as five kernels one after the other, so
// 40.3 (65.6 and 37.3 where state and records stay in the caches).
template <int MODE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MODE == kModeNoObs ? 6 : 1))) void k_rollout_parts(LaunchArgs a) {
  int i = 0;
  while (i + 1 < a.n_parts && (int)blockIdx.x >= a.part[i + 1].block_begin) ++i;
  i = uni(i);
  const LaunchArgs::Part &p = a.part[i];
  const int b0 = (int)blockIdx.x - p.block_begin;
  if (b0 >= p.n_blocks) return;   // (the gap before the next group)
  const int b = xcd_block(b0, p.n_blocks);
  const SegDev *segs = a.segs + p.seg_begin;
  const int n = p.n_segs;
  switch (p.pack) {
#define CX_PART(L, P)                                                                              \
  case part_id(L, P):                                                                              \
    rollout_body<L, P, true, false, false, 0, false, MODE>(a, segs, n, b);                         \
    break;
    CX_PART(4, 1) CX_PART(8, 1) CX_PART(16, 1) CX_PART(32, 1) CX_PART(64, 1)
    CX_PART(4, 2) CX_PART(8, 2) CX_PART(16, 2) CX_PART(32, 2) CX_PART(64, 2)
#undef CX_PART
    default: break;
  }
}

// Observation of empty stations at t_day = 0 for every env of one segment
// (env0: Philox index of its first env; g: the step the new episodes begin on).
__global__ void k_reset_obs(const ClassDev *cls, int64_t n_envs, float *obs, uint64_t seed, int64_t env0,
                            uint32_t g) {
  const int64_t dim = cls->obs_dim;
  const int N = cls->n_ports, n_days = cls->n_days, day_obs = cls->day_obs;
  const int64_t total = n_envs * dim;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t f = i % dim;
    float v = 0.f;
    if (f >= 6 * N && f < 6 * N + 3) v = cls->glob[f - 6 * N];
    if (cls->has_batt && f == 6 * N + 4) v = (float)cls->b_soc0;  // a battery starts the day at its initial SoC
    if (n_days > 0 && (f == 6 * N + 2 || f == day_obs || f == day_obs + 1)) {
      const int d = episode_day((uint32_t)(env0 + i / dim), g, (uint32_t)seed, (uint32_t)(seed >> 32), n_days);
      v = f == 6 * N + 2 ? cls->price_days[(int64_t)d * cls->steps_ep]
                         : f == day_obs ? (float)d * cls->inv_n_days : (d % 7 >= 5 ? 1.0f : 0.0f);
    }
    obs[i] = v;
  }
}

__global__ void k_fill_f64(double *p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

using KernelFn = void (*)(LaunchArgs);

// The kernels of one packing: general, SIMPLE, extended, SIMPLE with staged
// observations (which needs them; one step has no kernel of its own there).
#define CX_KINDS(L, P, M)                                                                           \
  &k_rollout<L, P, false, false, false, M>, &k_rollout<L, P, true, false, false, M>,                  \
      &k_rollout<L, P, false, true, false, M>,                                                        \
      &k_rollout<L, P, true, false, M != kModeNoObs, M == kModeNoObs ? kModeNoObs : kModeAny>
#define CX_KINDS_SIMPLE(L, P, M)                                                                    \
  &k_rollout<L, P, false, false, false, M>, &k_rollout_simple<L, P, false, M>,                        \
      &k_rollout<L, P, false, true, false, M>,                                                        \
      &k_rollout_simple<L, P, M != kModeNoObs, M == kModeNoObs ? kModeNoObs : kModeAny>
#define CX_ALL(M)                                                                                   \
  {CX_KINDS_SIMPLE(4, 1, M), CX_KINDS_SIMPLE(8, 1, M), CX_KINDS_SIMPLE(16, 1, M),                     \
   CX_KINDS_SIMPLE(32, 1, M), CX_KINDS_SIMPLE(64, 1, M), CX_KINDS_SIMPLE(4, 2, M),                    \
   CX_KINDS_SIMPLE(8, 2, M), CX_KINDS_SIMPLE(16, 2, M), CX_KINDS_SIMPLE(32, 2, M),                    \
   CX_KINDS_SIMPLE(64, 2, M), CX_KINDS(4, 4, M), CX_KINDS(8, 4, M), CX_KINDS(16, 4, M),               \
   CX_KINDS(32, 4, M), CX_KINDS(64, 4, M)}

// Kernel of each launch kind by mode: packing id (P index * 5 + L index, as
// pack_id()) times kNumKinds, plus the kernel kind (kKind*).
const KernelFn kKernels[3][kNumKinds * kNumPackings] = {CX_ALL(kModeAny), CX_ALL(kModeNoObs), CX_ALL(kModeStep)};
#undef CX_ALL
#undef CX_KINDS
#undef CX_KINDS_SIMPLE
int launch_mode(const LaunchArgs &a) {
  if (a.per_segment) return kModeAny;
  return a.T == 1 ? kModeStep : a.out_mode == CX_OUT_FULL && a.obs ? kModeAny : kModeNoObs;
}
const KernelFn &kernel_of(const LaunchArgs &a, int pack, int kind) {
  return kKernels[launch_mode(a)][kNumKinds * pack + kind];
}

// Waves of all groups of a launch.
int64_t total_waves(const LaunchGroup *groups, int n_groups) {
  int64_t n = 0;
  for (int i = 0; i < n_groups; ++i) n += (int64_t)groups[i].n_blocks * groups[i].wpb;
  return n;
}

// The kernel kind a group runs as in this launch: a SIMPLE class's observations
// go through the stage, asked for or not, in a launch of at least as many waves
// as the chip holds at once (8 per SIMD): its writes then set the pace, and the
// stage's whole lines are worth its barrier per step.  100 steps, every record,
// stage against lane stores: 16-port stations at 4,096 waves 0.202 / 0.179 ms,
// 8,192 0.330 / 0.353, 16,384 0.586 / 0.667; the mixture at 2,500 waves 0.414 /
// 0.342, 8,300 0.493 / 0.531, 27,300 1.280 / 1.594.
constexpr int64_t kStageMinWaves = 8192;
int launch_kind(const LaunchArgs &a, const LaunchGroup &g, int64_t waves) {
  if (g.kind != kKindSimple || a.per_segment || a.out_mode != CX_OUT_FULL || !a.obs || a.T < kLdsExoMinT ||
      waves < kStageMinWaves)
    return g.kind;
  return lds_plan(g.wpb, g.pack, g.max_obs_dim, g.max_dwell_log2, g.max_day_steps, true, false).bytes <= kMaxBlockLds
             ? kKindSimpleStaged
             : kKindSimple;
}

// Arguments of one group's launch as kernel kind `kind`: its slice of the
// segment table and its LDS.
// Records stored by the lanes themselves share their lines' halves with the next
// lanes', envs' and blocks', which meet in L2 only while the waves keep together:
// where the stores set the pace, a wave waits for a step's records before the next
// step.  Every record, free against paced: the mixture in one launch, 2,000 stations
// 0.507 / 0.483 ms, 10,000 0.630 / 0.605, 20,000 1.178 / 1.162; 10 DC + 6 AC
// ports, 144 steps, 8,192 waves 0.940 / 0.917, 16,384 1.160 / 1.126, but 2,000
// waves 0.161 / 0.176; extended classes, bound by their steps, 1.100 / 1.125
// (V2G, 8,192 waves).
bool paced(int kind, int64_t waves) { return kind == kKindGeneral && waves >= kStageMinWaves; }

LaunchArgs group_args(const LaunchArgs &a, const LaunchGroup &g, int kind, int64_t waves, size_t *lds) {
  LaunchArgs b = a;
  b.segs = a.segs + g.seg_begin;
  b.n_segs = g.n_segs;
  const bool stages =
      kind == kKindSimpleStaged && (a.per_segment || (a.out_mode == CX_OUT_FULL && a.obs != nullptr));
  const LdsPlan p = lds_plan(g.wpb, g.pack, g.max_obs_dim, g.max_dwell_log2, g.max_day_steps, stages,
                             kind == kKindExt);
  b.day_off = p.day_off;
  b.stage_off = p.stage_off;
  b.stage_floats = p.stage_floats;
  b.car_off = p.car_off;
  b.pace = paced(kind, waves) ? 1 : 0;
  *lds = p.bytes;
  return b;
}

}  // namespace

namespace {

// All groups in one launch (k_rollout_parts) when they are SIMPLE classes of one
// or two slots per lane with one block size and the launch is one step, keeps no
// observations, or has at most kPartsMaxWaves waves.  A graph of one kernel per
// packing costs 95 us of host time a launch and runs its kernels only partly at
// once, but keeps each packing's own registers (the shared kernel takes the
// largest, five waves per SIMD with observations) and the stage, which pays when
// the chip is full.  Uneven stations x 288 steps, every record (rewards only), one
// launch against the graph: 2,000 0.49 (0.30) / 0.80 (0.54) ms, 10,000 0.59 (0.35)
// / 0.87 (0.53), 20,000 (8,400 waves) 1.16 (0.57) / 1.20 (0.60), 28,000 (11,700)
// 1.58 (0.70) / 1.52 (0.73), 65,536 (27,300) 3.57 (1.46) / 3.55 (1.51).  One step:
// 300 stations 31.1 -> 8.3 us, 65,536 68.4 -> 40.3.  False: not such a launch.
constexpr int64_t kPartsMaxWaves = 10240;
bool launch_parts(const LaunchArgs &a, const LaunchGroup *groups, int n_groups, hipStream_t st, hipError_t *e) {
  if (n_groups < 2 || n_groups > LaunchArgs::kMaxParts || a.per_segment) return false;
  const int64_t waves = total_waves(groups, n_groups);
  // (and what the gaps between the parts add must fit one launch too)
  if (64 * (waves + 8 * n_groups * groups[0].wpb) > kMaxLaunchThreads) return false;
  if (launch_mode(a) == kModeAny && waves > kPartsMaxWaves) return false;
  LaunchArgs b = a;
  int blocks = 0, dwell = 1, days = 0;
  b.n_parts = 0;
  for (int i = 0; i < n_groups; ++i) {
    const LaunchGroup &g = groups[i];
    if ((g.kind != kKindSimple && g.kind != kKindSimpleStaged) || pack_per_lane(g.pack) > 2 || g.wpb != groups[0].wpb)
      return false;
    // a caller that asks for the stage gets it in every rollout that records observations
    if (g.kind == kKindSimpleStaged && launch_mode(a) == kModeAny) return false;
    if (g.n_blocks <= 0) continue;
    blocks = (blocks + 7) & ~7;
    b.part[b.n_parts++] = {blocks, g.n_blocks, g.seg_begin, g.n_segs,
                           part_id(pack_lanes(g.pack), pack_per_lane(g.pack))};
    blocks += g.n_blocks;
    dwell = std::max(dwell, g.max_dwell_log2);
    days = std::max(days, g.max_day_steps);
  }
  if (blocks == 0) {
    *e = hipSuccess;
    return true;
  }
  const LdsPlan p = lds_plan(groups[0].wpb, groups[0].pack, 0, dwell, a.T >= kLdsExoMinT ? days : 0, false, false);
  b.day_off = p.day_off;
  b.pace = 1;
  void *params[1] = {&b};
  static const KernelFn kParts[3] = {&k_rollout_parts<kModeAny>, &k_rollout_parts<kModeNoObs>,
                                     &k_rollout_parts<kModeStep>};
  const KernelFn f = kParts[launch_mode(a)];
  *e = hipLaunchKernel(reinterpret_cast<const void *>(f), dim3(blocks), dim3(64 * groups[0].wpb), params,
                       p.bytes, st);
  return true;
}

}  // namespace

hipError_t launch_groups(const LaunchArgs &a, const LaunchGroup *groups, int n_groups, hipStream_t st) {
  hipError_t pe;
  if (launch_parts(a, groups, n_groups, st, &pe)) return pe;
  const int64_t waves = total_waves(groups, n_groups);
  for (int i = 0; i < n_groups; ++i) {
    const LaunchGroup &g = groups[i];
    if (g.n_blocks <= 0) continue;
    size_t lds = 0;
    const int kind = launch_kind(a, g, waves);
    LaunchArgs b = group_args(a, g, kind, waves, &lds);
    void *params[1] = {&b};
    hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel_of(a, g.pack, kind)), dim3(g.n_blocks),
                                   dim3(64 * g.wpb), params, lds, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The fused policy rollout of one class: stations of 8 lanes (8, 16 or 32
// slots), 4 waves per block (32 stations, two 16-env tiles of the MLP), or of 16
// lanes (16 stations, one tile).  a.pol.HP:
// K-steps of 32 hidden units; the kernels are built for 2, 4 and 8 (a policy
// of 64 hidden units does a quarter of the matrix work of one of 256).
hipError_t launch_policy_rollout(const LaunchArgs &a, bool simple, int lanes, int per_lane, bool held, int n_blocks,
                                 size_t lds, hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  const int hp = a.pol.HP;
  // stations of 8 lanes with 1, 2 and 4 slots per lane, the same with their
  // weights held, and of 16 lanes, always held
#define CX_POL(K, L, P, H) {&K<L, P, 2, H>, &K<L, P, 4, H>, &K<L, P, 8, H>}
#define CX_POLS(K)                                                                                           \
  {CX_POL(K, 8, 1, false), CX_POL(K, 8, 2, false), CX_POL(K, 8, 4, false), CX_POL(K, 8, 1, true),             \
   CX_POL(K, 8, 2, true),  CX_POL(K, 8, 4, true),  CX_POL(K, 16, 1, true)}
  static const KernelFn kPol[2][7][3] = {CX_POLS(k_rollout_policy_general), CX_POLS(k_rollout_policy)};
#undef CX_POLS
#undef CX_POL
  if ((per_lane != 1 && per_lane != 2 && per_lane != 4) || hp < 1 || hp > 8) return hipErrorInvalidValue;
  if (lanes != 8 && (lanes != 16 || per_lane != 1 || !held)) return hipErrorInvalidValue;
  const int v = lanes == 16 ? 6 : (held ? 3 : 0) + (per_lane == 4 ? 2 : per_lane - 1);
  const KernelFn f = kPol[simple ? 1 : 0][v][hp <= 2 ? 0 : hp <= 4 ? 1 : 2];
  LaunchArgs b = a;
  void *params[1] = {&b};
  return hipLaunchKernel(reinterpret_cast<const void *>(f), dim3(n_blocks), dim3(64 * kPolRolloutWaves), params, lds,
                         st);
}

namespace {
void destroy_one(RolloutGraph &g) {
  if (g.exec) (void)hipGraphExecDestroy(g.exec);
  if (g.graph) (void)hipGraphDestroy(g.graph);
  g = RolloutGraph{};
}

// A new graph of n kernel nodes.
hipError_t build_graph(RolloutGraph &G, int n, const hipKernelNodeParams *p, const int (*shape)[4]) {
  hipError_t e = hipGraphCreate(&G.graph, 0);
  for (int i = 0; e == hipSuccess && i < n; ++i) e = hipGraphAddKernelNode(&G.node[i], G.graph, nullptr, 0, &p[i]);
  if (e == hipSuccess) e = hipGraphInstantiate(&G.exec, G.graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    destroy_one(G);
    return e;
  }
  G.n_nodes = n;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < 4; ++j) G.shape[i][j] = shape[i][j];
  return hipSuccess;
}
}  // namespace

hipError_t graph_rollout(RolloutGraphs &gs, const LaunchArgs &a, const LaunchGroup *groups, int n_groups,
                         hipStream_t st) {
  // one kernel is launched as it is; so are groups that share a launch
  hipError_t pe;
  if (n_groups == 1) return launch_groups(a, groups, n_groups, st);
  if (launch_parts(a, groups, n_groups, st, &pe)) return pe;
  LaunchArgs args[kNumKinds * kNumPackings];
  void *params[kNumKinds * kNumPackings][1];
  hipKernelNodeParams p[kNumKinds * kNumPackings];
  int shape[kNumKinds * kNumPackings][4] = {};
  int n = 0;
  const int64_t waves = total_waves(groups, n_groups);
  for (int i = 0; i < n_groups && n < kNumKinds * kNumPackings; ++i) {
    const LaunchGroup &g = groups[i];
    if (g.n_blocks <= 0) continue;
    size_t lds = 0;
    const int kind = launch_kind(a, g, waves);
    args[n] = group_args(a, g, kind, waves, &lds);
    params[n][0] = &args[n];
    p[n] = hipKernelNodeParams{};
    p[n].func = reinterpret_cast<void *>(kernel_of(a, g.pack, kind));
    p[n].gridDim = dim3(g.n_blocks);
    p[n].blockDim = dim3(64 * g.wpb);
    p[n].sharedMemBytes = (unsigned)lds;
    p[n].kernelParams = params[n];
    p[n].extra = nullptr;
    shape[n][0] = kNumKinds * (launch_mode(a) * kNumPackings + g.pack) + kind;
    shape[n][1] = g.n_blocks;
    shape[n][2] = g.wpb;
    shape[n][3] = (int)lds;
    ++n;
  }
  if (n == 0) return hipSuccess;
  hipError_t e;
  for (int k = 0; k < gs.n; ++k) {
    RolloutGraph &G = gs.g[k];
    bool same = G.n_nodes == n;
    for (int i = 0; same && i < n; ++i)
      for (int j = 0; j < 4; ++j) same = same && G.shape[i][j] == shape[i][j];
    if (!same) continue;
    for (int i = 0; i < n; ++i)
      if ((e = hipGraphExecKernelNodeSetParams(G.exec, G.node[i], &p[i])) != hipSuccess) return e;
    return hipGraphLaunch(G.exec, st);
  }
  if (gs.n == RolloutGraphs::kMax) {
    // (more shapes than a set of segments has: only the tuner's, of many sets)
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    graph_destroy(gs);
  }
  RolloutGraph &G = gs.g[gs.n];
  if ((e = build_graph(G, n, p, shape)) != hipSuccess) return e;
  ++gs.n;
  return hipGraphLaunch(G.exec, st);
}

void graph_destroy(RolloutGraphs &gs) {
  for (int k = 0; k < gs.n; ++k) destroy_one(gs.g[k]);
  gs.n = 0;
}

hipError_t launch_reset_obs_one(const ClassDev *cls_dev, int64_t n_envs, float *obs, uint64_t seed, int64_t env0,
                                uint32_t g, hipStream_t st) {
  if (n_envs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reset_obs, dim3(256), dim3(256), 0, st, cls_dev, n_envs, obs, seed, env0, g);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double *p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int blocks = (int)std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(k_fill_f64, dim3(blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace cx
