// cx_mlp.h -- device helpers of the policy MLP shared by the standalone
// policy kernel and the fused policy rollout, so that both compute the same
// logits and draw the same levels bit for bit.
//
// Layout of the two products (both computed transposed, so that no operand is
// shuffled between lanes): with D = A * B on 16 x 16 tiles of
// v_mfma_f32_16x16x32_bf16, lane l holds column l % 16 and rows 4 (l / 16) + i
// (i < 4) of D, and the 8 K-values 8 (l / 16) .. 8 (l / 16) + 7 of A's row
// l % 16 and of B's column l % 16.
//   h^T [hidden x env] = W1^T [hidden x obs] * obs^T [obs x env]
//   z^T [logit x env]  = W2^T [logit x hidden] * h^T [hidden x env]
// A lane ends the first product holding 8 hidden units of one env, exactly the
// B operand of the second (the host stores W2 in that order), and ends the
// second holding every level of one port of one env.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cx_device.h"
#include "cx_internal.h"

namespace cx {
namespace {

constexpr int kPolK1 = 8;  // K-steps of 32 observation features (obs_dim <= 256)
constexpr int kPolHP = 8;  // K-steps of 32 hidden units (hidden <= 256)
constexpr int kPolR = 3;   // tiles of 4 levels per port (levels + 1 <= 12)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Two FP32 values -> two BF16 (lo in the low half), rounded to nearest even:
// one v_cvt_pk_bf16_f32 on gfx950.
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                 0, 0, 0);
}

// tanh a = 1 - 2 / (e^{2a} + 1); saturates correctly at both ends.
__device__ __forceinline__ float tanh_f(float a) {
  const float e = __builtin_amdgcn_exp2f(a * 2.88539008177792681f);  // 2 / ln 2
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// The hidden units of one K-step of the second product from the two tiles of
// the first (c0: units 4 (l / 16) + i, c1: units 16 + 4 (l / 16) + i), bias
// added, tanh, rounded to BF16.
__device__ __forceinline__ u32x4 hidden_frag(f32x4 c0, f32x4 c1, f32x4 bA, f32x4 bB) {
  return u32x4{pack2(tanh_f(c0.x + bA.x), tanh_f(c0.y + bA.y)), pack2(tanh_f(c0.z + bA.z), tanh_f(c0.w + bA.w)),
               pack2(tanh_f(c1.x + bB.x), tanh_f(c1.y + bB.y)), pack2(tanh_f(c1.z + bB.z), tanh_f(c1.w + bB.w))};
}

// The uniform of a port's level draw from its Philox word: (top 24 bits + 1/2)
// 2^-24.  Port p takes word (p / 16) mod 4 of the call with counter index
// p mod 16 + 16 (p / 64): ports 16 apart share a call.
__device__ __forceinline__ float draw_uniform(uint32_t w) { return ((float)(w >> 8) + 0.5f) * 0x1p-24f; }
__device__ __forceinline__ uint32_t draw_index(int port) { return (uint32_t)(port % 16 + 16 * (port / 64)); }
__device__ __forceinline__ uint32_t draw_word(U4 w, int port) {
  const int k = (port / 16) % 4;
  return k == 0 ? w.x : k == 1 ? w.y : k == 2 ? w.z : w.w;
}

// The level drawn from softmax of a port's logits (level 4 r + i in c[r][i],
// L1 levels; the levels past them have the lowest float for a bias and weights 0,
// so their softmax weights are exactly 0): the first level whose
// cumulative softmax weight exceeds u times the total, i.e. the inverse of the
// distribution function at u (the last level where all of a port's logits are
// below -2.36e38 and the weights overflow; level 0 where a logit is NaN or none is
// finite).  The weights are 2^(z log2 e - zmax log2 e) (one
// fused multiply-add each); the running sums kept as they are formed are the
// cumulative weights.  Straight-line code, no test per level: with the levels
// in use selected one by one the draw took 110 vector and 35 scalar
// instructions, now 63 vector ones.
__device__ __forceinline__ int sample_level(const f32x4 (&c)[kPolR], int L1, float u) {
  constexpr float kLog2e = 1.44269504088896341f;
  float zmax = c[0][0];
#pragma unroll
  for (int r = 0; r < kPolR; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) zmax = __builtin_elementwise_maximum(zmax, (float)c[r][i]);
  const float zs = zmax * kLog2e;
  float cum[4 * kPolR];
#pragma unroll
  for (int l = 0; l < 4 * kPolR; ++l) {
    const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(c[l >> 2][l & 3], kLog2e, -zs));
    cum[l] = l ? cum[l - 1] + w : w;
  }
  const float target = u * cum[4 * kPolR - 1];
  int lev = 0;
#pragma unroll
  for (int l = 0; l < 4 * kPolR; ++l) lev += cum[l] <= target ? 1 : 0;
  return min(lev, L1 - 1);  // (u times the total may round to the total)
}

typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

// Weight fragments come in buffer loads: one resource per matrix, the
// fragment's offset a scalar, the lane's 16 bytes the vector offset (no 64-bit
// addresses).  Fragments are 1 KiB and padded to the largest sizes: W1^T
// [16 tiles][8 K-steps], W2^T [G][3 tiles][8 K-steps].
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frag_rsrc(const u32x4 *w, int n_frags) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(w), (short)0, n_frags * 1024, 0x00020000);
}
// Fragment i (wave-uniform).
__device__ __forceinline__ u32x4 frag(__amdgpu_buffer_rsrc_t w, int i) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(w, 16u * (uint32_t)__lane_id(), i * 1024, 0));
}

// Both products read their weight fragments through a ring of registers two
// K-steps deep: while step s is multiplied step s + 1 is in flight, and the ring
// is filled before the barrier or the draw that comes first.  The scheduling
// barriers keep the loads where they are written: left alone, the compiler
// sinks each load to its use to save registers, and every fragment then costs
// the L2's whole latency.  32-port stations, 262,144 x 288 steps: 39.5 ms a
// rollout so, 34.4 ms with the ring; 35.4 at depths 1 and 2, 37.5 at 3 and 4
// (spilled registers), 41.9 at 3 and 4 with two waves per SIMD and no spills.
constexpr int kRing = 2;
constexpr int ring_depth(int steps, int want) { return steps < want ? steps : want; }
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }

// The first product of a block of W waves and 16 NT envs, with the tanh: wave wv
// computes its pairs of 16-unit hidden tiles (HP pairs in all; with fewer pairs
// than waves, waves share a pair and split its env tiles) from the BF16
// observations xb (xrow fragments an env) into the hidden-unit fragments hb
// [HP][NT][64].  K1 K-steps of 32 features.  HELD: the ring holds every K-step's
// fragments and the biases too, and start() is called once for many run()s.
template <int W, int NT, int K1, int HP, bool HELD = false>
struct HiddenLayer {
  static constexpr int NI = HP >= W ? HP / W : 1;   // pairs of this wave
  static constexpr int SH = HP >= W ? 1 : W / HP;   // waves that share a pair
  static constexpr int NN = SH <= NT ? NT / SH : 1; // env tiles of this wave
  static constexpr int D = HELD ? K1 : ring_depth(K1, kRing);
  u32x4 a[D][NI][2];
  f32x4 bias[HELD ? NI : 1][2];   // HELD

  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t w1, int wv, int s) {
    const int mp0 = SH == 1 ? wv : wv % HP;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) a[s % D][i][h] = frag(w1, (2 * (mp0 + W * i) + h) * kPolK1 + s);
  }
  __device__ __forceinline__ void load_bias(const float *b1, int wv, int i, f32x4 (&b)[2]) {
    const int mp = (SH == 1 ? wv : wv % HP) + W * i, lg = __lane_id() >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) b[h] = gld(reinterpret_cast<const f32x4 *>(b1 + 32 * mp + 16 * h + 4 * lg), 0);
  }
  // the first K-steps' fragments, ahead of run()
  __device__ __forceinline__ void start(__amdgpu_buffer_rsrc_t w1, [[maybe_unused]] const float *b1, int wv) {
    pin();
#pragma unroll
    for (int s = 0; s < D; ++s) load(w1, wv, s);
    if constexpr (HELD) {
#pragma unroll
      for (int i = 0; i < NI; ++i) load_bias(b1, wv, i, bias[i]);
    }
    pin();
  }
  __device__ __forceinline__ void run(__amdgpu_buffer_rsrc_t w1, const float *b1, const lds_u32x4 *xb, int xrow,
                                      lds_u32x4 *hb, int wv) {
    const int lane = __lane_id(), col = lane & 15, lg = lane >> 4;
    const int mp0 = SH == 1 ? wv : wv % HP, n0 = SH == 1 ? 0 : (wv / HP) * NN;
    if (n0 >= NT) return;
    f32x4 c[NI][2][NN];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int n = 0; n < NN; ++n) c[i][0][n] = c[i][1][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < K1; ++s) {
#pragma unroll
      for (int n = 0; n < NN; ++n) {
        const u32x4 b = xb[(16 * (n0 + n) + col) * xrow + 4 * s + lg];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          c[i][0][n] = mfma_bf16(a[s % D][i][0], b, c[i][0][n]);
          c[i][1][n] = mfma_bf16(a[s % D][i][1], b, c[i][1][n]);
        }
      }
      if constexpr (!HELD) {
        pin();
        if (s + D < K1) load(w1, wv, s + D);
        pin();
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int mp = mp0 + W * i;
      f32x4 b[2];
      if constexpr (HELD) b[0] = bias[i][0], b[1] = bias[i][1];
      else load_bias(b1, wv, i, b);
#pragma unroll
      for (int n = 0; n < NN; ++n) hb[(mp * NT + n0 + n) * 64 + lane] = hidden_frag(c[i][0][n], c[i][1][n], b[0], b[1]);
    }
  }
};

// The logits of port groups grp (4 ports) for 16 NT envs: c[r][n] holds levels
// 4 r .. 4 r + 3 of port 4 grp + lane / 16 of env 16 n + lane % 16.  run()
// leaves the first K-steps of group `next` (if >= 0) in flight.  HELD: one group's
// fragments and biases, all of them, for many run()s.
template <int NT, int HP, bool HELD = false, int DEPTH = kRing>
struct LogitLayer {
  static constexpr int D = HELD ? HP : ring_depth(HP, DEPTH);   // divides HP
  u32x4 w[D][kPolR];
  f32x4 bias[HELD ? kPolR : 1];   // HELD

  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t w2, int grp, int s) {
#pragma unroll
    for (int r = 0; r < kPolR; ++r) w[s % D][r] = frag(w2, (grp * kPolR + r) * kPolHP + s);
  }
  __device__ __forceinline__ f32x4 load_bias(const float *b2f, int grp, int r) {
    return gld(reinterpret_cast<const f32x4 *>(b2f + (int64_t)(grp * kPolR + r) * 16 + 4 * (__lane_id() >> 4)), 0);
  }
  __device__ __forceinline__ void start(__amdgpu_buffer_rsrc_t w2, [[maybe_unused]] const float *b2f, int grp) {
    pin();
#pragma unroll
    for (int s = 0; s < D; ++s) load(w2, grp, s);
    if constexpr (HELD) {
#pragma unroll
      for (int r = 0; r < kPolR; ++r) bias[r] = load_bias(b2f, grp, r);
    }
    pin();
  }
  __device__ __forceinline__ void run(__amdgpu_buffer_rsrc_t w2, const float *b2f, const lds_u32x4 *hb, int grp, int next,
                                      f32x4 (&c)[kPolR][NT]) {
    const int lane = __lane_id();
#pragma unroll
    for (int r = 0; r < kPolR; ++r) {
      f32x4 b;
      if constexpr (HELD) b = bias[r];
      else b = load_bias(b2f, grp, r);
#pragma unroll
      for (int n = 0; n < NT; ++n) c[r][n] = b;
    }
#pragma unroll
    for (int s = 0; s < HP; ++s) {
      u32x4 hv[NT];
#pragma unroll
      for (int n = 0; n < NT; ++n) hv[n] = hb[(s * NT + n) * 64 + lane];
#pragma unroll
      for (int r = 0; r < kPolR; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n) c[r][n] = mfma_bf16(w[s % D][r], hv[n], c[r][n]);
      if constexpr (!HELD) {
        pin();
        if (s + D < HP) load(w2, grp, s + D);
        else if (next >= 0) load(w2, next, s + D - HP);
        pin();
      }
    }
  }
};

}  // namespace
}  // namespace cx
