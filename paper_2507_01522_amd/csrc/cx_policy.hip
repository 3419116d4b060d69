// cx_policy.hip -- policy-in-the-loop rollouts.
//   k_policy  obs -> BF16 -> W1 (tanh) -> W2 -> logits on the matrix cores
//             (v_mfma_f32_16x16x32_bf16, FP32 accumulation), then per port a
//             level drawn from softmax of its logits with one Philox uniform
//             (k_policy_few: the same for many rows of few ports).
// A rollout of a class of 8, 16 or 32 slots is one launch of the fused
// persistent kernel (the rollout kernel with this MLP between its steps,
// cx_kernels.hip): state in registers, observations only in LDS.  Other
// classes, and the rollout that allocates nothing, run two kernels per step:
// k_policy, then the one-step environment kernel with its levels as external
// actions, which writes the next observation.  k_observe gives the
// observation of the state a rollout starts from.
//
// The layout of the two products is described in cx_mlp.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <mutex>
#include <vector>

#include "cx_ctx.h"
#include "cx_device.h"
#include "cx_mlp.h"

namespace cx {

struct PolicyRt {
  int hidden = 0, in_dim = 0, N = 0, L1 = 0;
  int K1 = 0, HP = 0, G = 0;
  // weights in fragment order and FP32 biases, padded to the largest sizes
  // (features and W2 with zeros, hidden units with copies of the first, the biases
  // of levels past the class's with the lowest float): W1^T [16 tiles][8 K-steps][64],
  // b1 [256], W2^T [G][3][8][64], b2 [G][3][16]
  void *mem = nullptr;
  const u32x4 *w1p = nullptr;
  const float *b1p = nullptr;
  const u32x4 *w2p = nullptr;
  const float *b2p = nullptr;
  float *obs = nullptr;  // one step of observations (rollouts that do not return them)
  uint8_t *act = nullptr;  // one step of levels (rollouts that do not return them)
  int64_t scratch_envs = 0;
  // the fused rollout's segment table (stations of 8 or 16 lanes, 4 waves per block)
  SegDev *segs_dev = nullptr;
  int lanes = 8, n_segs = 0, n_blocks = 0;
};

namespace {

// One block of the standalone policy kernel: W waves, E = 16 NT observations.
// They are converted to BF16 fragments in LDS; the waves split the hidden units,
// then the port groups, as in the fused rollout, and read their weight
// fragments from L2 straight into the matrix-core operands.
template <int W, int NT, int K1, int HP>
__device__ __forceinline__ void policy_block(const PolicyArgs &a, lds_u32x4 *xb, lds_u32x4 *hb) {
  constexpr int E = 16 * NT, CPR = 4 * K1, XR = kPolXbRow;
  const int tid = threadIdx.x, lane = __lane_id(), wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, lg = lane >> 4;
  const int64_t e0 = (int64_t)blockIdx.x * E;
  const int n_e = (int)(a.n - e0 < E ? a.n - e0 : E);
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  const __amdgpu_buffer_rsrc_t w1 = frag_rsrc(a.w1f, 2 * kPolHP * kPolK1);
  HiddenLayer<W, NT, K1, HP> hid;
  hid.start(w1, a.b1, wv);
  const float *obs = a.obs + e0 * a.in_dim;
  for (int c = tid; c < E * CPR; c += 64 * W) {
    const int e = c / CPR, k = c % CPR, f = 8 * k;
    const float *row = obs + (int64_t)e * a.in_dim + f;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (e < n_e) {
      if (f + 8 <= a.in_dim) {
        const f4u x = gld(reinterpret_cast<const f4u *>(row), 0), y = gld(reinterpret_cast<const f4u *>(row + 4), 0);
        v = u32x4{pack2(x.x, x.y), pack2(x.z, x.w), pack2(y.x, y.y), pack2(y.z, y.w)};
      } else if (f < a.in_dim) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = f + j < a.in_dim ? gld(row, j) : 0.f;
        v = u32x4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
      }
    }
    xb[e * XR + k] = v;
  }
  __syncthreads();
  hid.run(w1, a.b1, xb, XR, hb, wv);
  const __amdgpu_buffer_rsrc_t w2 = frag_rsrc(a.w2f, a.G * kPolR * kPolHP);
  LogitLayer<NT, HP> logit;
  logit.start(w2, a.b2f, min(wv, a.G - 1));
  // the lane's ports are 4 wv + lg + 4 W i, a multiple of 16 apart: one Philox
  // call per observation serves them all
  U4 dw[NT];
  if (a.act) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
      dw[n] = philox((uint32_t)(a.env0 + e0 + 16 * n + col), a.g, draw_index(4 * wv + lg), kDomGum, (uint32_t)a.seed,
                     (uint32_t)(a.seed >> 32));
  }
  __syncthreads();
  // Levels and logits gather in LDS, over the observations, which are no longer
  // needed.  The levels leave as one contiguous run at the end; the logits of one
  // tile (16 observations) and W port groups leave together, each observation's
  // 4 W L1 floats (704 bytes at W = 4 and 11 levels) by one wave in 16-byte
  // stores: stored from the lanes that hold them, 44 bytes a lane at that
  // stride, 65,537 x 352 logits took 72 us a call, of which 29 the stores.
  __attribute__((address_space(3))) uint8_t *lev = (__attribute__((address_space(3))) uint8_t *)xb;
  __attribute__((address_space(3))) float *zs = (__attribute__((address_space(3))) float *)xb;
  constexpr int ZR = 4 * W * 4 * kPolR + 4;   // floats per observation's row
  static_assert(16 * ZR * 4 <= E * XR * 16, "the logits of a tile fit over the observations");
  for (int g0 = 0; g0 < a.G; g0 += W) {
    const int grp = min(g0 + wv, a.G - 1), port = 4 * (g0 + wv) + lg;
    f32x4 c[kPolR][NT];
    logit.run(w2, a.b2f, hb, grp, g0 + W < a.G ? min(g0 + W + wv, a.G - 1) : -1, c);
    if (a.logits) {
      const int n_z = min(4 * W, a.N - 4 * g0) * a.L1;   // floats per observation of these groups
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        if (port < a.N) {
          __attribute__((address_space(3))) float *z = zs + col * ZR + (4 * wv + lg) * a.L1;
#pragma unroll
          for (int l = 0; l < 4 * kPolR; ++l)
            if (l < a.L1) z[l] = c[l >> 2][n][l & 3];
        }
        __syncthreads();
        for (int r = wv; r < 16 && 16 * n + r < n_e; r += W) {
          float *out = a.logits + (e0 + 16 * n + r) * ((int64_t)a.N * a.L1) + (int64_t)4 * g0 * a.L1;
          const __attribute__((address_space(3))) float *row = zs + r * ZR;
          for (int i = 4 * lane; i + 4 <= n_z; i += 256)
            gst(reinterpret_cast<f4u *>(out + i), 0, (f4u){row[i], row[i + 1], row[i + 2], row[i + 3]});
          const int i = (n_z & ~3) + lane;
          if (i < n_z) gst(out, i, (float)row[i]);
        }
        __syncthreads();
      }
    }
    if (a.act && port < a.N) {
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const f32x4 cn[kPolR] = {c[0][n], c[1][n], c[2][n]};
        lev[(16 * n + col) * a.N + port] = (uint8_t)sample_level(cn, a.L1, draw_uniform(draw_word(dw[n], port)));
      }
    }
  }
  if (!a.act) return;
  __syncthreads();
  uint8_t *out = a.act + e0 * a.N;
  const int bytes = n_e * a.N;
  if ((reinterpret_cast<uintptr_t>(out) & 3u) == 0) {
    for (int i = tid; i < bytes >> 2; i += 64 * W)
      gst(reinterpret_cast<uint32_t *>(out), i, *reinterpret_cast<const __attribute__((address_space(3))) uint32_t *>(lev + 4 * i));
    const int i = (bytes & ~3) + tid;
    if (i < bytes) gst(out, i, (uint8_t)lev[i]);
  } else {
    for (int i = tid; i < bytes; i += 64 * W) gst(out, i, (uint8_t)lev[i]);
  }
}

template <int W, int NT>
__device__ __forceinline__ void policy_sizes(const PolicyArgs &a, lds_u32x4 *xb, lds_u32x4 *hb) {
  if (a.K1 <= 4) {  // up to 128 features (20 ports)
    if (a.HP <= 2) policy_block<W, NT, 4, 2>(a, xb, hb);
    else if (a.HP <= 4) policy_block<W, NT, 4, 4>(a, xb, hb);
    else policy_block<W, NT, 4, 8>(a, xb, hb);
  } else {
    if (a.HP <= 2) policy_block<W, NT, 8, 2>(a, xb, hb);
    else if (a.HP <= 4) policy_block<W, NT, 8, 4>(a, xb, hb);
    else policy_block<W, NT, 8, 8>(a, xb, hb);
  }
}

// 32 observations per block, whatever their number: 65,537 observations (32
// ports, 256 hidden units) take 43 us a draw; blocks of 64 take 46, of 16 62, and
// the blocks of 256 that this kernel had, one per CU and one block too many,
// 137.  300 observations: 11 us, 63 before.
constexpr int kPolWaves = 4, kPolNT = 2;
constexpr size_t kPolLds = (size_t)16 * kPolNT * kPolXbRow * 16 + (size_t)kPolHP * kPolNT * 1024;

__global__ __launch_bounds__(64 * kPolWaves) void k_policy(PolicyArgs a) {
  extern __shared__ u32x4 pol_lds[];
  lds_u32x4 *xb = (lds_u32x4 *)pol_lds;
  policy_sizes<kPolWaves, kPolNT>(a, xb, xb + 16 * kPolNT * kPolXbRow);
}

// Stations of up to 8 ports: one or two port groups leave most waves of such a
// block idle at the draw, and its barriers are most of its time.  Here a wave takes
// 16 NT observations through both products by itself: its lanes load them as the
// first product reads them, and the hidden units it leaves in a lane are what the
// second reads there.  The products are the block's, K-step by K-step in the same
// order, with the policy's own number of hidden units.  Bound by the draw and, at 256
// hidden units, the tanh; levels of 1,000,000 rows in blocks / here: 1 port, 32 hidden
// units 180 / 33 us, 256 263 / 106; 8 ports 186 / 61 and 281 / 160.  The bounds on
// waves keep the compiler from loading every fragment ahead: 74, 92 and 150 registers at
// 64, 128 and 256 hidden units, 96, 152 and 280 (one wave per SIMD) without them.
template <int NT, int K1, int HP>
__global__ __launch_bounds__(64 * kPolWaves)
__attribute__((amdgpu_waves_per_eu(HP == 8 ? 3 : HP == 4 ? 4 : 5))) void k_policy_few(PolicyArgs a) {
  const int lane = __lane_id(), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int col = lane & 15, lg = lane >> 4;
  const int64_t e0 = ((int64_t)blockIdx.x * kPolWaves + wv) * (16 * NT);
  if (e0 >= a.n) return;
  const int n_e = (int)(a.n - e0 < 16 * NT ? a.n - e0 : 16 * NT);
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  const __amdgpu_buffer_rsrc_t w1 = frag_rsrc(a.w1f, 2 * kPolHP * kPolK1);
  const __amdgpu_buffer_rsrc_t w2 = frag_rsrc(a.w2f, a.G * kPolR * kPolHP);
  const float *obs = a.obs + e0 * a.in_dim;
  u32x4 x[K1][NT];
#pragma unroll
  for (int s = 0; s < K1; ++s)
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int e = 16 * n + col, f = 32 * s + 8 * lg;
      const float *row = obs + (int64_t)e * a.in_dim + f;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (e < n_e) {
        if (f + 8 <= a.in_dim) {
          const f4u p = gld(reinterpret_cast<const f4u *>(row), 0), q = gld(reinterpret_cast<const f4u *>(row + 4), 0);
          v = u32x4{pack2(p.x, p.y), pack2(p.z, p.w), pack2(q.x, q.y), pack2(q.z, q.w)};
        } else if (f < a.in_dim) {
          float r[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) r[j] = f + j < a.in_dim ? gld(row, j) : 0.f;
          v = u32x4{pack2(r[0], r[1]), pack2(r[2], r[3]), pack2(r[4], r[5]), pack2(r[6], r[7])};
        }
      }
      x[s][n] = v;
    }
  u32x4 h[HP][NT];
#pragma unroll
  for (int m = 0; m < HP; ++m) {
    f32x4 c[2][NT], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      b[i] = gld(reinterpret_cast<const f32x4 *>(a.b1 + 32 * m + 16 * i + 4 * lg), 0);
#pragma unroll
      for (int n = 0; n < NT; ++n) c[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < K1; ++s) {
        const u32x4 w = frag(w1, (2 * m + i) * kPolK1 + s);
#pragma unroll
        for (int n = 0; n < NT; ++n) c[i][n] = mfma_bf16(w, x[s][n], c[i][n]);
      }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) h[m][n] = hidden_frag(c[0][n], c[1][n], b[0], b[1]);
  }
  for (int grp = 0; grp < a.G; ++grp) {
    const int port = 4 * grp + lg;
    f32x4 c[kPolR][NT];
#pragma unroll
    for (int r = 0; r < kPolR; ++r) {
      const f32x4 b = gld(reinterpret_cast<const f32x4 *>(a.b2f + (grp * kPolR + r) * 16 + 4 * lg), 0);
#pragma unroll
      for (int n = 0; n < NT; ++n) c[r][n] = b;
    }
#pragma unroll
    for (int s = 0; s < HP; ++s)
#pragma unroll
      for (int r = 0; r < kPolR; ++r) {
        const u32x4 w = frag(w2, (grp * kPolR + r) * kPolHP + s);
#pragma unroll
        for (int n = 0; n < NT; ++n) c[r][n] = mfma_bf16(w, h[s][n], c[r][n]);
      }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int e = 16 * n + col;
      if (port >= a.N || e >= n_e) continue;
      if (a.logits) {
        float *z = a.logits + ((e0 + e) * a.N + port) * (int64_t)a.L1;
#pragma unroll
        for (int l = 0; l < 4 * kPolR; ++l)
          if (l < a.L1) gst(z, l, (float)c[l >> 2][n][l & 3]);
      }
      if (a.act) {
        const U4 w = philox((uint32_t)(a.env0 + e0 + e), a.g, draw_index(port), kDomGum, (uint32_t)a.seed,
                            (uint32_t)(a.seed >> 32));
        const f32x4 cn[kPolR] = {c[0][n], c[1][n], c[2][n]};
        gst(a.act, (e0 + e) * a.N + port, (uint8_t)sample_level(cn, a.L1, draw_uniform(draw_word(w, port))));
      }
    }
  }
}
// Chosen by rows and ports: below about 16,384 rows its waves do not fill the chip and
// their longer chain shows (4,000 rows of 4 ports, 256 hidden units: levels 7.8 us in
// blocks, 9.6 here; 30,000 rows 14.2 and 9.7), and logits of more than one port group
// leave in larger pieces from a block (200,000 rows of 4 ports, 32 hidden units 45 us
// in blocks, 39 here, of 5 49 and 53, of 8 46 and 77).
constexpr int kFewNT = 2;
constexpr int64_t kFewRows = 16384;
bool few_ports(const PolicyArgs &a) { return a.n >= kFewRows && a.N <= (a.logits ? 4 : 8); }
static_assert((6 * 8 + 4 + 31) / 32 == 2, "k_policy_few is built for one and two K-steps of features");

// Observation of the current state (the features the step kernel records).
__global__ void k_observe(const ClassDev *cls, int64_t n_envs, const double *q, const float *u,
                          const float *p_last, const int16_t *dwell, const uint8_t *utype, const double *bsoc,
                          const float *bp, const float *rbar, int32_t t_day, uint64_t seed, int64_t env0, uint32_t g,
                          float *obs) {
  const ClassDev C = *cls;
  const int S = C.S, N = C.n_ports, dim = C.obs_dim;
  const int64_t total = n_envs * S;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t env = i / S;
    const int s = (int)(i - env * S);
    const int port = C.slot_port[s];
    if (port < 0) continue;
    const int dw = dwell[i];
    const bool cs = C.has_users && utype[i] != 0;
    const bool occ = dw > 0 || cs;
    const float qf = (float)q[i];
    float *o = obs + env * dim + port;
    o[0 * N] = occ ? 1.0f : 0.0f;
    o[1 * N] = occ ? 1.0f - qf : 0.0f;
    o[2 * N] = occ ? qf - u[i] : 0.0f;
    o[3 * N] = (float)dw * C.inv_steps_ep;
    float rh = fminf(1.0f, qf * C.inv_1mtau);
    if (C.n_models > 0) rh *= rbar[i] * C.slot_inv_pmax[s];  // the car's curve, as a share of the port maximum
    o[4 * N] = occ ? rh : 0.0f;
    o[5 * N] = p_last[i] * C.slot_inv_pmax[s];
    if (C.has_users) obs[env * dim + C.user_obs + port] = cs ? 1.0f : 0.0f;
  }
  for (int64_t env = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; env < n_envs;
       env += (int64_t)gridDim.x * blockDim.x) {
    int n_occ = 0;
    for (int s = 0; s < S; ++s)
      n_occ += (dwell[env * S + s] > 0 || (C.has_users && utype[env * S + s] != 0)) ? 1 : 0;
    float *o = obs + env * dim + 6 * N;
    o[0] = C.glob[t_day * 4 + 0];
    o[1] = C.glob[t_day * 4 + 1];
    o[2] = C.glob[t_day * 4 + 2];
    o[3] = (float)n_occ * (1.0f / (float)N);
    if (C.has_batt) {
      o[4] = (float)bsoc[env];
      o[5] = bp[env] * C.b_inv_rate;
    }
    if (C.n_days > 0) {  // the episode's price day, drawn at the step it began
      const int d = episode_day((uint32_t)(env0 + env), g - (uint32_t)t_day, (uint32_t)seed, (uint32_t)(seed >> 32),
                                C.n_days);
      o[2] = C.price_days[(int64_t)d * C.steps_ep + t_day];
      obs[env * dim + C.day_obs] = (float)d * C.inv_n_days;
      obs[env * dim + C.day_obs + 1] = d % 7 >= 5 ? 1.0f : 0.0f;
    }
  }
}

hipError_t launch_policy(const PolicyArgs &a, hipStream_t st) {
  // a launch has fewer than 2^32 threads: 537 M rows each
  const bool few = few_ports(a);
  const int64_t rows = few ? 16 * kFewNT * kPolWaves : 16 * kPolNT;
  const int64_t max_rows = kMaxLaunchThreads / (64 * kPolWaves) * rows;
  for (int64_t r = 0; r < a.n; r += max_rows) {
    PolicyArgs b = a;
    b.n = std::min(a.n - r, max_rows);
    b.obs += r * a.in_dim;
    if (b.act) b.act += r * a.N;
    if (b.logits) b.logits += r * a.N * a.L1;
    b.env0 += r;
    using Fn = void (*)(PolicyArgs);
    static const Fn kFew[2][4] = {
        {&k_policy_few<kFewNT, 1, 1>, &k_policy_few<kFewNT, 1, 2>, &k_policy_few<kFewNT, 1, 4>, &k_policy_few<kFewNT, 1, 8>},
        {&k_policy_few<kFewNT, 2, 1>, &k_policy_few<kFewNT, 2, 2>, &k_policy_few<kFewNT, 2, 4>, &k_policy_few<kFewNT, 2, 8>}};
    const Fn f = few ? kFew[a.K1 - 1][a.HP <= 1 ? 0 : a.HP <= 2 ? 1 : a.HP <= 4 ? 2 : 3] : &k_policy;
    void *params[1] = {&b};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(f), dim3((unsigned)((b.n + rows - 1) / rows)),
                                         dim3(64 * kPolWaves), params, few ? 0 : kPolLds, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_observe(const cx_ctx *ctx, float *obs, hipStream_t st) {
  for (const ClassRt &c : ctx->classes) {
    if (c.n_envs == 0) continue;
    const int64_t work = c.n_envs * c.comp.S;
    const int blocks = (int)std::min<int64_t>(4096, (work + 255) / 256);
    hipLaunchKernelGGL(k_observe, dim3(blocks), dim3(256), 0, st, c.dev, c.n_envs, ctx->q + c.slot_off,
                       ctx->u + c.slot_off, ctx->p_last + c.slot_off, ctx->dwell + c.slot_off,
                       ctx->utype + c.slot_off, ctx->bsoc + c.env_begin, ctx->bp + c.env_begin,
                       ctx->rbar + c.slot_off, ctx->t_day, ctx->seed, c.env_begin, ctx->g, obs + c.obs_off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

PolicyArgs policy_args(const cx_ctx *ctx, const float *obs, int64_t n) {
  const PolicyRt &p = *ctx->policy;
  PolicyArgs a{};
  a.obs = obs;
  a.n = n;
  a.in_dim = p.in_dim; a.K1 = p.K1; a.HP = p.HP; a.G = p.G; a.N = p.N; a.L1 = p.L1;
  a.w1f = p.w1p; a.b1 = p.b1p; a.w2f = p.w2p; a.b2f = p.b2p;
  a.seed = ctx->seed;
  a.env0 = ctx->classes[0].env_begin;
  return a;
}

double bf16_to_double(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

cx_status ensure_scratch(cx_ctx *ctx) {
  PolicyRt &p = *ctx->policy;
  if (p.scratch_envs >= ctx->n_envs) return CX_OK;
  if (p.obs) (void)hipFree(p.obs);
  if (p.act) (void)hipFree(p.act);
  p.obs = nullptr;
  p.act = nullptr;
  p.scratch_envs = 0;
  if (hipMalloc(&p.obs, sizeof(float) * ctx->obs_elems) != hipSuccess ||
      hipMalloc(&p.act, (size_t)ctx->total_ports) != hipSuccess)
    return fail_status(CX_E_OOM, "policy rollout: scratch allocation failed");
  p.scratch_envs = ctx->n_envs;
  return CX_OK;
}

}  // namespace

void free_policy(cx_ctx *ctx) {
  if (!ctx || !ctx->policy) return;
  PolicyRt *p = ctx->policy;
  if (p->mem) (void)hipFree(p->mem);
  if (p->segs_dev) (void)hipFree(p->segs_dev);
  if (p->obs) (void)hipFree(p->obs);
  if (p->act) (void)hipFree(p->act);
  delete p;
  ctx->policy = nullptr;
}

namespace {

// One policy rollout with the given scratch: obs_scr one step of observations
// (obs_elems floats), act_scr one step of levels (total_ports bytes).  Every
// element of both is written before it is read, so their contents on entry do
// not matter.
cx_status policy_step_with(cx_ctx *ctx, int32_t T, cx_out_mode out_mode, const cx_traj *out, float *obs_scr,
                           uint8_t *act_scr) {
  const bool ret_obs = out && out_mode == CX_OUT_FULL && out->obs;
  const bool ret_act = out && out_mode != CX_OUT_REWARD && out->actions;
  if (ret_obs && (reinterpret_cast<uintptr_t>(out->obs) & 15u) != 0)
    return fail_status(CX_E_INVALID, "policy rollout: obs buffer must be 16-byte aligned");
  hipError_t e = launch_observe(ctx, obs_scr, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "policy rollout: observation kernel");
  const float *obs_prev = obs_scr;
  for (int32_t t = 0; t < T; ++t) {
    float *obs_t = ret_obs ? out->obs + (int64_t)t * ctx->obs_elems : obs_scr;
    uint8_t *act_t = ret_act ? out->actions + (int64_t)t * ctx->total_ports : act_scr;
    PolicyArgs pa = policy_args(ctx, obs_prev, ctx->n_envs);
    pa.g = ctx->g + (uint32_t)t;
    pa.act = act_t;
    if ((e = launch_policy(pa, ctx->stream)) != hipSuccess) return hip_fail(ctx, e, "policy kernel");
    LaunchArgs a = base_args(ctx);
    a.T = 1;
    a.g0 = ctx->g + (uint32_t)t;
    a.t_day0 = (int32_t)(((int64_t)ctx->t_day + t) % ctx->steps_ep);
    a.mode = CX_ACT_EXTERNAL;
    a.out_mode = CX_OUT_FULL;
    a.act_in = act_t;
    a.obs = obs_t;
    a.act = nullptr;
    a.reward = out && out->reward ? out->reward + (int64_t)t * ctx->n_envs : nullptr;
    a.done = out && out->done ? out->done + (int64_t)t * ctx->n_envs : nullptr;
    if ((e = launch_groups(a, ctx->groups.data(), (int)ctx->groups.size(), ctx->stream)) !=
        hipSuccess)
      return hip_fail(ctx, e, "policy rollout: step kernel");
    obs_prev = obs_t;
  }
  // the next rollout starts from the observation kernel again (it does not
  // read obs_prev), so the clock is the only state carried here
  advance_clock(ctx, T);
  return CX_OK;
}

}  // namespace

// Scratch of the rollout that allocates nothing (cx_rollout_policy_noalloc):
// a fixed array of the device image, one per GPU the library runs on, held
// until the process ends.  In host code its name is only a stand-in for the
// device array: the address kernels take is looked up per device.
constexpr size_t kNoAllocScratchBytes = (size_t)CX_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on `device`, looked up on the first call for
// that device with the device current (each GPU has its own copy).
cx_status noalloc_scratch(int device, unsigned char **ptr) {
  if (device < 0 || device >= kMaxDevices) return fail_status(CX_E_INVALID, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return fail_status(CX_E_DEVICE, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess)
      return fail_status(CX_E_DEVICE, std::string("hipSetDevice: ") + hipGetErrorString(e));
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p)
      return fail_status(CX_E_DEVICE, std::string("hipGetSymbolAddress of the no-allocation scratch: ") +
                                          hipGetErrorString(e));
    g_scratch_ptr[device] = p;
  }
  *ptr = static_cast<unsigned char *>(g_scratch_ptr[device]);
  return CX_OK;
}

}  // namespace

namespace {

// The fused rollout runs classes of 8, 16 or 32 slots (stations of 8 lanes, 1, 2
// or 4 slots per lane); larger ones take the two kernels per step.  So do classes
// that are not SIMPLE in a packing of several slots per lane: their station sums
// are in that packing's order, the fused kernel's in the order of one slot per
// lane (the default), and records are those of the two kernels bit for bit.
bool fused_eligible(const cx_ctx *ctx) {
  const ClassRt &c = ctx->classes[0];
  const int S = c.comp.S, kind = c.host_view.kind;
  return (S == 8 || S == 16 || S == 32) && (kind == kKindSimple || (kind == kKindGeneral && c.lanes == S));
}

cx_status ensure_fused(cx_ctx *ctx) {
  PolicyRt &p = *ctx->policy;
  if (p.segs_dev) return CX_OK;
  const ClassRt &c = ctx->classes[0];
  std::vector<SegDev> segs;
  // 16-slot stations take 16 lanes each (16 stations a block) while that gives
  // every block a CU of its own: half the MLP and a shorter step per block (96
  // steps of 4,096 such envs, 256 hidden units, every record: 253 us, 383 with 8
  // lanes)
  int blocks = 0;
  for (p.lanes = c.comp.S == 16 ? 16 : 8;; p.lanes = 8) {
    segs.clear();
    class_segments(ctx, c, p.lanes, c.comp.S / p.lanes, &segs);
    blocks = 0;
    for (SegDev &sg : segs) {
      sg.block_begin = blocks;
      blocks += (sg.n_groups + kPolRolloutWaves - 1) / kPolRolloutWaves;
    }
    if (p.lanes == 8 || blocks <= kPolHeldBlocks) break;
  }
  void *d = nullptr;
  if (hipMalloc(&d, sizeof(SegDev) * std::max<size_t>(1, segs.size())) != hipSuccess)
    return fail_status(CX_E_OOM, "policy rollout: segment table allocation failed");
  hipError_t e = hipMemcpy(d, segs.data(), sizeof(SegDev) * segs.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(d);
    return hip_fail(ctx, e, "policy rollout: segment table upload");
  }
  p.segs_dev = static_cast<SegDev *>(d);
  p.n_segs = (int)segs.size();
  p.n_blocks = blocks;
  return CX_OK;
}

// One launch for the whole rollout: the observation the rollout starts from
// (into the scratch), then the persistent kernel with the MLP between steps.
cx_status fused_rollout(cx_ctx *ctx, int32_t T, cx_out_mode out_mode, const cx_traj *out) {
  PolicyRt &p = *ctx->policy;
  const ClassRt &c = ctx->classes[0];
  const bool ret_obs = out && out_mode == CX_OUT_FULL && out->obs;
  const bool ret_act = out && out_mode != CX_OUT_REWARD && out->actions;
  LaunchArgs::Pol lay{};
  int32_t stage_off = 0, stage_floats = 0;
  const auto plan = [&](bool over_stage) {
    return policy_rollout_lds(c.tab.dwell_log2, c.comp.obs_dim, c.comp.N, over_stage, &stage_off, &stage_floats,
                              &lay.hb_off, &lay.xb_off, &lay.act_off);
  };
  bool held = p.n_blocks <= kPolHeldBlocks;
  size_t lds = plan(!policy_dual(c.comp.S, held));
  if (lds > kMaxBlockLds) {   // 32 slots and a stay table of more than 1024 entries
    held = false;
    lds = plan(true);
  }
  hipError_t e = launch_observe(ctx, p.obs, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "policy rollout: observation kernel");
  LaunchArgs a = base_args(ctx);
  a.segs = p.segs_dev;
  a.n_segs = p.n_segs;
  a.T = T;
  a.mode = CX_ACT_POLICY;
  a.out_mode = out_mode;
  a.obs = ret_obs ? out->obs : nullptr;
  a.act = ret_act ? out->actions : nullptr;
  a.reward = out ? out->reward : nullptr;
  a.done = out ? out->done : nullptr;
  a.stage_off = stage_off;
  a.stage_floats = stage_floats;
  // launches with held weights keep the day's tables in LDS too, where they fit: a
  // step with all weights held then loads nothing from device memory and waits for no
  // record
  const size_t days = (size_t)ctx->steps_ep * 20;
  if (held && ctx->steps_ep <= kLdsExoSteps && lds + days <= kMaxBlockLds) {
    a.day_off = (int32_t)lds;
    lds += days;
  }
  a.pol = lay;
  a.pol.obs0 = p.obs;
  a.pol.w1f = p.w1p;
  a.pol.b1 = p.b1p;
  a.pol.w2f = p.w2p;
  a.pol.b2f = p.b2p;
  a.pol.in_dim = p.in_dim;
  a.pol.HP = p.HP;
  a.pol.G = p.G;
  a.pol.L1 = p.L1;
  if ((e = launch_policy_rollout(a, c.host_view.kind == kKindSimple, p.lanes, c.comp.S / p.lanes, held,
                                 p.n_blocks, lds, ctx->stream)) != hipSuccess)
    return hip_fail(ctx, e, "policy rollout kernel");
  advance_clock(ctx, T);
  return CX_OK;
}

}  // namespace

cx_status policy_step(cx_ctx *ctx, int32_t T, cx_out_mode out_mode, const cx_traj *out, bool graph) {
  (void)graph;
  if (!ctx->policy) return fail_status(CX_E_INVALID, "no policy set (cx_set_policy)");
  cx_status st = ensure_scratch(ctx);
  if (st != CX_OK) return st;
  if (fused_eligible(ctx)) {
    const bool ret_obs = out && out_mode == CX_OUT_FULL && out->obs;
    if (ret_obs && (reinterpret_cast<uintptr_t>(out->obs) & 15u) != 0)
      return fail_status(CX_E_INVALID, "policy rollout: obs buffer must be 16-byte aligned");
    const ClassRt &c = ctx->classes[0];
    LaunchArgs::Pol lay{};
    int32_t stage_off = 0, stage_floats = 0;
    const size_t lds = policy_rollout_lds(c.tab.dwell_log2, c.comp.obs_dim, c.comp.N, true, &stage_off,
                                          &stage_floats, &lay.hb_off, &lay.xb_off, &lay.act_off);
    if (lds <= kMaxBlockLds) {
      if (T == 0) return CX_OK;
      if ((st = ensure_fused(ctx)) != CX_OK) return st;
      return fused_rollout(ctx, T, out_mode, out);
    }
  }
  return policy_step_with(ctx, T, out_mode, out, ctx->policy->obs, ctx->policy->act);
}

}  // namespace cx

using namespace cx;

extern "C" {

cx_status cx_set_policy(cx_ctx *ctx, int32_t hidden, const uint16_t *w1, const uint16_t *b1,
                        const uint16_t *w2, const uint16_t *b2) {
  if (!ctx) return fail_status(CX_E_INVALID, "context is NULL");
  if (ctx->failed) return fail_status(CX_E_DEVICE, "context has a sticky device error");
  if (!w1 || !b1 || !w2 || !b2) return fail_status(CX_E_INVALID, "cx_set_policy: NULL weight array");
  if (ctx->classes.size() != 1) return fail_status(CX_E_INVALID, "cx_set_policy: single-class contexts only");
  const ClassRt &c = ctx->classes[0];
  if (c.comp.extended())
    return fail_status(CX_E_INVALID, "cx_set_policy: charging-only stations only (no V2G, no battery)");
  const int N = c.comp.N, L1 = c.spec.s.n_levels + 1, in_dim = 6 * N + 4;
  if (hidden < 32 || hidden > 32 * kPolHP || hidden % 32 != 0)
    return fail_status(CX_E_INVALID, "cx_set_policy: hidden must be a multiple of 32 in 32..256");
  if (in_dim > 32 * kPolK1)
    return fail_status(CX_E_INVALID, "cx_set_policy: observations longer than 256 (more than 42 ports)");
  if (L1 > 4 * kPolR) return fail_status(CX_E_INVALID, "cx_set_policy: at most 11 levels per port");
  const int K1 = (in_dim + 31) / 32, HP = hidden / 32, G = (N + 3) / 4;
  const int HP_kernel = HP <= 2 ? 2 : HP <= 4 ? 4 : 8;   // what the kernels are built for
  const int out_dim = N * L1;
  // W1^T fragments: tile m (hidden 16m..16m+15), K-step s at (m * 8 + s), lane l
  // -> hidden 16m + l % 16, features 32s + 8 (l / 16) + j.  Hidden units past the
  // policy's are copies of its first, with weights 0 in W2: zeros would make 0 x inf
  // of an infinite observation, whose own hidden units are +-1.
  std::vector<uint16_t> w1p((size_t)2 * kPolHP * kPolK1 * 64 * 8, 0);
  for (int m = 0; m < 2 * HP_kernel; ++m)
    for (int s = 0; s < K1; ++s)
      for (int l = 0; l < 64; ++l)
        for (int j = 0; j < 8; ++j) {
          const int f = 32 * s + 8 * (l >> 4) + j, hu = 16 * m + (l & 15);
          if (f < in_dim)
            w1p[(((size_t)m * kPolK1 + s) * 64 + l) * 8 + j] = w1[(size_t)f * hidden + (hu < hidden ? hu : 0)];
        }
  std::vector<float> b1p((size_t)32 * kPolHP, 0.f);
  for (int j = 0; j < 32 * HP_kernel; ++j) b1p[j] = (float)bf16_to_double(b1[j < hidden ? j : 0]);
  // W2^T fragments: tile (grp, r), K-step s at ((grp * 3 + r) * 8 + s), lane l ->
  // row l % 16 = port 4 grp + (l % 16) / 4, level 4 r + l % 4; slot j -> hidden
  // unit in the order the first product leaves them in a lane.  Levels past the
  // class's have weights 0 and the lowest bias, whose softmax weight is 0 (not -inf:
  // beside a port whose own logits are all that low, it would be the NaN of inf - inf).
  std::vector<uint16_t> w2p((size_t)G * kPolR * kPolHP * 64 * 8, 0);
  std::vector<float> b2p((size_t)G * kPolR * 16, 0.f);
  for (int grp = 0; grp < G; ++grp)
    for (int r = 0; r < kPolR; ++r) {
      const int tile = grp * kPolR + r;
      for (int row = 0; row < 16; ++row) {
        const int port = 4 * grp + (row >> 2), lev = 4 * r + (row & 3);
        if (lev >= L1) b2p[(size_t)tile * 16 + row] = -std::numeric_limits<float>::max();
        else if (port < N) b2p[(size_t)tile * 16 + row] = (float)bf16_to_double(b2[port * L1 + lev]);
      }
      for (int s = 0; s < HP; ++s)
        for (int l = 0; l < 64; ++l) {
          const int row = l & 15, q = l >> 4;
          const int port = 4 * grp + (row >> 2), lev = 4 * r + (row & 3);
          if (port >= N || lev >= L1) continue;
          const int o = port * L1 + lev;
          for (int j = 0; j < 8; ++j) {
            const int hu = 32 * s + (j < 4 ? 4 * q + j : 16 + 4 * q + (j - 4));
            w2p[((((size_t)tile * kPolHP + s) * 64 + l) * 8) + j] = w2[(size_t)hu * out_dim + o];
          }
        }
    }
  const size_t s_w1p = w1p.size() * 2, s_b1p = b1p.size() * 4, s_w2p = w2p.size() * 2, s_b2p = b2p.size() * 4;
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t o_b1p = al(s_w1p), o_w2p = o_b1p + al(s_b1p), o_b2p = o_w2p + al(s_w2p);
  const size_t bytes = o_b2p + al(s_b2p);
  void *mem = nullptr;
  if (hipMalloc(&mem, bytes) != hipSuccess) return fail_status(CX_E_OOM, "cx_set_policy: hipMalloc failed");
  unsigned char *b = static_cast<unsigned char *>(mem);
  hipError_t e;
  if ((e = hipMemcpy(b, w1p.data(), s_w1p, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(b + o_b1p, b1p.data(), s_b1p, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(b + o_w2p, w2p.data(), s_w2p, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(b + o_b2p, b2p.data(), s_b2p, hipMemcpyHostToDevice)) != hipSuccess) {
    (void)hipFree(mem);
    return hip_fail(ctx, e, "cx_set_policy upload");
  }
  // replacing a policy waits for work that may still read the old weights
  if ((e = hipStreamSynchronize(ctx->stream)) != hipSuccess) {
    (void)hipFree(mem);
    return hip_fail(ctx, e, "cx_set_policy synchronize");
  }
  PolicyRt *old = ctx->policy;
  PolicyRt *p = new PolicyRt();
  p->hidden = hidden; p->in_dim = in_dim; p->N = N; p->L1 = L1;
  p->K1 = K1; p->HP = HP; p->G = G;
  p->mem = mem;
  p->w1p = reinterpret_cast<const u32x4 *>(b);
  p->b1p = reinterpret_cast<const float *>(b + o_b1p);
  p->w2p = reinterpret_cast<const u32x4 *>(b + o_w2p);
  p->b2p = reinterpret_cast<const float *>(b + o_b2p);
  if (old) {  // keep the scratch buffers
    p->obs = old->obs; p->act = old->act; p->scratch_envs = old->scratch_envs;
    old->obs = nullptr; old->act = nullptr;
    ctx->policy = old;
    free_policy(ctx);
  }
  ctx->policy = p;
  return CX_OK;
}

cx_status cx_policy_logits(cx_ctx *ctx, const float *obs_dev, int64_t n, float *logits_dev) {
  if (!ctx) return fail_status(CX_E_INVALID, "context is NULL");
  if (ctx->failed) return fail_status(CX_E_DEVICE, "context has a sticky device error");
  if (!ctx->policy) return fail_status(CX_E_INVALID, "no policy set (cx_set_policy)");
  if (n < 0) return fail_status(CX_E_INVALID, "cx_policy_logits: n < 0");
  if (n > 0 && (!obs_dev || !logits_dev)) return fail_status(CX_E_INVALID, "cx_policy_logits: NULL buffer");
  if (n > 0 && (reinterpret_cast<uintptr_t>(obs_dev) & 15u) != 0)
    return fail_status(CX_E_INVALID, "cx_policy_logits: obs_dev must be 16-byte aligned");
  if (n == 0) return CX_OK;
  PolicyArgs a = policy_args(ctx, obs_dev, n);
  a.logits = logits_dev;
  hipError_t e = launch_policy(a, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "cx_policy_logits launch");
  return CX_OK;
}

cx_status cx_policy_sample(cx_ctx *ctx, const float *obs_dev, int64_t n, uint32_t g, uint8_t *act_dev) {
  if (!ctx) return fail_status(CX_E_INVALID, "context is NULL");
  if (ctx->failed) return fail_status(CX_E_DEVICE, "context has a sticky device error");
  if (!ctx->policy) return fail_status(CX_E_INVALID, "no policy set (cx_set_policy)");
  if (n < 0) return fail_status(CX_E_INVALID, "cx_policy_sample: n < 0");
  if (n > 0 && (!obs_dev || !act_dev)) return fail_status(CX_E_INVALID, "cx_policy_sample: NULL buffer");
  if (n > 0 && (reinterpret_cast<uintptr_t>(obs_dev) & 15u) != 0)
    return fail_status(CX_E_INVALID, "cx_policy_sample: obs_dev must be 16-byte aligned");
  if (n == 0) return CX_OK;
  PolicyArgs a = policy_args(ctx, obs_dev, n);
  a.g = g;
  a.act = act_dev;
  hipError_t e = launch_policy(a, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "cx_policy_sample launch");
  return CX_OK;
}

cx_status cx_rollout_policy_noalloc(cx_ctx *ctx, int32_t T, cx_out_mode out_mode, const cx_traj *out) {
  if (!ctx) return fail_status(CX_E_INVALID, "context is NULL");
  if (ctx->failed) return fail_status(CX_E_DEVICE, "context has a sticky device error");
  if (T < 0 || T > (1 << 24)) return fail_status(CX_E_INVALID, "T must be in 0..2^24");
  if (out_mode < CX_OUT_FULL || out_mode > CX_OUT_ACT_REWARD) return fail_status(CX_E_INVALID, "bad out mode");
  if (!ctx->policy) return fail_status(CX_E_INVALID, "no policy set (cx_set_policy)");
  // one step of observations (16-byte aligned for the policy kernel), then one of levels
  const size_t obs_bytes = ((size_t)ctx->obs_elems * sizeof(float) + 255) & ~(size_t)255;
  const size_t need = obs_bytes + (size_t)ctx->total_ports;
  if (need > kNoAllocScratchBytes)
    return fail_status(CX_E_INVALID, "cx_rollout_policy_noalloc: the context needs " + std::to_string(need) +
                                         " bytes of scratch per step, more than the fixed " +
                                         std::to_string(kNoAllocScratchBytes) + " bytes");
  if (T == 0) return CX_OK;
  unsigned char *base = nullptr;
  cx_status st = noalloc_scratch(ctx->device, &base);
  if (st != CX_OK) return st;
  return policy_step_with(ctx, T, out_mode, out, reinterpret_cast<float *>(base), base + obs_bytes);
}

cx_status cx_observe(cx_ctx *ctx, float *obs_dev) {
  if (!ctx) return fail_status(CX_E_INVALID, "context is NULL");
  if (ctx->failed) return fail_status(CX_E_DEVICE, "context has a sticky device error");
  if (!obs_dev) return fail_status(CX_E_INVALID, "cx_observe: obs_dev is NULL");
  hipError_t e = launch_observe(ctx, obs_dev, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "cx_observe launch");
  return CX_OK;
}

}  // extern "C"
