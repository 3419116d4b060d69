// drive_launches.cpp -- the choice of kernels and launch shapes on the fake HIP
// device (fake_hip.cpp), which checks every range a launch would touch (test
// infrastructure).
//
// Usage: drive_launches SECTION
//   horizons   a mixture that runs as a graph, calls of different kinds in turn
//   parts      mixtures of SIMPLE packings, in one launch and past its limits
//   stage      the observation stage chosen by a launch's size
//   policy     policy rollouts of every size of the fused kernels, and the two kernels
//   grids      calls of more than 2^32 threads
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "cx.h"
#include "cx_internal.h"

extern "C" long fake_hip_graph_destroys_in_flight();
extern "C" long fake_hip_live_allocations();
extern "C" long fake_hip_launches(const char *part);
extern "C" void fake_hip_only_count(bool on);

namespace {

[[noreturn]] void fail(const char *what, int line) {
  std::fprintf(stderr, "DRIVE FAILED: line %d: %s: %s\n", line, what, cx_last_error());
  std::fflush(stderr);
  std::exit(3);
}
#define CK(x)                                    \
  do {                                           \
    if ((x) != CX_OK) fail(#x, __LINE__);        \
  } while (0)
#define REQUIRE(x)                               \
  do {                                           \
    if (!(x)) fail(#x, __LINE__);                \
  } while (0)

// A station of n ports under splitters of four; uneven: ports of unequal
// efficiency (the general kind), v2g: bidirectional ports (the extended kind).
struct Station {
  cx_station_spec s{};
  std::vector<int32_t> node_parent, port_parent;
  std::vector<double> limit, node_eta, pmax, eta;
  explicit Station(int n, bool uneven = false, bool v2g = false) {
    node_parent.push_back(-1);
    limit.push_back(12.0 * n);
    for (int h = 0; h < (n + 3) / 4; ++h) {
      node_parent.push_back(0);
      limit.push_back(60.0);
    }
    node_eta.assign(limit.size(), 1.0);
    for (int i = 0; i < n; ++i) {
      port_parent.push_back(1 + i / 4);
      pmax.push_back(22.0);
      eta.push_back(uneven ? 0.9 + 0.01 * (i % 5) : 1.0);
    }
    s.n_ports = n;
    s.n_nodes = (int32_t)node_parent.size();
    s.node_parent = node_parent.data();
    s.node_limit_kw = limit.data();
    s.node_eta = node_eta.data();
    s.port_parent = port_parent.data();
    s.port_pmax_kw = pmax.data();
    s.port_eta = eta.data();
    s.dt_hours = 1.0 / 12;
    s.tau = 0.8;
    s.p_sell = 0.45;
    s.p_sell_grid = 0.25;
    s.steps_per_episode = 288;
    s.n_levels = 10;
    s.price_base = 0.25;
    s.price_amp = 0.1;
    s.price_sigma = 0.02;
    s.arrival_peak = 0.3;
    s.cap_lo = 40;
    s.cap_hi = 100;
    s.soc0_lo = 0.1;
    s.soc0_hi = 0.5;
    s.tgt_lo = 0.7;
    s.tgt_hi = 1.0;
    s.dwell_mu = 3.58;
    s.dwell_sigma = 0.5;
    s.dwell_max = 1024;
    s.v2g = v2g ? 1 : 0;
    s.battery_tau = 0.8;
    s.battery_soc0 = 0.5;
  }
  Station(const Station &) = delete;
};

// Device memory (not cleared: large buffers stay untouched pages).
struct Dev {
  void *p = nullptr;
  explicit Dev(size_t n) {
    if (hipMalloc(&p, n ? n : 1) != hipSuccess) fail("hipMalloc", __LINE__);
  }
  ~Dev() { (void)hipFree(p); }
};

struct Traj {
  std::vector<std::unique_ptr<Dev>> mem;
  cx_traj t{};
  Traj(const cx_info &i, int64_t T) {
    for (size_t n : {4 * (size_t)T * i.obs_elems, (size_t)T * i.total_ports, 4 * (size_t)T * i.n_envs,
                     (size_t)T * i.n_envs})
      mem.emplace_back(new Dev(n));
    t = cx_traj{static_cast<float *>(mem[0]->p), static_cast<uint8_t *>(mem[1]->p), static_cast<float *>(mem[2]->p),
                static_cast<uint8_t *>(mem[3]->p)};
  }
};

struct Context {
  cx_ctx *c = nullptr;
  cx_info info{};
  Context(const std::vector<const Station *> &st, const std::vector<int64_t> &counts) {
    std::vector<cx_station_spec> specs;
    std::vector<int32_t> ec;
    for (size_t i = 0; i < st.size(); ++i) {
      specs.push_back(st[i]->s);
      ec.insert(ec.end(), (size_t)counts[i], (int32_t)i);
    }
    CK(cx_create_multi(specs.data(), (int32_t)specs.size(), ec.data(), (int64_t)ec.size(), 7, &c));
    CK(cx_get_info(c, &info));
  }
  ~Context() { cx_destroy(c); }
  // launches of kernels named `part` that a call makes
  template <class F>
  long count(const char *part, F &&call) {
    CK(cx_synchronize(c));
    const long before = fake_hip_launches(part);
    CK(call());
    CK(cx_synchronize(c));
    return fake_hip_launches(part) - before;
  }
  cx_status rollout(int T, cx_out_mode mode, const Traj &tr) {
    return cx_rollout(c, T, CX_ACT_RANDOM, mode, nullptr, &tr.t);
  }
};

// Calls of different kinds in turn, none waited for: each launch shape has a graph
// of its own, and none is destroyed while its launch is in flight.  The large
// class brings the launch past the size at which the stage is chosen by itself.
void horizons() {
  const Station simple16(16), simple64(64), general(16, true), v2g(16, false, true);
  for (int64_t large : {5, 8200}) {
    for (int stage = 0; stage < 2; ++stage) {
      Context x({&simple16, &simple64, &general, &v2g}, {40, large, 9, 11});
      CK(cx_set_obs_stage(x.c, stage));
      Traj tr(x.info, 40);
      cx_traj bare = tr.t;
      bare.obs = nullptr;
      for (int k = 0; k < 4; ++k) {
        CK(cx_rollout(x.c, 40, CX_ACT_RANDOM, CX_OUT_FULL, nullptr, &tr.t));
        CK(cx_rollout(x.c, 24, CX_ACT_RANDOM, CX_OUT_FULL, nullptr, &tr.t));
        CK(cx_rollout(x.c, 1, CX_ACT_RANDOM, CX_OUT_FULL, nullptr, &tr.t));
        CK(cx_rollout(x.c, 1, CX_ACT_MAX, CX_OUT_REWARD, nullptr, &tr.t));
        CK(cx_rollout(x.c, 24, CX_ACT_MAX, CX_OUT_ACT_REWARD, nullptr, &tr.t));
        CK(cx_rollout(x.c, 40, CX_ACT_RANDOM, CX_OUT_FULL, nullptr, &bare));
        CK(cx_step_ex(x.c, CX_ACT_RANDOM, nullptr, &tr.t));
      }
      CK(cx_synchronize(x.c));
    }
  }
}

// Five packings of SIMPLE classes in every block size.
void parts() {
  Station s8(8), s16(16), s32(32), s64(64), s128(128), odd(16);
  odd.s.dwell_max = 4096;   // the launch's LDS holds the largest stay table and the longest day
  for (int steps : {288, 512, 600}) {   // (600: a day too long for the tables in LDS)
    for (Station *s : {&s8, &s16, &s32, &s64, &s128, &odd}) s->s.steps_per_episode = steps;
    Context x({&s8, &s16, &s32, &s64, &s128, &odd}, {70, 41, 9, 3, 2, 1});
    Traj tr(x.info, 40);
    Dev act_in((size_t)40 * x.info.total_ports);
    for (int wpb : {1, 2, 4, 8}) {
      for (int c = 0; c < x.info.n_classes; ++c) {
        cx_class_info ci{};
        CK(cx_get_class_info(x.c, c, &ci));
        CK(cx_set_packing(x.c, c, ci.slots == 128 || (ci.slots == 32 && wpb == 4) ? ci.slots / 2 : ci.slots, wpb));
      }
      for (int T : {1, 24, 40}) {
        for (cx_out_mode m : {CX_OUT_FULL, CX_OUT_ACT_REWARD, CX_OUT_REWARD})
          REQUIRE(x.count("k_rollout_parts<", [&] { return x.rollout(T, m, tr); }) == 1);
        CK(cx_rollout(x.c, T, CX_ACT_EXTERNAL, CX_OUT_FULL, static_cast<uint8_t *>(act_in.p), &tr.t));
      }
      REQUIRE(x.count("k_rollout_parts<2>", [&] { return cx_step_ex(x.c, CX_ACT_MAX, nullptr, &tr.t); }) == 1);
      // the stage asked for: rollouts that record observations take it, each packing
      // its own kernel; other calls have none
      CK(cx_set_obs_stage(x.c, 1));
      for (int T : {2, 24, 40}) {
        REQUIRE(x.count("k_rollout_parts<", [&] { return x.rollout(T, CX_OUT_FULL, tr); }) == 0);
        REQUIRE(x.count(", true, 0>", [&] { return x.rollout(T, CX_OUT_FULL, tr); }) >= 5);   // k_rollout_simple<., ., true, 0>
        REQUIRE(x.count("k_rollout_parts<1>", [&] { return x.rollout(T, CX_OUT_ACT_REWARD, tr); }) == 1);
      }
      REQUIRE(x.count("k_rollout_parts<2>", [&] { return x.rollout(1, CX_OUT_FULL, tr); }) == 1);
      CK(cx_set_obs_stage(x.c, 0));
    }
  }
  // every record: one launch up to 10,240 waves, past them a graph; one step and
  // calls without observations always one launch.  64-port stations take a wave
  // each, 16-port ones a quarter of one; blocks of 4 waves.
  for (Station *s : {&s16, &s64}) s->s.steps_per_episode = 288;
  for (int64_t n64 : {10240 - 4, 10240}) {
    Context x({&s16, &s64}, {16, n64});
    Traj tr(x.info, 33);
    const bool one = n64 + 4 <= 10240;
    REQUIRE(x.count("k_rollout_parts<0>", [&] { return x.rollout(33, CX_OUT_FULL, tr); }) == (one ? 1 : 0));
    REQUIRE(x.count("k_rollout_simple<64, 1, true, 0>", [&] { return x.rollout(33, CX_OUT_FULL, tr); }) == (one ? 0 : 1));
    REQUIRE(x.count("k_rollout_parts<1>", [&] { return x.rollout(33, CX_OUT_REWARD, tr); }) == 1);
    REQUIRE(x.count("k_rollout_parts<2>", [&] { return cx_step_ex(x.c, CX_ACT_MAX, nullptr, &tr.t); }) == 1);
  }
}

// One SIMPLE packing: every record of 32 steps or more goes through the stage from
// 8,192 waves (2,048 blocks of 4), below it and in shorter calls only when asked.
void stage() {
  const Station s64(64);
  for (int64_t n : {8192 - 4, 8192 - 3}) {
    Context x({&s64}, {n});
    Traj tr(x.info, 32);
    const long big = n == 8192 - 3;   // (a last block of one wave counts as four)
    const char *staged = "k_rollout_simple<64, 1, true, 0>";
    REQUIRE(x.count(staged, [&] { return x.rollout(32, CX_OUT_FULL, tr); }) == big);
    REQUIRE(x.count(staged, [&] { return x.rollout(31, CX_OUT_FULL, tr); }) == 0);
    REQUIRE(x.count(staged, [&] { return x.rollout(32, CX_OUT_ACT_REWARD, tr); }) == 0);
    CK(cx_set_obs_stage(x.c, 1));
    REQUIRE(x.count(staged, [&] { return x.rollout(31, CX_OUT_FULL, tr); }) == 1);
    REQUIRE(x.count(staged, [&] { return x.rollout(1, CX_OUT_FULL, tr); }) == 1);
  }
}

void policy_rollouts(const Station &st, int64_t n, int hidden, const char *kernel) {
  Context x({&st}, {n});
  const int in = 6 * st.s.n_ports + 4, out = st.s.n_ports * (st.s.n_levels + 1);
  const std::vector<uint16_t> w1((size_t)in * hidden, 0x3c00), b1(hidden, 0x3c00), w2((size_t)hidden * out, 0x3c00),
      b2(out, 0x3c00);
  CK(cx_set_policy(x.c, hidden, w1.data(), b1.data(), w2.data(), b2.data()));
  Traj tr(x.info, 40);
  auto run = [&](int T, cx_out_mode m) { return cx_rollout(x.c, T, CX_ACT_POLICY, m, nullptr, &tr.t); };
  for (cx_out_mode m : {CX_OUT_FULL, CX_OUT_ACT_REWARD, CX_OUT_REWARD}) {
    REQUIRE(x.count(kernel, [&] { return run(40, m); }) > 0);
    REQUIRE(x.count(kernel, [&] { return run(3, m); }) > 0);
  }
  CK(cx_step_ex(x.c, CX_ACT_POLICY, nullptr, &tr.t));
  Dev logits(4 * (size_t)n * out);
  CK(cx_policy_logits(x.c, tr.t.obs, n, static_cast<float *>(logits.p)));
  CK(cx_policy_sample(x.c, tr.t.obs, n, 3, tr.t.actions));
  CK(cx_rollout_policy_noalloc(x.c, 3, CX_OUT_FULL, &tr.t));
}

void policy() {
  for (int hidden : {32, 96, 128, 256}) {
    const int hp = hidden <= 64 ? 2 : hidden <= 128 ? 4 : 8;
    auto name = [&](bool general, int L, int P, bool held) {
      return std::string(general ? "k_rollout_policy_general<" : "k_rollout_policy<") + std::to_string(L) + ", " +
             std::to_string(P) + ", " + std::to_string(hp) + ", " + (held ? "true>" : "false>");
    };
    // 8, 16 and 32 slots: SIMPLE, and with padding slots and uneven ports.  Blocks
    // of 32 stations (8 lanes) or 16 (16 lanes); weights held up to 256 blocks.
    struct {
      int ports;
      bool uneven;
    } const stations[] = {{8, false}, {16, false}, {32, false}, {7, true}, {13, true}, {29, true}, {32, true}};
    for (const auto &c : stations) {
      const int S = c.ports <= 8 ? 8 : c.ports <= 16 ? 16 : 32;
      for (int dwell : {2, 1024, 4096}) {
        for (int steps : {288, 600}) {
          Station st(c.ports, c.uneven);
          st.s.dwell_max = dwell;
          st.s.steps_per_episode = steps;
          // (32 slots and a stay table of more than 1,024 entries: no LDS for the held layout)
          const bool held = S < 32 || dwell <= 1024;
          for (int64_t n : {1, 33})
            policy_rollouts(st, n, hidden, name(c.uneven, S == 16 ? 16 : 8, S == 16 ? 1 : S / 8, held).c_str());
        }
      }
      const Station st(c.ports, c.uneven);
      if (S == 16) {
        policy_rollouts(st, 4096, hidden, name(c.uneven, 16, 1, true).c_str());
        policy_rollouts(st, 4097, hidden, name(c.uneven, 8, 2, true).c_str());
      }
      policy_rollouts(st, 8192, hidden, name(c.uneven, 8, S / 8, true).c_str());
      policy_rollouts(st, 8193, hidden, name(c.uneven, 8, S / 8, false).c_str());
    }
  }
  // classes of other sizes take two kernels a step
  for (int ports : {3, 41}) policy_rollouts(Station(ports), 70, 128, "k_policy(");
  // ... with a kernel of its own for 16,384 stations and more of up to 8 ports
  policy_rollouts(Station(3), 16383, 32, "k_policy(");
  for (int hidden : {32, 64, 96, 256}) policy_rollouts(Station(3), 16384, hidden, "k_policy_few<");
  for (int ports : {1, 4, 5, 8, 9}) {
    const Station st(ports);
    Context x({&st}, {1});
    const int in = 6 * ports + 4, out = ports * 11, hidden = 96;
    const std::vector<uint16_t> w1((size_t)in * hidden), b1(hidden), w2((size_t)hidden * out), b2(out);
    CK(cx_set_policy(x.c, hidden, w1.data(), b1.data(), w2.data(), b2.data()));
    for (int64_t n : {16383, 16384, 16385, 40001}) {
      const Dev obs((size_t)n * in * 4), act((size_t)n * ports), logits(4 * (size_t)n * out);
      auto o = static_cast<const float *>(obs.p);
      REQUIRE(x.count("k_policy_few<", [&] { return cx_policy_sample(x.c, o, n, 3, static_cast<uint8_t *>(act.p)); }) ==
              (n >= 16384 && ports <= 8));
      REQUIRE(x.count("k_policy_few<", [&] { return cx_policy_logits(x.c, o, n, static_cast<float *>(logits.p)); }) ==
              (n >= 16384 && ports <= 4));
    }
  }
}

// A launch has fewer than 2^32 threads.
void grids() {
  // the policy's levels for 540 M observations of one port (21 GB)
  const Station st(1);
  Context x({&st}, {1});
  const int in = 10, out = 11, hidden = 32;
  const std::vector<uint16_t> w1(in * hidden), b1(hidden), w2(hidden * out), b2(out);
  CK(cx_set_policy(x.c, hidden, w1.data(), b1.data(), w2.data(), b2.data()));
  const int64_t n = 540'000'001;
  const Dev obs((size_t)n * in * 4), act((size_t)n);
  CK(cx_policy_sample(x.c, static_cast<const float *>(obs.p), n, 3, static_cast<uint8_t *>(act.p)));
  CK(cx_synchronize(x.c));
  // ... and for as many of nine ports, in blocks of 32 (125 GB, so only counted): two launches
  {
    const Station nine(9);
    Context y({&nine}, {1});
    const std::vector<uint16_t> v1((size_t)58 * hidden), v2((size_t)hidden * 99), c2(99);
    CK(cx_set_policy(y.c, hidden, v1.data(), b1.data(), v2.data(), c2.data()));
    fake_hip_only_count(true);
    REQUIRE(y.count("k_policy(", [&] {
      return cx_policy_sample(y.c, static_cast<const float *>(obs.p), n, 3, static_cast<uint8_t *>(act.p));
    }) == 2);
    fake_hip_only_count(false);
  }
  // two packings of 40 M blocks of a wave each, which fit one by one
  const cx::SegDev segs[2] = {};
  cx::LaunchArgs a{};
  a.segs = segs;
  a.T = 1;
  a.mode = CX_ACT_RANDOM;
  a.out_mode = CX_OUT_REWARD;
  cx::LaunchGroup g[2];
  for (int i = 0; i < 2; ++i) {
    g[i].kind = cx::kKindSimple;
    g[i].pack = cx::pack_id(i ? 64 : 32, 1);
    g[i].seg_begin = i;
    g[i].n_segs = 1;
    g[i].n_blocks = 40'000'000;
    g[i].wpb = 1;
  }
  fake_hip_only_count(true);
  const long before = fake_hip_launches("k_rollout");
  REQUIRE(cx::launch_groups(a, g, 2, nullptr) == hipSuccess);
  fake_hip_only_count(false);
  REQUIRE(fake_hip_launches("k_rollout") == before + 2);
}

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  const long live0 = fake_hip_live_allocations();
  if (what == "horizons") horizons();
  else if (what == "parts") parts();
  else if (what == "stage") stage();
  else if (what == "policy") policy();
  else if (what == "grids") grids();
  else return 2;
  std::printf("graph execs destroyed with launches in flight: %ld\n", fake_hip_graph_destroys_in_flight());
  std::printf("device allocations left: %ld\n", fake_hip_live_allocations() - live0);
  std::printf("DRIVE OK\n");
  return 0;
}
