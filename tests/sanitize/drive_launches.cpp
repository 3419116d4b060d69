// drive_launches.cpp -- the choice of kernels and launch shapes on the fake HIP
// device (fake_hip.cpp), which checks every range a launch would touch (test
// infrastructure).
//
// Usage: drive_launches SECTION
//   horizons   a mixture that runs as a graph, calls of different kinds in turn
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "cx.h"

extern "C" long fake_hip_graph_destroys_in_flight();
extern "C" long fake_hip_live_allocations();

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

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  const long live0 = fake_hip_live_allocations();
  if (what == "horizons") horizons();
  else return 2;
  std::printf("graph execs destroyed with launches in flight: %ld\n", fake_hip_graph_destroys_in_flight());
  std::printf("device allocations left: %ld\n", fake_hip_live_allocations() - live0);
  std::printf("DRIVE OK\n");
  return 0;
}
