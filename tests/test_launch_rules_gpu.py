"""The launch's own choice of the observation stage (rollouts of at least as many
waves as the GPU holds at once, 32 steps or more) against lane stores: the same
stations stepped in calls too short for it, record for record."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

WAVES = 8192


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return cx


@pytest.mark.parametrize("ports,extra", [(8, 0), (8, 5), (64, -1), (64, 3)])
def test_stage_chosen_by_size(cxm, ports, extra):
    """8 stations a wave (8 ports) or one (64): exactly WAVES waves, a ragged few
    more, and one fewer (lane stores in both)."""
    spec = W.fanout4_tree(ports, 2)
    n = WAVES * (64 // ports) + extra
    a, b = cxm.Env(spec, n_envs=n, seed=41), cxm.Env(spec, n_envs=n, seed=41)
    x = a.rollout(40, cxm.ACT_RANDOM)
    for t0 in (0, 20):
        y = b.rollout(20, cxm.ACT_RANDOM)
        for k in y:
            assert torch.equal(x[k][t0:t0 + 20], y[k]), (k, t0)
    assert a.get_state() == b.get_state()


@pytest.mark.parametrize("n,T", [(40, 1), (40, 45), (700, 33)])
def test_one_launch_for_all_packings(cxm, n, T):
    """Classes of five packings (8 to 128 ports, ragged env counts) in one launch
    against each class in a context of its own, where it is a launch of its own."""
    specs = [W.fanout4_tree(p, d) for p in (8, 16, 32, 64, 128) for d in (1, 3)]
    counts = [n + 3 * i for i in range(len(specs))]
    ec = np.repeat(np.arange(len(specs)), counts)
    env = cxm.Env(specs, env_class=ec, seed=43)
    env.rollout(140, cxm.ACT_MAX, cxm.OUT_REWARD)
    out = env.step(cxm.ACT_RANDOM) if T == 1 else env.rollout(T, cxm.ACT_RANDOM)
    # a context per class, its other envs in a second class that keeps the env indices
    for c, spec in enumerate(specs):
        pair = cxm.Env([spec, W.two_charger_types()], env_class=np.repeat([0, 1], [ec.size - 1, 1]), seed=43)
        pair.rollout(140, cxm.ACT_MAX, cxm.OUT_REWARD)
        ref = pair.step(cxm.ACT_RANDOM) if T == 1 else pair.rollout(T, cxm.ACT_RANDOM)
        ci = env.class_info(c)
        e0, e1 = ci.env_begin, min(ci.env_begin + ci.n_envs, ec.size - 1)   # same env index, same draws
        k = e1 - e0
        for key, off, width in (("reward", e0, 1), ("done", e0, 1), ("actions", ci.port_offset, ci.n_actions),
                                ("obs", ci.obs_offset, ci.obs_dim)):
            own = ref[key][:, e0 * width:e1 * width]
            assert torch.equal(out[key][:, off:off + k * width], own), (c, key)


MODE_SPECS = {"simple": lambda: W.fanout4_tree(32, 2), "general": lambda: W.fanout4_tree(31, 2).replace(alpha_sat=0.2),
              "dense": lambda: W.two_charger_types(), "v2g": lambda: W.v2g_station(alpha_degrad_cars=0.03),
              "users": lambda: W.user_station(), "exo": lambda: W.exo_station()}


@pytest.mark.parametrize("stage", [False, True])
@pytest.mark.parametrize("per_lane", [1, 2, 4])
@pytest.mark.parametrize("name", sorted(MODE_SPECS))
def test_modes_equal_full_records(cxm, name, per_lane, stage):
    """The kernels of calls without observation records and of one step against
    those of any call: the same levels, rewards, done flags, observations and state."""
    spec = MODE_SPECS[name]()
    n, T = 37, 5
    envs = [cxm.Env(spec, n_envs=n, seed=47) for _ in range(4)]
    for e in envs:
        e.set_packing(0, e.class_info(0).slots // per_lane, 2)
        e.set_obs_stage(stage)
        e.rollout(140, cxm.ACT_RANDOM)
    full, levels, rewards, steps = envs
    x = full.rollout(T, cxm.ACT_RANDOM)
    y = levels.rollout(T, cxm.ACT_RANDOM, cxm.OUT_ACT_REWARD)
    z = rewards.rollout(T, cxm.ACT_RANDOM, cxm.OUT_REWARD)
    assert set(z) < set(y) < set(x)
    for r in (y, z):
        for k in r:
            assert torch.equal(r[k], x[k]), k
    for t in range(T):
        w = steps.step(cxm.ACT_EXTERNAL, actions=x["actions"][t]) if t % 2 else steps.step(cxm.ACT_RANDOM)
        for k in w:
            assert torch.equal(w[k].reshape(-1), x[k][t].reshape(-1)), (k, t)
    for e in (levels, rewards, steps):
        assert e.get_state() == full.get_state()
