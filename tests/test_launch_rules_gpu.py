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
