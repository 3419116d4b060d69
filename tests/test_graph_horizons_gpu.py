"""A context whose rollouts are graphs (general and extended classes among its
packings), called with changing horizons and record sets, nothing waited for in
between: records and state equal those of the same steps taken one by one."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cxm():
    from paper_2507_01522_amd import cx
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    return cx


@pytest.mark.parametrize("stage", [False, True])
def test_alternating_calls(cxm, stage):
    specs = [W.fanout4_tree(16, 2), W.fanout4_tree(64, 3), W.two_charger_types(), W.v2g_station(), W.user_station()]
    ec = np.repeat(np.arange(len(specs)), [40, 9, 13, 7, 11])
    a, b = cxm.Env(specs, env_class=ec, seed=61), cxm.Env(specs, env_class=ec, seed=61)
    a.set_obs_stage(stage)
    full, act, rew = cxm.OUT_FULL, cxm.OUT_ACT_REWARD, cxm.OUT_REWARD
    calls = [(40, full), (1, full), (33, rew), (1, act), (24, full)] * 3
    outs = [a.rollout(T, cxm.ACT_RANDOM, mode) for T, mode in calls]
    for (T, _), out in zip(calls, outs):
        for t in range(T):
            ref = b.step(cxm.ACT_RANDOM)
            for k in out:
                assert torch.equal(out[k][t].reshape(-1), ref[k].reshape(-1)), (k, t)
    assert a.get_state() == b.get_state()
