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
