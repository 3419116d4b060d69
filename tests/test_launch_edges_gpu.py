"""Both sides of the sizes at which a launch's kernels change: 8,192 waves of one
packing (the observation stage, 32 steps or more) and 10,240 waves of several
(one launch below, a graph of staged kernels above).  Blocks are of 4 waves and a
64-port station takes a wave, so one station fewer can be a whole block fewer.
Records equal those of calls too short for the stage."""
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


@pytest.mark.parametrize("n16,n64", [(0, 8192 - 4), (0, 8192 - 3), (16, 10240 - 4), (16, 10240 - 3)])
def test_both_sides_of_the_launch_sizes(cxm, n16, n64):
    specs = [W.fanout4_tree(16, 2), W.fanout4_tree(64, 3)]
    if not n16:
        specs = specs[1:]
    ec = np.repeat(np.arange(len(specs)), [n16, n64][-len(specs):])
    a, b = (cxm.Env(specs, env_class=ec, seed=67) for _ in range(2))
    for e in (a, b):
        e.rollout(140, cxm.ACT_RANDOM, cxm.OUT_REWARD)
    x = a.rollout(33, cxm.ACT_RANDOM)
    for t0, T in ((0, 20), (20, 13)):
        y = b.rollout(T, cxm.ACT_RANDOM)
        for k in y:
            assert torch.equal(x[k][t0:t0 + T], y[k]), (k, t0)
    assert a.get_state() == b.get_state()
